// Max-hop 2-opt (objectives MAX and MAX_DIRECTED) for any 4 <= N <= 1024 and any entries: only the moves that can win
// are scored.  Move set, value and tie-break rules as stated in cc.h.
//
// Let V be the largest hop of the order and e its edge.  A move lowers the cost only if no hop of value V is left, so
//   * undirected: it removes e - N - 3 moves instead of N (N-3) / 2;
//   * directed: it removes e, or walks e the other way.  Exchanging the edges x and y (edge p joins ranks p-1 and p)
//     with the piece x+1 .. y-1 reversed keeps the forward hops f of y+1 .. x-1, takes the backward hops b of
//     x+1 .. y-1 and adds two new hops.  With e inside the reversed piece, x lies l >= 1 edges before e and y r >= 1
//     behind it, and no edge of the piece may have b >= V: that bounds l and r by the nearest such edges on either
//     side.  After s moves there are about s of them, so a sweep looks at about min(N, N / s)^2 pairs, about 2 N^2 over
//     a whole descent, where the exhaustive sweeps look at N^2 each.
// The winner (value, lowest id) is the exhaustive sweep's: every move that lowers the cost is scored, or dropped
// because a part of its value already exceeds the best one seen.
//
// One workgroup per restart; order and hops in LDS, carried through the moves; rows of the matrix through L2.  A sweep
// is a chain of latencies (two or three wave reductions, two LDS round trips, one gather, the move; about 8000 clocks
// directed at N = 100): no matrix staging, so any number of workgroups share a
// compute unit.  Whole searches, against the exhaustive kernels: undirected N = 50, 1197 restarts 587 -> 60 us, N = 256, 1024
// restarts 1456 -> 160 us, N = 700, 100 restarts 21 -> 0.26 ms; directed, inverse bandwidths that are eight times as small
// inside a rack, N = 100, 1000 restarts 2272 -> 205 us, N = 256, 1024 restarts 2656 -> 551 us, N = 350, 316 restarts
// 20.4 -> 0.71 ms, N = 1023, 41 restarts 141 -> 1.5 ms; directed on a symmetric matrix, N = 256, 1024 restarts 2350 -> 252 us
// (fewer sweeps).
#include "cc_device.h"
#include "cc_internal.h"
#include "cc_wave64.h"

namespace cc {
using namespace ccd;

namespace {

constexpr int kCostMax = (1 << 21) - 1;
constexpr int kNone = 0x7fffffff;

// Smallest (hi, lo) over the workgroup, lexicographically; every thread gets it.  `red`: one word pair per wave and
// parity, so that one barrier per call is enough.
template <int NW>
struct GroupMin {
    int (*red)[NW][2];
    int parity = 0;
    __device__ __forceinline__ static void in_wave(int& hi, int& lo) {
        const int h = wave_min(hi);
        const unsigned long long at = __ballot(hi == h);
        int l = __builtin_amdgcn_readlane(lo, (int)__builtin_ctzll(at));
        if (at & (at - 1)) l = wave_min(hi == h ? lo : kNone);
        hi = h;
        lo = l;
    }
    __device__ __forceinline__ void operator()(int& hi, int& lo, int wv, int lane) {
        in_wave(hi, lo);
        if (NW > 1) {
            if (lane == 0) {
                red[parity][wv][0] = hi;
                red[parity][wv][1] = lo;
            }
            __syncthreads();
            hi = red[parity][0][0];
            lo = red[parity][0][1];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                const int h = red[parity][w][0], l = red[parity][w][1];
                const bool less = h < hi || (h == hi && l < lo);
                hi = less ? h : hi;
                lo = less ? l : lo;
            }
            hi = __builtin_amdgcn_readfirstlane(hi);
            lo = __builtin_amdgcn_readfirstlane(lo);
            parity ^= 1;
        }
    }
};

template <int NW>
__device__ __forceinline__ void group_sync() {
    if (NW > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
}

// ----------------------------------------------------------------------------------------- undirected
// THREADS per restart, up to E ranks per thread (rank = thread + THREADS * k).
template <int THREADS, int E>
__global__ __launch_bounds__(THREADS) void twoopt_max_pruned_kernel(const int32_t* __restrict__ c, int N,
                                                                    int32_t* __restrict__ tours,
                                                                    int64_t* __restrict__ costs,
                                                                    int32_t* __restrict__ moves) {
    constexpr int NW = THREADS / 64;
    __shared__ int32_t t[THREADS * E], f[THREADS * E];
    __shared__ int red[2][NW][2];
    __shared__ int tops[2][NW][3];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.x;
    GroupMin<NW> group_min{red};
    int my_f[E], my_t[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int p = tid + THREADS * k;
        my_t[k] = p < N ? clampi(tours[r * N + p], 0, N - 1) : 0;
        if (p < N) t[p] = my_t[k];
    }
    group_sync<NW>();
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int p = tid + THREADS * k;
        my_f[k] = p < N ? clampi(c[my_t[k] * N + t[p ? p - 1 : N - 1]], 0, kCostMax) : 0;
        if (p < N) f[p] = my_f[k];
    }
    int applied = 0, parity = 0, cur;
    for (;;) {
        group_sync<NW>();
        // ---- the three largest hops: value << 10 | edge
        int key[E], k1 = -1, k2 = -1, k3 = -1;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = tid + THREADS * k;
            key[k] = p < N ? (my_f[k] << 10) | p : -1;
            k1 = max(k1, key[k]);
        }
        k1 = wave_max(k1);
#pragma unroll
        for (int k = 0; k < E; ++k) k2 = max(k2, key[k] == k1 ? -1 : key[k]);
        k2 = wave_max(k2);
#pragma unroll
        for (int k = 0; k < E; ++k) k3 = max(k3, key[k] == k1 || key[k] == k2 ? -1 : key[k]);
        k3 = wave_max(k3);
        if (NW > 1) {
            if (lane == 0) {
                tops[parity][wv][0] = k1;
                tops[parity][wv][1] = k2;
                tops[parity][wv][2] = k3;
            }
            __syncthreads();
            const int v = lane < 3 * NW ? (&tops[parity][0][0])[lane] : -1;
            k1 = wave_max(v);
            k2 = wave_max(v == k1 ? -1 : v);
            k3 = wave_max(v == k1 || v == k2 ? -1 : v);
            parity ^= 1;
        }
        cur = k1 >> 10;
        if ((k3 >> 10) == cur) break;              // three largest hops: no move removes them all
        const int e = k1 & 1023, second = k2 & 1023;
        const int rest = k2 >> 10, rest_without_second = k3 >> 10;
        // ---- the N - 3 moves that remove e
        const int32_t* row_before = c + (int64_t)t[e ? e - 1 : N - 1] * N;
        const int32_t* row_at = c + (int64_t)t[e] * N;
        int hi = cur, lo = kNone, x_best = 0, y_best = 0;
        int x[E], y[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int b = min(tid + THREADS * k, N - 1);
            x[k] = row_before[t[b ? b - 1 : N - 1]];
            y[k] = row_at[my_t[k]];
        }
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int b = tid + THREADS * k;
            const int x0 = clampi(x[k], 0, kCostMax), y0 = clampi(y[k], 0, kCostMax);
            const int value = max(max(x0, y0), b == second ? rest_without_second : rest);
            const int a = min(e, b), d = max(e, b);
            const int id = a ? a * N + d - 1 : d * N + N - 1;
            const bool fits = b < N && d - a >= 2 && d - a <= N - 2;
            if (fits && (value < hi || (value == hi && id < lo && value < cur))) {
                hi = value;
                lo = id;
                x_best = x0;
                y_best = y0;
            }
        }
        const int my_id = lo;
        group_min(hi, lo, wv, lane);
        if (hi >= cur) break;
        // ---- reverse ranks mi .. mj; hops follow, two are new (the winning thread has them)
        const int mi = lo / N, mj = lo - mi * N;
        const int after = mj + 1 == N ? 0 : mj + 1;
        int new_f[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = tid + THREADS * k;
            const bool inside = p >= mi && p <= mj;
            my_t[k] = inside ? t[mi + mj - p] : my_t[k];
            new_f[k] = inside && p > mi ? f[mi + mj + 1 - p] : my_f[k];
        }
        group_sync<NW>();
        if (my_id == lo) {
            f[mi] = x_best;
            f[after] = y_best;
        }
        group_sync<NW>();
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = tid + THREADS * k;
            my_f[k] = p == mi || p == after ? f[p < N ? p : 0] : new_f[k];
            if (p < N) {
                if (p >= mi && p <= mj) t[p] = my_t[k];
                f[p] = my_f[k];
            }
        }
        ++applied;
    }
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int p = tid + THREADS * k;
        if (p < N) tours[r * N + p] = my_t[k];
    }
    if (tid == 0) {
        costs[r] = (int64_t)cur;
        moves[r] = applied;
    }
}

// ------------------------------------------------------------------------------------------- directed
// Inclusive prefix maximum over the lanes of a wave (values >= 0).
__device__ __forceinline__ int wave_prefix_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));      // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));      // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));      // row_bcast:31
    return v;
}

// THREADS per restart, E consecutive edges per thread, N <= THREADS * E.  Edges are numbered from e: edge u of a sweep
// is edge (e + u) mod N of the order.
template <int THREADS, int E>
__global__ __launch_bounds__(THREADS) void twoopt_max_directed_pruned_kernel(const int32_t* __restrict__ c, int N,
                                                                             int with_flip,
                                                                             int32_t* __restrict__ tours,
                                                                             int64_t* __restrict__ costs,
                                                                             int32_t* __restrict__ moves) {
    constexpr int NW = THREADS / 64, kMax = THREADS * E;
    constexpr int kAhead = 2;                          // pairs of a thread whose loads are in flight together
    __shared__ int32_t t[kMax], f[kMax], b[kMax];
    // prefix maxima over the edges 1 .. u (index u) and the last m edges N-m .. N-1 (index m); 0 at index 0
    __shared__ int32_t b_right[kMax + 1], f_right[kMax + 1], b_left[kMax + 1], f_left[kMax + 1];
    __shared__ int32_t rn[kMax + 1];                   // nodes from e on: edge u joins rn[u] and rn[u + 1]
    // what a piece that ends r edges behind e, l edges before e brings with it (index r, l): its backward hops on that
    // side and the kept hops beyond, up to the cut z
    __shared__ int32_t right[kMax + 1], left[kMax + 1];
    __shared__ int red[2][NW][2];
    __shared__ int carry[NW][4];
    __shared__ int reach[2][NW][2], tops[NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.x;
    GroupMin<NW> group_min{red};
    auto C = [&](int from, int to) { return clampi(c[from * N + to], 0, kCostMax); };
    for (int p = tid; p < N; p += THREADS) t[p] = clampi(tours[r * N + p], 0, N - 1);
    if (tid == 0) b_right[0] = f_right[0] = b_left[0] = f_left[0] = 0;
    group_sync<NW>();
    for (int p = tid; p < N; p += THREADS) {
        const int q = t[p ? p - 1 : N - 1];
        f[p] = C(t[p], q);
        b[p] = C(q, t[p]);
    }
    int applied = 0, cur, parity = 0;
    for (;;) {
        group_sync<NW>();
        // ---- the largest hop and its edge
        int top = -1;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = tid + THREADS * k;
            if (p < N) top = max(top, (f[p] << 10) | p);
        }
        top = wave_max(top);
        if (NW > 1) {
            if (lane == 0) tops[wv] = top;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) top = max(top, tops[w]);
            top = __builtin_amdgcn_readfirstlane(top);
        }
        cur = top >> 10;
        const int e = top & 1023;
        auto edge = [&](int u) { const int p = e + u; return p >= N ? p - N : p; };          // 0 <= u < N
        const int b0 = b[e];
        // ---- prefix maxima from e to the right and to the left
        int v[4][E], turned_t[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int u = tid * E + k, m = N - 1 - u;                  // u-th edge from the left end, u-th from the right
            const int pr = edge(min(u, N - 1)), pl = edge(max(m, 0));
            const bool right = u >= 1 && u < N, left = m >= 1;         // e itself is in neither
            v[0][k] = right ? b[pr] : 0;
            v[1][k] = right ? f[pr] : 0;
            v[2][k] = left ? b[pl] : 0;
            v[3][k] = left ? f[pl] : 0;
            turned_t[k] = t[pr];
        }
        int before[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int k = 1; k < E; ++k) v[i][k] = max(v[i][k], v[i][k - 1]);
            before[i] = wave_prefix_max(v[i][E - 1]);
        }
        if (NW > 1) {
            if (lane == 63) {
#pragma unroll
                for (int i = 0; i < 4; ++i) carry[wv][i] = before[i];
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // what lies in front of this thread's edges
            before[i] = __builtin_amdgcn_update_dpp(0, before[i], w64::kDppWaveRor1, 0xf, 0xf, true);
            if (lane == 0) before[i] = 0;
            if (NW > 1)
#pragma unroll
                for (int w = 0; w < NW - 1; ++w) before[i] = max(before[i], w < wv ? carry[w][i] : 0);
        }
        // how far x and y can lie from e when e is inside the reversed piece: y = u + 1 while the edges 1 .. u have
        // b < cur, x = N - u - 2 while the last u + 1 have; the maxima grow with u, so counting is enough
        int l_most = 0, r_most = 0;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int u = tid * E + k;
            if (u < N) {
                const int br = max(v[0][k], before[0]), bl = max(v[2][k], before[2]);
                b_right[u] = br;
                rn[u + 1] = turned_t[k];
                if (u == N - 1) rn[0] = turned_t[k];
                f_right[u] = max(v[1][k], before[1]);
                b_left[u + 1] = bl;
                f_left[u + 1] = max(v[3][k], before[3]);
            }
            r_most += __popcll(__ballot(u < N && max(v[0][k], before[0]) < cur));
            l_most += __popcll(__ballot(u < N && max(v[2][k], before[2]) < cur));
        }
        if (NW > 1) {
            if (lane == 0) {
                reach[parity][wv][0] = l_most;
                reach[parity][wv][1] = r_most;
            }
        }
        group_sync<NW>();
        if (NW > 1) {
            l_most = r_most = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                l_most += reach[parity][w][0];
                r_most += reach[parity][w][1];
            }
            parity ^= 1;
        }
        // x = N - 1 leaves nothing between x and e
        l_most = b0 < cur ? __builtin_amdgcn_readfirstlane(min(l_most + 1, N - 3)) : 0;
        r_most = b0 < cur ? __builtin_amdgcn_readfirstlane(min(r_most, N - 3)) : 0;
        int hi = cur, lo = kNone;
        // the move that exchanges the edges x and y and reverses x+1 .. y-1
        auto move_id = [&](int x, int y) {
            const int px = edge(x), py = edge(y), a = min(px, py), d = max(px, py);
            const int o = a ? (px > py) : (px < py);
            return (a ? a * N + d - 1 : d * N + N - 1) * 2 + o;
        };
        auto take = [&](int value, int id) {
            const bool better = value < hi || (value == hi && value < cur && id < lo);
            hi = better ? value : hi;
            lo = better ? id : lo;
        };
        // ---- e removed: x = e (the piece runs from e + 1 to y - 1), or y = e (from x + 1 to e - 1)
        {
            // lanes that are out read one common entry: no branch, so the loads of all steps overlap
            const int t_before = rn[0], t_at = rn[1];
            int inner[2][E], hop[2][E][2];
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const int u = 2 + tid + THREADS * k;
                const bool in = u <= N - 2;
                const int uu = in ? u : 2;
                const int tn = rn[uu + 1], tp = rn[uu];
                inner[0][k] = in ? max(b_right[uu - 1], f_left[N - 1 - uu]) : cur;
                inner[1][k] = in ? max(b_left[N - 1 - uu], f_right[uu - 1]) : cur;
                const bool o1 = inner[0][k] < cur, o2 = inner[1][k] < cur;
                hop[0][k][0] = C(o1 ? tp : 0, o1 ? t_before : 0);
                hop[0][k][1] = C(o1 ? tn : 0, o1 ? t_at : 0);
                hop[1][k][0] = C(o2 ? t_before : 0, o2 ? tp : 0);
                hop[1][k][1] = C(o2 ? t_at : 0, o2 ? tn : 0);
            }
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const int u = 2 + tid + THREADS * k;
                take(max(inner[0][k], max(hop[0][k][0], hop[0][k][1])), move_id(0, min(u, N - 2)));
                take(max(inner[1][k], max(hop[1][k][0], hop[1][k][1])), move_id(min(u, N - 2), 0));
            }
        }
        if (with_flip && tid == 0) take(max(b0, b_right[N - 1]), (N + N - 1) * 2);
        // ---- e inside the piece: x = N - l, y = r, 1 <= l <= l_most, 1 <= r <= r_most.  The kept hops r+1 .. N-l-1 are cut
        // at edge z = N - l_most - 1; when every r is at most z (all sweeps but the first few, where hardly an edge has
        // b >= V) their maximum is that of two prefix maxima, and the pairs are scored in any order.
        if (l_most >= 1 && r_most >= 1) {
            // the wave's best so far is every lane's limit: most pairs tie with it and lose by their id, before any load
            GroupMin<NW>::in_wave(hi, lo);
            const int z = N - l_most - 1;
            {
                int g[2][E], in_front[2];
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const int i = tid * E + k, down = z - i, up = z + 1 + i;
                    g[0][k] = down >= 1 ? f[edge(down)] : 0;
                    g[1][k] = up < N ? f[edge(up)] : 0;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
#pragma unroll
                    for (int k = 1; k < E; ++k) g[j][k] = max(g[j][k], g[j][k - 1]);
                    in_front[j] = wave_prefix_max(g[j][E - 1]);
                }
                if (NW > 1) {
                    if (lane == 63) {
                        carry[wv][0] = in_front[0];
                        carry[wv][1] = in_front[1];
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    in_front[j] = __builtin_amdgcn_update_dpp(0, in_front[j], w64::kDppWaveRor1, 0xf, 0xf, true);
                    if (lane == 0) in_front[j] = 0;
                    if (NW > 1)
#pragma unroll
                        for (int w = 0; w < NW - 1; ++w) in_front[j] = max(in_front[j], w < wv ? carry[w][j] : 0);
                }
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    // kept hops z-i .. z belong to r = z-i-1, kept hops z+1 .. z+1+i to l = N-z-2-i
                    const int i = tid * E + k, r1 = z - i - 1, l1 = l_most - 1 - i;
                    if (r1 >= 1 && r1 <= r_most) right[r1] = max(max(g[0][k], in_front[0]), max(b0, b_right[r1 - 1]));
                    if (l1 >= 1) left[l1] = max(max(g[1][k], in_front[1]), b_left[l1 - 1]);
                    // nothing kept on that side of the cut
                    const int rz = z + i, lz = l_most + i;
                    if (rz <= r_most) right[rz] = max(b0, b_right[rz - 1]);
                    if (i == 0) left[lz] = b_left[lz - 1];
                }
                group_sync<NW>();
            }
            if (r_most <= z) {
                // lanes over r, as many rows of l at a time as fit
                int row_bits = 0;
                while ((1 << row_bits) < min(r_most, THREADS)) ++row_bits;
                const int rows = THREADS >> row_bits;
                for (int r0 = (tid & ((1 << row_bits) - 1)) + 1; r0 <= r_most; r0 += THREADS) {
                    const int tn = rn[r0 + 1], tp = rn[r0], fixed = right[r0];
                    for (int l0 = 1 + (tid >> row_bits); l0 <= l_most; l0 += kAhead * rows) {
                        const int limit = hi;
                        int inner[kAhead], id[kAhead], h1[kAhead], h2[kAhead];
#pragma unroll
                        for (int k = 0; k < kAhead; ++k) {
                            const int l = min(l0 + k * rows, l_most);
                            inner[k] = max(fixed, left[l]);
                            id[k] = move_id(N - l, r0);
                            const bool open = inner[k] - (id[k] < lo ? 1 : 0) < limit && inner[k] < cur && l + r0 <= N - 2;
                            if (!open) inner[k] = cur;
                            const int sp = rn[N - l], sn = rn[N - l + 1];
                            h1[k] = C(open ? tp : 0, open ? sp : 0);
                            h2[k] = C(open ? tn : 0, open ? sn : 0);
                        }
#pragma unroll
                        for (int k = 0; k < kAhead; ++k)
                            take(max(inner[k], max(h1[k], h2[k])), id[k]);
                    }
                }
            } else {
                // some r beyond the cut: l from l_most inwards, the kept hops gain one edge per step
                for (int r0 = tid + 1; r0 <= r_most; r0 += THREADS) {
                    const int tn = rn[r0 + 1], tp = rn[r0];
                    int range = right[r0];
                    for (int l0 = l_most; l0 >= 1; l0 -= kAhead) {
                        const int limit = hi;
                        int inner[kAhead], id[kAhead], h1[kAhead], h2[kAhead];
#pragma unroll
                        for (int k = 0; k < kAhead; ++k) {
                            const int l = max(l0 - k, 1);
                            if (l < l_most && l + r0 <= N - 2) range = max(range, f[edge(N - l - 1)]);
                            inner[k] = max(range, b_left[l - 1]);
                            id[k] = move_id(N - l, r0);
                            const bool open = inner[k] - (id[k] < lo ? 1 : 0) < limit && inner[k] < cur && l + r0 <= N - 2;
                            if (!open) inner[k] = cur;
                            const int sp = rn[N - l], sn = rn[N - l + 1];
                            h1[k] = C(open ? tp : 0, open ? sp : 0);
                            h2[k] = C(open ? tn : 0, open ? sn : 0);
                        }
#pragma unroll
                        for (int k = 0; k < kAhead; ++k)
                            take(max(inner[k], max(h1[k], h2[k])), id[k]);
                    }
                }
            }
        }
        group_min(hi, lo, wv, lane);
        if (hi >= cur) break;
        // ---- apply: new[p] = old[src(p)]; the hops go with the edges, turned round where the walk is
        const int o = lo & 1, mi = (lo >> 1) / N, mj = (lo >> 1) - mi * N;
        auto src = [&](int p) {
            const int p0 = o ? (p ? N - p : 0) : p;
            return p0 >= mi && p0 <= mj ? mi + mj - p0 : p0;
        };
        int nt[E], nf[E], nb[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = tid + THREADS * k;
            nt[k] = nf[k] = nb[k] = 0;
            if (p < N) {
                const int s0 = src(p), s1 = src(p ? p - 1 : N - 1);
                const bool same = s0 == (s1 + 1 == N ? 0 : s1 + 1), turned = s1 == (s0 + 1 == N ? 0 : s0 + 1);
                nt[k] = t[s0];
                if (same || turned) {
                    const int q = same ? s0 : s1;
                    const int fq = f[q], bq = b[q];
                    nf[k] = same ? fq : bq;
                    nb[k] = same ? bq : fq;
                } else {
                    const int tp = t[s1];
                    nf[k] = C(nt[k], tp);
                    nb[k] = C(tp, nt[k]);
                }
            }
        }
        group_sync<NW>();
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int p = tid + THREADS * k;
            if (p < N) {
                t[p] = nt[k];
                f[p] = nf[k];
                b[p] = nb[k];
            }
        }
        ++applied;
    }
    for (int p = tid; p < N; p += THREADS) tours[r * N + p] = t[p];
    if (tid == 0) {
        costs[r] = (int64_t)cur;
        moves[r] = applied;
    }
}

template <int THREADS, int E>
hipError_t launch(const int32_t* c, int N, bool directed, int restarts, bool with_flip, int32_t* tours, int64_t* costs,
                  int32_t* moves, hipStream_t s) {
    if (directed)
        hipLaunchKernelGGL((twoopt_max_directed_pruned_kernel<THREADS, E>), dim3(restarts), dim3(THREADS), 0, s, c, N,
                           with_flip ? 1 : 0, tours, costs, moves);
    else
        hipLaunchKernelGGL((twoopt_max_pruned_kernel<THREADS, E>), dim3(restarts), dim3(THREADS), 0, s, c, N, tours, costs,
                           moves);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_2opt_max_pruned(const int32_t* c, int N, bool directed, int restarts, bool with_flip, int32_t* tours,
                                  int64_t* costs, int32_t* moves, hipStream_t s) {
    // Wider workgroups shorten a sweep's phases until their barriers cost more, and take room from other restarts.  The directed
    // searches of the head of this file: N = 100, 1000 restarts 205 us with 128 threads, 261 with 64, 221 with 256; N = 256, 1024
    // restarts 551 us with 256, 684 with 128, 823 with 512; N = 300, 256 restarts 604 us with 512, 735 with 256, 839 with 1024, 1000 restarts
    // 961 / 800 / 2163; N = 512, 256 restarts 872 / 1156 / 1147; N = 1024, 32 restarts 2027 / 2992 / 2064.  Undirected: N = 100, 1000
    // restarts 120 us with 64, 155 with 256; N = 256, 256 restarts 139 us with 256, 150 with 128, 1000 restarts 173 / 190; N = 512, 256
    // restarts 236 us with 512, 226 with 256; N = 1024, 256 restarts 314 / 330.
    const bool few = restarts <= 512;
    if (N <= 64) return launch<64, 1>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
    if (N <= 128) {
        if (directed) return launch<128, 1>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
        return launch<64, 2>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
    }
    if (N <= 256) {
        if (directed || restarts <= 1024) return launch<256, 1>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
        return launch<128, 2>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
    }
    if (N <= 512) {
        if (directed && few) return launch<512, 1>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
        return launch<256, 2>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
    }
    if (few) return launch<512, 2>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
    return launch<256, 4>(c, N, directed, restarts, with_flip, tours, costs, moves, s);
}

}  // namespace cc
