// Descent over segment insertions (Or-opt), with or without the 2-opt moves, ring sum, for any 4 <= N <= 1024 and any
// entries: only the moves that can be the best one are scored.  Move set, ids, values and tie-breaks as in cc.h
// (cc_local_search); symmetric matrix, read through its upper triangle.
//
// The scheme is that of cc_2opt_sum_pruned.hip.  Taking the segment s .. e out saves
// R = f[s] + f[e+1] - c(t[s-1], t[e+1]); putting it between the ranks g and g+1 adds two edges, each between an end of
// the segment and a node of the gap, and saves the gap's hop f[g+1]:
//     delta = [c(end, gap node) - (f[g+1] + R) / 2] + [c(other end, other gap node) - (f[g+1] + R) / 2].
// If some move changes the cost by D, the best one has a bracket of at most D / 2, so its new edge (x, y) has
// c(x, y) <= max(value of x, value of y) + D / 2, where the value of a node is the longest hop at it or the largest R of the
// five segments it ends (L = 1, 2, 3, at either end), whichever is larger.  The pairs up to that cost come from the
// partner lists, each looked at by the node with the larger value; a pair that passes with the best of its hops and
// segments is scored in all its roles: 20 insertions (either node ends the segment, five segments, the gap on either
// side of the other) and the two 2-opt moves.  D comes from the candidates remembered from earlier sweeps.
//
// What bounds it: instruction issue and look-up latency; scoring 64 pairs in all roles is about 650 instructions (4000
// clocks alone on a SIMD; 10000 while every move waited for its own look-ups), one or two of these per 64 nodes and sweep.
// Against the general kernel (cc_local.hip), 2-opt and insertion: N = 32, 1024 restarts 381 -> 174 us; N = 100, 512 restarts
// 4.9 -> 0.99 ms; N = 150, 512 restarts 13.1 -> 1.6 ms; N = 292, 228 restarts 53 -> 5.0 ms; N = 1000, 20 restarts 1371 -> 33 ms;
// against the exhaustive multi-rank kernel at N = 256, 250 restarts 9.6 -> 3.0 ms.  Matrices of few values are handed over to
// those kernels (hand_over).
#include <type_traits>

#include "cc_device.h"
#include "cc_internal.h"
#include "cc_pruned.h"

namespace cc {
using namespace ccd;

namespace {

using namespace pruned;
constexpr int kNoSegment = -(1 << 28);  // R of a segment that does not exist

// LDS of one restart: per node {hop in << 10 | rank, hop out} and {longest hop, largest R}, R of the segments of length
// 1, 2, 3 by first rank, the nodes of the ranks -1 .. N
__host__ __device__ constexpr size_t local_order_bytes(int N) {
    return ((size_t)N * 28 + (size_t)(N + 2) * 2 + 15) & ~(size_t)15;
}

template <int WAVES, int K, int ROOM, bool WITH_2OPT, typename COUNT, class MAT>
__device__ __forceinline__ void descend(const MAT mat, int N, const uint32_t* __restrict__ lists, int M,
                                        const COUNT* __restrict__ counts, int scale0, const uint16_t* scales,
                                        unsigned char* order_mem, unsigned char* wave_mem,
                                        unsigned long long (*red)[WAVES], int wv, int lane, int32_t* __restrict__ tour,
                                        int64_t* __restrict__ cost_out, int32_t* __restrict__ moves_out) {
    constexpr int THREADS = 64 * WAVES;
    uint2* info = (uint2*)order_mem;                           // [N] by node
    int2* value = (int2*)(info + N);                           // [N] by node
    int32_t* saved = (int32_t*)(value + N);                    // [3][N] R by first rank
    uint16_t* t = (uint16_t*)(saved + 3 * N) + 1;              // t[-1] = t[N-1], t[N] = t[0]
    uint16_t* owner = (uint16_t*)wave_mem;                     // [ROOM] stamp << 6 | lane
    uint32_t* passed = (uint32_t*)(wave_mem + ROOM * 2);       // [kPassed] x | place << 10 (as in the 2-opt kernel)
    const int tid = wv * 64 + lane;
    auto sync = [] { if (WAVES > 1) __syncthreads(); else __builtin_amdgcn_wave_barrier(); };
    auto hop_in = [](uint2 w) { return (int)(w.x >> 10); };
    auto hop_out = [](uint2 w) { return (int)w.y; };
    auto rank_of = [](uint2 w) { return (int)(w.x & 1023u); };
    const int longest = min(3, N - 3);                         // of the segments

    int t0[K], applied = 0, parity = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = tid + THREADS * k;
        t0[k] = p < N ? clampi(tour[p], 0, N - 1) : 0;
        if (p < N) {
            t[p] = (uint16_t)t0[k];
            if (p == N - 1) t[-1] = (uint16_t)t0[k];
            if (p == 0) t[N] = (uint16_t)t0[k];
        }
    }
    for (int i = lane; i < ROOM; i += 64) owner[i] = 0;
    sync();
    int sum = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = min(tid + THREADS * k, N - 1);
        const uint2 w = make_uint2(((unsigned)mat(t0[k], t[p - 1]) << 10) | (unsigned)p, (unsigned)mat(t0[k], t[p + 1]));
        if (tid + THREADS * k < N) {
            info[t0[k]] = w;
            sum += hop_in(w);
        }
    }
    sync();
    // An order that is no permutation (a data error) is left as it is: the node-wise hops would not describe it.
    bool good = true;
#pragma unroll
    for (int k = 0; k < K; ++k) good = good && (tid + THREADS * k >= N || rank_of(info[t0[k]]) == tid + THREADS * k);
    bool search = __ballot(!good) == 0;
    if (WAVES > 1) {
        // over the wavefronts of this restart alone: the workgroup's others have ended, which a plain barrier allows and a
        // workgroup-wide reduction of the library need not
        if (lane == 0) red[parity][wv] = search ? 1u : 0u;
        __syncthreads();
        search = __ballot(red[parity][min(lane, WAVES - 1)] == 0) == 0;
        parity ^= 1;
    }

    // the move a lane remembers: a pair and how it is used.  Use: length of the segment x ends (0: a 2-opt move) << 2 |
    // x is its last rank << 1 | y stands behind the gap (2-opt: the edges before x and y).  At first the nearest partner
    // of its first node.
    int rx = min(64 * wv * K + lane, N - 1), ry = (int)(lists[(size_t)rx * M] & 1023u);
    int r_use = WITH_2OPT ? 0 : 4, r_value = 0;
    unsigned stamp = 0;
    while (search) {
        int hi = 0, lo = -1;                                   // best move so far; none: 0 and an id nothing undercuts
        int sweep_best = kNone;
        auto take = [&](int delta, int id, int x, int y, int use) {
            const bool better = delta < hi || (delta == hi && id < lo);
            hi = better ? delta : hi;
            lo = better ? id : lo;
            if (delta < sweep_best) {
                sweep_best = r_value = delta;
                rx = x;
                ry = y;
                r_use = use;
            }
        };
        auto group_min = [&] {
            int h = wave_min(hi);
            const unsigned long long at = __ballot(hi == h);
            int l = __builtin_amdgcn_readlane(lo, (int)__builtin_ctzll(at));
            if (at & (at - 1)) l = wave_min(hi == h ? lo : kNone);
            if (WAVES > 1) {
                if (lane == 0) red[parity][wv] = ((unsigned long long)(unsigned)(h + (1 << 30)) << 32) | (unsigned)l;
                __syncthreads();
                const unsigned long long v = red[parity][min(lane, WAVES - 1)];
                const int vh = (int)(v >> 32) - (1 << 30), vl = (int)(unsigned)v;
                h = wave_min(vh);
                const unsigned long long who = __ballot(vh == h);
                l = __builtin_amdgcn_readlane(vl, (int)__builtin_ctzll(who));
                if (who & (who - 1)) l = wave_min(vh == h ? vl : kNone);
                parity ^= 1;
            }
            hi = h;
            lo = l;
        };
        // ---- what the segments that start at each rank save, and the nodes' values
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int s = tid + THREADS * k;
            if (s < N) {
                const int before = t[s - 1], f = hop_in(info[t[s]]);
#pragma unroll
                for (int L = 1; L <= 3; ++L) {
                    const bool has = s >= 1 && s + L <= N && L <= longest;
                    const int behind = t[has ? s + L : 0];
                    const int r = f + hop_in(info[behind]) - mat(before, behind);
                    saved[(L - 1) * N + s] = has ? r : kNoSegment;
                }
            }
        }
        sync();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int p = tid + THREADS * k;
            if (p < N) {
                const int x = t[p];
                const uint2 w = info[x];
                int r = max(saved[p], max(saved[N + p], saved[2 * N + p]));
                if (p >= 1) r = max(r, saved[N + p - 1]);
                if (p >= 2) r = max(r, saved[2 * N + p - 2]);
                value[x] = make_int2(max(hop_in(w), hop_out(w)), r);
            }
        }
        // ---- D from the remembered moves; a reversal turns one into its mirror image
        {
            const bool worth = r_value <= 0;
            const int x = rx, y = ry, use = r_use, L = use >> 2;
            const uint2 ix = info[x], iy = info[y];
            const int p = rank_of(ix), q = rank_of(iy), d = p < q ? q - p : p - q;
            const int cost = mat(worth ? x : 1, worth ? y : 0);
            r_value = kNone;
#pragma unroll
            for (int mirror = 0; mirror < 2; ++mirror) {
                const int last = ((use >> 1) & 1) ^ mirror, side = (use & 1) ^ mirror;
                // the segment and its gap; for a 2-opt move (L = 0) the edges before or behind x and y
                const int s0 = last ? p - L + 1 : p, e = s0 + L - 1, g = side ? (q ? q - 1 : N - 1) : q;
                const bool fits = L ? s0 >= 1 && e < N && (g < s0 - 1 || g > e) && L <= longest : d >= 2 && d <= N - 2;
                const bool open = worth && fits;
                const int w = t[open ? (L ? (last ? s0 : e) : (side ? p - 1 : p + 1)) : 1], z = t[open ? (side ? q - 1 : q + 1) : 0];
                const int fy = side ? hop_in(iy) : hop_out(iy);
                const int gain = fy + (L ? saved[open ? (L - 1) * N + s0 : 0] : side ? hop_in(ix) : hop_out(ix));
                const int delta = cost + mat(w, z) - gain;
                int a = side ? p : p + 1, b = side ? q : q + 1;
                a = a == N ? 0 : a;
                b = b == N ? 0 : b;
                const int i = min(a, b), j = max(a, b), variant = L <= 1 ? 0 : 2 * L - 3 + (last != side ? 1 : 0);
                const int id = L ? (N * (1 + variant) + s0) * N + g : i ? i * N + j - 1 : j * N + N - 1;
                if (open) take(delta, id, x, y, (L << 2) | (last << 1) | side);
            }
        }
        group_min();                                           // its barrier also covers `value`
        if (WAVES == 1) __builtin_amdgcn_wave_barrier();
        // only a move that lowers the cost is wanted: its value is -1 or less
        const int D = min(hi, -1);
        int n_passed = 0;
        // scores n passed pairs in all their roles
        auto score = [&](int from, int n) {
            const bool live = lane < n;
            const uint32_t w = passed[from + (live ? lane : 0)];
            int x = (int)(w & 1023u);
            const int place = (int)(w >> 10);
            const bool listed = place < M;
            const uint32_t e = lists[(size_t)x * M + (listed ? place : 0)];
            int y = listed ? (int)(e & 1023u) : place - M;
            int cost = (int)(e >> 10);
            if (__ballot(!listed)) cost = listed ? cost : mat(x, y);
            uint2 ix = info[x], iy = info[y];
            int p = rank_of(ix), q = rank_of(iy);
            const bool open = live && x != y;
            // the best of the pair's moves; all look-ups of a role are in flight together
            int bd = kNone, bid = kNone, bx = x, by = y, buse = 0;
            auto better = [&](bool ok, int delta, int id, int use) {
                ok = ok && (delta < bd || (delta == bd && id < bid));
                bd = ok ? delta : bd;
                bid = ok ? id : bid;
                buse = ok ? use : buse;
                return ok;
            };
            if (WITH_2OPT) {
                const int d = p < q ? q - p : p - q;
                const bool fits = open && d >= 2 && d <= N - 2;
                const int out = cost + mat(t[p + 1], t[q + 1]) - hop_out(ix) - hop_out(iy);
                const int in = cost + mat(t[p - 1], t[q - 1]) - hop_in(ix) - hop_in(iy);
                const int lo_r = min(p, q), hi_r = max(p, q);              // lo_r + 1 < hi_r when it fits
                better(fits, in, lo_r ? lo_r * N + hi_r - 1 : hi_r * N + N - 1, 1);
                better(fits, out, hi_r + 1 < N ? (lo_r + 1) * N + hi_r : (lo_r + 1) * N + N - 1, 0);
            }
#pragma unroll 1
            for (int role = 0; role < 2; ++role) {
                // the five segments that x ends: first rank, what they save, the node at their other end
                const int z[2] = {t[q + 1], t[q - 1]};
                const int f[2] = {hop_out(iy), hop_in(iy)};
                int first[5], save[5], other[5];
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const int L = i == 0 ? 1 : (i + 3) >> 1, last = i == 2 || i == 4 ? 1 : 0;
                    first[i] = last ? p - L + 1 : p;
                    save[i] = saved[(L - 1) * N + max(first[i], 0)];
                    if (first[i] < 1) save[i] = kNoSegment;
                    other[i] = t[last ? max(first[i], 0) : min(p + L - 1, N - 1)];
                }
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const int L = i == 0 ? 1 : (i + 3) >> 1, last = i == 2 || i == 4 ? 1 : 0;
#pragma unroll
                    for (int side = 0; side < 2; ++side) {
                        const int g = side ? (q ? q - 1 : N - 1) : q;
                        const int delta = cost + mat(other[i], z[side]) - f[side] - save[i];
                        const int variant = L == 1 ? 0 : 2 * L - 3 + (last != side ? 1 : 0);
                        const bool ok = open && save[i] != kNoSegment && (g < first[i] - 1 || g > first[i] + L - 1);
                        if (better(ok, delta, (N * (1 + variant) + first[i]) * N + g, (L << 2) | (last << 1) | side)) {
                            bx = x;
                            by = y;
                        }
                    }
                }
                const int tx = x, tp = p;
                x = y; y = tx;
                p = q; q = tp;
                const uint2 ti = ix;
                ix = iy; iy = ti;
            }
            if (bd != kNone) take(bd, bid, bx, by, buse);
        };
        auto pass = [&](bool ok, int x, int place) {
            const unsigned long long mask = __ballot(ok);
            if (ok) passed[n_passed + lanes_below(mask)] = (unsigned)x | ((unsigned)place << 10);
            n_passed += __popcll(mask);
        };
        auto flush = [&] {
            __builtin_amdgcn_wave_barrier();
            while (n_passed >= 64) {
                n_passed -= 64;
                score(n_passed, 64);
            }
            __builtin_amdgcn_wave_barrier();
        };
        // the node with the larger value looks at the pair
        auto worth_scoring = [&](int x, int2 vx, int y, int2 vy, int twice) {
            const int mx = max(vx.x, vx.y), my = max(vy.x, vy.y);
            int most = max(vx.x + vy.y, vx.y + vy.x);
            if (WITH_2OPT) most = max(most, vx.x + vy.x);
            return (mx > my || (mx == my && x < y)) && twice - most <= D;
        };
#pragma unroll 1
        for (int k = 0; k < K; ++k) {
            // ---- how far the thresholds of 64 nodes reach; their candidates end to end
            const int x_first = 64 * (wv * K + k), x = x_first + lane;
            const int2 vx = value[min(x, N - 1)];
            const int reach = max(vx.x, vx.y) + (D >> 1);
            const int scale = K == 1 ? scale0 : (int)scales[min(x, N - 1)];
            const int bucket = bucket_of(max(reach, 0), scale);
            int count = (int)counts[(size_t)min(x, N - 1) * kBuckets + max(0, min(bucket, kBuckets - 2))];
            count = bucket >= kBuckets - 1 ? N - 1 : count;
            count = x < N && reach >= 0 && bucket >= 0 ? count : 0;
            bool all = count > M;                              // beyond the list: scanned against every node below
            count = all ? 0 : count;
            int end = wave_prefix_sum(count);
            int total = __builtin_amdgcn_readlane(end, 63);
            if (total > ROOM) {
                const bool out = end > ROOM;
                all = all || (out && count > 0);
                count = out ? 0 : count;
                total = wave_max(out ? 0 : end);
            }
            const int start = end - count;
            if (++stamp == 1024) {
                stamp = 1;
                for (int i = lane; i < ROOM; i += 64) owner[i] = 0;
                __builtin_amdgcn_wave_barrier();
            }
            if (count > 0) {
                const uint16_t mark = (uint16_t)((stamp << 6) | (unsigned)lane);
                owner[start] = mark;
                for (int i = (start | 63) + 1; i < start + count; i += 64) owner[i] = mark;     // every 64 start anew
            }
            __builtin_amdgcn_wave_barrier();
            // ---- brackets, U times 64 candidates with their LDS and list reads in flight together
            auto brackets = [&](auto u_const, int i0) {
                constexpr int U = decltype(u_const)::value;
                unsigned src[U];
                int from[U];
                int2 jx[U], jy[U];
                uint32_t e[U];
#pragma unroll
                for (int u = 0; u < U; ++u) src[u] = owner[i0 + 64 * u + lane];
#pragma unroll
                for (int u = 0; u < U; ++u) src[u] = wave_prefix_max(src[u]) & 63u;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    from[u] = __builtin_amdgcn_ds_bpermute((int)(src[u] << 2), start);
                    jx[u] = value[min(x_first + (int)src[u], N - 1)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + 64 * u + lane;
                    e[u] = lists[(size_t)((x_first + (int)src[u]) * M + i - from[u]) * (i < total ? 1 : 0)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) jy[u] = value[e[u] & 1023u];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + 64 * u + lane, nx = x_first + (int)src[u];
                    pass(i < total && worth_scoring(nx, jx[u], (int)(e[u] & 1023u), jy[u], 2 * (int)(e[u] >> 10)), nx,
                         i - from[u]);
                }
            };
            for (int i0 = 0; i0 < total; i0 += 256) {
                if (total - i0 > 128) brackets(std::integral_constant<int, 4>{}, i0);
                else if (total - i0 > 64) brackets(std::integral_constant<int, 2>{}, i0);
                else brackets(std::integral_constant<int, 1>{}, i0);
                flush();
            }
            // ---- nodes scanned against every node
            unsigned long long rest = __ballot(all);
            while (rest) {
                const int nx = x_first + (int)__builtin_ctzll(rest);
                rest &= rest - 1;
                const int2 jx = value[nx];
                for (int y0 = 0; y0 < N; y0 += 256) {
                    int cost[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) cost[u] = mat(nx, min(y0 + 64 * u + lane, N - 1));
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int y = y0 + 64 * u + lane;
                        pass(y < N && worth_scoring(nx, jx, y, value[min(y, N - 1)], 2 * cost[u]), nx, M + y);
                    }
                    flush();
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (n_passed) score(0, n_passed);
        group_min();
        if (hi >= 0) break;
        // ---- apply: new[p] = old[src(p)]; a hop between nodes that were neighbours goes with them, the new ones are
        // looked up
        int node[K];
        uint2 w[K];
        const MoveSource source(lo, N);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int p = min(tid + THREADS * k, N - 1);
            const int s0 = source(p), sb = source(p ? p - 1 : N - 1), sa = source(p + 1 == N ? 0 : p + 1);
            node[k] = t[s0];
            const uint2 old = info[node[k]];
            auto hop = [&](int other) {
                if (other == (s0 ? s0 - 1 : N - 1)) return hop_in(old);
                if (other == (s0 + 1 == N ? 0 : s0 + 1)) return hop_out(old);
                return mat(node[k], t[other]);
            };
            const int in = hop(sb), out = hop(sa);
            w[k] = make_uint2(((unsigned)in << 10) | (unsigned)p, (unsigned)out);
        }
        sync();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int p = tid + THREADS * k;
            if (p < N) {
                t[p] = (uint16_t)node[k];
                if (p == N - 1) t[-1] = (uint16_t)node[k];
                info[node[k]] = w[k];
            }
        }
        sum += tid == 0 ? hi : 0;
        ++applied;
        sync();
    }
    // ---- results
    sum = wave_sum(sum);
    if (WAVES > 1) {
        if (lane == 0) red[parity][wv] = (unsigned long long)(unsigned)sum;
        __syncthreads();
        sum = 0;
        for (int i = 0; i < WAVES; ++i) sum += (int)red[parity][i];
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tid + THREADS * k < N) tour[tid + THREADS * k] = (int)t[tid + THREADS * k];
    if (tid == 0) {
        *cost_out = (int64_t)sum;
        *moves_out = applied;
    }
}

// Whether the kernel behind this one does the work (see TieHandover).  Where many partners cost the same, most pairs pass
// their brackets in one role or another, and scoring them costs more than the exhaustive sweeps.
__device__ __forceinline__ bool hand_over(const TieHandover& ties, int tied, int highest) {
    if (!ties.flags) return false;
    const bool hand = tied > ties.most && (!ties.to_16bit || highest < (1 << 16));
    if (blockIdx.x == 0 && threadIdx.x == 0) ties.flags[0] = hand == ties.to_16bit ? 0 : 1 << 16;
    return hand;
}

// N <= 64 K, as twoopt_sum_pruned_kernel: lists (and the matrix) in LDS, for `waves` restarts of one wavefront each or
// (WAVES > 1) one restart of WAVES wavefronts.
template <int K, int WAVES, bool WITH_2OPT>
__global__ __launch_bounds__(1024) void local_pruned_kernel(const int32_t* __restrict__ c, int N, int M, int lds_matrix,
                                                            int waves, TieHandover ties, int restarts,
                                                            int32_t* __restrict__ tours, int64_t* __restrict__ costs,
                                                            int32_t* __restrict__ moves) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int largest[16], tied[16];
    __shared__ unsigned long long red[2][WAVES];
    uint32_t* lists = (uint32_t*)smem;                         // [N][M]
    unsigned char* counts = smem + (size_t)N * M * 4;          // [N][kBuckets]
    uint16_t* scales = (uint16_t*)(counts + (size_t)N * kBuckets);      // [N]
    uint16_t* m16 = scales + N;                                 // [N][N]
    unsigned char* rest = smem + shared_bytes(N, M, lds_matrix);
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    {
        int* hist = (int*)rest + kBuckets * wv;                // where the restarts' state comes later
        int high = 0, tied_here = 0;
        for (int x = wv; x < N; x += nw) {
            int row_max;
            const int scale = make_list<(WAVES > 1 ? WAVES : K)>(c, N, x, M, lists + (size_t)x * M, counts + (size_t)x * kBuckets,
                                                             hist, lane, row_max, [&](int y, int cost) {
                                                                 if (lds_matrix) m16[x * N + y] = (uint16_t)cost;
                                                             });
            if (lane == 0) scales[x] = (uint16_t)scale;
            high = max(high, row_max);
            tied_here += counts[(size_t)x * kBuckets];
        }
        if (lane == 0) {
            largest[wv] = high;
            tied[wv] = tied_here;
        }
    }
    __syncthreads();
    int high = 0, tied_in_all = 0;
    for (int w = 0; w < nw; ++w) {
        high = max(high, largest[w]);
        tied_in_all += tied[w];
    }
    high = __builtin_amdgcn_readfirstlane(high);
    if (hand_over(ties, __builtin_amdgcn_readfirstlane(tied_in_all), high)) return;
    if (wv >= waves) return;                                   // barriers below wait for the remaining wavefronts only
    const bool in_lds = lds_matrix && high < (1 << 16);
    const int64_t r = WAVES > 1 ? blockIdx.x : (int64_t)blockIdx.x * waves + wv;
    if (r >= restarts) return;
    const int mine = WAVES > 1 ? 0 : wv, part = WAVES > 1 ? wv : 0;
    unsigned char* order_mem = rest + (size_t)mine * (local_order_bytes(N) + wave_bytes(kRoom));
    unsigned char* wave_mem = order_mem + local_order_bytes(N) + (size_t)part * wave_bytes(kRoom);
    const int scale0 = (int)scales[min(64 * part + lane, N - 1)];
    if (in_lds)
        descend<WAVES, K, kRoom, WITH_2OPT>(LdsMatrix{m16, N}, N, lists, M, counts, scale0, scales, order_mem, wave_mem, red, part,
                                            lane, tours + r * N, costs + r, moves + r);
    else
        descend<WAVES, K, kRoom, WITH_2OPT>(CallersMatrix{c, N}, N, lists, M, counts, scale0, scales, order_mem, wave_mem, red,
                                            part, lane, tours + r * N, costs + r, moves + r);
}

// N > 256: lists in the workspace
template <int WAVES, bool WITH_2OPT>
__global__ __launch_bounds__(64 * WAVES) void local_pruned_group_kernel(const int32_t* __restrict__ c, int N, int M,
                                                                        const uint32_t* __restrict__ lists,
                                                                        const uint16_t* __restrict__ counts,
                                                                        TieHandover ties, int32_t* __restrict__ tours,
                                                                        int64_t* __restrict__ costs,
                                                                        int32_t* __restrict__ moves) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ unsigned long long red[2][WAVES];
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    {
        const int x = threadIdx.x;
        const int tied = wave_sum(x < N ? (int)counts[(size_t)x * kBuckets] : 0);
        if (lane == 0) red[0][wv] = (unsigned long long)tied;
        __syncthreads();
        int tied_in_all = 0;
        for (int w = 0; w < WAVES; ++w) tied_in_all += (int)red[0][w];
        if (hand_over(ties, __builtin_amdgcn_readfirstlane(tied_in_all), 0)) return;
    }
    const int scale = (int)counts[(size_t)min(64 * wv + lane, N - 1) * kBuckets + kBuckets - 1];
    descend<WAVES, 1, kGroupRoom, WITH_2OPT>(CallersMatrix{c, N}, N, lists, M, counts, scale, nullptr, smem,
                                             smem + local_order_bytes(N) + wv * wave_bytes(kGroupRoom), red, wv, lane,
                                             tours + r * N, costs + r, moves + r);
}

template <int K, int WAVES, bool WITH_2OPT>
hipError_t launch_lds(const int32_t* c, int N, const LdsPlan& plan, const TieHandover& ties, int restarts, int32_t* tours,
                      int64_t* costs, int32_t* moves, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute((const void*)local_pruned_kernel<K, WAVES, WITH_2OPT>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan.bytes);
    if (e != hipSuccess) return e;
    const int grid = WAVES > 1 ? restarts : (restarts + plan.waves - 1) / plan.waves;
    hipLaunchKernelGGL((local_pruned_kernel<K, WAVES, WITH_2OPT>), dim3(grid), dim3(64 * (plan.waves > 8 ? plan.waves : 8)),
                       plan.bytes, s, c, N, plan.M, plan.lds_matrix, plan.waves, ties, restarts, tours, costs, moves);
    return hipGetLastError();
}

template <int K, bool WITH_2OPT>
hipError_t launch_waves(const int32_t* c, int N, const TieHandover& ties, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        hipStream_t s) {
    const LdsPlan plan = lds_plan(N, K, restarts, local_order_bytes(N), K, local_order_bytes(N) + K * wave_bytes(kRoom));
    if constexpr (K > 1)
        if (plan.together) return launch_lds<1, K, WITH_2OPT>(c, N, plan, ties, restarts, tours, costs, moves, s);
    return launch_lds<K, 1, WITH_2OPT>(c, N, plan, ties, restarts, tours, costs, moves, s);
}

template <int WAVES, bool WITH_2OPT>
hipError_t launch_group(const int32_t* c, int N, void* room, const TieHandover& ties, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        hipStream_t s) {
    int M;
    const uint32_t* lists;
    const uint16_t* counts;
    hipError_t e = launch_partner_lists(c, N, room, M, lists, counts, s);
    if (e != hipSuccess) return e;
    const size_t lds = local_order_bytes(N) + WAVES * wave_bytes(kGroupRoom);
    e = hipFuncSetAttribute((const void*)local_pruned_group_kernel<WAVES, WITH_2OPT>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((local_pruned_group_kernel<WAVES, WITH_2OPT>), dim3(restarts), dim3(64 * WAVES), lds, s, c, N, M, lists,
                       counts, ties, tours, costs, moves);
    return hipGetLastError();
}

template <bool WITH_2OPT>
hipError_t launch(const int32_t* c, int N, void* room, const TieHandover& ties, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                  hipStream_t s) {
    if (N <= 64) return launch_waves<1, WITH_2OPT>(c, N, ties, restarts, tours, costs, moves, s);
    if (N <= 128) return launch_waves<2, WITH_2OPT>(c, N, ties, restarts, tours, costs, moves, s);
    if (N <= 192) return launch_waves<3, WITH_2OPT>(c, N, ties, restarts, tours, costs, moves, s);
    if (N <= 256) return launch_waves<4, WITH_2OPT>(c, N, ties, restarts, tours, costs, moves, s);
    if (N <= 320) return launch_group<5, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
    if (N <= 384) return launch_group<6, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
    if (N <= 512) return launch_group<8, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
    if (N <= 768) return launch_group<12, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
    return launch_group<16, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
}

}  // namespace

hipError_t launch_local_pruned(const int32_t* c, int N, bool with_2opt, void* room, const TieHandover& ties, int restarts,
                               int32_t* tours, int64_t* costs, int32_t* moves, hipStream_t s) {
    return with_2opt ? launch<true>(c, N, room, ties, restarts, tours, costs, moves, s)
                     : launch<false>(c, N, room, ties, restarts, tours, costs, moves, s);
}

}  // namespace cc
