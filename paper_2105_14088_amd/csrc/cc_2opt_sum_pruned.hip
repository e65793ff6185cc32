// Ring-sum 2-opt for 65 <= N <= 1024 and any entries: only the moves that can be the best one are scored.  Move set,
// value and tie-break rules as stated in cc.h; symmetric matrix, read through its upper triangle.
//
// Exchanging the ring edges a and b (edge p joins ranks p-1 and p) changes the cost by
//     delta = [c(t[a-1], t[b-1]) - (f[a] + f[b]) / 2] + [c(t[a], t[b]) - (f[a] + f[b]) / 2],
// one bracket per new edge.  If some move of the sweep is known to change the cost by D, the best move has a bracket of at
// most D / 2, and then its new edge (x, y) has c(x, y) <= max(f_x, f_y) + D / 2, f_x and f_y the removed edges at x and
// y.  So for every node x only the partners y up to that cost are looked at, from a list of the node's partners in rising
// order of cost, each by its bracket first (three words in LDS) and with the second new edge's entry only if the bracket
// passes.  D comes from the candidates that were good in the sweep before: most of them still stand, so D is the best
// move's value or close to it.  On hierarchies of hosts and racks a sweep looks at about 6 N partners (N = 1000; 4 N at
// N = 256) where the exhaustive sweep has N (N-3) / 2 moves.  Equal values are looked at too (<=, not <), so the winner
// (value, lowest id) is the exhaustive sweep's.
//
// Lists: the partners of a node in buckets of cost (16, 8 or 4 per octave, as the spread of the row asks: the top bits of
// 2 cost + 1 as a float), with the number of partners up to each bucket: how far a threshold reaches is one look-up, and
// order inside a bucket does not matter.  A list holds the nearest M partners; a node whose threshold reaches further,
// or whose candidates exceed the room for them, is scanned against every node instead.
//   * N <= 256: lists in LDS, made by the workgroup itself; up to 256 (N <= 192: mostly 512) restarts one workgroup of a
//     wavefront per 64 nodes each, beyond that up to 16 restarts of one wavefront each around one copy of the lists.
//   * N > 256: one workgroup per restart, a wavefront per 64 nodes, lists in the workspace (M = (N - 128) / 2), made by a
//     kernel of their own.
// The candidates of 64 nodes are laid out end to end (prefix sum of their counts) and taken 64 at a time, up to four
// times 64 with their look-ups in flight together; those whose bracket passes are collected in LDS and scored 64 at a
// time.
//
// What bounds it: instruction issue, about 60 instructions per 64 candidates and 180 per 64 scored ones, and with 16
// wavefronts per restart the barriers (N = 1000: 17000 clocks a sweep, 6000 of them brackets, 4000 waiting for the
// slowest wavefront).  Costs of few values or from 0 on take no longer than others (see cc_pruned.h and where D is known).  Measured against the exhaustive kernels: N = 1000, 128 restarts 494 -> 11 ms; N = 583, 47 restarts
// 112 -> 4.6 ms; N = 345, 2140 restarts 239 -> 7.5 ms; N = 1024, 256 restarts 57.9 -> 12 ms (a kernel that streamed the
// matrix through LDS row by row, gone since); N = 512, 768 restarts 19.2 -> 6.1 ms; N = 240, 1024 restarts 7.1 -> 3.4 ms;
// N = 256, 4096 restarts 7.8 -> 5.2 ms.
#include <type_traits>

#include "cc_device.h"
#include "cc_internal.h"
#include "cc_pruned.h"

namespace cc {
using namespace ccd;

namespace {

using namespace pruned;

// LDS of one restart (WAVES wavefronts): per node {hop into it << 10 | its rank, hop out of it}, the nodes of the ranks
// -1 .. N, and per wave the laid out candidates' owners and the candidates whose bracket passed.
__host__ __device__ constexpr size_t order_bytes(int N) { return ((size_t)N * 8 + (size_t)(N + 2) * 2 + 15) & ~(size_t)15; }

// One descent.  A node's scale (of its buckets) is scale0 (one node per lane) or scales[node].  Wave `wv` of the restart
// owns the nodes 64 * (wv * K + k) + lane.
template <int WAVES, int K, int ROOM, typename COUNT, class MAT>
__device__ __forceinline__ void descend(const MAT mat, int N, const uint32_t* __restrict__ lists, int M,
                                        const COUNT* __restrict__ counts, int scale0, const uint16_t* scales, unsigned char* order_mem,
                                        unsigned char* wave_mem, unsigned long long (*red)[WAVES], int wv, int lane,
                                        int32_t* __restrict__ tour, int64_t* __restrict__ cost_out,
                                        int32_t* __restrict__ moves_out) {
    constexpr int THREADS = 64 * WAVES;
    uint2* info = (uint2*)order_mem;                           // [N] by node
    uint16_t* t = (uint16_t*)(info + N) + 1;                   // t[-1] = t[N-1], t[N] = t[0]
    uint16_t* owner = (uint16_t*)wave_mem;                     // [ROOM] stamp << 6 | lane
    // [kPassed] x | place << 10 | sides << 21; place: in the list of x, or M + y for a node scanned against every node
    uint32_t* passed = (uint32_t*)(wave_mem + ROOM * 2);
    const int tid = wv * 64 + lane;
    auto sync = [] { if (WAVES > 1) __syncthreads(); else __builtin_amdgcn_wave_barrier(); };
    auto hop_in = [](uint2 w) { return (int)(w.x >> 10); };
    auto hop_out = [](uint2 w) { return (int)w.y; };
    auto rank_of = [](uint2 w) { return (int)(w.x & 1023u); };

    // ---- order, hops, ranks
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
    uint2 own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int p = min(tid + THREADS * k, N - 1);
        own[k].x = ((unsigned)mat(t0[k], t[p - 1]) << 10) | (unsigned)p;
        own[k].y = (unsigned)mat(t0[k], t[p + 1]);
        if (tid + THREADS * k < N) {
            info[t0[k]] = own[k];
            sum += hop_in(own[k]);
        }
    }
    sync();
    // An order that is no permutation (a data error) is left as it is: the node-wise hops below would not describe it.
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

    // the candidate a lane remembers from an earlier sweep; at first the nearest partner of its first node
    int rx = min(64 * wv * K + lane, N - 1), ry = (int)(lists[(size_t)rx * M] & 1023u);
    int r_value = 0;                                           // what it was worth
    unsigned stamp = 0;
    while (search) {
        int hi = 0, lo = -1;                                   // best move so far; none: 0 and an id nothing undercuts
        int sweep_best = kNone;                                // this lane's own best of the sweep, for rx and ry
        // edges a and b exchanged
        auto take = [&](int delta, int a, int b) {
            a = a >= N ? a - N : a;
            b = b >= N ? b - N : b;
            const int p = min(a, b), q = max(a, b);
            const int id = p ? p * N + q - 1 : q * N + N - 1;
            const bool better = delta < hi || (delta == hi && id < lo);
            hi = better ? delta : hi;
            lo = better ? id : lo;
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
        // ---- D from the remembered candidates, on both sides (a reversal turns one into the other)
        {
            const bool worth = r_value <= 0;
            const uint2 ix = info[rx], iy = info[ry];
            const int p = rank_of(ix), q = rank_of(iy), d = p < q ? q - p : p - q;
            const int cxy = mat(worth ? rx : 1, worth ? ry : 0);
            const int cp = mat(worth ? t[p + 1] : 1, worth ? t[q + 1] : 0), cm = mat(worth ? t[p - 1] : 1, worth ? t[q - 1] : 0);
            if (worth && d >= 2 && d <= N - 2) {
                const int behind = cxy + cp - hop_out(ix) - hop_out(iy), before = cxy + cm - hop_in(ix) - hop_in(iy);
                take(behind, p + 1, q + 1);
                take(before, p, q);
                sweep_best = min(behind, before);
            }
            r_value = sweep_best;
        }
        group_min();
        // only a move that lowers the cost is wanted: its value is -1 or less
        const int D = min(hi, -1);
        // A move of value D has one bracket below D / 2, or two of D / 2.  In the second case both new edges cost
        // (f_x + f_y + D) / 2: within less than half of D of the longer removed edge, or, where the two are equal, within
        // exactly half of D of both.  The move then counts only with an id below lo, its lower edge e has e N <= lo, and the
        // node at rank e finds the pair; all other nodes look for less than half of D.  (Two zones of equal costs: all moves
        // of a sweep were scored, N = 512, 768 restarts 34 ms, now 1.9.)
        int n_passed = 0;
        // scores the n passed candidates from `from` on; a lane's candidate may stand on both sides
        auto score = [&](int from, int n) {
            const bool live = lane < n;
            const uint32_t w = passed[from + (live ? lane : 0)];
            const int x = (int)(w & 1023u), place = (int)((w >> 10) & 2047u), sides = (int)(w >> 21);
            const bool listed = place < M;
            const uint32_t e = lists[(size_t)x * M + (listed ? place : 0)];
            const int y = listed ? (int)(e & 1023u) : place - M;
            int cost = (int)(e >> 10);
            if (__ballot(!listed)) cost = listed ? cost : mat(x, y);
            const uint2 ix = info[x], iy = info[y];
            const int p = rank_of(ix), q = rank_of(iy), d = p < q ? q - p : p - q;
            const bool fits = live && d >= 2 && d <= N - 2;
            auto side = [&](bool out) {
                const int a = out ? p + 1 : p, b = out ? q + 1 : q;
                const int delta = cost + mat(t[out ? p + 1 : p - 1], t[out ? q + 1 : q - 1]) -
                                  (out ? hop_out(ix) + hop_out(iy) : hop_in(ix) + hop_in(iy));
                if (fits) {
                    take(delta, a, b);
                    if (delta < sweep_best) {
                        sweep_best = delta;
                        r_value = delta;
                        rx = x;
                        ry = y;
                    }
                }
            };
            side(sides & 1);
            if (__ballot(live && sides == 3)) side(sides != 3);        // the other side of those; of the others, any
        };
        // side bits: 1 the edges behind x and y, 2 those before
        auto pass = [&](int sides, int x, int place) {
            const unsigned long long mask = __ballot(sides != 0);
            if (sides) passed[n_passed + lanes_below(mask)] = (unsigned)x | ((unsigned)place << 10) | ((unsigned)sides << 21);
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
        // the node with the longer removed edge looks at the pair
        auto sides_of = [&](uint2 ix, uint2 iy, int twice) {
            const int ox = hop_out(ix), oy = hop_out(iy), nx = hop_in(ix), ny = hop_in(iy);
            return (ox >= oy && twice - oy <= ox + D ? 1 : 0) | (nx >= ny && twice - ny <= nx + D ? 2 : 0);
        };
#pragma unroll 1
        for (int k = 0; k < K; ++k) {
            // ---- how far the thresholds of 64 nodes reach; their candidates end to end
            const int x_first = 64 * (wv * K + k), x = x_first + lane;
            const uint2 ix = info[min(x, N - 1)];
            const bool equals = (unsigned)(rank_of(ix) * N) <= (unsigned)lo;      // lo is -1 where no move is known
            const int reach = max(hop_in(ix), hop_out(ix)) + ((equals ? D : D - 1) >> 1);
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
                uint2 jx[U], jy[U];
                uint32_t e[U];
#pragma unroll
                for (int u = 0; u < U; ++u) src[u] = owner[i0 + 64 * u + lane];
                // marks of earlier layouts are smaller than this one's, and the first of the 64 is always marked
#pragma unroll
                for (int u = 0; u < U; ++u) src[u] = wave_prefix_max(src[u]) & 63u;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    from[u] = __builtin_amdgcn_ds_bpermute((int)(src[u] << 2), start);
                    jx[u] = info[min(x_first + (int)src[u], N - 1)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + 64 * u + lane;
                    e[u] = lists[(size_t)((x_first + (int)src[u]) * M + i - from[u]) * (i < total ? 1 : 0)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) jy[u] = info[e[u] & 1023u];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + 64 * u + lane;
                    const int sides = sides_of(jx[u], jy[u], 2 * (int)(e[u] >> 10));
                    pass(i < total ? sides : 0, x_first + (int)src[u], i - from[u]);
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
                const uint2 jx = info[nx];
                for (int y0 = 0; y0 < N; y0 += 256) {
                    int cost[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) cost[u] = mat(nx, min(y0 + 64 * u + lane, N - 1));
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int y = y0 + 64 * u + lane;
                        pass(y < N ? sides_of(jx, info[min(y, N - 1)], 2 * cost[u]) : 0, nx, M + y);
                    }
                    flush();
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (n_passed) score(0, n_passed);
        group_min();
        if (hi >= 0) break;
        // ---- reverse ranks mi .. mj: the nodes inside swap the hops in and out, two hops are new
        const int mi = lo / N, mj = lo - mi * N;
        const int n_before = t[mi - 1], n_first = t[mi], n_last = t[mj], n_after = t[mj + 1];
        const int h_first = mat(n_before, n_last), h_after = mat(n_first, n_after);
        int node[K];
        uint2 w[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int p = tid + THREADS * k;
            node[k] = t[p >= mi && p <= mj ? mi + mj - p : min(p, N - 1)];
            w[k] = info[node[k]];
        }
        sync();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int p = tid + THREADS * k;
            if (p >= mi && p <= mj) {
                const int in = p == mi ? h_first : hop_out(w[k]), out = p == mj ? h_after : hop_in(w[k]);
                t[p] = (uint16_t)node[k];
                if (p == N - 1) t[-1] = (uint16_t)node[k];
                info[node[k]] = make_uint2(((unsigned)in << 10) | (unsigned)p, (unsigned)out);
            } else if (p < N) {
                if (node[k] == n_before) w[k].y = (unsigned)h_first;
                if (node[k] == n_after) w[k].x = ((unsigned)h_after << 10) | (unsigned)p;
                if (node[k] == n_before || node[k] == n_after) info[node[k]] = w[k];
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

// N <= 64 K: a workgroup holds the lists in LDS (and the matrix as 16-bit entries when lds_matrix is set and its entries
// allow) for `waves` restarts of one wavefront each, or (WAVES > 1) for one restart of WAVES wavefronts.
template <int K, int WAVES>
__global__ __launch_bounds__(1024) void twoopt_sum_pruned_kernel(const int32_t* __restrict__ c, int N, int M, int lds_matrix,
                                                                 int waves, int restarts, int32_t* __restrict__ tours,
                                                                 int64_t* __restrict__ costs,
                                                                 int32_t* __restrict__ moves,
                                                                 const int32_t* __restrict__ skip_if_small) {
    // when the exhaustive 16-bit kernel is launched beside this one, the matrix maximum decides which of them runs
    if (skip_if_small && skip_if_small[0] < (1 << 16)) return;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int largest[16];
    __shared__ unsigned long long red[2][WAVES];
    uint32_t* lists = (uint32_t*)smem;                         // [N][M]
    unsigned char* counts = smem + (size_t)N * M * 4;          // [N][kBuckets]
    uint16_t* scales = (uint16_t*)(counts + (size_t)N * kBuckets);     // [N]
    uint16_t* m16 = scales + N;                                 // [N][N]
    unsigned char* rest = smem + shared_bytes(N, M, lds_matrix);
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    {
        // the lists are made by all wavefronts of the workgroup, those without a restart included; the histograms
        // lie where the restarts' state comes later
        int* hist = (int*)rest + kBuckets * wv;
        int high = 0;
        for (int x = wv; x < N; x += nw) {
            int row_max;
            const int scale = make_list<(WAVES > 1 ? WAVES : K)>(c, N, x, M, lists + (size_t)x * M, counts + (size_t)x * kBuckets,
                                                             hist, lane, row_max, [&](int y, int cost) {
                                                                 if (lds_matrix) m16[x * N + y] = (uint16_t)cost;
                                                             });
            if (lane == 0) scales[x] = (uint16_t)scale;
            high = max(high, row_max);
        }
        if (lane == 0) largest[wv] = high;
    }
    __syncthreads();
    if (wv >= waves) return;                                   // barriers below wait for the remaining wavefronts only
    int high = 0;
    for (int w = 0; w < nw; ++w) high = max(high, largest[w]);
    const bool in_lds = lds_matrix && __builtin_amdgcn_readfirstlane(high) < (1 << 16);
    const int64_t r = WAVES > 1 ? blockIdx.x : (int64_t)blockIdx.x * waves + wv;
    if (r >= restarts) return;
    const int mine = WAVES > 1 ? 0 : wv, part = WAVES > 1 ? wv : 0;
    unsigned char* order_mem = rest + (size_t)mine * (order_bytes(N) + wave_bytes(kRoom));
    unsigned char* wave_mem = order_mem + order_bytes(N) + (size_t)part * wave_bytes(kRoom);
    const int scale0 = (int)scales[min(64 * part + lane, N - 1)];
    if (in_lds)
        descend<WAVES, K, kRoom>(LdsMatrix{m16, N}, N, lists, M, counts, scale0, scales, order_mem, wave_mem, red, part, lane,
                          tours + r * N, costs + r, moves + r);
    else
        descend<WAVES, K, kRoom>(CallersMatrix{c, N}, N, lists, M, counts, scale0, scales, order_mem, wave_mem, red, part, lane,
                          tours + r * N, costs + r, moves + r);
}

// N > 256.  Workspace, 2 N^2 bytes: lists [N][M] of 4 bytes, counts [N][kBuckets] of 2 bytes.
constexpr int group_list(int N) { return (N - kBuckets) / 2; }

// The lists of all nodes, one workgroup of four wavefronts per four nodes.
__global__ __launch_bounds__(256) void partner_lists_kernel(const int32_t* __restrict__ c, int N, int M,
                                                            uint32_t* __restrict__ lists, uint16_t* __restrict__ counts) {
    __shared__ int hist[4][kBuckets];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, x = blockIdx.x * 4 + wv;
    if (x >= N) return;
    uint16_t* mine = counts + (size_t)x * kBuckets;
    int high;
    const int scale = N <= 512 ? make_list<8>(c, N, x, M, lists + (size_t)x * M, mine, hist[wv], lane, high, [](int, int) {})
                           : make_list<16>(c, N, x, M, lists + (size_t)x * M, mine, hist[wv], lane, high, [](int, int) {});
    if (lane == 63) mine[kBuckets - 1] = (uint16_t)scale;      // the last bucket's count is N - 1: the scale has its place
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void twoopt_sum_pruned_group_kernel(const int32_t* __restrict__ c, int N, int M,
                                                                             const uint32_t* __restrict__ lists,
                                                                             const uint16_t* __restrict__ counts,
                                                                             int32_t* __restrict__ tours,
                                                                             int64_t* __restrict__ costs,
                                                                             int32_t* __restrict__ moves) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ unsigned long long red[2][WAVES];
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    const int scale = (int)counts[(size_t)min(64 * wv + lane, N - 1) * kBuckets + kBuckets - 1];
    descend<WAVES, 1, kGroupRoom>(CallersMatrix{c, N}, N, lists, M, counts, scale, nullptr, smem,
                                  smem + order_bytes(N) + wv * wave_bytes(kGroupRoom), red, wv, lane, tours + r * N, costs + r,
                                  moves + r);
}

template <int K, int WAVES>
hipError_t launch_lds(const int32_t* c, int N, const LdsPlan& plan, int restarts, int32_t* tours, int64_t* costs,
                      int32_t* moves, const int32_t* skip_if_small, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute((const void*)twoopt_sum_pruned_kernel<K, WAVES>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan.bytes);
    if (e != hipSuccess) return e;
    const int grid = WAVES > 1 ? restarts : (restarts + plan.waves - 1) / plan.waves;
    hipLaunchKernelGGL((twoopt_sum_pruned_kernel<K, WAVES>), dim3(grid), dim3(64 * (plan.waves > 8 ? plan.waves : 8)), plan.bytes,
                       s, c, N, plan.M, plan.lds_matrix, plan.waves, restarts, tours, costs, moves, skip_if_small);
    return hipGetLastError();
}

template <int K>
hipError_t launch_waves(const int32_t* c, int N, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        const int32_t* skip_if_small, hipStream_t s) {
    const LdsPlan plan = lds_plan(N, K, restarts, order_bytes(N));
    return plan.together ? launch_lds<1, K>(c, N, plan, restarts, tours, costs, moves, skip_if_small, s)
                         : launch_lds<K, 1>(c, N, plan, restarts, tours, costs, moves, skip_if_small, s);
}

template <int WAVES>
hipError_t launch_group(const int32_t* c, int N, void* room, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        hipStream_t s) {
    int M;
    const uint32_t* lists;
    const uint16_t* counts;
    hipError_t e = launch_partner_lists(c, N, room, M, lists, counts, s);
    if (e != hipSuccess) return e;
    const size_t lds = order_bytes(N) + WAVES * wave_bytes(kGroupRoom);
    e = hipFuncSetAttribute((const void*)twoopt_sum_pruned_group_kernel<WAVES>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((twoopt_sum_pruned_group_kernel<WAVES>), dim3(restarts), dim3(64 * WAVES), lds, s, c, N, M, lists,
                       counts, tours, costs, moves);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_partner_lists(const int32_t* c, int N, void* room, int& M, const uint32_t*& lists, const uint16_t*& counts,
                                hipStream_t s) {
    M = group_list(N);
    lists = (const uint32_t*)room;
    counts = (const uint16_t*)(lists + (size_t)N * M);
    hipLaunchKernelGGL(partner_lists_kernel, dim3((N + 3) / 4), dim3(256), 0, s, c, N, M, (uint32_t*)lists, (uint16_t*)counts);
    return hipGetLastError();
}

hipError_t launch_2opt_sum_pruned(const int32_t* c, int N, void* room, int restarts, int32_t* tours, int64_t* costs,
                                  int32_t* moves, const int32_t* skip_if_small, hipStream_t s) {
    if (N <= 128) return launch_waves<2>(c, N, restarts, tours, costs, moves, skip_if_small, s);
    if (N <= 192) return launch_waves<3>(c, N, restarts, tours, costs, moves, skip_if_small, s);
    if (N <= 256) return launch_waves<4>(c, N, restarts, tours, costs, moves, skip_if_small, s);
    if (N <= 320) return launch_group<5>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 384) return launch_group<6>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 448) return launch_group<7>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 512) return launch_group<8>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 640) return launch_group<10>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 768) return launch_group<12>(c, N, room, restarts, tours, costs, moves, s);
    return launch_group<16>(c, N, room, restarts, tours, costs, moves, s);
}

}  // namespace cc
