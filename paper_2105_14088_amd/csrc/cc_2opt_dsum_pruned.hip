// 2-opt descent under the directed ring sum (costs differ by direction) for any N and any entries: only the moves that can be the best
// one are looked up.  Move set, ids, values and tie-breaks as in cc.h.
//
// Reversing the ranks i .. j, q = j + 1, with f the hops as walked, b the same edges the other way and P the prefix sums of b - f, changes
// the cost by
//     c(t[j], t[i-1]) + c(t[q], t[i]) - f[i] - f[q] + P[j] - P[i],                                 or, walked the other way,
//     c(t[i-1], t[j]) + c(t[i], t[q]) - b[i] - b[q] - (P[j] - P[i]) + (sum b - sum f).
// An entry is at least the smallest of its row and of its column, so either is at least U[i] + V[j] with U and V known per rank: a move is
// one addition and a comparison, and only those that can be worth the threshold T are looked up, 64 at a time through L2.  Along a good
// order f is below b, so P grows and all but short pieces, or short rests, fall out.  T is a quarter of the last move's value (the first sweep:
// any that lowers the cost) and shrinks to the best value found as a sweep goes on; when no move is worth T, T is an eighth of it, and no move
// worth -1 ends the descent.
//
// What bounds it: a sweep of N^2 / 64 additions over the workgroup's wavefronts, then look-ups, 64 in a chain of LDS, L2 and a wave
// minimum at a time.  The general kernel, which looks every move up -> this one, inverse bandwidths that are eight times as small inside a
// rack: N = 70, 300 restarts 0.77 -> 0.39 ms; N = 100, 1000 restarts 2.7 -> 1.0, 4000 restarts 7.8 -> 2.5; N = 150, 500 restarts 6.6 -> 1.4, 2000
// restarts 15.9 -> 4.0; N = 220, 500 restarts 16.0 -> 2.7; N = 300, 300 restarts 27 -> 4.2; N = 512, 100 restarts 54 -> 7.0; N = 1000, 16 restarts
// 286 -> 33; N = 256, 1000 restarts (costs beyond the exhaustive kernel's keys) 60 -> 5.4.  A zero in every row and column, where the smallest
// entries say nothing: N = 100, 1000 restarts 2.7 -> 0.95, N = 512, 100 restarts 53 -> 6.8.  Symmetric costs, where P is flat and hardly a
// move falls out by it: N = 100, 1000 restarts 3.9 -> 2.9, N = 512, 100 restarts 134 -> 64.  Two values or two zones of equal costs: 1.3 to 9 times as
// fast.  T nearer to the last value costs sweeps that find nothing: N = 220, 500 restarts with 15/16 of it 6.8 ms,
// 3/4 4.7, 1/2 4.0; two values alone are the faster for it (3.9, 3/4 3.3).  The matrix as 16-bit entries in LDS gained nothing.
#include "cc_device.h"
#include "cc_dsum_bounds.h"
#include "cc_internal.h"
#include "cc_pruned.h"

namespace cc {
using namespace ccd;

namespace {

using pruned::kCostMax;
using pruned::kNone;
using pruned::lanes_below;
using pruned::wave_prefix_sum;

constexpr int kDsumItems = 192;      // of a wave: 63, and what 64 lanes add for both directions

// A thread per rank at least, N <= 64 WAVES.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void twoopt_dsum_pruned_kernel(const int32_t* __restrict__ c, int N, int with_flip,
                                                                        int32_t* __restrict__ tours, int64_t* __restrict__ costs,
                                                                        int32_t* __restrict__ moves, const int32_t* __restrict__ skip_if_small,
                                                                        int small_limit) {
    if (skip_if_small && skip_if_small[0] < small_limit) return;
    constexpr int THREADS = 64 * WAVES;
    __shared__ int32_t t[THREADS], f[THREADS], b[THREADS], prefix[THREADS], row_min[THREADS], col_min[THREADS];
    __shared__ int2 u_of[THREADS], v_of[THREADS];               // of both directions
    __shared__ uint32_t items[WAVES][kDsumItems];               // i << 11 | j << 1 | direction
    __shared__ int sums[WAVES][2], words[WAVES], best_value[2];
    __shared__ unsigned long long key[2];
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    auto C = [&](int from, int to) { return clampi(c[__umul24((unsigned)from, (unsigned)N) + (unsigned)to], 0, kCostMax); };
    t[tid] = tid < N ? clampi(tours[r * N + tid], 0, N - 1) : 0;
    f[tid] = -1;
    row_min[tid] = col_min[tid] = kCostMax;
    if (tid < 2) {
        key[tid] = ~0ull;
        best_value[tid] = 0;
    }
    __syncthreads();
    if (tid < N) f[t[tid]] = tid;
    __syncthreads();
    // an order that is no permutation (a data error) can hold a node beside itself: entries are then at least 0
    const bool twice = __ballot(tid < N && f[t[tid]] != tid) != 0;
    if (lane == 0) words[wv] = twice ? 1 : 0;
    __syncthreads();
    bool whole = true;
    for (int w = 0; w < WAVES; ++w) whole = whole && words[w] == 0;
    if (whole) {
        int col[WAVES];
#pragma unroll
        for (int k = 0; k < WAVES; ++k) col[k] = kCostMax;
        for (int x = wv; x < N; x += WAVES) {
            int row = kCostMax;
#pragma unroll
            for (int k = 0; k < WAVES; ++k) {
                const int y = lane + 64 * k;
                const int e = y < N && y != x ? C(x, y) : kCostMax;
                col[k] = min(col[k], e);
                row = min(row, e);
            }
            row = wave_min(row);
            if (lane == 0) row_min[x] = row;
        }
#pragma unroll
        for (int k = 0; k < WAVES; ++k)
            if (lane + 64 * k < N) atomicMin(&col_min[lane + 64 * k], col[k]);
    } else {
        row_min[tid] = col_min[tid] = 0;
    }
    __syncthreads();

    const int blocks = (N + 63) >> 6, q_own = tid + 1 < N ? tid + 1 : 0;
    int applied = 0, turn = 0, cur = 0, T = -1;
    for (;;) {
        // ---- hops both ways, their prefix sums, what the bounds take from each rank
        int own_f = 0, own_b = 0;
        const int node = t[tid], node_before = t[tid ? tid - 1 : N - 1];
        if (tid < N) {
            own_f = C(node, node_before);
            own_b = C(node_before, node);
            f[tid] = own_f;
            b[tid] = own_b;
        }
        int upto = wave_prefix_sum(own_b - own_f);
        const int sum_f = wave_sum(own_f);
        if (lane == 63) {
            sums[wv][0] = upto;
            sums[wv][1] = sum_f;
        }
        __syncthreads();
        int turned = 0;                                          // sum b - sum f
        cur = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            upto += w < wv ? sums[w][0] : 0;
            turned += sums[w][0];
            cur += sums[w][1];
        }
        prefix[tid] = upto;
        if (tid < N) {
            const int qn = t[q_own], f_q = f[q_own], b_q = b[q_own];
            const dsum::Terms u = dsum::term_of_first((col_min[node_before] + col_min[node]) >> 1, (row_min[node_before] + row_min[node]) >> 1,
                                                      own_f, own_b, upto);
            const dsum::Terms v = dsum::term_of_last((row_min[node] + row_min[qn]) >> 1, (col_min[node] + col_min[qn]) >> 1, f_q, b_q, upto, turned);
            u_of[tid] = make_int2(u.kept, u.other);
            v_of[tid] = make_int2(v.kept, v.other);
        }
        __syncthreads();
        int hi, lo;
        for (;;) {
            hi = T;
            lo = kNone;
            if (with_flip && tid == 0 && turned <= T) {          // every hop the other way
                hi = turned;
                lo = (N + N - 1) * 2;
            }
            int limit = T, n_items = 0;
            // the last n of the wave's items, a move per lane
            auto score = [&](int n) {
                const uint32_t item = items[wv][n_items + min(lane, n - 1)];
                const int i = (int)(item >> 11), j = (int)(item >> 1 & 1023u), o = (int)(item & 1u), q = j + 1 < N ? j + 1 : 0;
                const int ti = t[i], tim = t[i - 1], tj = t[j], tq = t[q];
                const int x = C(o ? tim : tj, o ? tj : tim), y = C(o ? ti : tq, o ? tq : ti);
                const int inner = prefix[j] - prefix[i];
                const int delta = x + y + (o ? turned - inner - b[i] - b[q] : inner - f[i] - f[q]);
                const int id = (int)((__umul24((unsigned)i, (unsigned)N) + (unsigned)j) * 2u) + o;
                if (lane < n && (i != 1 || j != N - 1) && (delta < hi || (delta == hi && id < lo))) {
                    hi = delta;
                    lo = id;
                }
                const int h = wave_min(hi);
                if (h < limit) {
                    limit = h;
                    if (lane == 0) atomicMin(&best_value[turn & 1], h);
                }
            };
            // ---- 64 j by sixteen i at a time, dealt out to the wavefronts
            int deal = wv;
            for (int jb = 0; jb < blocks; ++jb) {
                const int j = 64 * jb + lane, last_i = min(64 * jb + 62, N - 2), chunks = (last_i + 15) >> 4;       // i = 1 .. last_i
                const unsigned long long real = __ballot(j >= 2 && j < N);
                const int2 v = v_of[min(j, N - 1)];
                int chunk = deal;
                for (; chunk < chunks; chunk += WAVES) {
                    limit = min(limit, *(volatile int*)&best_value[turn & 1]);
                    limit = __builtin_amdgcn_readfirstlane(limit);
                    const int i0 = 1 + 16 * chunk;
#pragma unroll 4
                    for (int k = 0; k < 16; ++k) {
                        const int i = i0 + k;
                        const int2 u = u_of[min(i, N - 1)];
                        // i < j: from the block's first j on one lane fewer for each i
                        const int over = i - 64 * jb;
                        const unsigned long long open = over < 0 ? real : over > 62 ? 0ull : real & ~((2ull << over) - 1ull);
                        const unsigned long long kept = __ballot(dsum::together(u.x, v.x) <= limit) & open,
                                                 other = __ballot(dsum::together(u.y, v.y) <= limit) & open;
                        if (kept | other) {
                            if (kept >> lane & 1) items[wv][n_items + lanes_below(kept)] = (uint32_t)(i << 11 | j << 1);
                            n_items += __popcll(kept);
                            if (other >> lane & 1) items[wv][n_items + lanes_below(other)] = (uint32_t)(i << 11 | j << 1 | 1);
                            n_items += __popcll(other);
                            __builtin_amdgcn_wave_barrier();
                            while (n_items >= 64) {
                                n_items -= 64;
                                score(64);
                            }
                            __builtin_amdgcn_wave_barrier();
                        }
                    }
                }
                deal = chunk - chunks;
            }
            if (n_items) {
                const int n = n_items;
                n_items = 0;
                score(n);
            }
            // ---- the best of all: value, id
            int h = wave_min(hi);
            const int l = wave_min(hi == h ? lo : kNone);
            if (lane == 0) {
                if (l != kNone) atomicMin(&key[turn & 1], ((unsigned long long)((unsigned)h ^ 0x80000000u) << 32) | (unsigned)l);
            }
            __syncthreads();
            const unsigned long long k = key[turn & 1];
            ++turn;
            if (tid == 0) {
                key[turn & 1] = ~0ull;
                best_value[turn & 1] = 0;
            }
            lo = k == ~0ull ? kNone : __builtin_amdgcn_readfirstlane((int)(unsigned)k);
            hi = __builtin_amdgcn_readfirstlane((int)((unsigned)(k >> 32) ^ 0x80000000u));
            __syncthreads();
            if (lo != kNone || T == -1) break;
            T = -max(1, -(T / 8));
        }
        if (lo == kNone) break;                                  // no move lowers the cost
        T = min(-1, (int)((long long)hi / 4));
        // ---- apply: new[p] = old[src(p)]
        const int o = lo & 1, move = lo >> 1, mi = move / N, mj = move - mi * N;
        const int p0 = o ? (tid == 0 ? 0 : N - tid) : tid, src = p0 >= mi && p0 <= mj ? mi + mj - p0 : p0;
        const int val = t[tid < N ? src : 0];
        __syncthreads();
        if (tid < N) t[tid] = val;
        ++applied;
        __syncthreads();
    }
    if (tid < N) tours[r * N + tid] = t[tid];
    if (tid == 0) {
        costs[r] = (int64_t)cur;
        moves[r] = applied;
    }
}

template <int WAVES>
hipError_t launch(const int32_t* c, int N, bool with_flip, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                  const int32_t* skip_if_small, int small_limit, hipStream_t s) {
    hipLaunchKernelGGL(twoopt_dsum_pruned_kernel<WAVES>, dim3(restarts), dim3(64 * WAVES), 0, s, c, N, with_flip ? 1 : 0, tours, costs, moves,
                       skip_if_small, small_limit);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_2opt_dsum_pruned(const int32_t* c, int N, bool with_flip, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                                   const int32_t* skip_if_small, int small_limit, hipStream_t s) {
    // (4 / 8 / 16 wavefronts: N = 70, 100 restarts 434 / 349 / 289 us, 500 restarts 492 / 398 / 546; N = 100, 100 restarts 772 / 608 / 492, 500 restarts
    // 808 / 677 / 912, 1000 restarts 992 / 1132 / 1697; N = 150, 100 restarts 2.0 / 1.3 / 1.0 ms, 500 restarts 2.0 / 1.4 / 1.8, 2000 restarts 3.8 / 4.0 /
    // 6.3; N = 220, 500 restarts 4.1 / 2.7 / 3.3; N = 256, 1000 restarts 6.0 / 5.4 / 7.2; N = 300, 300 restarts - / 4.2 / 4.8; N = 400, 200
    // restarts - / 6.4 / 4.5; N = 512, 100 restarts - / 9.8 / 7.0, 600 restarts - / 16.7 / 19.2)
    const int per_unit = (restarts + 255) / 256;
    if (N > 512 || (N > 64 && per_unit == 1)) return launch<16>(c, N, with_flip, restarts, tours, costs, moves, skip_if_small, small_limit, s);
    if (N > 128 || (N > 64 && per_unit == 2)) return launch<8>(c, N, with_flip, restarts, tours, costs, moves, skip_if_small, small_limit, s);
    return launch<4>(c, N, with_flip, restarts, tours, costs, moves, skip_if_small, small_limit, s);
}

}  // namespace cc
