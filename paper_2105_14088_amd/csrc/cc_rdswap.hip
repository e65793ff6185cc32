// Multi-start pair-swap local search under the halving-doubling cost model (Section 4.1 equation
// C_hd with the pairing of Section 2.2; neighbour "permute a pair" of Section 4.3; move set, value and
// tie-break rules as stated in cc.h, cc_rd_swap_search).
//
// In round k ranks i and i xor 2^k form a LINK whose value is the larger of its two directed costs; a
// round costs its largest link.  Swapping ranks p and q touches, per round, only the links of p and of q
// (one link, with unchanged value, when q = p xor 2^k).  The new round cost is therefore
//     max( link of p re-evaluated, link of q re-evaluated, largest link among all the others ),
// and "largest among the others" is one of the round's three largest links.
//
// General kernel: one workgroup per restart, one thread per rank p scanning q = p+1 .. N-1; matrix
// gathered through L2; 64-bit keys (value << 32 | move id) min-reduced over the workgroup.
// Pruned kernel: one workgroup per restart, any power of two; scores only the swaps that can win.
#include <type_traits>

#include "cc_device.h"
#include "cc_internal.h"

namespace cc {
using namespace ccd;

namespace {

constexpr int kCostMax = (1 << 21) - 1;
constexpr int kMaxStages = 10;
constexpr unsigned long long kNoMove = ~0ull;

// ------------------------------------------------------------------------------------- general kernel
__global__ void rdswap_general_kernel(const int32_t* __restrict__ c, int N, int32_t* __restrict__ tours,
                                      int64_t* __restrict__ costs, int32_t* __restrict__ moves) {
    extern __shared__ int32_t sm[];
    int32_t* t = sm;                 // [N]
    int32_t* w = sm + N;             // [N] directed cost of each rank in the round being prepared
    __shared__ int top_v[kMaxStages][3], top_l[kMaxStages][3], top_n[kMaxStages];
    __shared__ unsigned long long red[16];
    __shared__ unsigned long long winner;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nwv = blockDim.x >> 6;
    const int64_t r = blockIdx.x;
    auto C = [&](int a, int b) { return clampi(c[a * N + b], 0, kCostMax); };
    if (tid < N) t[tid] = clampi(tours[r * N + tid], 0, N - 1);
    __syncthreads();

    auto block_max_u64 = [&](unsigned long long key) {   // every thread gets the maximum
        unsigned long long v = key;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            const unsigned long long o = __shfl_xor(v, m, kWave);
            v = o > v ? o : v;
        }
        __syncthreads();
        if (lane == 0) red[wv] = v;
        __syncthreads();
        v = red[0];
        for (int k = 1; k < nwv; ++k) v = red[k] > v ? red[k] : v;
        return v;
    };

    int applied = 0;
    long long cur = 0;
    for (;;) {
        // ---- per round: link values and the three largest links
        int stages = 0;
        cur = 0;
        for (int bit = 1; bit < N; bit <<= 1, ++stages) {
            if (tid < N) w[tid] = C(t[tid], t[tid ^ bit]);
            __syncthreads();
            int lv = -1;
            if (tid < N && !(tid & bit)) lv = max(w[tid], w[tid | bit]);
            int taken[3] = {-1, -1, -1};
            int n = 0;
            for (int round = 0; round < 3; ++round) {
                const bool mine = lv >= 0 && tid != taken[0] && tid != taken[1];
                // key: value, then a preference for the lower link id (any choice among equal values is valid)
                const unsigned long long key = mine ? (((unsigned long long)(unsigned)lv << 32) | (unsigned)(N - tid)) : 0ull;
                const unsigned long long best = block_max_u64(key);
                if (best == 0ull) break;
                taken[round] = N - (int)(best & 0xffffffffu);
                if (tid == 0) {
                    top_v[stages][round] = (int)(best >> 32);
                    top_l[stages][round] = taken[round];
                }
                ++n;
            }
            if (tid == 0) top_n[stages] = n;
            __syncthreads();
            cur += top_v[stages][0];
        }
        // ---- score swaps (p, q), q > p, for p = tid
        unsigned long long best = kNoMove;
        const int p = tid;
        if (p < N - 1) {
            const int tp = t[p];
            for (int q = p + 1; q < N; ++q) {
                const int tq = t[q];
                int total = 0;
                int k = 0;
                for (int bit = 1; bit < N; bit <<= 1, ++k) {
                    if (q == (p ^ bit)) { total += top_v[k][0]; continue; }
                    const int lp = p & ~bit, lq = q & ~bit;
                    int others = 0;
                    for (int m = 0; m < top_n[k]; ++m)
                        if (top_l[k][m] != lp && top_l[k][m] != lq) { others = top_v[k][m]; break; }
                    const int pb = t[p ^ bit], qb = t[q ^ bit];
                    const int link_p = max(C(tq, pb), C(pb, tq));      // rank p now holds t[q]
                    const int link_q = max(C(tp, qb), C(qb, tp));      // rank q now holds t[p]
                    total += max(others, max(link_p, link_q));
                }
                best = min(best, ((unsigned long long)(unsigned)total << 32) | (unsigned)(p * N + q));
            }
        }
        best = wave_min_u64(best);
        __syncthreads();
        if (lane == 0) red[wv] = best;
        __syncthreads();
        if (tid == 0) {
            unsigned long long m = red[0];
            for (int k = 1; k < nwv; ++k) m = min(m, red[k]);
            winner = m;
        }
        __syncthreads();
        const unsigned long long win = winner;
        if (win == kNoMove || (long long)(win >> 32) >= cur) break;
        const unsigned id = (unsigned)(win & 0xffffffffu);
        const int sp = (int)(id / (unsigned)N), sq = (int)(id % (unsigned)N);
        if (tid == 0) {
            const int a = t[sp];
            t[sp] = t[sq];
            t[sq] = a;
        }
        __syncthreads();
        ++applied;
    }
    if (tid < N) tours[r * N + tid] = t[tid];
    if (tid == 0) {
        costs[r] = cur;
        moves[r] = applied;
    }
}

// 16-bit matrix with both directed entries of a pair folded into both places, max(c[x][y], c[y][x]): a link is then
// one gather.  For the sizes whose matrix does not fit LDS; skipped when an entry needs more than 16 bits.
__global__ __launch_bounds__(256) void fold_to_u16_kernel(const int32_t* __restrict__ c, int n,
                                                          uint16_t* __restrict__ c16,
                                                          const int32_t* __restrict__ flags) {
    if (flags[0] >= (1 << 16)) return;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n * n; e += gridDim.x * 256) {
        const int x = e / n, y = e - x * n;
        c16[e] = (uint16_t)max(clampi(c[e], 0, 0xffff), clampi(c[y * n + x], 0, 0xffff));
    }
}

// ------------------------------------------------------------------------------------- pruned kernel
// A round keeps its cost unless the swap touches its largest link, so a swap that lowers the total has to move an
// end of the largest link of some round: of the N (N-1) / 2 swaps only those with p among the 2 log2 N ends of
// those links can win (20 of 1024 ranks at N = 1024).  Two bounds cut these further, both taken from the three
// largest links (values v1 >= v2 >= v3) of every round:
//   * an end p and any q off every round's two largest links: total >= cur - G(p), G(p) = the sum of v1 - v2 over
//     the rounds whose largest link is p's.  Ends are scanned in falling order of G while cur - G(p) can still reach
//     the best total seen (equal totals are scored too: the lowest id wins them), usually one link's two ends.
//   * an end p and a q on the second largest link of p's round, or two ends: total >= cur - the sum of v1 - the
//     largest other link over the rounds where p or q touch the largest link; no matrix entry is needed to test it,
//     and few of the 4 log2 N + 2 log2^2 N pairs pass.
// The result (value, lowest id) is that of the exhaustive sweep.  Link values live in LDS from sweep to sweep: a swap
// changes 2 log2 N of them, and a round's three largest are found anew only if one of them changed or was passed.
//
// What bounds a sweep is latency: LDS round trips, wave reductions, two barriers.  N = 256, 256 restarts: 10000 clocks a sweep and 306
// vector instructions per wavefront, VALU a third and LDS a quarter of the time busy, the wavefronts waiting for more than half of it.
// So the pairs are looked at beside the first scan, every wave renews the links of the rounds whose largest it keeps, and the order has
// a second copy for the swap, with no barrier between (pairs behind the scans, one wave for the swap, five barriers: 1.27 ms, now 1.01).
// Against the
// exhaustive sweeps before it, matrices of the benchmark's hierarchy: N = 1024, 32 restarts 394 -> 3.3 ms; N = 512, 136 restarts
// 95.7 -> 3.1 ms; N = 256, 58 restarts 9.4 -> 0.98 ms, 788 restarts 31.7 -> 3.0 ms; N = 128, 600 restarts 4.6 -> 0.75 ms; N = 32, 300
// restarts 2.4 -> 0.09 ms.
//
// Where entries come from: N <= 128 folded int32 in LDS (64 KiB at 128), N = 256 folded 16-bit in LDS (128 KiB), else
// the folded 16-bit copy of the workspace through L2, where a scan of p reads only log2 N + 1 rows: the mates' rows in
// node order (coalesced) and p's own row staged in LDS.  Entries from 2^16 up at N >= 256: the caller's matrix.

struct LdsWords {                       // folded int32 in LDS
    const int32_t* m;
    int log_n;
    __device__ __forceinline__ int at(int x, int y) const { return m[(x << log_n) | y]; }
    static constexpr bool kRows = false;
    static constexpr bool kScattered = false;
};
struct LdsHalves {                      // folded 16-bit in LDS
    const uint16_t* m;
    int log_n;
    __device__ __forceinline__ int at(int x, int y) const { return m[(x << log_n) | y]; }
    static constexpr bool kRows = false;
    static constexpr bool kScattered = false;
};
struct GlobalHalves {                   // folded 16-bit copy in the workspace
    const uint16_t* m;
    int log_n;
    __device__ __forceinline__ int at(int x, int y) const { return m[(x << log_n) | y]; }
    static constexpr bool kRows = true;
    static constexpr bool kScattered = false;
};
struct GlobalWords {                    // the caller's matrix, folded as it is read
    const int32_t* m;
    int log_n;
    __device__ __forceinline__ int at(int x, int y) const {
        return max(clampi(m[(x << log_n) | y], 0, kCostMax), clampi(m[(y << log_n) | x], 0, kCostMax));
    }
    static constexpr bool kRows = true;
    static constexpr bool kScattered = true;      // some look-ups take a cache line per lane
};

// LDS words of a workgroup besides the matrix: order, link values, inverse order (the two orders twice) and rows of two scanned
// ranks
constexpr size_t swap_state_words(int log_n, bool rows) {
    const size_t n = (size_t)1 << log_n;
    return 2 * n + (size_t)log_n * (n / 2) + (rows ? 4 * n : 0);
}

// Read before any of them is used: left alone, each is waited for before the next is asked for.
template <int K>
__device__ __forceinline__ void in_flight(int (&x)[K], int (&y)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) asm volatile("" : "+v"(x[k]), "+v"(y[k]));
}

// A link is named by its upper rank (bit k set), a value other than 0; link keys are value << 10 | name, 0 = no link.
// SCAN threads scan, PAIRS more look at the pairs meanwhile (0: the same, afterwards); every wave keeps some rounds' links.
template <int LOGN, int SCAN, int PAIRS, class MAT>
__device__ __forceinline__ void descend_pruned(const MAT mat, int32_t* state, int32_t* __restrict__ tour,
                                               int64_t* __restrict__ cost_out, int32_t* __restrict__ moves_out) {
    constexpr int THREADS = SCAN + PAIRS, N = 1 << LOGN, HALF = N / 2, NW = THREADS / 64, SW = SCAN / 64, M = (HALF + 63) / 64;
    constexpr int kEnds = 2 * LOGN, kNone = 0x7fffffff;
    constexpr int kPicks = 2;                          // ends scanned at a time; the waves share them
    constexpr int kScanThreads = SW > 1 ? SCAN / 2 : 64;
    constexpr int kPairThreads = PAIRS ? PAIRS : THREADS, kPairs = 4 * LOGN + kEnds * (kEnds / 2);
    constexpr int kPairLanes = 2 * kPairs <= kPairThreads ? 2 : 1;     // that share a pair's rounds
    static_assert((SW > 1) == (NW > 1), "one wavefront for everything, or a scanned end for half of them");
    __shared__ int top[3][LOGN];                       // keys of every round's three largest links
    __shared__ int4 gaps[LOGN];                        // {name 1, value 1 - value 2, name 2, value 2 - value 3}
    __shared__ int4 scan_a[SW][kPicks][LOGN];          // for a scanned end: {largest other link's name, its value, the next value, mate's node}
    __shared__ int scan_b[SW][kPicks][LOGN];           // value 1
    __shared__ unsigned long long red[3];
    // the order, and what it becomes while every wave still reads the nodes that move; it is a swap behind (one wave: the same)
    int32_t *t = state, *t_next = NW > 1 ? t + N : t;  // [N]
    int32_t* links = t + 2 * N;                        // [LOGN][HALF] keys
    int32_t *pos = links + LOGN * HALF, *pos_next = pos + N;           // [N] (kRows) rank of a node, -1: none
    int32_t* rows = pos_next + N;                      // [kPicks][N] (kRows)
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto sync = [] { if (NW > 1) __syncthreads(); else __builtin_amdgcn_wave_barrier(); };
    auto upper_of = [](int link, int k) { return ((link >> k) << (k + 1)) | (1 << k) | (link & ((1 << k) - 1)); };
    auto link_of = [](int p, int k) { return ((p >> (k + 1)) << k) | (p & ((1 << k) - 1)); };

    for (int p = tid; p < N; p += THREADS) {
        t[p] = clampi(tour[p], 0, N - 1);
        if (NW > 1) t_next[p] = t[p];
        if (MAT::kRows) pos[p] = -1;
    }
    if (tid < 3) red[tid] = ~0ull;
    __syncthreads();
    if (MAT::kRows) {
        for (int p = tid; p < N; p += THREADS) pos[t[p]] = p;
        __syncthreads();
        for (int p = tid; p < N; p += THREADS) pos_next[p] = pos[p];
    }
#pragma unroll
    for (int k = 0; k < LOGN; ++k)
        for (int l = tid; l < HALF; l += THREADS) {
            const int up = upper_of(l, k);
            links[k * HALF + l] = (mat.at(t[up ^ (1 << k)], t[up]) << 10) | up;
        }
    __syncthreads();

    int cell = 0;
    // smallest (hi, lo) over the workgroup; every thread gets it
    auto block_min = [&](int& hi, int& lo) {
        int h = wave_min(hi);
        const unsigned long long at = __ballot(hi == h);
        int l = __builtin_amdgcn_readlane(lo, (int)__builtin_ctzll(at));
        if (at & (at - 1)) l = wave_min(hi == h ? lo : kNone);
        if (NW > 1) {
            if (lane == 0) atomicMin(&red[cell], ((unsigned long long)(unsigned)h << 32) | (unsigned)l);
            if (tid == 0) red[cell == 2 ? 0 : cell + 1] = ~0ull;    // last read before the previous barrier
            __syncthreads();
            const unsigned long long v = red[cell];
            h = __builtin_amdgcn_readfirstlane((int)(v >> 32));
            l = __builtin_amdgcn_readfirstlane((int)(unsigned)v);
            cell = cell == 2 ? 0 : cell + 1;
        }
        hi = h;
        lo = l;
    };

    constexpr int kPerWave = (LOGN + NW - 1) / NW;     // rounds whose largest links a wave keeps up to date
    constexpr int kBatch = kPerWave < 3 ? kPerWave : 3;
    unsigned dirty = (1u << LOGN) - 1u;                // of this wave's rounds
    // Pairs beside the first scan are bounded by less than pairs behind the last one.  Where their look-ups share the caches with those
    // of many restarts, they come last (entries from 2^16 up, beside / last: N = 1024, 16 restarts 6.93 / 7.17 ms, 64 restarts 8.34 /
    // 8.12, 256 restarts 13.9 / 12.6; N = 512, 64 restarts 5.2 / 5.8, 256 restarts 7.9 / 7.5, 1024 restarts 23.8 / 22.8).  A wavefront
    // alone, 4096 restarts: N = 32 237 / 232 us, but N = 16 88 / 96 and N = 8 32.4 / 32.7.
    const bool pairs_beside = NW == 1 ? LOGN != 5 : !MAT::kScattered || LOGN < 9 || gridDim.x <= (LOGN == 9 ? 128 : 32);
    int applied = 0, cur = -1, last_p = 0, last_q = 0, last_a = t[0], last_b = t[0];
    for (;;) {
        // ---- the three largest links of the rounds that may have new ones
#pragma unroll 1
        for (int k0 = wv * kPerWave; k0 < min((wv + 1) * kPerWave, LOGN); k0 += kBatch) {
            if (!((dirty >> k0) & ((1u << kBatch) - 1u))) continue;
            int key[kBatch][M], kk[3][3];
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const int l = lane + 64 * m, k = min(k0 + j, LOGN - 1);
                    key[j][m] = (HALF >= 64 || l < HALF) ? links[k * HALF + l] : 0;
                }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    int v = 0;
                    if (j < kBatch)
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            int& x = key[j < kBatch ? j : 0][m];
                            if (i > 0 && x == kk[i - 1][j]) x = 0;
                            v = max(v, x);
                        }
                    kk[i][j] = v;
                }
                if (kBatch == 1) kk[i][0] = wave_max(kk[i][0]);
                else wave_max3(kk[i][0], kk[i][1], kk[i][2]);
            }
            if (lane == 0) {
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (k0 + j < LOGN) {
                        const int k = k0 + j;
#pragma unroll
                        for (int i = 0; i < 3; ++i) top[i][k] = kk[i][j];
                        gaps[k] = make_int4(kk[0][j] & 1023, (kk[0][j] >> 10) - (kk[1][j] >> 10), kk[1][j] & 1023,
                                            (kk[1][j] >> 10) - (kk[2][j] >> 10));
                    }
            }
        }
        sync();
        if (cur < 0) cur = wave_sum(lane < LOGN ? top[0][min(lane, LOGN - 1)] >> 10 : 0);
        // lanes 0 .. 2 LOGN - 1: the ends of the largest links; the next 2 LOGN lanes: those of the second largest
        const int round = min(lane >> 1, 2 * LOGN - 1);
        const int name = (&top[0][0])[round] & 1023;
        const int end_rank = (lane & 1) ? name : name & ~(1 << (round >= LOGN ? round - LOGN : round));
        int gain = 0, both = 0;                        // G; what moving a second large link of its rounds can add
#pragma unroll
        for (int k = 0; k < LOGN; ++k) {
            const int4 g = gaps[k];
            const int up = end_rank | (1 << k);
            gain += up == g.x ? g.y : 0;
            both += (up == g.x || up == g.z) ? g.w : 0;
        }
        // ---- scans: two ends at a time, in falling order of G, against every rank
        bool seen = lane >= kEnds;
        int best_hi = cur, best_id = 0;                // a winner has a total below cur
        for (bool pairs_left = true;;) {
            int pick[kPicks] = {};
            int n = 0;
            if (__ballot(!seen && gain > 0 && cur - gain <= best_hi))
#pragma unroll
            for (int s = 0; s < kPicks; ++s) {
                const int g = wave_max(seen ? 0 : (gain << 6) | lane);
                pick[s] = 0;
                if ((g >> 6) > 0 && cur - (g >> 6) <= best_hi) {
                    pick[s] = __builtin_amdgcn_readlane(end_rank, g & 63);
                    seen = seen || end_rank == pick[s];
                    n = s + 1;
                }
            }
            const bool pairs_now = pairs_left && (pairs_beside || n == 0);
            const unsigned long long left = pairs_now ? __ballot(!seen) : 0;
            pairs_left = pairs_left && !pairs_now;
            if (n == 0 && !left) break;
            if (MAT::kRows && n) {
                for (int i = tid; i < n * N; i += THREADS) rows[i] = mat.at(t[i < N ? pick[0] : pick[1]], i & (N - 1));
                sync();
            }
            int hi = best_hi, id = best_id;
#pragma unroll
            for (int s0 = 0; s0 < (NW > 1 ? 1 : kPicks); ++s0) {
                const int s = NW > 1 ? wv / (SW > 1 ? SW / 2 : 1) : s0;
                if (s >= n) break;                     // also the pairs' waves
                const int p = s ? pick[1] : pick[0];
                const int tp = __builtin_amdgcn_readfirstlane(t[p]);
                if (lane < LOGN) {
                    // round `lane`: its largest link that is not p's, and the value that replaces it when it is q's
                    const int k1 = top[0][lane], k2 = top[1][lane], k3 = top[2][lane], up = p | (1 << lane);
                    const bool one = (k1 & 1023) == up, two = (k2 & 1023) == up;
                    const int first = one ? k2 : k1, second = (one || two) ? k3 : k2;
                    scan_a[wv][s0][lane] = make_int4(first & 1023, first >> 10, second >> 10, t[p ^ (1 << lane)]);
                    scan_b[wv][s0][lane] = k1 >> 10;
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll 1
                for (int i = tid & (kScanThreads - 1); i < N; i += kScanThreads) {
                    const int q = MAT::kRows ? pos[i] : i;         // kRows: i is the node, so that rows are read in order
                    const int tq = MAT::kRows ? i : t[i];
                    if (q < 0) continue;
                    int total = 0, x[LOGN], y[LOGN];
#pragma unroll
                    for (int k = 0; k < LOGN; ++k) {
                        const int tm = t[q ^ (1 << k)];
                        x[k] = mat.at(scan_a[wv][s0][k].w, tq);
                        y[k] = MAT::kRows ? rows[s * N + tm] : mat.at(tp, tm);
                    }
                    if constexpr (LOGN == 10) in_flight(x, y);
#pragma unroll
                    for (int k = 0; k < LOGN; ++k) {
                        const int4 w = scan_a[wv][s0][k];
                        const int v = scan_b[wv][s0][k], up = q | (1 << k);
                        const int cost = max(up == w.x ? w.z : w.y, max(x[k], y[k]));
                        total += up == (p | (1 << k)) ? v : cost;  // the mate: the link stays, and with it the round
                    }
                    const int move = min(p, q) * N + max(p, q);
                    const bool better = q != p && (total < hi || (total == hi && move < id));
                    hi = better ? total : hi;
                    id = better ? move : id;
                }
                __builtin_amdgcn_wave_barrier();
            }
            // ---- pairs that move two large links at once: an end of a round's largest and one of its second largest link, or
            // two ends of largest links; pairs with an end scanned before or beside them are known already
            if (left && (PAIRS == 0 || wv >= SW)) {
                constexpr int kSameRound = 4 * LOGN, kAtOnce = kPairThreads / kPairLanes;
                const int bound = PAIRS ? hi : wave_min(hi);
                constexpr int kRounds = (LOGN + kPairLanes - 1) / kPairLanes;
#pragma unroll 1
                for (int i0 = 0; i0 < kPairs; i0 += kAtOnce) {
                    const int at = PAIRS ? tid - SCAN : tid, i = i0 + at / kPairLanes, u = max(i - kSameRound, 0);
                    int e1 = u % kEnds, e2 = e1 + 1 + u / kEnds;
                    e2 = e2 >= kEnds ? e2 - kEnds : e2;
                    const bool same = i < kSameRound;
                    e1 = same ? ((i >> 2) << 1) | (i & 1) : e1;
                    e2 = same ? kEnds + (((i >> 2) << 1) | ((i >> 1) & 1)) : e2;
                    const int p = __shfl(end_rank, e1), q = __shfl(end_rank, e2);
                    const int reach = __shfl(gain, e1) + __shfl(gain, e2) + min(__shfl(both, e1), __shfl(both, e2));
                    if (i >= kPairs || !((left >> e1) & 1) || (!same && !((left >> e2) & 1)) || p == q || cur - reach > bound ||
                        reach == 0)
                        continue;
                    const int tp = t[p], tq = t[q];
                    int total = 0;
#pragma unroll
                    for (int j = 0; j < kRounds; ++j) {
                        const int k = min(at % kPairLanes * kRounds + j, LOGN - 1);
                        const int k1 = top[0][k], k2 = top[1][k], k3 = top[2][k], up = p | (1 << k), uq = q | (1 << k);
                        const bool one = ((k1 & 1023) == up) | ((k1 & 1023) == uq), two = ((k2 & 1023) == up) | ((k2 & 1023) == uq);
                        const int other = (one ? (two ? k3 : k2) : k1) >> 10;
                        const int cost = max(other, max(mat.at(tq, t[p ^ (1 << k)]), mat.at(tp, t[q ^ (1 << k)])));
                        const bool counts = kRounds * kPairLanes == LOGN || at % kPairLanes * kRounds + j < LOGN;
                        total += counts ? (up == uq ? k1 >> 10 : cost) : 0;
                    }
                    if (kPairLanes == 2) total += __builtin_amdgcn_update_dpp(0, total, 0xB1, 0xf, 0xf, true);       // quad_perm 1, 0, 3, 2
                    const int move = min(p, q) * N + max(p, q);
                    const bool better = total < hi || (total == hi && move < id);
                    hi = better ? total : hi;
                    id = better ? move : id;
                }
            }
            block_min(hi, id);
            best_hi = hi;
            best_id = id;
        }
        if (best_hi >= cur) break;
        // ---- the swap: every wave renews the links of its rounds, the first one moves the two nodes
        const int sp = best_id >> LOGN, sq = best_id & (N - 1), a = t[sp], b = t[sq];
        dirty = 0;
        {
            const int k0 = wv * kPerWave, k = min(k0 + (lane >> 1), LOGN - 1);
            const int rank = (lane & 1) ? sq : sp, mate = rank ^ (1 << k), tr = (lane & 1) ? a : b;
            int tm = t[mate];
            tm = mate == sp ? b : (mate == sq ? a : tm);
            bool touched = false;
            if (lane < 2 * min(kPerWave, LOGN - k0)) {
                const int up = rank | (1 << k), key = (mat.at(tr, tm) << 10) | up, l = link_of(rank, k);
                const int k3 = top[2][k];
                touched = key > k3 || links[k * HALF + l] >= k3;
                links[k * HALF + l] = key;
            }
            const unsigned long long bits = __ballot(touched);
#pragma unroll
            for (int j = 0; j < kPerWave; ++j) dirty |= ((bits >> (2 * j)) & 3) ? 1u << (k0 + j) : 0u;
        }
        if (NW == 1) {
            if (lane < 2) t[lane ? sq : sp] = lane ? a : b;
        } else if (wv == 0) {
            if (lane < 4) {
                // this swap and the one before, which the other copy has not seen
                const int x = lane & 2 ? (lane & 1 ? sq : sp) : (lane & 1 ? last_q : last_p);
                const int node = x == sp ? b : x == sq ? a : t[x];
                t_next[x] = node;
                if (MAT::kRows) {
                    const int y = lane & 2 ? (lane & 1 ? b : a) : (lane & 1 ? last_b : last_a);
                    pos_next[y] = y == a ? sq : y == b ? sp : pos[y];
                }
            }
            last_p = sp;
            last_q = sq;
            last_a = a;
            last_b = b;
        }
        if (NW > 1) {
            int32_t* const was = t;
            t = t_next;
            t_next = was;
            if (MAT::kRows) {
                int32_t* const were = pos;
                pos = pos_next;
                pos_next = were;
            }
        }
        ++applied;
        cur = best_hi;
        __builtin_amdgcn_wave_barrier();
    }
    for (int p = tid; p < N; p += THREADS) tour[p] = t[p];
    if (tid == 0) {
        *cost_out = (int64_t)cur;
        *moves_out = applied;
    }
}

// ON_SIMD: wavefronts that find room on a SIMD at least
template <int LOGN, int SCAN, int PAIRS, int ON_SIMD>
__global__ __launch_bounds__(SCAN + PAIRS, ON_SIMD) void rdswap_pruned_kernel(const int32_t* __restrict__ c,
                                                                const uint16_t* __restrict__ folded,
                                                                int32_t* __restrict__ tours, int64_t* __restrict__ costs,
                                                                int32_t* __restrict__ moves,
                                                                const int32_t* __restrict__ flags) {
    constexpr int N = 1 << LOGN, THREADS = SCAN + PAIRS;
    extern __shared__ __attribute__((aligned(16))) int32_t sm[];
    const int tid = threadIdx.x;
    const int64_t r = blockIdx.x;
    int32_t* tour = tours + r * N;
    if constexpr (LOGN <= 8) {
        using E = typename std::conditional<LOGN <= 7, int32_t, uint16_t>::type;
        E* m = (E*)(sm + swap_state_words(LOGN, LOGN == 8));
        __shared__ int wave_top[THREADS / 64];
        int mx = 0;
        for (int e = tid; e < N * N; e += THREADS) {
            const int v = clampi(c[e], 0, kCostMax);
            mx = max(mx, v);
            m[e] = (E)v;
        }
        if constexpr (LOGN == 8) {
            mx = wave_max(mx);
            if ((tid & 63) == 0) wave_top[tid >> 6] = mx;
        }
        __syncthreads();
        if constexpr (LOGN == 8) {
            for (int w = 0; w < THREADS / 64; ++w) mx = max(mx, wave_top[w]);
            if (mx >= (1 << 16)) {
                descend_pruned<LOGN, SCAN, PAIRS>(GlobalWords{c, LOGN}, sm, tour, costs + r, moves + r);
                return;
            }
        }
        // a link costs the larger of its two directed entries: fold the two into both places, every unordered pair
        // once, neighbouring threads on neighbouring columns
        for (int i = tid; i < N * (N / 2); i += THREADS) {
            const int x = i & (N - 1), j = 1 + (i >> LOGN), y = (x + j) & (N - 1);
            if (j < N / 2 || x < N / 2) {
                const E both = max(m[x * N + y], m[y * N + x]);
                m[x * N + y] = both;
                m[y * N + x] = both;
            }
        }
        __syncthreads();
        if constexpr (LOGN <= 7) descend_pruned<LOGN, SCAN, PAIRS>(LdsWords{m, LOGN}, sm, tour, costs + r, moves + r);
        else descend_pruned<LOGN, SCAN, PAIRS>(LdsHalves{m, LOGN}, sm, tour, costs + r, moves + r);
    } else {
        if (flags[0] < (1 << 16)) descend_pruned<LOGN, SCAN, PAIRS>(GlobalHalves{folded, LOGN}, sm, tour, costs + r, moves + r);
        else descend_pruned<LOGN, SCAN, PAIRS>(GlobalWords{c, LOGN}, sm, tour, costs + r, moves + r);
    }
}

template <int LOGN, int SCAN, int PAIRS, int ON_SIMD = LOGN <= 6 ? 5 : 1>
hipError_t rdswap_pruned_launch(const int32_t* c, const uint16_t* folded, int restarts, int32_t* tours, int64_t* costs,
                                int32_t* moves, const int32_t* flags, hipStream_t s) {
    constexpr size_t N = (size_t)1 << LOGN;
    const size_t lds = swap_state_words(LOGN, LOGN >= 8) * 4 + (LOGN <= 7 ? 4 * N * N : LOGN == 8 ? 2 * N * N : 0);
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)rdswap_pruned_kernel<LOGN, SCAN, PAIRS, ON_SIMD>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((rdswap_pruned_kernel<LOGN, SCAN, PAIRS, ON_SIMD>), dim3(restarts), dim3(SCAN + PAIRS), lds, s, c, folded, tours, costs,
                       moves, flags);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fold_to_u16(const int32_t* c, int N, uint16_t* folded, const int32_t* flags, hipStream_t s) {
    hipLaunchKernelGGL(fold_to_u16_kernel, dim3(512), dim3(256), 0, s, c, N, folded, flags);
    return hipGetLastError();
}

hipError_t launch_rdswap(const int32_t* c, int N, int restarts, uint64_t seed, bool tours_hold_init, int32_t* tours,
                         int64_t* costs, int32_t* moves, int32_t* flags, uint16_t* mat16, hipStream_t s) {
    if (!tours_hold_init) {
        hipError_t e = launch_init_tours(N, 0, restarts, seed, tours, s);
        if (e != hipSuccess) return e;
    }
    if (force_general_path()) {
        const int threads = ((N + 63) / 64) * 64;
        hipLaunchKernelGGL(rdswap_general_kernel, dim3(restarts), dim3(threads), sizeof(int32_t) * 2 * (size_t)N, s, c, N,
                           tours, costs, moves);
        return hipGetLastError();
    }
    if (N > 256) {
        hipError_t e = launch_matrix_max(c, N, flags, s);
        if (e == hipSuccess) e = launch_fold_to_u16(c, N, mat16, flags, s);
        if (e != hipSuccess) return e;
    }
    // A sweep is a chain of latencies: more wavefronts per restart, and others for the pairs beside them, shorten it until the compute
    // units run out of room for restarts.  (Wavefronts that scan + those for the pairs, 0: the same; us.)  N = 8, 1024 restarts
    // 1+0 28, 2+1 24, 4096 restarts 35 / 41; N = 16, 1024 restarts 1+0 98, 2+2 66, 2+1 73, 2+0 77, 2048 restarts 98 / 82 / 75 / 77, 4096
    // 105 / 120 / 116 / 107; N = 32, 768 restarts 1+0 177, 2+3 118, 2+2 128, 2+0 137, 2048 restarts 227 / 243 / 186 / 171; N = 64, 256
    // restarts 2+3 199, 2+2 204, 2+0 238, 1+0 320, 1280 restarts 385 / 286 / 298 / 392, 2048 restarts 559 / 402 / 327 / 398; N = 128,
    // 256 restarts 4+4 425, 4+2 482, 4+0 501, 2048 restarts 1591 / 1942 / 1799; N = 512, 256 restarts 8+4 3168, 8+0 3550, 4+4
    // 3862, 512 restarts 5663 / 3999 / 4081; N = 1024, 256 restarts 8+4 3990, 8+0 4546, 512 restarts 7295 / 6358.
    // Two or three wavefronts each are the faster as long as all restarts are on the chip at once: 9 of three on a unit at N = 8 (2+1 /
    // 1+0: 2304 restarts 27.5 / 28.0, 3072 32.9 / 28.5), 10 of two at N = 32 (2+0 / 1+0: 2560 restarts 163 / 199, 3072 229 / 229).
    // At N = 64 registers for five wavefronts on a SIMD are three to six too few; four, where that is room enough (five / four: 256 restarts
    // 273 / 258, 512 285 / 270, 768 301 / 395; 2+2 1280 restarts 317 / 393; 2+0 2048 restarts 371 / 368, 4096 643 / 629).
#define CC_SWAP(LOGN, SCAN, ...) rdswap_pruned_launch<LOGN, SCAN, __VA_ARGS__>(c, mat16, restarts, tours, costs, moves, flags, s)
    switch (N) {
        case 2: return CC_SWAP(1, 64, 0);
        case 4: return CC_SWAP(2, 64, 0);
        case 8: return restarts <= 2304 ? CC_SWAP(3, 128, 64) : CC_SWAP(3, 64, 0);
        case 16: return restarts <= 1536 ? CC_SWAP(4, 128, 128) : restarts <= 3072 ? CC_SWAP(4, 128, 0) : CC_SWAP(4, 64, 0);
        case 32: return restarts <= 768 ? CC_SWAP(5, 128, 192) : restarts <= 2560 ? CC_SWAP(5, 128, 0) : CC_SWAP(5, 64, 0);
        case 64:
            if (restarts <= 512) return CC_SWAP(6, 128, 192, 4);
            return restarts <= 768 ? CC_SWAP(6, 128, 192) : restarts <= 1280 ? CC_SWAP(6, 128, 128) : CC_SWAP(6, 128, 0, 4);
        case 128: return CC_SWAP(7, 256, 256);
        case 256: return CC_SWAP(8, 512, 320);
        case 512: return restarts <= 256 ? CC_SWAP(9, 512, 256) : CC_SWAP(9, 512, 0);
        default: return restarts <= 256 ? CC_SWAP(10, 512, 256) : CC_SWAP(10, 512, 0);
    }
#undef CC_SWAP
}

}  // namespace cc
