// Ring-sum 2-opt, one workgroup per restart: the pairs that can carry the best move are kept from sweep to sweep.  Move set, value
// and tie-break rules as stated in cc.h; symmetric matrix, read through its upper triangle, any entries.
//
// Exchanging the ring edges a and b (edge p joins ranks p-1 and p) changes the cost by
//     delta = [c(t[a-1], t[b-1]) - (f[a] + f[b]) / 2] + [c(t[a], t[b]) - (f[a] + f[b]) / 2],
// one bracket per new edge, so a move of value T or less has a bracket of T / 2 or less: its new edge (x, y) has
//     2 c(x, y) - H(x) - H(y) <= T,      H(x) = the longer of the two hops at x.
// The workgroup keeps all pairs for which that holds in LDS (each wavefront its share, with the cost).  A sweep scores the kept
// pairs on both sides: if the best of them is T or less it is the best move of all, ties included.  A move changes H at four nodes; where
// one grew beyond what the pairs were made for, that node's row is looked through for the pairs that come in, and pairs that no
// longer qualify stay until the next making.  When no kept pair gives T or less, no move does, and the pairs are made anew for alpha / 16
// of T, down to T = -1, where the descent ends; alpha is 8 to 14 by N and restarts (launch_2opt_sum_kept).  Where the pairs do not fit, a
// wavefront scores what it has, starts over and the next sweep makes them anew with T = the value just found, and alpha is one more
// from then on, up to 15: slower, the same moves.
//
// On hierarchies of hosts and racks with 30 % of noise N = 100 keeps some 380 pairs and makes them 12 times in 121 sweeps with alpha 8 (270 and
// 17 of 126 with 10), N = 256 1100 and 17 of 333 with 10, N = 1000 2900 and 56 of 1400 with 14; every third or fourth move lets a row in
// (counted in a model of the algorithm on the CPU).
//
// What bounds it: a sweep is a chain of LDS round trips (pair, its two nodes, the second new edge, the waves' best, the move) between two
// barriers: 3700 clocks at N = 100, 4000 at 128, 4900 at 256, 6000 at 512 and 7800 at 1000 with one restart per unit (4400, 4800, 6300 with four at
// 100, 128, 256).  A sweep that makes the pairs anew takes 8200, 10100, 29900, 22900 and 32300, 15 to 27 % of the time (29 to 39 % with four restarts per unit).
// N = 1000: 271 vector instructions per wavefront and sweep, VALU 49 % busy, wavefronts waiting for 55 % of their time.  Lists of candidates laid out anew on
// every sweep (cc_2opt_sum_pruned.hip, cc_2opt_multi.hip) -> this one: N = 1000, 128 restarts 10.4 -> 5.2 ms; N = 512, 745 restarts 5.65 ->
// 3.16; N = 300, 745 restarts 2.23 -> 1.41; N = 256, 200 restarts 1.22 -> 0.89, 1024 restarts 3.5 -> 1.7; N = 128, 256 restarts 0.60 -> 0.33;
// N = 100, 32 restarts 0.37 -> 0.23.  Slower were: rows of the triangle instead of all its entries end to end (N = 128, 256 restarts 0.33 -> 0.40),
// lists of every node in LDS up to N = 256 (0.39).
//
// Matrices of few values without noise, whose pairs are mostly equal, gain less or lose, by up to 2.7 times where an exhaustive kernel had
// the matrix in LDS (before -> now, two zones: N = 100, 1000 restarts 0.15 -> 0.21 ms, 2048 restarts 0.23 -> 0.35, N = 150, 2000 restarts 0.46 ->
// 0.67, N = 192, 1024 restarts 0.35 -> 0.94, N = 256, 1024 restarts 0.86 -> 1.5, N = 1000, 64 restarts 2.4 -> 2.8; three levels: N = 100, 1000
// restarts 0.29 -> 0.28, N = 256, 1024 restarts 2.3 -> 1.2, 2048 restarts 3.2 -> 4.3; zones of eight: N = 256, 1024 restarts 2.1 -> 0.94).
// Without the large steps over gaps between such values (N <= 256), and handed over above N = 176 only: two zones, N = 100, 1000 restarts 0.26, 2048 restarts
// 0.87, N = 150, 2000 restarts 2.4.
#include <type_traits>

#include "cc_device.h"
#include "cc_internal.h"
#include "cc_pruned.h"

namespace cc {
using namespace ccd;

namespace {

using namespace pruned;

// Above this N a descent is left to the kernel that keeps no pairs: from partner lists after so many sweeps whose pairs did not fit, or at
// once if the first ones, those of the longest hops, do not; from the triangle, whose makings are cheap, after two in a row, as costs
// of few values have them.  In a row / all and at once: racks with 3 % of noise, N = 256, 1024 restarts 1.85 / 5.7 ms, uniform costs, 2048
// restarts 3.8 / 5.9, but racks of equal costs, 2048 restarts 4.3 / 3.3; lists, N = 300, 1500 restarts, 3 % 6.6 / 5.2, two zones 1.67 / 1.36.
// Below, the launch that a hand-over needs costs more than it would give.
constexpr int kStaysMaxN = 128, kMostUnkept = 12, kLeft = -1;

// What becomes of an order that is no permutation: left as it is, taken down rank by rank, or that if no entry needs more than 16 bits.
enum ByRank { kLeftAlone, kByRank, kByRank16 };

// What each wave's best move is, used in turn: value (kNone: none), id, the new hops into the reversed ranks and behind them; the top bit
// of the last says that the wave could not keep all its pairs.
template <int WAVES>
struct KeptWords {
    int4 best[2][WAVES];
    int word[WAVES];
};

__host__ __device__ constexpr size_t align16(size_t n) { return (n + 15) & ~(size_t)15; }
// By node {hop in, hop out, nodes before and behind it, rank}, and the order: two copies, a move reads one and writes the other.  H of
// every node.
__host__ __device__ constexpr size_t kept_info_bytes(int N) { return (size_t)N * 16; }
__host__ __device__ constexpr size_t kept_order_bytes(int N) { return align16((size_t)N * 2); }
__host__ __device__ constexpr size_t kept_state_bytes(int N) {
    return 2 * (kept_info_bytes(N) + kept_order_bytes(N)) + align16((size_t)N * 4);
}

// A kept pair: in 32 bits where node names have eight and costs sixteen.
struct WidePair {
    uint2 w;                                // cost << 10 | y, x
    __device__ __forceinline__ int x() const { return (int)w.y; }
    __device__ __forceinline__ int y() const { return (int)(w.x & 1023u); }
    __device__ __forceinline__ int cost() const { return (int)(w.x >> 10); }
    static __device__ __forceinline__ WidePair of(int x, int y, int cost) { return {make_uint2(((unsigned)cost << 10) | (unsigned)y, (unsigned)x)}; }
};
struct ShortPair {
    uint32_t w;                             // cost << 16 | x << 8 | y
    __device__ __forceinline__ int x() const { return (int)(w >> 8 & 255u); }
    __device__ __forceinline__ int y() const { return (int)(w & 255u); }
    __device__ __forceinline__ int cost() const { return (int)(w >> 16); }
    static __device__ __forceinline__ ShortPair of(int x, int y, int cost) { return {((unsigned)cost << 16) | (unsigned)(x << 8 | y)}; }
};

struct PartnerLists {
    const uint32_t* lists;                  // [N][M] cost << 10 | node
    const uint16_t* counts;                 // [N][kBuckets] partners up to a bucket of cost, the last one holds the scale
    int M;
};

// LISTS: pairs come from partner lists (N > 256), else from the whole upper triangle.
template <int WAVES, bool LISTS, class MAT>
__device__ __forceinline__ void descend_kept(const MAT mat, int N, const PartnerLists lists, int room, int alpha, int by_rank, unsigned char* state, void* pairs_mem,
                                             KeptWords<WAVES>* group, int wv, int lane, int32_t* __restrict__ tour,
                                             int64_t* __restrict__ cost_out, int32_t* __restrict__ moves_out) {
    using Pair = std::conditional_t<MAT::kScattered, WidePair, ShortPair>;
    const int tid = wv * 64 + lane;
    unsigned char* infos = state;                                               // two of uint4 [N]
    unsigned char* orders = infos + 2 * kept_info_bytes(N);                     // two of uint16 [N]
    int* covered = (int*)(orders + 2 * kept_order_bytes(N));                    // [N] the H that the kept pairs stand for
    Pair* pairs = (Pair*)pairs_mem + wv * room;             // [room]
    int side = 0;
    uint4* info = (uint4*)infos;
    uint16_t* t = (uint16_t*)orders;
    auto hop_in = [](uint4 w) { return (int)w.x; };
    auto hop_out = [](uint4 w) { return (int)w.y; };
    auto before = [](uint4 w) { return (int)(w.z & 0xffffu); };
    auto behind = [](uint4 w) { return (int)(w.z >> 16); };
    auto longer = [&](uint4 w) { return max(hop_in(w), hop_out(w)); };
    auto over_waves = [&](int v) {                              // the least of all waves' words
        if (lane == 0) group->word[wv] = v;
        __syncthreads();
        int all = group->word[0];
        for (int w = 1; w < WAVES; ++w) all = min(all, group->word[w]);
        return __builtin_amdgcn_readfirstlane(all);
    };
    auto looser = [&](int v) { return -max((int)((long long)-v * alpha >> 4), 1); };

    // ---- order, hops, ranks; a thread per rank
    const int p0 = min(tid, N - 1), p_before = p0 ? p0 - 1 : N - 1, p_behind = p0 + 1 == N ? 0 : p0 + 1;
    const int t0 = clampi(tour[p0], 0, N - 1);
    if (tid < N) t[tid] = (uint16_t)t0;
    __syncthreads();
    int sum = 0;
    bool few = !LISTS;                                         // 24 of the first 64 ranks' hops cost the same
    {
        const int u = t[p_before], v = t[p_behind];
        const int in = mat(t0, u), out = mat(t0, v);
        if (tid < N) {
            info[t0] = make_uint4((unsigned)in, (unsigned)out, (unsigned)(u | v << 16), (unsigned)tid);
            sum = in;
        }
        if (!LISTS && wv == 0) {
            few = false;
#pragma unroll
            for (int l = 0; l < 8; ++l) few = few || __popcll(__ballot(in == __builtin_amdgcn_readlane(in, l))) >= 24;
        }
    }
    __syncthreads();
    // An order that is no permutation (a data error) is left as it is, or taken down rank by rank below: node-wise hops would not describe it.
    const int start = over_waves(__ballot(tid < N && (int)info[t0].w != tid) == 0 ? few ? 2 : 1 : 0);
    const bool search = start != 0;

    int applied = 0, turn = 0, n_pairs = 0, unkept = 0;        // LISTS: sweeps whose pairs did not fit, else the last of them
    int T = !LISTS && start == 2 ? 1 : 0;                      // none chosen yet; 1: costs of few values
    bool make = true, partial = false;
    int changed = 0, changed_H = 0, changed_before = kNone;    // lanes 0 .. 3: the nodes whose hops the last move changed
    const int units_per_step = 64 * WAVES / (N - 1), rest_per_step = 64 * WAVES - units_per_step * (N - 1);
    while (search) {
        int hi = T, lo = kNone;                                // best move so far: of T or less, none yet
        int first_hop = 0, after_hop = 0;                      // the hops into the reversed ranks and behind them
        // edges a and b exchanged; the new hops before and behind what lies between them
        auto take = [&](int delta, int a, int b, int new_before, int new_behind) {
            if (delta <= hi) {
                a = a >= N ? a - N : a;
                b = b >= N ? b - N : b;
                const int p = min(a, b), q = max(a, b);
                const int id = (int)__umul24((unsigned)(p ? p : q), (unsigned)N) + (p ? q : N) - 1;
                const bool better = delta < hi || id < lo;
                hi = delta;
                lo = better ? id : lo;
                first_hop = better ? new_before : first_hop;
                after_hop = better ? new_behind : after_hop;
            }
        };
        // Scores the wave's pairs from i on, U times 64 with their look-ups in flight together.  Neighbours in the order come out as 0: the
        // edges that they would get are the ones that go.
        auto score_some = [&](auto u_const, int i) {
            constexpr int U = decltype(u_const)::value;
            Pair pr[U];
            uint4 ix[U], iy[U];
            bool in[U], out[U];
            int raw_out[U], raw_in[U], d_out[U], d_in[U], best = kNone;
#pragma unroll
            for (int u = 0; u < U; ++u) pr[u] = pairs[min(i + 64 * u + lane, n_pairs - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ix[u] = info[pr[u].x()];
                iy[u] = info[pr[u].y()];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int least = 2 * pr[u].cost() - T;
                out[u] = hop_out(ix[u]) + hop_out(iy[u]) >= least;
                in[u] = hop_in(ix[u]) + hop_in(iy[u]) >= least;
                raw_out[u] = mat.raw(out[u], mat.row(behind(ix[u])), behind(iy[u]));
                raw_in[u] = mat.raw(in[u], mat.row(before(ix[u])), before(iy[u]));
            }
            // no branch before all are known: a load that moved into one waited on its own
#pragma unroll
            for (int u = 0; u < U; ++u) {
                d_out[u] = out[u] ? pr[u].cost() + mat.cost(raw_out[u]) - (hop_out(ix[u]) + hop_out(iy[u])) : kNone;
                d_in[u] = in[u] ? pr[u].cost() + mat.cost(raw_in[u]) - (hop_in(ix[u]) + hop_in(iy[u])) : kNone;
                best = min(best, min(d_out[u], d_in[u]));
            }
            if (best <= hi) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    take(d_out[u], (int)ix[u].w + 1, (int)iy[u].w + 1, pr[u].cost(), mat.cost(raw_out[u]));
                    take(d_in[u], (int)ix[u].w, (int)iy[u].w, mat.cost(raw_in[u]), pr[u].cost());
                }
            }
        };
        auto put = [&](unsigned long long mask, bool ok, int x, int y, int cost) {
            if (ok) pairs[n_pairs + lanes_below(mask)] = Pair::of(x, y, cost);
            n_pairs += __popcll(mask);
        };
        // ---- pairs come in a part at a time, as far as there is room (scoring stands here once: the code of a sweep has to fit the
        // instruction cache)
        const int H_own = make ? longer(info[p0]) : 0;
        int listed = 0;                                        // LISTS: entries of this lane's node to look at
        unsigned long long more = 0, far = 0;                  // nodes with more than sixteen of them; with partners beyond the list
        int unit = 0, entry_in = 0;                            // of the triangle
        bool listing = true;
        int at = 0;                                            // how far the making, or the node at hand, has got
        if (make) {
            n_pairs = 0;
            if (tid < N) covered[tid] = H_own;
            __syncthreads();
            if constexpr (LISTS) {
                // no bracket is smaller than that of a node's nearest partner beside another hop as long as its own
                if (T == 0) hi = T = looser(over_waves(wave_min(2 * ((int)(lists.lists[p0 * lists.M] >> 10) - H_own))));
                const int reach = H_own + (T >> 1);
                const int bucket = bucket_of(max(reach, 0), (int)lists.counts[p0 * kBuckets + kBuckets - 1]);
                listed = (int)lists.counts[p0 * kBuckets + max(0, min(bucket, kBuckets - 2))];
                listed = bucket >= kBuckets - 1 ? N - 1 : listed;
                listed = tid < N && reach >= 0 && bucket >= 0 ? listed : 0;
                far = __ballot(listed > lists.M);
                listed = listed > lists.M ? 0 : listed;
                more = __ballot(listed > 16);
            } else {
                if (T >= 0) {
                    // Costs of few values leave gaps in which no pair comes in: T takes them in large steps.  (Said by T and alpha, which are
                    // there anyway; a word of its own, or the pairs that came in counted, took 1 to 2 % at N <= 150 with other matrices.)
                    const int later = T == 1 ? 2 : alpha;
                    hi = T = looser(over_waves(-2 * wave_max(H_own)));
                    alpha = later;
                }
                unit = tid / (N - 1);
                entry_in = tid - unit * (N - 1);
            }
            changed_before = kNone;
        } else {
            changed_before = covered[changed];
            more = __ballot(lane < 4 && changed_H > changed_before);
        }
        const unsigned long long all_grew = more;
        // One part; false: no room.  Of two nodes the one with the longer hop finds the pair.
        auto finds = [&](int x, int Hx, int y, int Hy, int cost) {
            return 2 * cost - Hx - Hy <= T && (Hx > Hy || (Hx == Hy && x < y));
        };
        // every node for one whose partners are beyond its list
        auto far_part = [&](int x_first, int H_lane) {
            constexpr int U = 4;
            const int l = (int)__builtin_ctzll(far), x = x_first + l, Hx = __builtin_amdgcn_readlane(H_lane, l);
            int y[U], cost[U], n = 0;
            unsigned long long mask[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                y[u] = min(at + 64 * u + lane, N - 1);
                cost[u] = mat(x, y[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mask[u] = __ballot(at + 64 * u + lane < N && y[u] != x && finds(x, Hx, y[u], covered[y[u]], cost[u]));
                n += __popcll(mask[u]);
            }
            if (n_pairs + n > room) return false;
#pragma unroll
            for (int u = 0; u < U; ++u) put(mask[u], mask[u] >> lane & 1, x, y[u], cost[u]);
            at += 64 * U;
            if (at >= N) {
                at = 0;
                far &= far - 1;
            }
            return true;
        };
        auto lists_part = [&](bool& done) {
            constexpr int U = 8;
            const int M = lists.M, sub = lane & 15, quarter = lane >> 4;
            // the first sixteen partners of 32 nodes, sixteen lanes per node; then the others, 64 of eight nodes at a time
            const bool first = at < 16;
            if (listing && !first && !more) {
                listing = false;
                at = 0;                                        // counts the nodes of a row from here on
            }
            if (!listing) {
                done = !far;
                return done || far_part(64 * wv, H_own);
            }
            uint32_t e[U];
            int x[U], Hx[U], Hy[U], n = 0, most = 0;
            bool ok[U];
            unsigned long long mask[U], rest = more;
            if (first) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int l = 4 * (at + u) + quarter;
                    x[u] = 64 * wv + l;
                    Hx[u] = __builtin_amdgcn_ds_bpermute(l << 2, H_own);
                    ok[u] = sub < __builtin_amdgcn_ds_bpermute(l << 2, listed);
                    e[u] = lists.lists[ok[u] ? (unsigned)(x[u] * M + sub) : 0u];
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int l = rest ? (int)__builtin_ctzll(rest) : 0, end = rest ? __builtin_amdgcn_readlane(listed, l) : 0;
                    rest &= rest - 1;
                    most = max(most, end);
                    x[u] = 64 * wv + l;
                    Hx[u] = __builtin_amdgcn_readlane(H_own, l);
                    ok[u] = at + lane < end;
                    e[u] = lists.lists[ok[u] ? (unsigned)(x[u] * M + at + lane) : 0u];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) Hy[u] = covered[e[u] & 1023u];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ok[u] = ok[u] && finds(x[u], Hx[u], (int)(e[u] & 1023u), Hy[u], (int)(e[u] >> 10));
                mask[u] = __ballot(ok[u]);
                n += __popcll(mask[u]);
            }
            if (n_pairs + n > room) return false;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (mask[u]) put(mask[u], ok[u], x[u], (int)(e[u] & 1023u), (int)(e[u] >> 10));
            at += first ? U : 64;
            if (!first && at >= most) {
                at = 16;
                more = rest;
            }
            return true;
        };
        // Rows x and N - 1 - x of the upper triangle have N - 1 entries together: a unit.  All units end to end, four entries per thread.
        auto triangle_part = [&](bool& done) {
            constexpr int U = 4, THREADS = 64 * WAVES;
            const int total = N * (N - 1) / 2;
            done = at + 64 * wv >= total;
            if (done) return true;
            int x[U], y[U], raw[U], H[U], n = 0, un = unit, i = entry_in;
            unsigned long long mask[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool live = at + tid + THREADS * u < total, low = i < N - 1 - un;
                x[u] = live ? low ? un : N - 1 - un : 0;
                y[u] = live ? low ? un + 1 + i : i + 1 : 1;
                raw[u] = mat.above(x[u], y[u]);
                H[u] = covered[x[u]] + covered[y[u]];
                i += rest_per_step;
                un += units_per_step;
                const bool over = i >= N - 1;
                i -= over ? N - 1 : 0;
                un += over ? 1 : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                raw[u] = mat.cost(raw[u]);
                mask[u] = __ballot(2 * raw[u] - H[u] <= T && at + tid + THREADS * u < total);
                n += __popcll(mask[u]);
            }
            if (n_pairs + n > room) return false;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (mask[u]) put(mask[u], 2 * raw[u] - H[u] <= T && at + tid + THREADS * u < total, x[u], y[u], raw[u]);
            unit = un;
            entry_in = i;
            at += THREADS * U;
            return true;
        };
        // the row of a node whose longer hop grew beyond what the pairs stand for: the pairs that come in
        auto grown_part = [&](bool& done) {
            done = more == 0;
            if (done) return true;
            if (n_pairs + 64 > room) return false;
            const int k = (int)__builtin_ctzll(more);
            const int x = __builtin_amdgcn_readlane(changed, k), Hx = __builtin_amdgcn_readlane(changed_H, k),
                      H_was = __builtin_amdgcn_readlane(changed_before, k);
            more &= more - 1;
            const int cost = mat(x, p0);
            int Hy = covered[p0];
            for (unsigned long long before = all_grew & ((1ull << k) - 1); before; before &= before - 1) {
                const int l = (int)__builtin_ctzll(before);
                Hy = p0 == __builtin_amdgcn_readlane(changed, l) ? __builtin_amdgcn_readlane(changed_H, l) : Hy;
            }
            const bool ok = tid < N && p0 != x && 2 * cost - Hx - Hy <= T && 2 * cost - H_was - Hy > T;
            put(__ballot(ok), ok, x, p0, cost);
            return true;
        };
        for (bool done = false;;) {
            if (!make) {
                while (grown_part(done) && !done) {}
            } else if constexpr (LISTS) {
                while (lists_part(done) && !done) {}
            } else {
                while (triangle_part(done) && !done) {}
            }
            __builtin_amdgcn_wave_barrier();
            int i = 0;
            for (; n_pairs - i > 64; i += 128) score_some(std::integral_constant<int, 2>{}, i);
            if (n_pairs > i) score_some(std::integral_constant<int, 1>{}, i);
            __builtin_amdgcn_wave_barrier();
            if (done) break;
            n_pairs = 0;                                       // what there was has been scored; the rest
            partial = true;
        }
        // ---- the best move of all lanes, then of all waves
        int value, id, h_first, h_after;
        bool again;
        {
            const int h = wave_min(hi);
            unsigned long long at = __ballot(hi == h);
            if (at & (at - 1)) {
                const int l = wave_min(hi == h ? lo : kNone);
                at = __ballot(hi == h && lo == l);
            }
            const int holder = (int)__builtin_ctzll(at);
            if (lane == holder)
                group->best[turn & 1][wv] = make_int4(lo == kNone ? kNone : hi, lo, first_hop, after_hop | (partial ? 1 << 31 : 0));
            __syncthreads();
            const int4 b = group->best[turn & 1][min(lane & 15, WAVES - 1)];
            int v = b.x;
            v = min(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, true));
            v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, true));
            v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, true));
            v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, true));
            value = __builtin_amdgcn_readfirstlane(v);
            at = __ballot(b.x == value);
            if ((at & 0xffffu) & ((at & 0xffffu) - 1)) {
                const int l = wave_min(b.x == value ? b.y : kNone);
                at = __ballot(b.x == value && b.y == l);
            }
            const int w = (int)__builtin_ctzll(at);
            id = __builtin_amdgcn_readlane(b.y, w);
            h_first = __builtin_amdgcn_readlane(b.z, w);
            h_after = __builtin_amdgcn_readlane(b.w, w) & 0x7fffffff;
            again = __ballot(b.w < 0) != 0;
        }
        ++turn;
        partial = false;
        if (value == kNone && T == -1) break;
        if constexpr (LISTS) {                                  // (N is above it; without the comparison N = 1000 takes 1 % longer)
            if (again && N > kStaysMaxN && (unkept += turn == 1 ? kMostUnkept + 1 : 1) > kMostUnkept) break;
        } else if (again && N > kStaysMaxN) {
            const bool in_a_row = unkept == turn - 1 && turn > 1;
            unkept = in_a_row ? kLeft : turn;
            if (in_a_row) break;
        }
        if (value == kNone) {                                   // no move is worth T
            T = looser(T);
            make = true;
            continue;
        }
        make = again;
        if (again) {
            T = value;
            alpha = min(alpha + 1, 15);
        }
        if (wv == 0 && lane < 4 && changed_H > changed_before) covered[changed] = changed_H;
        // ---- reverse ranks mi .. mj: the nodes inside swap the hops and nodes before and behind them, two hops are new
        const int mi = id / N, mj = id - mi * N, after = mj + 1 == N ? 0 : mj + 1;
        {
            const bool inside = tid >= mi && tid <= mj;
            const int node = t[inside ? mi + mj - tid : p0];
            const int n_before = t[mi - 1], n_first = t[mi], n_last = t[mj], n_after = t[after];
            changed = lane == 0 ? n_before : lane == 1 ? n_first : lane == 2 ? n_last : n_after;
            const uint4 w = info[node], was = info[changed];
            changed_H = max(lane == 0 || lane == 2 ? h_first : h_after, lane == 0 || lane == 2 ? hop_in(was) : hop_out(was));
            side ^= 1;
            info = (uint4*)(infos + side * kept_info_bytes(N));
            t = (uint16_t*)(orders + side * kept_order_bytes(N));
            int in = inside ? hop_out(w) : hop_in(w), out = inside ? hop_in(w) : hop_out(w);
            int nb = inside ? behind(w) : before(w), na = inside ? before(w) : behind(w);
            if (tid == mi) in = h_first, nb = n_before;
            if (tid == mj) out = h_after, na = n_after;
            if (tid == mi - 1) out = h_first, na = n_last;
            if (tid == after) in = h_after, nb = n_first;
            if (tid < N) {
                t[tid] = (uint16_t)node;
                info[node] = make_uint4((unsigned)in, (unsigned)out, (unsigned)(nb | na << 16), (unsigned)tid);
            }
        }
        sum += tid == 0 ? value : 0;
        ++applied;
        __syncthreads();
    }
    if constexpr (!LISTS) {
        // The exhaustive kernels go by ranks and descend from such an order as from any; where one serves N as well, so does this.
        bool descends = !search && by_rank != kLeftAlone;
        if (descends && by_rank == kByRank16) {
            int high = 0;
            for (int e = tid; e < N * N; e += 64 * WAVES) {
                const int x = e / N, y = e - x * N;
                high = max(high, mat(x, y));
            }
            __syncthreads();                                   // the words of `search` have been read
            descends = over_waves(-wave_max(high)) > -(1 << 16);
        }
        while (descends) {
            unsigned long long key = ~0ull;
            for (int e = tid; e < N * N; e += 64 * WAVES) {
                const int i = e / N, j = e - i * N, q = j + 1 == N ? 0 : j + 1;
                if (i < 1 || i >= j || (i == 1 && j == N - 1)) continue;
                const int delta = mat(t[j], t[i - 1]) + mat(t[q], t[i]) - mat(t[i], t[i - 1]) - mat(t[q], t[j]);
                const unsigned long long k = ((unsigned long long)(unsigned)(delta + (1 << 30)) << 32) | (unsigned)e;
                key = k < key ? k : key;
            }
            key = wave_min_u64(key);
            __syncthreads();
            if (lane == 0) group->best[0][wv] = make_int4((int)(key >> 32), (int)key, 0, 0);
            __syncthreads();
            for (int w = 0; w < WAVES; ++w) {
                const int4 b = group->best[0][w];
                const unsigned long long k = ((unsigned long long)(unsigned)b.x << 32) | (unsigned)b.y;
                key = k < key ? k : key;
            }
            const int value = (int)(key >> 32) - (1 << 30), id = (int)key, mi = id / N, mj = id - mi * N;
            if (key == ~0ull || value >= 0) break;
            const int node = t[tid >= mi && tid <= mj ? mi + mj - tid : p0];
            __syncthreads();
            if (tid < N) t[tid] = (uint16_t)node;
            sum += tid == 0 ? value : 0;
            ++applied;
            __syncthreads();
        }
    }
    // ---- results
    sum = wave_sum(sum);
    __syncthreads();
    if (lane == 0) group->word[wv] = sum;
    __syncthreads();
    sum = 0;
    for (int i = 0; i < WAVES; ++i) sum += group->word[i];
    if (tid < N) tour[tid] = (int)t[tid];
    if (tid == 0) {
        *cost_out = (LISTS ? unkept > kMostUnkept : unkept == kLeft) ? -1 : (int64_t)sum;
        *moves_out = applied;
    }
}

// N <= 64 WAVES.  lds_matrix: the matrix as 16-bit entries in LDS where its entries allow.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void twoopt_sum_kept_kernel(const int32_t* __restrict__ c, int N, int lds_matrix, int room,
                                                                     int alpha, int by_rank, int32_t* __restrict__ tours,
                                                                     int64_t* __restrict__ costs, int32_t* __restrict__ moves) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ KeptWords<WAVES> group;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    const PartnerLists none{nullptr, nullptr, 0};
    void* pairs = smem + kept_state_bytes(N);
    if (lds_matrix) {
        uint16_t* m16 = (uint16_t*)(smem + kept_state_bytes(N) + (size_t)WAVES * room * 4);
        int high = 0;
        for (int x = wv; x < N; x += WAVES)
            for (int y = x + lane; y < N; y += 64) {
                const int v = entry(c, N, x, y);
                high = max(high, v);
                m16[x * N + y] = (uint16_t)v;
                m16[y * N + x] = (uint16_t)v;
            }
        high = wave_max(high);
        if (lane == 0) group.word[wv] = high;
        __syncthreads();
        high = 0;
        for (int w = 0; w < WAVES; ++w) high = max(high, group.word[w]);
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(high) < (1 << 16)) {
            descend_kept<WAVES, false>(LdsMatrix{m16, N}, N, none, room, alpha, by_rank, smem, pairs, &group, wv, lane, tours + r * N, costs + r,
                                       moves + r);
            return;
        }
    }
    // wider pairs; the matrix's room is theirs
    descend_kept<WAVES, false>(CallersMatrix{c, N}, N, none, room, alpha, by_rank, smem, pairs, &group, wv, lane, tours + r * N, costs + r, moves + r);
}

// N > 256: partner lists in the workspace.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES <= 8 ? 6 : 4))) void twoopt_sum_kept_lists_kernel(const int32_t* __restrict__ c, int N, int M,
                                                                           const uint32_t* __restrict__ lists,
                                                                           const uint16_t* __restrict__ counts, int room, int alpha,
                                                                           int32_t* __restrict__ tours, int64_t* __restrict__ costs,
                                                                           int32_t* __restrict__ moves) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ KeptWords<WAVES> group;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    descend_kept<WAVES, true>(CallersMatrix{c, N}, N, PartnerLists{lists, counts, M}, room, alpha, kLeftAlone, smem,
                               (void*)(smem + kept_state_bytes(N)), &group, wv, lane, tours + r * N,
                              costs + r, moves + r);
}

template <int WAVES>
hipError_t launch_kept(const int32_t* c, int N, bool lds_matrix, int room, int alpha, int restarts, int32_t* tours, int64_t* costs,
                       int32_t* moves, hipStream_t s) {
    if (N > 64 * WAVES || room < 256) return hipErrorInvalidValue;       // a thread per rank; a part of a making fits
    const size_t wide = (size_t)WAVES * room * 8, brief = (size_t)WAVES * room * 4 + (size_t)N * N * 2;
    const size_t lds = kept_state_bytes(N) + (lds_matrix && brief > wide ? brief : wide);
    hipError_t e = hipFuncSetAttribute((const void*)twoopt_sum_kept_kernel<WAVES>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // 192 and 256: the restarts that the exhaustive kernels of these sizes are the alternative for
    const int by_rank = N <= 128 ? kByRank : (N == 192 || N == 256) && restarts > 256 && restarts <= 1536 ? kByRank16 : kLeftAlone;
    hipLaunchKernelGGL((twoopt_sum_kept_kernel<WAVES>), dim3(restarts), dim3(64 * WAVES), lds, s, c, N, lds_matrix ? 1 : 0, room, alpha, by_rank,
                       tours, costs, moves);
    return hipGetLastError();
}

template <int WAVES>
hipError_t launch_kept_lists(const int32_t* c, int N, int room, int alpha, void* workspace, int restarts, int32_t* tours, int64_t* costs,
                             int32_t* moves, hipStream_t s) {
    if (N > 64 * WAVES || room < 512) return hipErrorInvalidValue;       // a thread per rank; a part of a making fits
    int M;
    const uint32_t* lists;
    const uint16_t* counts;
    hipError_t e = launch_partner_lists(c, N, workspace, M, lists, counts, s);
    if (e != hipSuccess) return e;
    const size_t lds = kept_state_bytes(N) + (size_t)WAVES * room * 8;
    e = hipFuncSetAttribute((const void*)twoopt_sum_kept_lists_kernel<WAVES>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((twoopt_sum_kept_lists_kernel<WAVES>), dim3(restarts), dim3(64 * WAVES), lds, s, c, N, M, lists, counts, room, alpha,
                       tours, costs, moves);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_2opt_sum_kept(const int32_t* c, int N, void* room, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                                hipStream_t s) {
    // Up to 256 restarts a unit has one: as many wavefronts as shorten a sweep (N = 128, 256 restarts, 4 / 8 wavefronts 383 / 331 us, N = 256
    // 1411 / 943, N = 512 8 / 12 / 16 2096 / 2104 / 2183), T loosened in larger steps where a making costs more than longer sweeps do.
    // Pairs have the rest of the LDS: with less, matrices of few values make them anew on every sweep.
    const int per_unit = (restarts + 255) / 256;
    auto room_for = [&](int waves, int at_a_time, bool lds_matrix) {
        const int all = 152 * 1024 / at_a_time - 1024 - (int)kept_state_bytes(N);
        const int wide = all / (waves * 8), brief = (all - N * N * 2) / (waves * 4);
        const int fit = lds_matrix && brief < wide ? brief : wide, most = N * (N - 1) / waves;   // all pairs, and as many that came in later
        const int room = fit < most ? fit : most, least = N <= 256 ? 256 : 512;                  // a part of a making fits
        return room > least ? room : least;
    };
    if (N <= 128) {
        if (per_unit == 1) return launch_kept<8>(c, N, true, room_for(8, 1, true), 8, restarts, tours, costs, moves, s);
        if (per_unit <= 4) {
            const bool lds_matrix = per_unit <= 2 || N <= 112;
            return launch_kept<4>(c, N, lds_matrix, room_for(4, per_unit, lds_matrix), 10, restarts, tours, costs, moves, s);
        }
        return launch_kept<2>(c, N, false, room_for(2, 8, false), 10, restarts, tours, costs, moves, s);
    }
    if (N <= 256) {
        // the matrix in LDS where two workgroups with it fit a unit (N = 170, 512 restarts 635 us, through L2 650; N = 192 1122, 742)
        if (per_unit <= 2) return launch_kept<8>(c, N, N <= 176, room_for(8, per_unit, N <= 176), 10, restarts, tours, costs, moves, s);
        return launch_kept<4>(c, N, false, room_for(4, per_unit < 6 ? per_unit : 6, false), 11, restarts, tours, costs, moves, s);
    }
    // three workgroups of eight wavefronts or four of five are what a unit's registers hold
    if (N <= 320 && per_unit > 2) return launch_kept_lists<5>(c, N, room_for(5, per_unit < 4 ? per_unit : 4, false), 13, room, restarts, tours, costs, moves, s);
    if (N <= 512) return launch_kept_lists<8>(c, N, room_for(8, per_unit < 3 ? per_unit : 3, false), 13, room, restarts, tours, costs, moves, s);
    if (N <= 640) return launch_kept_lists<12>(c, N, room_for(12, 1, false), 13, room, restarts, tours, costs, moves, s);
    return launch_kept_lists<16>(c, N, room_for(16, 1, false), 14, room, restarts, tours, costs, moves, s);
}

bool sum_kept_leaves_restarts(int N) { return N > kStaysMaxN; }

}  // namespace cc
