// Ring-sum 2-opt for 97 <= N <= 1024 and any entries, where restarts are too many, or pairs, for cc_2opt_sum_kept.hip: only the moves
// that can be the best one are scored.  Move set, value and tie-break rules as stated in cc.h; symmetric matrix, read through its upper
// triangle.
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
//   * N <= 256: lists in LDS, made by the workgroup itself, up to 16 restarts of one wavefront each around one copy of them.  Up to 256
//     (N <= 192: mostly 512) restarts, which come here from N = 129 on and only as far as cc_2opt_sum_kept.hip left them, one workgroup of
//     eight (four) wavefronts each.
//   * N > 256, only restarts that cc_2opt_sum_kept.hip left: one workgroup per restart, lists in the workspace (M = (N - 128) / 2), which
//     have been made for that kernel.
// The candidates of 64 nodes are laid out end to end (prefix sum of their counts) and taken 64 at a time, up to four
// times 64 with their look-ups in flight together; those whose bracket passes are collected in LDS and scored 64 at a
// time.  The wavefronts of one restart take the 64s of all nodes in turn (the nodes of one wavefront have two or three times the
// candidates of another's, and the passed ones lie together), so there may be more wavefronts than nodes / 64.
//
// What bounds it: instruction issue (with 16 wavefronts, N = 1000, about 740 vector instructions per wavefront and sweep, 70 % of the
// SIMDs' rate), and with few wavefronts the latency of each one's own.  All times here are of whole searches by this kernel, also at the
// sizes where it now has only what is left.  Exhaustive kernels -> this one: N = 1000, 128 restarts 494 ->
// 10.6 ms; N = 583, 47 restarts 112 -> 4.4 ms; N = 345, 2140 restarts 239 -> 7.4 ms; N = 1024, 256 restarts 57.9 -> 11.3 ms; N = 512, 768
// restarts 19.2 -> 5.6 ms; N = 256, 4096 restarts 7.8 -> 5.2 ms.  Every wavefront its own nodes' candidates, one per 64 nodes -> shared,
// more wavefronts: N = 1000, 128 restarts 11.5 -> 10.6 ms, N = 700, 100 restarts 6.4 -> 5.5, N = 400, 64 restarts 2.77 -> 2.23, N = 300,
// 250 restarts 1.89 -> 1.53, N = 200, 256 restarts 1.24 -> 0.96, N = 150, 500 restarts 0.88 -> 0.70.  Slower were: two or four nodes per lane
// and half or a quarter of the wavefronts (N = 1000 13.2, 21.2 ms); a D of each wavefront's own without the barrier (N = 1000 10.4 ms, but
// two zones of equal costs, N = 1024, 64 restarts 2.9 -> 5.3 ms: fewer equal moves are ruled out).
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

// Several waves per restart: besides, where each node's candidates begin.
__host__ __device__ constexpr size_t group_order_bytes(int N) { return order_bytes(N) + (((size_t)N * 2 + 15) & ~(size_t)15); }
constexpr int kGroupAtOnce = 3;         // times 64 candidates
constexpr int kGroupPassed = 64 * (kGroupAtOnce + 1);
// entries: a passed candidate is kept with its entry of the list (eight bytes), else by its place in the lists (four)
__host__ __device__ constexpr size_t group_wave_bytes(int room, bool entries) {
    return (size_t)room * 2 + kGroupPassed * (entries ? 8 : 4);
}

// What the waves of one restart tell each other
template <int WAVES>
struct GroupWords {
    unsigned long long key[4];              // of the best move, used in turn: value, id, wave
    uint2 hops[2][WAVES];                   // the hops each wave's best move makes
    int laid_out[WAVES];                    // candidates
    int word[WAVES];
};

// One descent.  A node's scale (of its buckets) is scale0 (one node per lane) or scales[node].  Wave `wv` of the restart
// owns the nodes 64 * (wv * K + k) + lane.
template <int WAVES, int K, int ROOM, bool ENTRIES, typename COUNT, class MAT>
__device__ __forceinline__ void descend(const MAT mat, int N, const uint32_t* __restrict__ lists, int M,
                                        const COUNT* __restrict__ counts, int scale0, const uint16_t* scales, unsigned char* order_mem,
                                        unsigned char* wave_mem, GroupWords<WAVES>* group, int wv, int lane, int applied,
                                        int32_t* __restrict__ tour, int64_t* __restrict__ cost_out,
                                        int32_t* __restrict__ moves_out) {
    constexpr int THREADS = 64 * WAVES;
    // The waves of a restart share the candidates of all its nodes, and what a look-up through L2 has brought is kept: a passed
    // candidate's entry of the list, the hops that the best move makes.
    constexpr bool GROUP = WAVES > 1;
    static_assert(!GROUP || K == 1, "a group's wave owns 64 nodes at most");
    uint2* info = (uint2*)order_mem;                           // [N] by node
    uint16_t* t = (uint16_t*)(info + N) + 1;                   // t[-1] = t[N-1], t[N] = t[0]
    uint16_t* owner = (uint16_t*)wave_mem;                     // [ROOM] stamp << 6 | lane
    // [kPassed] x | place << 10 | sides << 21; place: in the list of x, or M + y for a node scanned against every node
    uint32_t* passed = (uint32_t*)(wave_mem + ROOM * 2);
    uint2* passed_entries = (uint2*)passed;                    // ENTRIES: [kGroupPassed] x | sides << 21, cost << 10 | y
    uint16_t* starts = (uint16_t*)(order_mem + order_bytes(N));                    // GROUP: [N] place of a node's first candidate
    const int tid = wv * 64 + lane;
    auto list_entry = [&](unsigned at) { return *(const uint32_t*)((const char*)lists + at * 4u); };
    auto sync = [] { if (WAVES > 1) __syncthreads(); else __builtin_amdgcn_wave_barrier(); };
    auto hop_in = [](uint2 w) { return (int)(w.x >> 10); };
    auto hop_out = [](uint2 w) { return (int)w.y; };
    auto rank_of = [](uint2 w) { return (int)(w.x & 1023u); };

    // ---- order, hops, ranks
    int t0[K], turn = 0;
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
    // the candidate a lane remembers from an earlier sweep; at first the nearest partner of its first node
    int rx = min(64 * wv * K + lane, N - 1);
    const uint32_t nearest = lists[(size_t)rx * M];
    int ry = (int)(nearest & 1023u), r_cost = (int)(nearest >> 10);
    int r_value = 0;                                           // what it was worth
    if (GROUP) {
        // over the wavefronts of this restart alone: the workgroup's others have ended, which a plain barrier allows and a
        // workgroup-wide reduction of the library need not
        if (lane == 0) group->word[wv] = search ? 1 : 0;
        if (tid < 4) group->key[tid] = ~0ull;
        __syncthreads();
        search = __ballot(group->word[min(lane, WAVES - 1)] == 0) == 0;
    }
    unsigned stamp = 0;
    int last_start = 0;
    while (search) {
        int hi = 0, lo = -1;                                   // best move so far; none: 0 and an id nothing undercuts
        int sweep_best = kNone;                                // this lane's own best of the sweep, for rx and ry
        int first_hop = 0, after_hop = 0;                      // GROUP: the hops into the reversed ranks and behind them
        // edges a and b exchanged; the new hops before and behind what lies between them
        auto take = [&](int delta, int a, int b, int before, int behind) {
            a = a >= N ? a - N : a;
            b = b >= N ? b - N : b;
            const int p = min(a, b), q = max(a, b);
            const int id = (int)__umul24((unsigned)(p ? p : q), (unsigned)N) + (p ? q : N) - 1;
            const bool better = delta < hi || (delta == hi && id < lo);
            hi = better ? delta : hi;
            lo = better ? id : lo;
            if (GROUP) {
                first_hop = better ? before : first_hop;
                after_hop = better ? behind : after_hop;
            }
        };
        // the best move of all lanes
        auto group_best = [&] {
            const int h = wave_min(hi);
            const unsigned long long at = __ballot(hi == h);
            int holder = (int)__builtin_ctzll(at), l = __builtin_amdgcn_readlane(lo, holder);
            if (at & (at - 1)) {
                l = wave_min(hi == h ? lo : kNone);
                holder = (int)__builtin_ctzll(__ballot(hi == h && lo == l));
            }
            hi = h;
            lo = l;
            if (GROUP) {
                first_hop = __builtin_amdgcn_readlane(first_hop, holder);
                after_hop = __builtin_amdgcn_readlane(after_hop, holder);
                if (lane == 0) {
                    group->hops[turn & 1][wv] = make_uint2((unsigned)first_hop, (unsigned)after_hop);
                    atomicMin(&group->key[turn & 3], ((unsigned long long)(unsigned)(hi + (1 << 30)) << 24) |
                                                         (unsigned)((lo & 0xfffff) << 4) | (unsigned)wv);
                    group->key[(turn + 2) & 3] = ~0ull;          // read by all before the last barrier, used again after the next
                }
                __syncthreads();
                const unsigned long long key = group->key[turn & 3];
                const uint2 hops = group->hops[turn & 1][(int)key & 15];
                hi = __builtin_amdgcn_readfirstlane((int)(key >> 24)) - (1 << 30);
                lo = hi < 0 ? __builtin_amdgcn_readfirstlane((int)((unsigned)key >> 4 & 0xfffffu)) : -1;
                first_hop = (int)hops.x;
                after_hop = (int)hops.y;
                ++turn;
            }
        };
        // ---- D from the remembered candidates, on both sides (a reversal turns one into the other)
        {
            const bool worth = r_value <= 0;
            const uint2 ix = info[rx], iy = info[ry];
            const int p = rank_of(ix), q = rank_of(iy), d = p < q ? q - p : p - q;
            const int cxy = GROUP ? r_cost : mat(worth ? rx : 1, worth ? ry : 0);
            const int cp = mat(worth ? t[p + 1] : 1, worth ? t[q + 1] : 0), cm = mat(worth ? t[p - 1] : 1, worth ? t[q - 1] : 0);
            if (worth && d >= 2 && d <= N - 2) {
                const int behind = cxy + cp - hop_out(ix) - hop_out(iy), before = cxy + cm - hop_in(ix) - hop_in(iy);
                take(behind, p + 1, q + 1, cxy, cp);
                take(before, p, q, cm, cxy);
                sweep_best = min(behind, before);
            }
            r_value = sweep_best;
        }
        group_best();
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
            int x, y, sides, cost;
            if (ENTRIES) {
                const uint2 w = passed_entries[from + (live ? lane : 0)];
                x = (int)(w.x & 1023u);
                sides = (int)(w.x >> 21);
                y = (int)(w.y & 1023u);
                cost = (int)(w.y >> 10);
            } else {
                const uint32_t w = passed[from + (live ? lane : 0)];
                const int place = (int)((w >> 10) & 2047u);
                x = (int)(w & 1023u);
                sides = (int)(w >> 21);
                const bool listed = place < M;
                const uint32_t e = list_entry(__umul24((unsigned)x, (unsigned)M) + (unsigned)(listed ? place : 0));
                y = listed ? (int)(e & 1023u) : place - M;
                cost = (int)(e >> 10);
                if (__ballot(!listed)) cost = listed ? cost : mat(x, y);
            }
            const uint2 ix = info[x], iy = info[y];
            const int p = rank_of(ix), q = rank_of(iy), d = p < q ? q - p : p - q;
            const bool fits = live && d >= 2 && d <= N - 2;
            auto side = [&](bool out) {
                const int a = out ? p + 1 : p, b = out ? q + 1 : q;
                const int other = mat(t[out ? p + 1 : p - 1], t[out ? q + 1 : q - 1]);
                const int delta = cost + other - (out ? hop_out(ix) + hop_out(iy) : hop_in(ix) + hop_in(iy));
                if (fits) {
                    take(delta, a, b, out ? cost : other, out ? other : cost);
                    if (delta < sweep_best) {
                        sweep_best = delta;
                        r_value = delta;
                        rx = x;
                        ry = y;
                        r_cost = cost;
                    }
                }
            };
            side(sides & 1);
            if (__ballot(live && sides == 3)) side(sides != 3);        // the other side of those; of the others, any
        };
        // Notes the pair x, y of cost e >> 10 if a bracket of it passes; the node with the longer removed edge looks at it.  Side bits: 1
        // the edges behind x and y, 2 those before; place: where the list has y (ENTRIES: unused).  No branches but the store:
        // with one per condition a candidate took half as many instructions again.
        auto look = [&](bool live, uint2 ix, uint2 iy, uint32_t e, int x, int place) {
            const int ox = hop_out(ix), oy = hop_out(iy), nx = hop_in(ix), ny = hop_in(iy), least = (int)((e >> 9) & ~1u) - D;
            const bool out = live & (ox >= oy) & (ox + oy >= least), in = live & (nx >= ny) & (nx + ny >= least);
            const unsigned long long mask = __ballot(out | in);
            if (out | in) {
                const unsigned at = (unsigned)(n_passed + lanes_below(mask));
                const unsigned who = (unsigned)x | (out ? 1u << 21 : 0u) | (in ? 2u << 21 : 0u);
                if (ENTRIES) passed_entries[at] = make_uint2(who, e);
                else passed[at] = who | ((unsigned)place << 10);
            }
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
        // ---- how far the threshold of node x (one per lane) reaches; the candidates of the 64 nodes end to end from place `from` on.
        // Returns where they end; all: x is scanned against every node instead, its partners are beyond the list or the room.
        auto lay_out = [&](int x, int scale, int from, unsigned mark, bool& all) {
            const uint2 ix = info[min(x, N - 1)];
            const bool equals = __umul24((unsigned)rank_of(ix), (unsigned)N) <= (unsigned)lo;      // lo is -1 where no move is known
            const int reach = max(hop_in(ix), hop_out(ix)) + ((equals ? D : D - 1) >> 1);
            const int bucket = bucket_of(max(reach, 0), scale);
            int count = (int)*(const COUNT*)((const char*)counts + (unsigned)sizeof(COUNT) * (unsigned)(min(x, N - 1) * kBuckets + max(0, min(bucket, kBuckets - 2))));
            count = bucket >= kBuckets - 1 ? N - 1 : count;
            count = x < N && reach >= 0 && bucket >= 0 ? count : 0;
            all = count > M;
            count = all ? 0 : count;
            int end = from + wave_prefix_sum(count);
            int total = __builtin_amdgcn_readlane(end, 63);
            if (total > ROOM) {
                const bool out = end > ROOM;
                all = all || (out && count > 0);
                count = out ? 0 : count;
                total = wave_max(out ? from : end);
            }
            const int start = end - count;
            if (count > 0) {
                owner[start] = (uint16_t)mark;
                for (int i = (start | 63) + 1; i < start + count; i += 64) owner[i] = (uint16_t)mark;     // every 64 start anew
            }
            if (GROUP && x < N) starts[x] = (uint16_t)start;
            last_start = start;
            return total;
        };
        auto next_stamp = [&] {
            if (++stamp == 1024) {
                stamp = 1;
                for (int i = lane; i < ROOM; i += 64) owner[i] = 0;
                __builtin_amdgcn_wave_barrier();
            }
        };
        auto scan_all = [&](bool all, int x_first) {
            unsigned long long rest = __ballot(all);
            while (rest) {
                const int nx = x_first + (int)__builtin_ctzll(rest);
                rest &= rest - 1;
                const uint2 jx = info[nx];
                constexpr int U = GROUP ? 2 : 4;               // four times 64 nodes of N = 256 (three at a time: N = 225, 300 restarts 1.47 ms, 1.41)
                for (int y0 = 0; y0 < N; y0 += 64 * U) {
                    int cost[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) cost[u] = mat(nx, min(y0 + 64 * u + lane, N - 1));
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int y = y0 + 64 * u + lane;
                        look(y < N, jx, info[min(y, N - 1)], ((unsigned)cost[u] << 10) | (unsigned)y, nx, M + y);
                    }
                    flush();
                }
            }
        };
        if constexpr (GROUP) {
            // ---- an equal share of all nodes' candidates for every wave, 64 at a time
            bool all;
            next_stamp();
            const int total = lay_out(64 * wv + lane, scale0, 0, stamp * 64 + (unsigned)lane, all);
            if (lane == 0) group->laid_out[wv] = total;
            __syncthreads();
            const int laid_out = lane < WAVES ? group->laid_out[lane] : 0;
            const int upto = wave_prefix_sum((laid_out + 63) >> 6);          // of the waves up to this lane's
            const int blocks = __builtin_amdgcn_readlane(upto, 63);
            auto brackets = [&](auto u_const, int g0) {
                constexpr int U = decltype(u_const)::value;
                unsigned src[U];
                int from[U], place[U], first[U], live[U];
                uint2 jx[U], jy[U];
                uint32_t e[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int g = g0 + WAVES * u, w = __popcll(__ballot(upto <= g));         // whose candidates these are
                    const int i0 = 64 * (g - (w ? __builtin_amdgcn_readlane(upto, w - 1) : 0));
                    first[u] = 64 * w;
                    live[u] = __builtin_amdgcn_readlane(laid_out, w) - i0;
                    place[u] = i0 + lane;
                    src[u] = ((const uint16_t*)(wave_mem + (w - wv) * (int)group_wave_bytes(ROOM, ENTRIES)))[place[u]];
                }
                // marks of earlier layouts are smaller than this one's, and the first of the 64 is always marked
#pragma unroll
                for (int u = 0; u < U; ++u) src[u] = min((unsigned)first[u] + (wave_prefix_max(src[u]) & 63u), (unsigned)N - 1);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    from[u] = starts[src[u]];
                    jx[u] = info[src[u]];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) e[u] = list_entry(lane < live[u] ? __umul24(src[u], (unsigned)M) + (unsigned)(place[u] - from[u]) : 0u);
#pragma unroll
                for (int u = 0; u < U; ++u) jy[u] = info[e[u] & 1023u];
#pragma unroll
                for (int u = 0; u < U; ++u) look(lane < live[u], jx[u], jy[u], e[u], (int)src[u], place[u] - from[u]);
            };
            // one after the other in turn: the candidates of a node that most is scored of lie side by side
            for (int g = wv; g < blocks; g += kGroupAtOnce * WAVES) {
                if (blocks - g > 2 * WAVES) brackets(std::integral_constant<int, 3>{}, g);
                else if (blocks - g > WAVES) brackets(std::integral_constant<int, 2>{}, g);
                else brackets(std::integral_constant<int, 1>{}, g);
                flush();
            }
            scan_all(all, 64 * wv);
        } else {
#pragma unroll 1
            for (int k = 0; k < K; ++k) {
                const int x_first = 64 * (wv * K + k);
                bool all;
                next_stamp();
                const int total = lay_out(x_first + lane, K == 1 ? scale0 : (int)scales[min(x_first + lane, N - 1)], 0,
                                          stamp * 64 + (unsigned)lane, all);
                const int start = last_start;
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
                        e[u] = list_entry(i < total ? __umul24((unsigned)x_first + src[u], (unsigned)M) + (unsigned)(i - from[u]) : 0u);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) jy[u] = info[e[u] & 1023u];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = i0 + 64 * u + lane;
                        look(i < total, jx[u], jy[u], e[u], x_first + (int)src[u], i - from[u]);
                    }
                };
                for (int i0 = 0; i0 < total; i0 += 256) {
                    if (total - i0 > 128) brackets(std::integral_constant<int, 4>{}, i0);
                    else if (total - i0 > 64) brackets(std::integral_constant<int, 2>{}, i0);
                    else brackets(std::integral_constant<int, 1>{}, i0);
                    flush();
                }
                scan_all(all, x_first);
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (n_passed) score(0, n_passed);
        group_best();
        if (hi >= 0) break;
        // ---- reverse ranks mi .. mj: the nodes inside swap the hops in and out, two hops are new
        const int mi = lo / N, mj = lo - mi * N;
        const int n_before = t[mi - 1], n_first = t[mi], n_last = t[mj], n_after = t[mj + 1];
        const int h_first = GROUP ? first_hop : mat(n_before, n_last), h_after = GROUP ? after_hop : mat(n_first, n_after);
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
    if (GROUP) {
        __syncthreads();
        if (lane == 0) group->word[wv] = sum;
        __syncthreads();
        sum = 0;
        for (int i = 0; i < WAVES; ++i) sum += group->word[i];
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
template <int E, int WAVES, bool ENTRIES>
__global__ __launch_bounds__(1024) void twoopt_sum_pruned_kernel(const int32_t* __restrict__ c, int N, int M, int lds_matrix,
                                                                 int waves, int restarts, int32_t* __restrict__ tours,
                                                                 int64_t* __restrict__ costs,
                                                                 int32_t* __restrict__ moves,
                                                                 const int32_t* __restrict__ skip_if_small, int left_over) {
    constexpr int K = WAVES > 1 ? 1 : E;                        // nodes per lane
    // when the exhaustive 16-bit kernel is launched beside this one, the matrix maximum decides which of them runs
    if (skip_if_small && skip_if_small[0] < (1 << 16)) return;
    if (left_over) {
        // behind the kernel that keeps pairs: only restarts that it left
        bool any = false;
        const int64_t first = WAVES > 1 ? blockIdx.x : (int64_t)blockIdx.x * waves;
        for (int i = 0; i < (WAVES > 1 ? 1 : waves); ++i) any = any || costs[min(first + i, (int64_t)restarts - 1)] < 0;
        if (!any) return;
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int largest[16];
    __shared__ GroupWords<WAVES> group;
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
            const int scale = make_list<E>(c, N, x, M, lists + (size_t)x * M, counts + (size_t)x * kBuckets,
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
    if (r >= restarts || (left_over && costs[r] >= 0)) return;
    const int applied = left_over ? moves[r] : 0;
    const int mine = WAVES > 1 ? 0 : wv, part = WAVES > 1 ? wv : 0;
    unsigned char* order_mem = rest + (size_t)mine * (order_bytes(N) + wave_bytes(kRoom));
    unsigned char* wave_mem = WAVES > 1 ? order_mem + group_order_bytes(N) + (size_t)part * group_wave_bytes(kRoom, ENTRIES)
                                        : order_mem + order_bytes(N);
    const int scale0 = (int)scales[min(64 * part + lane, N - 1)];
    if (in_lds)
        descend<WAVES, K, kRoom, ENTRIES>(LdsMatrix{m16, N}, N, lists, M, counts, scale0, scales, order_mem, wave_mem, &group, part, lane, applied,
                          tours + r * N, costs + r, moves + r);
    else
        descend<WAVES, K, kRoom, ENTRIES>(CallersMatrix{c, N}, N, lists, M, counts, scale0, scales, order_mem, wave_mem, &group, part, lane, applied,
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

// More than 80 scalar registers leave room for fewer wavefronts than the vector registers do (N = 1024, 512 restarts, two
// workgroups per unit: 84 of them 22.0 ms, 78 17.2).
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_num_sgpr(80))) void twoopt_sum_pruned_group_kernel(const int32_t* __restrict__ c, int N, int M,
                                                                             const uint32_t* __restrict__ lists,
                                                                             const uint16_t* __restrict__ counts,
                                                                             int32_t* __restrict__ tours,
                                                                             int64_t* __restrict__ costs,
                                                                             int32_t* __restrict__ moves) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ GroupWords<WAVES> group;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    if (costs[r] >= 0) return;                                  // only restarts that the kernel that keeps pairs left
    const int scale = (int)counts[(size_t)min(64 * wv + lane, N - 1) * kBuckets + kBuckets - 1];
    descend<WAVES, 1, kGroupRoom, true>(CallersMatrix{c, N}, N, lists, M, counts, scale, nullptr, smem,
                                  smem + group_order_bytes(N) + wv * group_wave_bytes(kGroupRoom, true), &group, wv, lane, moves[r],
                                  tours + r * N, costs + r, moves + r);
}

template <int E, int WAVES, bool ENTRIES>
hipError_t launch_lds(const int32_t* c, int N, const LdsPlan& plan, int restarts, int32_t* tours, int64_t* costs,
                      int32_t* moves, const int32_t* skip_if_small, bool left_over, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute((const void*)twoopt_sum_pruned_kernel<E, WAVES, ENTRIES>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan.bytes);
    if (e != hipSuccess) return e;
    const int grid = WAVES > 1 ? restarts : (restarts + plan.waves - 1) / plan.waves;
    hipLaunchKernelGGL((twoopt_sum_pruned_kernel<E, WAVES, ENTRIES>), dim3(grid), dim3(64 * (plan.waves > 8 ? plan.waves : 8)), plan.bytes,
                       s, c, N, plan.M, plan.lds_matrix, plan.waves, restarts, tours, costs, moves, skip_if_small, left_over ? 1 : 0);
    return hipGetLastError();
}

template <int E>
hipError_t launch_waves(const int32_t* c, int N, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        const int32_t* skip_if_small, bool left_over, hipStream_t s) {
    // A wave's own instructions bound a sweep, so more of them than the 64 nodes each would need are the faster as long as the unit has
    // room (4 / 8 / 12 / 16 waves: N = 150, 200 restarts 612 / 579 / 610 / 650 us; N = 256, 200 restarts 1526 / 1335 / 1319 / 1550; two
    // restarts per unit: N = 150, 500 restarts 696 / 723 / 876 / 1230).
    constexpr int kOne = 8, kTwo = 4;
    // Two restarts per unit above N = 208: what passes is noted by its place, so that the lists have room for four to six partners more
    // per node (with the entry / by place: N = 200, 300 restarts 1082 / 1091 us, zones of equal costs 425 / 439; N = 225 1411 / 1354, zones
    // 484 / 498; N = 250 2048 / 1856; N = 255, whose lists would be too short for two at a time, zones 898 / 580).
    const bool places = E == 4 && N > 208;
    auto state = [&](int waves, bool entries) { return group_order_bytes(N) + waves * group_wave_bytes(kRoom, entries); };
    const LdsPlan plan = lds_plan(N, restarts, order_bytes(N), Groups{2, false, {kOne, kTwo}, {state(kOne, true), state(kTwo, !places)}});
    if constexpr (E > 2) {                                      // N <= 128 comes here with more than 1024 restarts
        if (plan.together && plan.waves == kOne)
            return launch_lds<E, kOne, true>(c, N, plan, restarts, tours, costs, moves, skip_if_small, left_over, s);
        if constexpr (E == 4)
            if (plan.together && places)
                return launch_lds<E, kTwo, false>(c, N, plan, restarts, tours, costs, moves, skip_if_small, left_over, s);
        if (plan.together) return launch_lds<E, kTwo, true>(c, N, plan, restarts, tours, costs, moves, skip_if_small, left_over, s);
    }
    return launch_lds<E, 1, false>(c, N, plan, restarts, tours, costs, moves, skip_if_small, left_over, s);
}

// Where the lists lie in `room`, and how long they are.
void partner_lists_at(int N, void* room, int& M, const uint32_t*& lists, const uint16_t*& counts) {
    M = group_list(N);
    lists = (const uint32_t*)room;
    counts = (const uint16_t*)(lists + (size_t)N * M);
}

template <int WAVES>
hipError_t launch_group(const int32_t* c, int N, void* room, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        hipStream_t s) {
    int M;
    const uint32_t* lists;
    const uint16_t* counts;
    partner_lists_at(N, room, M, lists, counts);
    const size_t lds = group_order_bytes(N) + WAVES * group_wave_bytes(kGroupRoom, true);
    const hipError_t e = hipFuncSetAttribute((const void*)twoopt_sum_pruned_group_kernel<WAVES>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((twoopt_sum_pruned_group_kernel<WAVES>), dim3(restarts), dim3(64 * WAVES), lds, s, c, N, M, lists,
                       counts, tours, costs, moves);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_partner_lists(const int32_t* c, int N, void* room, int& M, const uint32_t*& lists, const uint16_t*& counts,
                                hipStream_t s) {
    partner_lists_at(N, room, M, lists, counts);
    hipLaunchKernelGGL(partner_lists_kernel, dim3((N + 3) / 4), dim3(256), 0, s, c, N, M, (uint32_t*)lists, (uint16_t*)counts);
    return hipGetLastError();
}

hipError_t launch_2opt_sum_pruned(const int32_t* c, int N, void* room, int restarts, int32_t* tours, int64_t* costs,
                                  int32_t* moves, const int32_t* skip_if_small, bool left_over, hipStream_t s) {
    if (N <= 128) return launch_waves<2>(c, N, restarts, tours, costs, moves, skip_if_small, left_over, s);
    if (N <= 192) return launch_waves<3>(c, N, restarts, tours, costs, moves, skip_if_small, left_over, s);
    if (N <= 256) return launch_waves<4>(c, N, restarts, tours, costs, moves, skip_if_small, left_over, s);
    if (!left_over) return hipErrorInvalidValue;                // the kernel that keeps pairs is in front of it at any number of restarts
    // at least a wave per 64 nodes; more where the compute units have room for them (a wave per 64 nodes / 8 / 12 / 16 waves: N = 300, 250
    // restarts 1782 / 1590 / 1534 / 1620 us, 500 restarts 1982 / 1867 / 2022 / 2300, 1000 restarts 2523 / 3219 / 3786; N = 512, 250
    // restarts 3621 / - / 3340 / 3330, 500 restarts 4431 / - / 4605 / 4900)
    if (restarts <= 256) {
        if (N <= 768) return launch_group<12>(c, N, room, restarts, tours, costs, moves, s);
    } else if (restarts <= 512) {
        if (N <= 512) return launch_group<8>(c, N, room, restarts, tours, costs, moves, s);
    }
    if (N <= 320) return launch_group<5>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 384) return launch_group<6>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 448) return launch_group<7>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 512) return launch_group<8>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 640) return launch_group<10>(c, N, room, restarts, tours, costs, moves, s);
    if (N <= 768) return launch_group<12>(c, N, room, restarts, tours, costs, moves, s);
    return launch_group<16>(c, N, room, restarts, tours, costs, moves, s);
}

}  // namespace cc
