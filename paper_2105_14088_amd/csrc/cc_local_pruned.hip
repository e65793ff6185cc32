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
// What bounds it: a sweep is a chain of phases, each a few LDS look-ups deep, with a barrier behind it.  Up to 512 restarts 4 to 16
// wavefronts share a restart: its candidates, 64 at a time in turn, and then both halves of the pairs that passed, 32 pairs at a
// time.  N = 150, 512 restarts (8 wavefronts each, two restarts per compute unit): 16900 clocks a sweep and 690 vector instructions per
// wavefront, VALU 57 % and LDS 23 % of the time busy, the wavefronts waiting for half of it (a wavefront per 64 nodes, each of which
// scored what its own nodes had passed: 1.58 ms, now 1.08).  There the matrix is in LDS as a triangle; a look-up through the cache costs a line
// per lane, which bounds N > 256 (N = 700, before only the moves with a bracket of their own were looked up: 16.1 ms, now 11.3).  One
// wavefront per restart: instruction issue.
// Against the general kernel (cc_local.hip), 2-opt and insertion: N = 32, 1024 restarts 381 -> 165 us; N = 100, 512 restarts
// 4.9 -> 0.62 ms; N = 150, 512 restarts 13.1 -> 1.1 ms; N = 292, 228 restarts 53 -> 2.3 ms; N = 1000, 20 restarts 1371 -> 23 ms;
// against the exhaustive multi-rank kernel at N = 256, 250 restarts 9.6 -> 2.0 ms.  Matrices of few values are handed over to
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
constexpr int kNodesLeft = 1 << 16;     // in GroupWords::laid_out: nodes of the wavefront had no room

// LDS of one restart: per node {hop in << 10 | rank, hop out} and {longest hop, largest R}, R of the segments of length
// 1, 2, 3 by first rank, the nodes of the ranks -1 .. N
__host__ __device__ constexpr size_t local_order_bytes(int N) {
    return ((size_t)N * 28 + (size_t)(N + 2) * 2 + 15) & ~(size_t)15;
}

// and of the wavefronts that share a restart: the first candidate's place by node, the passed candidates (of 128 per wavefront and a
// rest), ROOM candidates for each that owns nodes.  N <= 256: a passed candidate by its place in the lists, which are in LDS too;
// above with the list's entry.
constexpr int group_passed(int waves) { return 160 * waves; }
constexpr int passed_bytes(int room) { return room == kRoom ? 4 : 8; }
__host__ __device__ constexpr size_t group_bytes(int N, int room, int waves) {
    return local_order_bytes(N) + (((size_t)N * 2 + 7) & ~(size_t)7) + (size_t)group_passed(waves) * passed_bytes(room) +
           (size_t)((N + 63) / 64) * room * 2;
}
template <int WAVES>
struct GroupWords {
    unsigned long long key[4];              // of the best move, used in turn: value, id
    unsigned long long scanned[WAVES];      // nodes that are scanned against every node, a bit each
    int laid_out[WAVES];                    // candidates
    int word[WAVES];
    int passed[2];                          // candidates, used in turn
};

// One descent of WAVES wavefronts; wave `wv` owns the nodes 64 * (wv * K + k) + lane.  Several wavefronts share the candidates of
// all nodes, and then what is scored of them.
template <int WAVES, int K, int ROOM, bool WITH_2OPT, typename COUNT, class MAT>
__device__ __forceinline__ void descend(const MAT mat, int N, const uint32_t* __restrict__ lists, int M,
                                        const COUNT* __restrict__ counts, int scale0, const uint16_t* scales,
                                        unsigned char* order_mem, GroupWords<WAVES>* group, int wv, int lane,
                                        int32_t* __restrict__ tour, int64_t* __restrict__ cost_out, int32_t* __restrict__ moves_out) {
    constexpr int THREADS = 64 * WAVES;
    constexpr bool GROUP = WAVES > 1;
    static_assert(!GROUP || K == 1, "a group's wave owns 64 nodes at most");
    uint2* info = (uint2*)order_mem;                           // [N] by node
    int2* value = (int2*)(info + N);                           // [N] by node
    int32_t* saved = (int32_t*)(value + N);                    // [3][N] R by first rank
    uint16_t* t = (uint16_t*)(saved + 3 * N) + 1;              // t[-1] = t[N-1], t[N] = t[0]
    // one wavefront: [ROOM] stamp << 6 | lane; [kPassed] x | place << 10, as in the 2-opt kernel
    unsigned char* wave_mem = order_mem + local_order_bytes(N);
    uint16_t* owner = (uint16_t*)wave_mem;
    uint32_t* passed = (uint32_t*)(wave_mem + ROOM * 2);
    // several: the first candidate's place by node, the passed ones as above or as {x, cost << 10 | y}, `owner` of every wave with nodes
    constexpr bool ENTRIES = passed_bytes(ROOM) == 8;
    uint16_t* starts = (uint16_t*)wave_mem;
    unsigned char* shared = wave_mem + ((N * 2 + 7) & ~7);
    uint16_t* owners = (uint16_t*)(shared + group_passed(WAVES) * passed_bytes(ROOM));
    const bool owns = 64 * wv * K < N;
    if (GROUP) {
        passed = (uint32_t*)shared;
        owner = owners + (owns ? wv : 0) * ROOM;
    }
    const int tid = wv * 64 + lane;
    auto sync = [] { if (WAVES > 1) __syncthreads(); else __builtin_amdgcn_wave_barrier(); };
    auto hop_in = [](uint2 w) { return (int)(w.x >> 10); };
    auto hop_out = [](uint2 w) { return (int)w.y; };
    auto rank_of = [](uint2 w) { return (int)(w.x & 1023u); };
    const int longest = min(3, N - 3);                         // of the segments

    int t0[K], applied = 0, turn = 0;
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
    if (owns)
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
    if (GROUP) {
        // over the wavefronts of this restart alone: the workgroup's others have ended, which a plain barrier allows and a
        // workgroup-wide reduction of the library need not
        if (lane == 0) group->word[wv] = search ? 1 : 0;
        if (tid < 4) group->key[tid] = ~0ull;
        if (tid < 2) group->passed[tid] = 0;
        __syncthreads();
        search = __ballot(group->word[min(lane, WAVES - 1)] == 0) == 0;
    }

    // the move a lane remembers: a pair and how it is used.  Use: length of the segment x ends (0: a 2-opt move) << 2 |
    // x is its last rank << 1 | y stands behind the gap (2-opt: the edges before x and y).  At first the nearest partner
    // of its first node.
    int rx = min(64 * wv * K + lane, N - 1), ry = (int)(lists[(size_t)rx * M] & 1023u);
    int r_use = WITH_2OPT ? 0 : 4, r_value = owns ? 0 : kNone;
    unsigned stamp = 0;
    int list = 0;                                              // which of group->passed counts
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
            if (GROUP) {
                if (lane == 0) {
                    atomicMin(&group->key[turn & 3], ((unsigned long long)(unsigned)(h + (1 << 30)) << 32) | (unsigned)l);
                    group->key[(turn + 2) & 3] = ~0ull;          // read by all before the last barrier, used again after the next
                }
                __syncthreads();
                const unsigned long long key = group->key[turn & 3];
                h = __builtin_amdgcn_readfirstlane((int)(key >> 32)) - (1 << 30);
                l = __builtin_amdgcn_readfirstlane((int)(unsigned)key);
                ++turn;
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
        // scores a passed pair in half of its roles, one pair per lane: the ten insertions of a segment that x ends beside y, and the
        // 2-opt move behind x and y, or (second half) before them; the other half is that of y and x.  All look-ups are in flight
        // together.  Where a look-up costs a cache line, only the moves whose own bracket at this pair passes make one: the best move has
        // such a bracket at one of its pairs (N = 400, 500 restarts 9.9 -> 7.1 ms, N = 1000, 300 restarts 78 -> 51 ms).
        auto score = [&](bool live, int x, int y, int cost, bool second) {
            constexpr int kOut = 1 << 28;                      // of a move that does not exist or is not looked up: no value below 0
            const uint2 ix = info[x], iy = info[y];
            const int p = rank_of(ix), q = rank_of(iy);
            live = live && x != y;
            const int most = min(hi, -1), behind = t[q + 1], before = t[q - 1];
            int least[11], entry[11];                          // a move's value without the entry of its other edge, and that
            auto look_up = [&](int i, bool ok, int value, decltype(mat.row(0)) row, int z) {
                ok = ok && (!MAT::kScattered || value + cost <= most);
                least[i] = ok ? value : kOut;
                entry[i] = mat.raw(ok, row, z);
            };
            // the five segments that x ends: what they save, the node at their other end
            int less[5];
            decltype(mat.row(0)) other[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                const int L = i == 0 ? 1 : (i + 3) >> 1, last = i == 2 || i == 4 ? 1 : 0, first = max(last ? p - L + 1 : p, 0);
                less[i] = saved[(L - 1) * N + first];          // of a segment that does not exist: so little that none counts
                other[i] = mat.row(t[last ? first : min(p + L - 1, N - 1)]);
            }
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int g = side ? (q ? q - 1 : N - 1) : q, z = side ? before : behind;
                const int apart = g - p, more = cost - (side ? hop_in(iy) : hop_out(iy));
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const int L = i == 0 ? 1 : (i + 3) >> 1, last = i == 2 || i == 4 ? 1 : 0;
                    // the gaps first - 1 .. first + L - 1 are those of the segment itself
                    look_up(5 * side + i, live & ((unsigned)(apart + (last ? L : 1)) > (unsigned)L), more - less[i], other[i], z);
                }
            }
            if (WITH_2OPT) {
                const int d = p < q ? q - p : p - q, f = second ? hop_in(ix) + hop_in(iy) : hop_out(ix) + hop_out(iy);
                look_up(10, live & (d >= 2) & (d <= N - 2), cost - f, mat.row(t[second ? p - 1 : p + 1]), second ? before : behind);
            } else {
                least[10] = kOut;
                entry[10] = 0;
            }
            // without this each entry was waited for before the next was asked for
            asm volatile("" : "+v"(entry[0]), "+v"(entry[1]), "+v"(entry[2]), "+v"(entry[3]), "+v"(entry[4]), "+v"(entry[5]), "+v"(entry[6]),
                         "+v"(entry[7]), "+v"(entry[8]), "+v"(entry[9]), "+v"(entry[10]));
            int bd = kNone, bid = kNone, buse = 0;
            auto better = [&](int i, int id, int use) {
                const int delta = least[i] + mat.cost(entry[i]);
                const bool ok = (delta < bd) | ((delta == bd) & (id < bid));
                bd = ok ? delta : bd;
                bid = ok ? id : bid;
                buse = ok ? use : buse;
            };
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int g = side ? (q ? q - 1 : N - 1) : q, at = (int)__umul24((unsigned)p, (unsigned)N) + g;
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const int L = i == 0 ? 1 : (i + 3) >> 1, last = i == 2 || i == 4 ? 1 : 0;
                    const int variant = L == 1 ? 0 : 2 * L - 3 + (last != side ? 1 : 0);
                    better(5 * side + i, at + (N * (1 + variant) - (last ? L - 1 : 0)) * N, (L << 2) | (last << 1) | side);
                }
            }
            if (WITH_2OPT) {
                // ranks lo_r .. hi_r reversed, or around rank 0 those that are left
                const int lo_r = min(p, q) + (second ? 0 : 1), hi_r = max(p, q) - (second ? 1 : 0);
                better(10, second ? (lo_r ? lo_r * N + hi_r : (hi_r + 1) * N + N - 1) : lo_r * N + (hi_r + 1 < N ? hi_r : N - 1), second ? 1 : 0);
            }
            if (bd < kOut / 2) take(bd, bid, x, y, buse);
        };
        // the passed pairs from .. from + n, at most 32, both halves side by side
        auto score_listed = [&](int from, int n) {
            const int i = lane >> 1, at = from + min(i, n - 1);
            const bool live = i < n, second = lane & 1;
            int x, y, cost;
            if (GROUP && ENTRIES) {
                const uint2 w = ((const uint2*)shared)[at];
                x = (int)w.x;
                y = (int)(w.y & 1023u);
                cost = (int)(w.y >> 10);
            } else {
                const uint32_t w = passed[at];
                const int place = (int)(w >> 10);
                x = (int)(w & 1023u);
                const bool listed = place < M;
                const uint32_t e = lists[__umul24((unsigned)x, (unsigned)M) + (unsigned)(listed ? place : 0)];
                y = listed ? (int)(e & 1023u) : place - M;
                cost = (int)(e >> 10);
                if (__ballot(!listed)) cost = listed ? cost : mat(x, y);
            }
            score(live, second ? y : x, second ? x : y, cost, second);
        };
        // notes the pairs that passed, U per lane
        auto pass = [&](auto u_const, const bool* ok, const int* x, const uint32_t* e, const int* place) {
            constexpr int U = decltype(u_const)::value;
            unsigned long long mask[U];
            int n = 0, from = n_passed;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mask[u] = __ballot(ok[u]);
                n += __popcll(mask[u]);
            }
            if (GROUP) {
                if (!n) return;
                from = __builtin_amdgcn_readfirstlane(lane == 0 ? atomicAdd(&group->passed[list], n) : 0);
            }
            n_passed += n;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int at = from + lanes_below(mask[u]);
                if (ok[u]) {
                    if (GROUP && ENTRIES) ((uint2*)shared)[at] = make_uint2((unsigned)x[u], e[u]);
                    else passed[at] = (unsigned)x[u] | ((unsigned)place[u] << 10);
                }
                from += __popcll(mask[u]);
            }
            if (!GROUP) {
                __builtin_amdgcn_wave_barrier();
                while (n_passed >= 32) {
                    n_passed -= 32;
                    score_listed(n_passed, 32);
                }
                __builtin_amdgcn_wave_barrier();
            }
        };
        // the node with the larger value looks at the pair
        auto worth_scoring = [&](int x, int2 vx, int y, int2 vy, int twice) {
            const int mx = max(vx.x, vx.y), my = max(vy.x, vy.y);
            int most = max(vx.x + vy.y, vx.y + vy.x);
            if (WITH_2OPT) most = max(most, vx.x + vy.x);
            return (mx > my || (mx == my && x < y)) && twice - most <= D;
        };
        // ---- how far the threshold of node x (one per lane) reaches; the candidates of 64 nodes end to end, of those that are left.
        // Returns where they end, with kNodesLeft if nodes are left; all: x is scanned against every node instead, its partners are beyond
        // the list; left: not 0, for another time, they are beyond the room (a list is shorter than the room: of the nodes that are
        // left one fits).
        auto lay_out = [&](int x, int scale, int& start, bool& all, int& left) {
            const int2 vx = value[min(x, N - 1)];
            const int reach = max(vx.x, vx.y) + (D >> 1);
            const int bucket = bucket_of(max(reach, 0), scale);
            int count = (int)counts[(size_t)min(x, N - 1) * kBuckets + max(0, min(bucket, kBuckets - 2))];
            count = bucket >= kBuckets - 1 ? N - 1 : count;
            count = left && reach >= 0 && bucket >= 0 ? count : 0;
            left = 0;
            all = count > M;
            count = all ? 0 : count;
            int end = wave_prefix_sum(count);
            int total = __builtin_amdgcn_readlane(end, 63);
            if (total > ROOM) {
                const bool out = end > ROOM;
                left = out ? count : 0;
                count = out ? 0 : count;
                total = wave_max(out ? 0 : end) | kNodesLeft;
            }
            start = end - count;
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
            return total;
        };
        // node nx against the nodes from y0 on, 64 U at a time
        auto scan = [&](auto u_const, int nx, int y0) {
            constexpr int U = decltype(u_const)::value;
            const int2 jx = value[nx];
            int x[U], place[U];
            uint32_t e[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int y = min(y0 + 64 * u + lane, N - 1);
                e[u] = ((unsigned)mat(nx, y) << 10) | (unsigned)y;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int y = y0 + 64 * u + lane;
                x[u] = nx;
                place[u] = M + y;
                ok[u] = y < N && worth_scoring(nx, jx, y, value[min(y, N - 1)], 2 * (int)(e[u] >> 10));
            }
            pass(u_const, ok, x, e, place);
        };
        if constexpr (GROUP) {
            // ---- an equal share of all nodes' candidates for every wave, 64 at a time.  What the room does not hold follows in a turn of
            // its own: with barriers between them, scans of those nodes against every node took longer than they had within one
            // wavefront (32 zones of equal costs, N = 1000, 16 restarts 61 -> 91 ms when the candidates came to be shared, now 43; 16
            // zones 87 -> 123, now 52; hosts and racks without noise 37 -> 34, now 20).
            int left = 64 * wv + lane < N ? 1 : 0, words;      // in vector registers: the scalar ones are spilled as it is
            do {
                bool all = false;
                if (owns) {
                    int start;
                    const int x = 64 * wv + lane, total = lay_out(x, scale0, start, all, left);
                    if (x < N) starts[x] = (uint16_t)start;
                    if (lane == 0) group->laid_out[wv] = total;
                } else if (lane == 0) {
                    group->laid_out[wv] = 0;
                }
                const unsigned long long scanned_here = __ballot(all);
                if (lane == 0) group->scanned[wv] = scanned_here;
                __syncthreads();
                words = lane < WAVES ? group->laid_out[lane] : 0;
                const int laid_out = words & (kNodesLeft - 1);
                asm volatile("" : "+v"(left), "+v"(words));
                const int upto = wave_prefix_sum((laid_out + 63) >> 6);          // of the waves up to this lane's
                const int listed = __builtin_amdgcn_readlane(upto, 63);
                const int chunks = (N + 63) >> 6, scans_upto = wave_prefix_sum(lane < WAVES ? __popcll(group->scanned[lane]) : 0);
                const int blocks = listed + __builtin_amdgcn_readlane(scans_upto, 63) * chunks;
                auto brackets = [&](auto u_const, int g0) {
                    constexpr int U = decltype(u_const)::value;
                    unsigned src[U];
                    int from[U], place[U], first[U], live[U], x[U];
                    int2 jx[U], jy[U];
                    uint32_t e[U];
                    bool ok[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int g = g0 + WAVES * u, w = __popcll(__ballot(upto <= g));         // whose candidates these are
                        const int i0 = 64 * (g - (w ? __builtin_amdgcn_readlane(upto, w - 1) : 0));
                        first[u] = 64 * w;
                        live[u] = __builtin_amdgcn_readlane(laid_out, w) - i0;
                        place[u] = i0 + lane;
                        src[u] = owners[w * ROOM + place[u]];
                    }
                    // marks of earlier layouts are smaller than this one's, and the first of the 64 is always marked
#pragma unroll
                    for (int u = 0; u < U; ++u) src[u] = min((unsigned)first[u] + (wave_prefix_max(src[u]) & 63u), (unsigned)N - 1);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        from[u] = starts[src[u]];
                        jx[u] = value[src[u]];
                        x[u] = (int)src[u];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        place[u] -= from[u];                         // in the list of x
                        e[u] = lists[lane < live[u] ? __umul24(src[u], (unsigned)M) + (unsigned)place[u] : 0u];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) jy[u] = value[e[u] & 1023u];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        ok[u] = lane < live[u] && worth_scoring(x[u], jx[u], (int)(e[u] & 1023u), jy[u], 2 * (int)(e[u] >> 10));
                    pass(u_const, ok, x, e, place);
                };
                auto scan_block = [&](int g) {
                    const int i = (g - listed) / chunks, w = __popcll(__ballot(scans_upto <= i));
                    const unsigned long long nodes = group->scanned[w];
                    const int skip = i - (w ? __builtin_amdgcn_readlane(scans_upto, w - 1) : 0);
                    const unsigned long long at = __ballot((nodes >> lane & 1) && lanes_below(nodes) == skip);
                    scan(std::integral_constant<int, 1>{}, 64 * w + (int)__builtin_ctzll(at), 64 * (g - listed - i * chunks));
                };
                // two blocks for each wave at a time; then what passed is scored if it is enough to give every wave 32 pairs, or the last
                int g = wv;
                do {
                    if (g + WAVES < listed) {
                        brackets(std::integral_constant<int, 2>{}, g);
                    } else {
                        if (g < listed) brackets(std::integral_constant<int, 1>{}, g);
                        else if (g < blocks) scan_block(g);
                        if (g + WAVES < blocks) scan_block(g + WAVES);
                    }
                    g += 2 * WAVES;
                    const bool more = g - wv < blocks;
                    __syncthreads();
                    const int pairs = __builtin_amdgcn_readfirstlane(group->passed[list]);
                    if (more && pairs <= 32 * WAVES) {
                        __syncthreads();
                        continue;
                    }
                    if (tid == 0) group->passed[list ^ 1] = 0;       // for the next ones
                    list ^= 1;
                    for (int i0 = 32 * wv; i0 < pairs; i0 += 32 * WAVES) score_listed(i0, pairs - i0);
                    if (more) __syncthreads();
                } while (g - wv < blocks);
            } while (__ballot(words >= kNodesLeft));
        } else {
#pragma unroll 1
            for (int k = 0; k < K; ++k) {
                const int x_first = 64 * (wv * K + k), x = x_first + lane;
                int start;
                bool all;
                int left = x < N ? 1 : 0;
                const int total = lay_out(x, K == 1 ? scale0 : (int)scales[min(x, N - 1)], start, all, left) & (kNodesLeft - 1);
                __builtin_amdgcn_wave_barrier();
                // ---- brackets, U times 64 candidates with their LDS and list reads in flight together
                auto brackets = [&](auto u_const, int i0) {
                    constexpr int U = decltype(u_const)::value;
                    unsigned src[U];
                    int from[U], nx[U], place[U];
                    int2 jx[U], jy[U];
                    uint32_t e[U];
                    bool ok[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) src[u] = owner[i0 + 64 * u + lane];
#pragma unroll
                    for (int u = 0; u < U; ++u) src[u] = wave_prefix_max(src[u]) & 63u;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        from[u] = __builtin_amdgcn_ds_bpermute((int)(src[u] << 2), start);
                        nx[u] = x_first + (int)src[u];
                        jx[u] = value[min(nx[u], N - 1)];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        place[u] = i0 + 64 * u + lane - from[u];
                        e[u] = lists[i0 + 64 * u + lane < total ? __umul24((unsigned)nx[u], (unsigned)M) + (unsigned)place[u] : 0u];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) jy[u] = value[e[u] & 1023u];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        ok[u] = i0 + 64 * u + lane < total &&
                                worth_scoring(nx[u], jx[u], (int)(e[u] & 1023u), jy[u], 2 * (int)(e[u] >> 10));
                    pass(u_const, ok, nx, e, place);
                };
                for (int i0 = 0; i0 < total; i0 += 256) {
                    if (total - i0 > 128) brackets(std::integral_constant<int, 4>{}, i0);
                    else if (total - i0 > 64) brackets(std::integral_constant<int, 2>{}, i0);
                    else brackets(std::integral_constant<int, 1>{}, i0);
                }
                unsigned long long rest = __ballot(all || left != 0);
                while (rest) {
                    const int nx = x_first + (int)__builtin_ctzll(rest);
                    rest &= rest - 1;
                    for (int y0 = 0; y0 < N; y0 += 256) scan(std::integral_constant<int, 4>{}, nx, y0);
                }
            }
            if (n_passed) score_listed(0, n_passed);
        }
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

// Whether the kernel behind this one does the work (see TieHandover).  Where many partners cost the same, most pairs pass
// their brackets in one role or another, and scoring them costs more than the exhaustive sweeps.
__device__ __forceinline__ bool hand_over(const TieHandover& ties, int tied, int level, int highest) {
    if (!ties.flags) return false;
    const bool hand = (tied > ties.most || level > ties.most_level) && (!ties.to_16bit || highest < (1 << 16));
    if (blockIdx.x == 0 && threadIdx.x == 0) ties.flags[0] = hand == ties.to_16bit ? 0 : 1 << 16;
    return hand;
}

// N <= 256, N <= 64 E, as twoopt_sum_pruned_kernel: lists (and the matrix, or one triangle of it) in LDS, for `waves` restarts of one
// wavefront each or (WAVES > 1) one restart of WAVES wavefronts.
template <int E, int WAVES, bool WITH_2OPT>
__global__ __launch_bounds__(1024) void local_pruned_kernel(const int32_t* __restrict__ c, int N, int M, int lds_matrix,
                                                            int waves, TieHandover ties, int restarts,
                                                            int32_t* __restrict__ tours, int64_t* __restrict__ costs,
                                                            int32_t* __restrict__ moves) {
    constexpr int K = WAVES > 1 ? 1 : E;                       // nodes per lane
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int largest[16], tied[16], level[16];
    __shared__ GroupWords<WAVES> group;
    uint32_t* lists = (uint32_t*)smem;                         // [N][M]
    unsigned char* counts = smem + (size_t)N * M * 4;          // [N][kBuckets]
    uint16_t* scales = (uint16_t*)(counts + (size_t)N * kBuckets);      // [N]
    uint16_t* m16 = scales + N;                                 // [N][N], or its lower triangle
    unsigned char* rest = smem + shared_bytes(N, M, lds_matrix);
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    {
        int* hist = (int*)rest + kBuckets * wv;                // where the restarts' state comes later
        int high = 0, tied_here = 0, level_here = 0;
        for (int x = wv; x < N; x += nw) {
            int row_max;
            const int scale = make_list<E>(c, N, x, M, lists + (size_t)x * M, counts + (size_t)x * kBuckets, hist, lane, row_max,
                                           [&](int y, int cost) {
                                               if (lds_matrix == 1) m16[x * N + y] = (uint16_t)cost;
                                               else if (lds_matrix && y <= x) m16[(x * x + x) / 2 + y] = (uint16_t)cost;
                                           });
            if (lane == 0) scales[x] = (uint16_t)scale;
            high = max(high, row_max);
            const unsigned char* upto = counts + (size_t)x * kBuckets;
            tied_here += upto[0];
            if (ties.to_16bit) {
                // a move to a cost that many partners have in common ties with many others, the row's largest cost is none to move to
                const int below = lane ? upto[2 * lane - 1] : 0, first = upto[2 * lane], second = upto[2 * lane + 1];
                level_here += wave_max(max(first < N - 1 ? first - below : 0, second < N - 1 ? second - first : 0));
            }
        }
        if (lane == 0) {
            largest[wv] = high;
            tied[wv] = tied_here;
            level[wv] = level_here;
        }
    }
    __syncthreads();
    int high = 0, tied_in_all = 0, level_in_all = 0;
    for (int w = 0; w < nw; ++w) {
        high = max(high, largest[w]);
        tied_in_all += tied[w];
        level_in_all += level[w];
    }
    high = __builtin_amdgcn_readfirstlane(high);
    if (hand_over(ties, __builtin_amdgcn_readfirstlane(tied_in_all), __builtin_amdgcn_readfirstlane(level_in_all), high)) return;
    if (wv >= waves) return;                                   // barriers below wait for the remaining wavefronts only
    const int in_lds = high < (1 << 16) ? lds_matrix : 0;
    const int64_t r = WAVES > 1 ? blockIdx.x : (int64_t)blockIdx.x * waves + wv;
    if (r >= restarts) return;
    const int mine = WAVES > 1 ? 0 : wv, part = WAVES > 1 ? wv : 0;
    unsigned char* order_mem = rest + (size_t)mine * (local_order_bytes(N) + wave_bytes(kRoom));
    const int scale0 = (int)scales[min(64 * part + lane, N - 1)];
    auto search = [&](const auto mat) {
        descend<WAVES, K, kRoom, WITH_2OPT>(mat, N, lists, M, counts, scale0, scales, order_mem, &group, part, lane, tours + r * N,
                                            costs + r, moves + r);
    };
    if (in_lds == 1) search(LdsMatrix{m16, N});
    else if (WAVES > 1 && in_lds) search(LdsTriangle{m16});
    else search(CallersMatrix{c, N});
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
    __shared__ GroupWords<WAVES> group;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    {
        const int x = threadIdx.x;
        const int tied = wave_sum(x < N ? (int)counts[(size_t)x * kBuckets] : 0);
        if (lane == 0) group.word[wv] = tied;
        __syncthreads();
        int tied_in_all = 0;
        for (int w = 0; w < WAVES; ++w) tied_in_all += group.word[w];
        if (hand_over(ties, __builtin_amdgcn_readfirstlane(tied_in_all), 0, 0)) return;
        __syncthreads();
    }
    const int scale = (int)counts[(size_t)min(64 * wv + lane, N - 1) * kBuckets + kBuckets - 1];
    descend<WAVES, 1, kGroupRoom, WITH_2OPT>(CallersMatrix{c, N}, N, lists, M, counts, scale, nullptr, smem, &group, wv, lane,
                                             tours + r * N, costs + r, moves + r);
}

template <int E, int WAVES, bool WITH_2OPT>
hipError_t launch_lds(const int32_t* c, int N, const LdsPlan& plan, const TieHandover& ties, int restarts, int32_t* tours,
                      int64_t* costs, int32_t* moves, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute((const void*)local_pruned_kernel<E, WAVES, WITH_2OPT>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan.bytes);
    if (e != hipSuccess) return e;
    const int grid = WAVES > 1 ? restarts : (restarts + plan.waves - 1) / plan.waves;
    hipLaunchKernelGGL((local_pruned_kernel<E, WAVES, WITH_2OPT>), dim3(grid), dim3(64 * (plan.waves > 8 ? plan.waves : 8)),
                       plan.bytes, s, c, N, plan.M, plan.lds_matrix, plan.waves, ties, restarts, tours, costs, moves);
    return hipGetLastError();
}

template <int E, bool WITH_2OPT>
hipError_t launch_waves(const int32_t* c, int N, const TieHandover& ties, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        hipStream_t s) {
    // Wavefronts for one restart (one / 4 / 8 / 12 / 16 of them): N = 20, 256 restarts 84 / 92 / 91 us; N = 48 246 / 206 / 207; N = 100
    // 1137 / 632 / 521 / 517 / 536; N = 150 2206 / 1113 / 834 / 825 / 853; N = 256 6617 / 2975 / 2175 / 1994 / 2007.  Two restarts
    // per unit at a time (one / 4 / 6 / 8): N = 48, 512 restarts 259 / 224 / 229 / 236; N = 100 1167 / 653 / 634 / 614; N = 200 4142 /
    // 2327 / 2151 / 2039; further restarts wait for a unit: N = 56, 768 restarts 319 (one) / 458; N = 100, 768 restarts 1195 / 1020,
    // 1024 1184 / 1135, 1536 1254 / 1610; N = 256, 1024 restarts, one at a time 8301 / 7619, 1536 8716 / 11094.
    constexpr int kMany = E > 2 ? 12 : E > 1 ? 8 : 4, kTwo = E > 1 ? 8 : 4, E2 = E > 2 ? 4 : E;
    auto state = [&](int waves) { return group_bytes(N, kRoom, waves); };
    const LdsPlan plan = lds_plan(N, restarts, local_order_bytes(N),
                                  Groups{N <= 32 ? 0 : N <= 64 ? 2 : 4, true, {kMany, kTwo}, {state(kMany), state(kTwo)}});
    if (!plan.together) return launch_lds<E, 1, WITH_2OPT>(c, N, plan, ties, restarts, tours, costs, moves, s);
    return plan.waves == kMany ? launch_lds<E2, kMany, WITH_2OPT>(c, N, plan, ties, restarts, tours, costs, moves, s)
                               : launch_lds<E2, kTwo, WITH_2OPT>(c, N, plan, ties, restarts, tours, costs, moves, s);
}

template <int WAVES, bool WITH_2OPT>
hipError_t launch_group(const int32_t* c, int N, void* room, const TieHandover& ties, int restarts, int32_t* tours, int64_t* costs, int32_t* moves,
                        hipStream_t s) {
    int M;
    const uint32_t* lists;
    const uint16_t* counts;
    hipError_t e = launch_partner_lists(c, N, room, M, lists, counts, s);
    if (e != hipSuccess) return e;
    const size_t lds = group_bytes(N, kGroupRoom, WAVES);
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
    // (5 / 8 / 12 / 16 wavefronts: N = 292, 256 restarts 3.60 / 2.82 / 2.55 / 2.36 ms, 512 restarts 4.27 / 3.57 / 4.94 / 4.65; N = 400 - /
    // 5.14 / 4.35 / 4.34, 512 restarts - / 6.4 / 8.4 / 8.4; N = 600 - / - / 9.3 / 8.7, 512 restarts - / - / 18.3 / 17.1)
    if (restarts <= 256) return launch_group<16, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
    if (N <= 512) return launch_group<8, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
    return launch_group<16, WITH_2OPT>(c, N, room, ties, restarts, tours, costs, moves, s);
}

}  // namespace

hipError_t launch_local_pruned(const int32_t* c, int N, bool with_2opt, void* room, const TieHandover& ties, int restarts,
                               int32_t* tours, int64_t* costs, int32_t* moves, hipStream_t s) {
    return with_2opt ? launch<true>(c, N, room, ties, restarts, tours, costs, moves, s)
                     : launch<false>(c, N, room, ties, restarts, tours, costs, moves, s);
}

}  // namespace cc
