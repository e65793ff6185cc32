// What the pruned descents (cc_2opt_sum_pruned.hip, cc_local_pruned.hip) share: partner lists by cost, matrix access,
// wave prefixes.
#pragma once
#include "cc_device.h"

namespace cc {
namespace pruned {
using namespace ccd;

constexpr int kCostMax = (1 << 21) - 1;
constexpr int kNone = 0x7fffffff;
constexpr int kBuckets = 128;           // of cost per node; the last one holds no partner
constexpr int kRoom = 512;              // candidates of 64 nodes laid out at a time, N <= 256
constexpr int kGroupRoom = 1024;        // and above
constexpr int kPassed = 320;            // candidates whose bracket passed: four times 64 and a rest below 64

// A cost on a logarithmic scale, 0 included: the bits of 2 cost + 1 as a float, its exponent from 0 on.
__device__ __forceinline__ unsigned key_of(int cost) { return __float_as_uint((float)(2 * cost + 1)) - (127u << 23); }
// The buckets of a node: 16, 8 or 4 per octave, the most with which its row's smallest to largest cost (22 octaves at most)
// fit.  Kept as first bucket | step << 12.  Sixteen per octave of the cost itself from the smallest on, everything beyond
// 8 octaves in the last, sent every node with one partner at cost 0 to the scan against every node: ring sum, one such
// partner per node, N = 256, 4096 restarts 79 ms, now 4.8; N = 512, 768 restarts 145 ms, now 6.2; N = 1000, 32 restarts 222 ms,
// now 10.5.
__device__ __forceinline__ int scale_of(int lowest, int highest) {
    const unsigned low = key_of(lowest), high = key_of(highest);
    int step = 0;
    while ((high >> (19 + step)) - (low >> (19 + step)) > kBuckets - 2) ++step;
    return (int)(low >> (19 + step)) | (step << 12);
}
// negative: below the row's smallest cost
__device__ __forceinline__ int bucket_of(int cost, int scale) { return (int)(key_of(cost) >> (19 + (scale >> 12))) - (scale & 4095); }

__device__ __forceinline__ int wave_prefix_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);      // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // row_bcast:31
    return v;
}
// unsigned: 0, what a lane without a source reads, is then the maximum's neutral element and a step is one instruction
__device__ __forceinline__ unsigned wave_prefix_max(unsigned v) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
    return v;
}
__device__ __forceinline__ int lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
}
__device__ __forceinline__ int entry(const int32_t* __restrict__ c, int N, int x, int y) {
    // 24-bit products and 32-bit offsets: a full-rate multiply, one address register
    const unsigned at = __umul24((unsigned)min(x, y), (unsigned)N) + (unsigned)max(x, y);
    return clampi(*(const int32_t*)((const char*)c + at * 4u), 0, kCostMax);
}
// Where a descent looks entries up: the caller's matrix, or both triangles as 16-bit entries in LDS.
struct CallersMatrix {
    static constexpr bool kScattered = true;                    // a cache line per lane that reads
    const int32_t* c;
    int N;
    __device__ __forceinline__ int operator()(int x, int y) const { return entry(c, N, x, y); }
    __device__ __forceinline__ int row(int x) const { return x; }
    __device__ __forceinline__ int above(int x, int y) const { return c[__umul24((unsigned)x, (unsigned)N) + (unsigned)y]; }      // raw, x < y
    // for several look-ups at once: what is read, and then the cost
    __device__ __forceinline__ int raw(bool ok, int row, int y) const {
        const unsigned at = __umul24((unsigned)min(row, y), (unsigned)N) + (unsigned)max(row, y);
        return *(const int32_t*)((const char*)c + (ok ? at : 0u) * 4u);
    }
    __device__ __forceinline__ int cost(int raw) const { return clampi(raw, 0, kCostMax); }
};
struct LdsMatrix {
    static constexpr bool kScattered = false;
    const uint16_t* m;
    int N;
    __device__ __forceinline__ int operator()(int x, int y) const { return m[__umul24((unsigned)x, (unsigned)N) + (unsigned)y]; }
    __device__ __forceinline__ const uint16_t* row(int x) const { return m + __umul24((unsigned)x, (unsigned)N); }
    __device__ __forceinline__ int above(int x, int y) const { return (*this)(x, y); }
    __device__ __forceinline__ int raw(bool, const uint16_t* row, int y) const { return row[(unsigned)y]; }
    __device__ __forceinline__ int cost(int raw) const { return raw; }
};
// the lower triangle with the diagonal, row by row: row x begins at (x x + x) / 2
struct LdsTriangle {
    static constexpr bool kScattered = false;
    const uint16_t* m;
    __device__ __forceinline__ int operator()(int x, int y) const {
        const unsigned high = (unsigned)max(x, y), low = (unsigned)min(x, y);
        return *(const uint16_t*)((const char*)m + (__umul24(high, high) + high) + 2u * low);
    }
    __device__ __forceinline__ int row(int x) const { return x; }
    __device__ __forceinline__ int raw(bool, int row, int y) const { return (*this)(row, y); }
    __device__ __forceinline__ int cost(int raw) const { return raw; }
};

// Makes the list of node x with one wavefront: list[0 .. M): cost << 10 | node, counts[b]: partners up to bucket b (the
// last one N - 1).  Returns the node's scale; row_max: the largest cost.  hist: kBuckets words of LDS of
// this wave.  each(y, cost): every entry of the row.
template <int E, typename COUNT, class EACH>
__device__ __forceinline__ int make_list(const int32_t* __restrict__ c, int N, int x, int M, uint32_t* list, COUNT* counts,
                                         int* hist, int lane, int& row_max, EACH each) {
    int cost[E], low = kNone, high = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int y = lane + 64 * k;
        const bool in = y < N && y != x;
        cost[k] = in ? entry(c, N, x, y) : -1;
        low = min(low, in ? cost[k] : kNone);
        high = max(high, cost[k]);
    }
    row_max = wave_max(high);
    const int scale = scale_of(wave_min(low), row_max);
    static_assert(kBuckets == 128, "two buckets per lane");
    hist[lane] = hist[lane + 64] = 0;
    __builtin_amdgcn_wave_barrier();
    int at[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        at[k] = cost[k] >= 0 ? atomicAdd(&hist[bucket_of(cost[k], scale)], 1) : 0;
        if (lane + 64 * k < N) each(lane + 64 * k, max(cost[k], 0));
    }
    __builtin_amdgcn_wave_barrier();
    const int here0 = hist[2 * lane], here1 = hist[2 * lane + 1], up_to = wave_prefix_sum(here0 + here1);
    counts[2 * lane] = (COUNT)(up_to - here1);
    counts[2 * lane + 1] = (COUNT)up_to;
    __builtin_amdgcn_wave_barrier();
    hist[2 * lane] = up_to - here1 - here0;
    hist[2 * lane + 1] = up_to - here1;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < E; ++k)
        if (cost[k] >= 0) {
            const int i = hist[bucket_of(cost[k], scale)] + at[k];
            if (i < M) list[i] = ((unsigned)cost[k] << 10) | (unsigned)(lane + 64 * k);
        }
    __builtin_amdgcn_wave_barrier();
    return scale;
}

// LDS the restarts of a workgroup share (N <= 256): lists, counts, scales, matrix
__host__ __device__ constexpr size_t shared_bytes(int N, int M, int lds_matrix) {
    return ((size_t)N * (M * 4 + kBuckets + 2 + (lds_matrix ? lds_matrix > 1 ? N + 1 : 2 * N : 0)) + 15) & ~(size_t)15;
}
__host__ __device__ constexpr size_t wave_bytes(int room) { return (size_t)room * 2 + kPassed * 4; }

// How the restarts of a search with N <= 256 share the chip.
struct LdsPlan {
    int waves;              // wavefronts with work per workgroup
    bool together;          // they share one restart
    int M, lds_matrix;      // list length; matrix in LDS, 2: one triangle of it
    size_t bytes;           // LDS per workgroup
};
// Wavefronts that share a restart.
struct Groups {
    int most_per_unit;      // restarts per compute unit up to which they do, 0: never
    bool triangle;          // the kernel can read one
    int waves[2];           // with one and with two workgroups per unit at a time
    size_t state[2];        // bytes of LDS they need then
};
// order_bytes: LDS of one restart's order.  Few restarts: a group of wavefronts each, one or two workgroups per compute unit at a
// time (a sweep then takes a fifth to a half of the time that one wavefront needs; four workgroups per unit at a time were slower:
// their lists are short and made four times).  Many: one wavefront per restart, up to 16 around one copy of the lists, but no more
// than keeps all 256 compute units busy.
// Lists of less than 32 partners would send too many nodes to the scan against every node; beyond 96 they add nothing.
inline LdsPlan lds_plan(int N, int restarts, size_t order_bytes, const Groups& groups) {
    constexpr size_t kLds = 160 * 1024 - 1024;
    LdsPlan p;
    const int per_unit = (restarts + 255) / 256;
    auto longest = [&](size_t room, int lds_matrix) {
        const size_t fixed = shared_bytes(N, 0, lds_matrix);
        const int m = room > fixed ? (int)((room - fixed) / ((size_t)N * 4)) : 0;
        return m < 96 ? m : 96;
    };
    auto finish = [&](size_t state) {
        p.M = p.M < N - 1 ? p.M : N - 1;
        p.bytes = shared_bytes(N, p.M, p.lds_matrix) + state;
        // at least eight wavefronts make the lists, with a histogram each
        const size_t makers = shared_bytes(N, p.M, p.lds_matrix) + (size_t)(p.waves > 8 ? p.waves : 8) * kBuckets * 4;
        p.bytes = p.bytes < makers ? makers : p.bytes;
    };
    if (per_unit <= groups.most_per_unit)
        for (int at_a_time = per_unit > 1 ? 2 : 1; at_a_time >= 1; --at_a_time) {
            // 1024 bytes for a unit's words outside the plan
            const size_t state = groups.state[at_a_time - 1], all = (kLds - 1024) / at_a_time, room = all > state ? all - state : 0;
            p.together = true;
            p.waves = groups.waves[at_a_time - 1];
            const int forms[3] = {1, groups.triangle ? 2 : 0, 0};
            for (int form : forms) {
                p.lds_matrix = form;
                p.M = longest(room, form);
                if (p.M >= (form == 1 ? 64 : 32) || p.M >= N - 1) {
                    finish(state);
                    return p;
                }
            }
        }
    p.together = false;
    p.M = N <= 128 ? 64 : 48;
    p.waves = per_unit < 16 ? per_unit : 16;
    const size_t slice = order_bytes + wave_bytes(kRoom);
    p.M = p.M < N - 1 ? p.M : N - 1;
    p.lds_matrix = shared_bytes(N, p.M, 1) + slice * (size_t)p.waves <= kLds ? 1 : 0;
    const int fit = (int)((kLds - shared_bytes(N, p.M, p.lds_matrix)) / slice);
    p.waves = p.waves < fit ? p.waves : fit;
    const int more = longest(kLds - slice * (size_t)p.waves, p.lds_matrix);
    p.M = more > p.M ? more : p.M;
    finish(slice * (size_t)p.waves);
    return p;
}

}  // namespace pruned
}  // namespace cc
