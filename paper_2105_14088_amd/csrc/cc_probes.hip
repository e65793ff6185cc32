// Cost matrix from latency probes (Section 4.2): per ordered pair of nodes the RTT at a given percentile
// of its K samples (nearest rank), then c[a][b] <- max(c[a][b], c[b][a]).
//
// Every sample is read from HBM exactly once and then lives in a register.  One wavefront per ordered
// pair loads the pair's K samples (up to 256 per lane, all loads in flight together).  The two directions of a
// pair are the two waves of one workgroup, which meet once, through LDS, for the symmetrisation.
//
// K <= 1024: the sample of rank k is found by descending over the value's bits from the top set bit of the largest
// sample: with candidate x = prefix | bit, the bit is kept iff fewer than k samples are below x.
//
// K > 1024: counting every sample once per value bit is what bounded this kernel (15 bits of two instructions per
// 64 samples: N = 64, K = 10000 77 us).  So a pilot of 256 to 1024 of the samples, taken evenly over the whole of them,
// gives a bracket that holds the wanted rank but for about one pair in a thousand; one pass counts the samples below the bracket
// and collects those inside it in LDS (each lane its own, so there is no traffic between lanes); and the descent over the bits
// runs over these few.  Where the rank lies outside, the next bracket is the one beside; where a lane has more samples inside
// than there is room (many equal samples), or after three brackets, the descent runs over all samples, within what the
// counts left over.
//
// What bounds it now: HBM, and what a wave computes once its last sample is there (about 1700 instructions at K = 10000; two
// waves per SIMD, both load first).  Counting every bit over every sample -> now, one call among others, 10th percentile: N = 64,
// K = 10000 72 -> 41 us (4.0 TB/s); N = 90, K = 4900 90 -> 36 us; N = 70, K = 8100 64 -> 39 us; N = 150, K = 1750 50 -> 38 us; N = 50,
// K = 16000 90 -> 58 us (one wave per SIMD); N = 8, K = 5000 13 -> 7.6 us; with a drift larger than the noise N = 64 80 -> 45 us, three values
// 66 -> 36 us.  Up to K = 1024 a bracket costs as many instructions as it saves; there the registers are counted by compare,
// mask and scalar population count instead of add-with-carry and a lane reduction per bit: N = 256, K = 300 73 -> 35 us,
// K = 610 79 -> 58 us.
#include "cc_device.h"
#include "cc_internal.h"

namespace cc {
using namespace ccd;

namespace {

constexpr int kCostMax = (1 << 21) - 1;
constexpr int kPad = 0x7fffffff;         // no candidate exceeds it: padding never counts as "below"

// sixteen bytes of samples, aligned as samples are
typedef int sample4 __attribute__((ext_vector_type(4), aligned(4)));

// acc += (v.x < cand) + (v.y < cand) + (v.z < cand) + (v.w < cand) per lane: each term is a compare into the carry
// flag and an add-with-carry.
__device__ __forceinline__ void count_below(int& acc, const int4& v, int cand) {
    asm("v_cmp_lt_i32 vcc, %1, %5\n\t"
        "v_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
        "v_cmp_lt_i32 vcc, %2, %5\n\t"
        "v_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
        "v_cmp_lt_i32 vcc, %3, %5\n\t"
        "v_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
        "v_cmp_lt_i32 vcc, %4, %5\n\t"
        "v_addc_co_u32 %0, vcc, 0, %0, vcc"
        : "+v"(acc)
        : "v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w), "v"(cand)
        : "vcc");
}
// d = x - low; acc += x < low: the borrow is the count (x and low from 0 on)
__device__ __forceinline__ unsigned above(int& acc, int x, int low) {
    unsigned d;
    asm("v_subrev_co_u32 %0, vcc, %3, %2\n\t"
        "v_addc_co_u32 %1, vcc, 0, %1, vcc"
        : "=&v"(d), "+v"(acc)
        : "v"(x), "v"(low)
        : "vcc");
    return d;
}
__device__ __forceinline__ int below_in_wave(int x, int cand) { return __popcll(__ballot(x < cand)); }
__device__ __forceinline__ int bits_of(int x) { return x > 0 ? 32 - __clz(x) : 0; }

// The pairs a < b of N nodes on a grid of full rows: row y holds the pairs of node y and, in the columns these leave, those of
// the node as far from the other end.
__host__ __device__ constexpr int pair_columns(int N) { return (N - 1) | 1; }
__host__ __device__ constexpr int pair_rows(int N) { return N / 2; }
__device__ __forceinline__ void pair_of(int x, int y, int N, int& a, int& b) {
    // with N odd N columns, the N - 1 - y pairs of node y and the y + 1 of node N - 2 - y; with N even N - 1, the y pairs of node
    // N - 1 - y instead; every workgroup has a pair
    const int first = N - 1 - y;
    a = x < first ? y : (N & 1 ? N - 2 - y : N - 1 - y);
    b = x < first ? y + 1 + x : a + 1 + x - first;
}

// Chunk of 256 samples that pilot register i takes its sample from in the lanes whose number is j modulo 16 / PILOT: sixteen
// chunks, evenly over all of them, so that samples that drift in time are met in all their states (one chunk per register,
// from the first ones alone: drifting samples, N = 150, K = 1750 81 us, now 37).
template <int CH, int PILOT>
__host__ __device__ constexpr int pilot_chunk(int i, int j) {
    return PILOT ? (i * (16 / PILOT) + j) * CH / 16 : 0;
}
template <int CH, int PILOT>
__host__ __device__ constexpr bool in_pilot(int u) {
    for (int r = 0; r < 16; ++r)
        if (r * CH / 16 == u) return PILOT > 0;
    return false;
}

struct PilotRanks {
    int low, high;           // ranks of the bracket's ends among the pilot's samples; 0 and beyond `held`: open ends
    int held;
};

// CH: int4 registers per lane (the wave holds up to 256 * CH samples).  FROM: the smallest K this form is launched with.
// PILOT: samples per lane that give the bracket (0: no bracket).  ROOM: samples inside the bracket a lane has room for.
template <int CH, int FROM, int PILOT, int ROOM>
__global__ __launch_bounds__(128, CH <= 48 ? (CH <= 24 ? 3 : 2) : 1) void probes_percentile_kernel(const int32_t* __restrict__ samples, int N, int K,
                                                                int rank, PilotRanks pilot, int symmetrize,
                                                                int32_t* __restrict__ out) {
    __shared__ int direction_result[2];
    __shared__ unsigned inside_all[2][PILOT ? ROOM + 4 : 1][64];
    const int lane = threadIdx.x & 63, dir = threadIdx.x >> 6;
    int a, b;
    pair_of(blockIdx.x, blockIdx.y, N, a, b);
    const int from = dir ? b : a, to = dir ? a : b;
    const int32_t* src = samples + ((int64_t)from * N + to) * K;
    int4 v[CH];
    // the last chunks are fetched from a clamped (valid) address; what a lane then has twice or should not have is padded
    constexpr int kWhole = FROM / 256;       // chunks of 256 that every K of this form fills
    auto load = [&](int u) {
        if (FROM >= 4) {
            const int e = u * 256 + lane * 4;
            const sample4 w = *(const sample4*)(src + (u < kWhole ? e : min(e, K - 4)));
            v[u] = make_int4(w.x, w.y, w.z, w.w);
        } else {
            const int e = u * 256 + lane;
            v[u] = make_int4(src[min(e, K - 1)], src[min(e + 64, K - 1)], src[min(e + 128, K - 1)], src[min(e + 192, K - 1)]);
        }
    };
    // the pilot's chunks first: the bracket is found while the others are on their way
#pragma unroll
    for (int u = 0; u < CH; ++u)
        if (in_pilot<CH, PILOT>(u)) load(u);
#pragma unroll
    for (int u = 0; u < CH; ++u)
        if (!in_pilot<CH, PILOT>(u)) load(u);

    // samples outside 0 .. kCostMax are data errors and count as the nearer end
    auto tidy = [&](int u) {
        v[u] = make_int4(clampi(v[u].x, 0, kCostMax), clampi(v[u].y, 0, kCostMax), clampi(v[u].z, 0, kCostMax),
                         clampi(v[u].w, 0, kCostMax));
        if (u < kWhole) return;
        if (FROM >= 4) {
            const int e = u * 256 + lane * 4, at = min(e, K - 4);
            v[u].x = at >= e ? v[u].x : kPad;
            v[u].y = at + 1 >= e ? v[u].y : kPad;
            v[u].z = at + 2 >= e ? v[u].z : kPad;
            v[u].w = at + 3 >= e ? v[u].w : kPad;
        } else {
            const int e = u * 256 + lane;
            v[u].x = e < K ? v[u].x : kPad;
            v[u].y = e + 64 < K ? v[u].y : kPad;
            v[u].z = e + 128 < K ? v[u].z : kPad;
            v[u].w = e + 192 < K ? v[u].w : kPad;
        }
        // the compiler would make every later compare with a padded register a compare and a test of the padding's condition
        asm("" : "+v"(v[u].x), "+v"(v[u].y), "+v"(v[u].z), "+v"(v[u].w));
    };
    int result;
    // the sample of rank `want` among those from `base` on, given that it is below base + 2^bits and `want` counts all samples
    auto descend = [&](int base, int bits, int want) {
        int found = base;
        for (int bit = bits - 1; bit >= 0; --bit) {
            const int cand = found + (1 << bit);
            int below = 0;
            if (CH <= 4) {
                // few registers: counted by the scalar unit, no reduction over the lanes
#pragma unroll
                for (int u = 0; u < CH; ++u)
                    below += (below_in_wave(v[u].x, cand) + below_in_wave(v[u].y, cand)) +
                             (below_in_wave(v[u].z, cand) + below_in_wave(v[u].w, cand));
            } else {
#pragma unroll
                for (int u = 0; u < CH; ++u) count_below(below, v[u], cand);
                below = wave_sum(below);
            }
            if (below < want) found = cand;          // the wanted sample is at least cand
        }
        return found;
    };
    if (PILOT == 0) {
#pragma unroll
        for (int u = 0; u < CH; ++u) tidy(u);
        int top = 0;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            // padding is above every sample
            top = max(max(top, v[u].x == kPad ? 0 : v[u].x), max(v[u].y == kPad ? 0 : v[u].y, max(v[u].z == kPad ? 0 : v[u].z, v[u].w == kPad ? 0 : v[u].w)));
        }
        result = descend(0, bits_of(wave_max(top)), rank);
    } else {
        // ---- the bracket [low, high] from the pilot's ranks
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (in_pilot<CH, PILOT>(u)) tidy(u);
        int p[PILOT > 0 ? PILOT : 1];
        int top = 0;
#pragma unroll
        for (int i = 0; i < PILOT; ++i) {
            constexpr int kWays = PILOT ? 16 / PILOT : 1;
            int w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int4 four = v[pilot_chunk<CH, PILOT>(i, j % kWays)];
                w[j] = (i & 3) == 0 ? four.x : (i & 3) == 1 ? four.y : (i & 3) == 2 ? four.z : four.w;
            }
            const int even = kWays > 2 && (lane & 2) ? w[2] : w[0], odd = kWays > 2 && (lane & 2) ? w[3] : w[1];
            p[i] = kWays > 1 && (lane & 1) ? odd : even;
            top = max(top, p[i] == kPad ? 0 : p[i]);
        }
        top = bits_of(wave_max(top));
        unsigned(*inside)[64] = inside_all[dir];
        int rank_low = pilot.low, rank_high = pilot.high, least = 0, most = kCostMax;      // least, most: what is known of the result
        int want = 0, low = 0, width = 0, here = 0, longest = 0;        // of the bracket that holds the wanted sample
#pragma unroll 1
        for (int attempt = 0; attempt < 3 && least <= most; ++attempt) {
            int high = 0;
            low = 0;
            for (int bit = top - 1; bit >= 0; --bit) {
                const int cand_low = low + (1 << bit), cand_high = high + (1 << bit);
                int below_low = 0, below_high = 0;
#pragma unroll
                for (int i = 0; i < PILOT; ++i) {
                    below_low += below_in_wave(p[i], cand_low);
                    below_high += below_in_wave(p[i], cand_high);
                }
                low = below_low < rank_low ? cand_low : low;
                high = below_high < rank_high ? cand_high : high;
            }
            low = rank_low > 0 ? max(low, least) : least;
            high = rank_high <= pilot.held ? min(high, most) : most;
            high = max(low, high);
            // ---- below the bracket: counted; inside: each lane's own column in LDS
            width = high - low + 1;
            here = 0;
            int below = 0;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                if (!in_pilot<CH, PILOT>(u)) tidy(u);    // as they arrive (a second time changes nothing)
                const int x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                here = min(here, ROOM);
                __builtin_amdgcn_sched_barrier(0);       // one chunk's differences at a time: all at once take twice the registers
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned d = above(below, x[j], low);
                    inside[here][lane] = d;
                    here += d < (unsigned)width ? 1 : 0;
                }
            }
            below = wave_sum(below);
            longest = wave_max(here);
            const int found = wave_sum(here), span = rank_high - rank_low;
            if (rank <= below) {
                most = low - 1;
                rank_high = rank_low;
                rank_low -= span;
                continue;
            }
            least = low;
            if (longest >= ROOM) {
                // how many there are inside is not known: counted, and the descent over all samples does the rest
                int upto = 0;
#pragma unroll
                for (int u = 0; u < CH; ++u) count_below(upto, v[u], high + 1);
                if (wave_sum(upto) >= rank) most = high;
                else least = high + 1;
                break;
            }
            if (rank > below + found) {
                least = high + 1;
                rank_low = rank_high;
                rank_high += span;
                continue;
            }
            want = rank - below;
            break;
        }
        if (want > 0) {
            int4 c[ROOM ? ROOM / 4 : 1];
#pragma unroll
            for (int i = 0; i < ROOM / 4; ++i) {
                c[i].x = 4 * i < here ? (int)inside[4 * i][lane] : kPad;
                c[i].y = 4 * i + 1 < here ? (int)inside[4 * i + 1][lane] : kPad;
                c[i].z = 4 * i + 2 < here ? (int)inside[4 * i + 2][lane] : kPad;
                c[i].w = 4 * i + 3 < here ? (int)inside[4 * i + 3][lane] : kPad;
            }
            int at = 0, span = width - 1;
            if (rank_high > pilot.held) {
                // an open bracket is as wide as costs may be, what was found in it is not (99th percentile, descending over its width /
                // over what was found: N = 9, K = 3073 9.2 / 6.9 us, N = 64, K = 2049 14.0 / 11.7, N = 100, K = 1100 25.8 / 21.6)
                span = 0;
#pragma unroll
                for (int i = 0; i < ROOM / 4; ++i)
                    if (4 * i < longest)
                        span = max(max(span, c[i].x == kPad ? 0 : c[i].x), max(c[i].y == kPad ? 0 : c[i].y, max(c[i].z == kPad ? 0 : c[i].z, c[i].w == kPad ? 0 : c[i].w)));
                span = wave_max(span);
            }
            for (int bit = bits_of(span) - 1; bit >= 0; --bit) {
                const int cand = at + (1 << bit);
                int n = 0;
#pragma unroll
                for (int i = 0; i < ROOM / 4; i += 2) {
                    if (4 * i < longest) {
                        count_below(n, c[i], cand);
                        count_below(n, c[i + 1], cand);
                    }
                }
                if (wave_sum(n) < want) at = cand;
            }
            result = low + at;
        } else {
            // the spread of what is left: no sample is beyond the largest one
            int largest = 0;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                largest = max(max(largest, v[u].x == kPad ? 0 : v[u].x), v[u].y == kPad ? 0 : v[u].y);
                largest = max(max(largest, v[u].z == kPad ? 0 : v[u].z), v[u].w == kPad ? 0 : v[u].w);
            }
            most = min(most, wave_max(largest));
            result = descend(least, bits_of(most - least), rank);
        }
    }
    if (lane == 0) direction_result[dir] = result;
    __syncthreads();
    if (lane == 0) {
        const int value = symmetrize ? max(direction_result[0], direction_result[1]) : result;
        out[(int64_t)from * N + to] = value;
        // the diagonal: node a's by the pair (a, a + 1), the last node's beside it
        if (b == a + 1 && (dir == 0 || b == N - 1)) out[(int64_t)from * N + from] = 0;
    }
}

__global__ void zero_cost_kernel(int32_t* out) { out[0] = 0; }

}  // namespace

template <int CH, int FROM, int PILOT, int ROOM>
static hipError_t probes_launch(const int32_t* samples, int N, int K, int rank, bool symmetrize, int32_t* out,
                                hipStream_t s) {
    // what the pilot holds: its chunks may lie beyond K
    int held = 0;
    for (int i = 0; i < PILOT; ++i)
        for (int j = 0; j < 16 / (PILOT ? PILOT : 1); ++j) {
            const int left = (K - 256 * pilot_chunk<CH, PILOT>(i, j)) / 4, lanes = left < 0 ? 0 : left < 64 ? left : 64;
            held += lanes * PILOT / 16;
        }
    // The ends lie 3.3 standard deviations of the pilot's rank of the wanted sample from it, and one more.
    const double q = (double)rank / K, spread = 3.3 * sqrt(held * q * (1.0 - q));
    PilotRanks pilot;
    pilot.low = (int)(held * q - spread) - 1;
    pilot.low = pilot.low < 1 ? 0 : pilot.low;
    pilot.high = (int)(held * q + spread) + 2;
    pilot.held = held;
    hipLaunchKernelGGL((probes_percentile_kernel<CH, FROM, PILOT, ROOM>), dim3(pair_columns(N), pair_rows(N)), dim3(128), 0, s,
                       samples, N, K, rank, pilot, symmetrize ? 1 : 0, out);
    return hipGetLastError();
}

// K <= 16384 (checked by the caller).  A form for every 1000 to 4000 samples: registers that K leaves empty cost loads and counts
// like full ones (K = 4900 in the form for 10240: 90 us, in its own 36).  The room holds what a bracket of the widest pilot, that of the median, leaves per lane
// (K = 10240: 23 on average) and five standard deviations more.
hipError_t launch_probes_percentile(const int32_t* samples, int N, int K, int rank, bool symmetrize, int32_t* out,
                                    hipStream_t s) {
    if (N == 1) {
        hipLaunchKernelGGL(zero_cost_kernel, dim3(1), dim3(1), 0, s, out);
        return hipGetLastError();
    }
    if (K <= 256) return probes_launch<1, 1, 0, 0>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 512) return probes_launch<2, 257, 0, 0>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 1024) return probes_launch<4, 513, 0, 0>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 2048) return probes_launch<8, 1025, 4, 24>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 3072) return probes_launch<12, 2049, 4, 32>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 4096) return probes_launch<16, 3073, 4, 32>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 6144) return probes_launch<24, 4097, 8, 32>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 8192) return probes_launch<32, 6145, 8, 40>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 10240) return probes_launch<40, 8193, 8, 48>(samples, N, K, rank, symmetrize, out, s);
    if (K <= 12288) return probes_launch<48, 10241, 16, 48>(samples, N, K, rank, symmetrize, out, s);
    return probes_launch<64, 12289, 16, 48>(samples, N, K, rank, symmetrize, out, s);
}

}  // namespace cc
