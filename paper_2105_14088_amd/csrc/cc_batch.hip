// Batched evaluation of the ring and halving-doubling cost models (Section 4.1) over candidate rank
// orders, plus the seeded initial-order generator and the matrix contract check.
//
// Ring, N a power of two in [8, 128]: the cost matrix (<= 64 KiB int32) is staged in LDS once per
// workgroup; the order stream is read from HBM as 16-byte vectors, N/4 lanes per order, several
// vector loads in flight per wave; each lane gathers its four hops from LDS and the N/4 lanes of an
// order are combined with a butterfly.  The stream is read exactly once, so the kernel is bound by
// HBM bandwidth (4N bytes in + 8 bytes out per order).
// Other N up to 280, large batches: 16-bit matrix in LDS, sixteen lanes per order; max-hop above: marked entries in LDS.
// The rest: one wave per order, hops gathered from the L2-resident matrix.
#include "cc_device.h"
#include "cc_internal.h"
#include "cc_wave64.h"

#include <type_traits>

namespace cc {
using namespace ccd;

constexpr int kMaxRoundWeight = 1 << 30;   // round weights are clamped to [0, 2^30]: weight * cost stays below 2^51

// A threshold that about `wanted` of 64 U entries reach, from 1024 U sampled ones, U per thread of a 1024-thread workgroup: every
// wave takes the wanted-th largest of its 64 U, the result is the one of the sixteen values that ABOVE of them exceed.  `v` are
// not negative; per_wave: 16 words of LDS.  (A bit-by-bit search over all 4096, a barrier per bit, took 10 us longer.)
template <int ABOVE = 8, int U>
__device__ __forceinline__ int sampled_threshold(int (&v)[U], int wanted, int* per_wave) {
    int T = 0;
    for (int seen = 0; seen < wanted;) {
        int largest = v[0];
#pragma unroll
        for (int i = 1; i < U; ++i) largest = max(largest, v[i]);
        T = wave_max(largest);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            seen += __popcll(__ballot(v[i] == T));
            if (v[i] == T) v[i] = -1;
        }
    }
    if (lane_id() == 0) per_wave[threadIdx.x >> 6] = T;
    __syncthreads();
    const int sub = lane_id() & 15, mine = per_wave[sub];
    int above = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) above += per_wave[k] > mine || (per_wave[k] == mine && k < sub);
    return __builtin_amdgcn_readlane(mine, __ffsll((unsigned long long)__ballot(above == ABOVE)) - 1);
}

// four ranks of an order, aligned as a rank is
typedef int ranks4 __attribute__((ext_vector_type(4), aligned(4)));

// The caller's matrix into LDS, by all threads of the workgroup, sixteen loads of each in flight; returns the thread's share
// of the largest entry (a negative one counts as too large).  16 bits: what is too large for them is staged as 0xffff.
template <typename ENTRY>
__device__ __forceinline__ unsigned stage_matrix(const int32_t* __restrict__ c, int entries, ENTRY* staged) {
    constexpr int U = 16;
    unsigned top = 0;
    const int threads = blockDim.x;
    for (int e0 = threadIdx.x; e0 < entries; e0 += U * threads) {
        unsigned v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = (unsigned)c[min(e0 + u * threads, entries - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            top = max(top, v[u]);
            if (e0 + u * threads < entries) staged[e0 + u * threads] = (ENTRY)(sizeof(ENTRY) == 2 ? min(v[u], 0xffffu) : v[u]);
        }
    }
    return top;
}

// ------------------------------------------------------------------------------------------ ring
template <int N, bool IS_MAX>
__global__ __launch_bounds__(256) void ring_batch_lds_kernel(const int32_t* __restrict__ c,
                                                             const int4* __restrict__ perms4, int64_t B,
                                                             int64_t* __restrict__ out) {
    __shared__ int32_t m[N * N];
    for (int e = threadIdx.x; e < N * N; e += 256) m[e] = c[e];
    __syncthreads();

    constexpr int LP = N / 4;     // lanes that share one order
    constexpr int PPW = 64 / LP;  // orders covered by one 1 KiB wave-load
    constexpr int U = 4;          // wave-loads in flight
    constexpr int M = N - 1;
    const int lane = lane_id();
    const int sub = lane & (LP - 1);
    const int prev_lane = (lane & ~(LP - 1)) | ((sub + LP - 1) & (LP - 1));
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    const int64_t nloads = (B + PPW - 1) / PPW;

    for (int64_t base = wave * U; base < nloads; base += nwaves * U) {
        int4 v[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ld = base + u;
            const int64_t b = ld * PPW + lane / LP;
            ok[u] = ld < nloads && b < B;
            v[u] = ok[u] ? perms4[ld * 64 + lane] : make_int4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int x = v[u].x & M, y = v[u].y & M, z = v[u].z & M, w = v[u].w & M;
            const int pw = __shfl(w, prev_lane, kWave);   // last node of the previous lane (cyclic in the order)
            const int h0 = m[x * N + pw], h1 = m[y * N + x], h2 = m[z * N + y], h3 = m[w * N + z];
            int acc = IS_MAX ? max(max(h0, h1), max(h2, h3)) : h0 + h1 + h2 + h3;
#pragma unroll
            for (int s = LP / 2; s >= 1; s >>= 1) {
                const int o = __shfl_xor(acc, s, kWave);
                acc = IS_MAX ? max(acc, o) : acc + o;
            }
            if (ok[u] && sub == 0) out[(base + u) * PPW + lane / LP] = (int64_t)acc;
        }
    }
}

template <bool IS_MAX>
__global__ __launch_bounds__(256) void ring_batch_generic_kernel(const int32_t* __restrict__ c, int N,
                                                                 const int32_t* __restrict__ perms, int64_t B,
                                                                 int64_t* __restrict__ out) {
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t b = wave; b < B; b += nwaves) {
        const int32_t* pi = perms + b * N;
        long long acc = 0;
        for (int p = lane; p < N; p += kWave) {
            const int a = clampi(pi[p], 0, N - 1);
            const int q = clampi(pi[p ? p - 1 : N - 1], 0, N - 1);
            const long long hop = c[(int64_t)a * N + q];
            acc = IS_MAX ? (hop > acc ? hop : acc) : acc + hop;
        }
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            const long long o = __shfl_xor(acc, s, kWave);
            acc = IS_MAX ? (o > acc ? o : acc) : acc + o;
        }
        if (lane == 0) out[b] = acc;
    }
}

// Orders stored one byte per rank (N <= 256): a quarter of the HBM bytes per order.  N in {16, 32, 64, 128}: matrix
// in LDS; one lane fetches 16 ranks as an int4, N/16 adjacent lanes share an order, a wave-load covers 1024/N
// orders.  The hop into a lane's first rank needs the last rank of the lane before it (cyclically within the
// order's lanes), fetched with one lane permute.
template <int N, bool IS_MAX>
__global__ __launch_bounds__(256) void ring_batch_u8_lds_kernel(const int32_t* __restrict__ c,
                                                                const int4* __restrict__ perms16, int64_t B,
                                                                int64_t* __restrict__ out) {
    __shared__ int32_t m[N * N];
    for (int e = threadIdx.x; e < N * N; e += 256) m[e] = c[e];
    __syncthreads();

    constexpr int LP = N / 16;    // lanes that share one order
    constexpr int PPW = 64 / LP;  // orders covered by one 1 KiB wave-load
    constexpr int U = 2;          // wave-loads in flight
    constexpr unsigned M4 = (unsigned)(N - 1) * 0x01010101u;
    const int lane = lane_id();
    const int sub = lane & (LP - 1);
    const int prev_lane = (lane & ~(LP - 1)) | ((sub + LP - 1) & (LP - 1));
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    const int64_t nloads = (B + PPW - 1) / PPW;

    for (int64_t base = wave * U; base < nloads; base += nwaves * U) {
        int4 v[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t ld = base + u;
            const int64_t b = ld * PPW + lane / LP;
            ok[u] = ld < nloads && b < B;
            v[u] = ok[u] ? perms16[ld * 64 + lane] : make_int4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned w[4] = {(unsigned)v[u].x & M4, (unsigned)v[u].y & M4, (unsigned)v[u].z & M4,
                                   (unsigned)v[u].w & M4};
            int prev = (int)(w[3] >> 24);
            prev = LP > 1 ? __shfl(prev, prev_lane, kWave) : prev;   // last rank of the previous lane (or of this order)
            int acc = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int node = (int)((w[k >> 2] >> (8 * (k & 3))) & 0xffu);
                const int hop = m[node * N + prev];
                acc = IS_MAX ? max(acc, hop) : acc + hop;
                prev = node;
            }
#pragma unroll
            for (int s = LP / 2; s >= 1; s >>= 1) {
                const int o = __shfl_xor(acc, s, kWave);
                acc = IS_MAX ? max(acc, o) : acc + o;
            }
            if (ok[u] && sub == 0) out[(base + u) * PPW + lane / LP] = (int64_t)acc;
        }
    }
}

// Orders stored one byte or two bytes per rank, any N: one wave per order, matrix through L2.
template <typename RANK, bool IS_MAX>
__global__ __launch_bounds__(256) void ring_batch_narrow_generic_kernel(const int32_t* __restrict__ c, int N,
                                                                        const RANK* __restrict__ perms, int64_t B,
                                                                        int64_t* __restrict__ out) {
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t b = wave; b < B; b += nwaves) {
        const RANK* pi = perms + b * N;
        long long acc = 0;
        for (int p = lane; p < N; p += kWave) {
            const int a = min((int)pi[p], N - 1);
            const int q = min((int)pi[p ? p - 1 : N - 1], N - 1);
            const long long hop = c[(int64_t)a * N + q];
            acc = IS_MAX ? (hop > acc ? hop : acc) : acc + hop;
        }
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            const long long o = __shfl_xor(acc, s, kWave);
            acc = IS_MAX ? (o > acc ? o : acc) : acc + o;
        }
        if (lane == 0) out[b] = acc;
    }
}

// Any N up to kRingRowsMaxN, orders of 1, 2 or 4 bytes per rank: the matrix as 16-bit entries in LDS, sixteen lanes per
// order (a DPP row), four orders per wave.  A step takes sixteen consecutive ranks of each order, so whatever N and the
// alignment are the loads of a step are four short runs and those of the next steps lie in the same cache lines; the hop
// into a lane's rank uses the node of the lane before it (one DPP rotation; lane 0 takes lane 15's node of the step
// before, in the first step the order's last node).  Eight steps are in flight per wave.  The workgroup finds the matrix
// maximum while staging; with an entry outside 0 .. 2^16 - 1 it gathers from the caller's matrix through L2 instead.
// One order per wave through L2 (the generic kernels) runs at the L2's request rate, or for short orders at the cost of
// its 64-bit reductions.  Measured, generic -> rows: N = 9, 10^6 orders 154 -> 35 us; N = 20, 10^6 orders 150 -> 38 us;
// N = 100, 100000 orders 33 -> 12 us, 600000 orders 187 -> 46 us (5.3 TB/s of the order stream); N = 180, 300000 orders
// of two bytes a rank 200 -> 39 us; N = 270, 200000 orders 228 -> 64 us.
// The ranks in flight are held as int whatever their type: as 16-bit values each was masked, and so waited for, in the
// conditional block of its own load (58 us for the two-byte case; 82 instead of 55 us in ring_batch_max_marked_kernel).
constexpr int kRingRowsMaxN = 280;              // 2 N^2 bytes and the waves' maxima in 160 KiB

template <typename RANK, bool IS_MAX>
__global__ __launch_bounds__(1024) void ring_batch_rows_kernel(const int32_t* __restrict__ c, int N,
                                                               const RANK* __restrict__ perms, int64_t B,
                                                               int64_t* __restrict__ out) {
    constexpr int U = 8;                        // steps in flight
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_rows[];
    unsigned* wave_top = (unsigned*)smem_rows;                  // [16]
    uint16_t* m16 = (uint16_t*)(smem_rows + 64);                // [N * N]
    const int lane = lane_id(), wv = threadIdx.x >> 6, sub = lane & 15;
    unsigned top = 0;
    for (int e = threadIdx.x; e < N * N; e += 1024) {
        const unsigned v = (unsigned)c[e];                      // a negative entry counts as too large
        top = max(top, v);
        m16[e] = (uint16_t)v;
    }
    top = (unsigned)wave_max((int)min(top, 0x7fffffffu));
    if (lane == 0) wave_top[wv] = top;
    __syncthreads();
    unsigned all_top = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) all_top = max(all_top, wave_top[k]);
    auto node = [&](int r) { return sizeof(RANK) == 4 ? clampi(r, 0, N - 1) : min(r, N - 1); };
    // total: all hops of an order in 32 bits when they come from LDS (at most 280 * 65535), in 64 bits otherwise
    auto score = [&](auto in_lds, auto zero) {
        using Acc = decltype(zero);
        const int64_t waves = (int64_t)gridDim.x * 16;
        for (int64_t w = (int64_t)blockIdx.x * 16 + wv; w * 4 < B; w += waves) {
            const int64_t b = w * 4 + (lane >> 4);
            const RANK* pi = perms + (b < B ? b : B - 1) * N;
            int before = node(pi[N - 1]);                       // of lane 0: the node of the rank before this step's first
            Acc acc = 0;
            for (int p0 = 0; p0 < N; p0 += 16 * U) {
                int r[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (p0 + 16 * u < N) r[u] = (int)pi[min(p0 + 16 * u + sub, N - 1)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (p0 + 16 * u < N) {
                        const int x = node(r[u]);
                        const int rot = __builtin_amdgcn_update_dpp(x, x, 0x121, 0xf, 0xf, true);      // row_ror:1
                        const int e = x * N + (sub == 0 ? before : rot);
                        before = rot;
                        const int hop = in_lds ? (int)m16[e] : c[e];
                        if (p0 + 16 * u + sub < N) acc = IS_MAX ? max(acc, (Acc)hop) : acc + hop;
                    }
                }
            }
            if constexpr (sizeof(Acc) == 4) {
#define CC_ROW_STEP(ctrl)                                                                     \
    {                                                                                         \
        const int o = __builtin_amdgcn_update_dpp(acc, acc, ctrl, 0xf, 0xf, true);            \
        acc = IS_MAX ? max(acc, o) : acc + o;                                                 \
    }
                CC_ROW_STEP(0xB1) CC_ROW_STEP(0x4E) CC_ROW_STEP(0x141) CC_ROW_STEP(0x140)
#undef CC_ROW_STEP
            } else {
#pragma unroll
                for (int m = 8; m >= 1; m >>= 1) {
                    const Acc o = __shfl_xor(acc, m, kWave);
                    acc = IS_MAX ? max(acc, o) : acc + o;
                }
            }
            if (sub == 0 && b < B) out[b] = (int64_t)acc;
        }
    };
    if (all_top < (1u << 16)) score(std::true_type{}, 0);
    else score(std::false_type{}, 0ll);
}

static int batch_grid(int64_t work_items_per_block_pass, int64_t total) {
    int64_t blocks = (total + work_items_per_block_pass - 1) / work_items_per_block_pass;
    const int64_t cap = 256 * 8;  // 8 workgroups of 4 waves per compute unit
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (int)blocks;
}

template <int N>
static hipError_t ring_lds(const int32_t* c, bool is_max, const int32_t* perms, int64_t B, int64_t* out,
                           hipStream_t s) {
    constexpr int PPW = 64 / (N / 4);
    const int grid = batch_grid((int64_t)PPW * 4 * 4, B);
    if (is_max)
        hipLaunchKernelGGL((ring_batch_lds_kernel<N, true>), dim3(grid), dim3(256), 0, s, c, (const int4*)perms, B, out);
    else
        hipLaunchKernelGGL((ring_batch_lds_kernel<N, false>), dim3(grid), dim3(256), 0, s, c, (const int4*)perms, B, out);
    return hipGetLastError();
}

// N = 256 for large batches: the matrix as 16-bit entries in LDS (128 KiB, one 1024-thread workgroup per compute
// unit), one wave per order: a 1 KiB wave-load is the order, four ranks per lane, the hop into a lane's first rank
// uses the previous lane's last node (cyclic), four LDS gathers per lane and one wave reduction per order.  Through
// L2 (generic kernel) the same batch runs at the L2's request rate, 256 scattered requests per order.  The workgroup
// finds the matrix maximum while staging; with an entry outside 0 .. 2^16 - 1 it scores its orders through L2 instead.
template <bool IS_MAX>
__global__ __launch_bounds__(1024) void ring_batch_n256_kernel(const int32_t* __restrict__ c,
                                                               const int4* __restrict__ perms4, int64_t B,
                                                               int64_t* __restrict__ out) {
    constexpr int N = 256, U = 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem256[];
    uint16_t* m16 = (uint16_t*)smem256;
    __shared__ unsigned wave_top[16];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    unsigned top = 0;
    for (int e = threadIdx.x; e < N * N; e += 1024) {
        const unsigned v = (unsigned)c[e];                 // a negative entry counts as too large
        top = max(top, v);
        m16[e] = (uint16_t)v;
    }
    top = (unsigned)wave_max((int)min(top, 0x7fffffffu));
    if (lane == 0) wave_top[wv] = top;
    __syncthreads();
    unsigned all_top = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) all_top = max(all_top, wave_top[k]);
    const bool in_lds = all_top < (1u << 16);
    const int64_t wave = (int64_t)blockIdx.x * 16 + wv;
    const int64_t nwaves = (int64_t)gridDim.x * 16;
    const char* mbytes = (const char*)m16;
    for (int64_t base = wave * U; base < B; base += nwaves * U) {
        int4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t b = base + u < B ? base + u : B - 1;
            v[u] = perms4[b * 64 + lane];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int x = v[u].x & 255, y = v[u].y & 255, z = v[u].z & 255, w = v[u].w & 255;
            const int pw = __builtin_amdgcn_update_dpp(w, w, 0x13C, 0xf, 0xf, true);   // lane p <- lane p - 1, cyclic
            int h0, h1, h2, h3;
            if (in_lds) {
                h0 = *(const uint16_t*)(mbytes + ((x << 9) | (pw << 1)));
                h1 = *(const uint16_t*)(mbytes + ((y << 9) | (x << 1)));
                h2 = *(const uint16_t*)(mbytes + ((z << 9) | (y << 1)));
                h3 = *(const uint16_t*)(mbytes + ((w << 9) | (z << 1)));
            } else {
                h0 = c[x * N + pw]; h1 = c[y * N + x]; h2 = c[z * N + y]; h3 = c[w * N + z];
            }
            long long total;
            if (IS_MAX) {
                total = max(wave_max(max(max(h0, h1), max(h2, h3))), 0);
            } else if (in_lds) {
                total = wave_sum(h0 + h1 + h2 + h3);       // at most 256 * 65535
            } else {
                total = wave_sum64((long long)h0 + h1 + h2 + h3);
            }
            if (lane == 0 && base + u < B) out[base + u] = total;
        }
    }
}

template <bool IS_MAX>
static hipError_t ring_n256_launch(const int32_t* c, const int32_t* perms, int64_t B, int64_t* out, hipStream_t s) {
    const size_t lds = sizeof(uint16_t) * 256 * 256;
    hipError_t e = hipFuncSetAttribute((const void*)ring_batch_n256_kernel<IS_MAX>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int64_t blocks = (B + 16 * 4 - 1) / (16 * 4);
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(ring_batch_n256_kernel<IS_MAX>, dim3((int)blocks), dim3(1024), lds, s, c, (const int4*)perms, B,
                       out);
    return hipGetLastError();
}

template <typename RANK, bool IS_MAX>
static hipError_t ring_rows_launch(const int32_t* c, int N, const RANK* perms, int64_t B, int64_t* out, hipStream_t s) {
    const size_t lds = 64 + sizeof(uint16_t) * (size_t)N * N;
    hipError_t e = hipFuncSetAttribute((const void*)ring_batch_rows_kernel<RANK, IS_MAX>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t at_once = lds <= 80 * 1024 ? 512 : 256;       // two workgroups of 16 waves fill a compute unit
    int64_t blocks = (B + 63) / 64;
    if (blocks > at_once) blocks = at_once;
    hipLaunchKernelGGL((ring_batch_rows_kernel<RANK, IS_MAX>), dim3((int)blocks), dim3(1024), lds, s, c, N, perms, B, out);
    return hipGetLastError();
}

// Staging N^2 entries per workgroup against L2 gathers: both forms take a call's launch time (7 us) up to about 2^20 hops;
// beyond that the rows kernel is ahead from 35 N orders (generic / rows at N = 270: 8000 orders 10.9 / 12.8 us, 16000
// orders 19.5 / 13.1) or 48 N (N = 180: 12000 orders 9.5 / 8.4), at N = 256, whose 1 KiB rows meet in the same memory
// channels, from 85 N (17000 orders 19.7 / 23.4, 25000 orders 27.7 / 23.5).
static bool ring_rows_pays(int N, int64_t B) {
    return N <= kRingRowsMaxN && B * N >= (1 << 20) && B >= (N == 256 ? 96 : 64) * (int64_t)N;
}

// Max-hop, 280 < N <= 1024: only hops among the matrix's largest entries have to be looked up exactly.  Every workgroup
// marks in LDS, one bit per entry (32 KiB at N = 500, 128 KiB at N = 1024), the entries that are T or more; T is chosen
// from 4096 sampled hops of the batch's orders so that about ln N of an order's N hops carry the bit (where the exact look-ups and the orders
// without a marked hop, which are looked up whole, cost the same).  Any T gives the right result, only the time depends on
// it.  One order per wave, its ranks in a wide load or two, two orders ahead; the marked hops' entries are read together, the others'
// lanes at one common place.  Where all marked entries are the largest one nothing is read, and an order with many marked hops ends
// at the first of the largest, so a matrix of few values ends early.
// The generic kernels ask L2 for every hop and run at its request rate; here what is left is the marking (N = 500: 1 MB read per
// compute unit, 14 us), sampling (3 us), the order stream and a chain of LDS and L2 latencies per order, two orders' overlapping.
// Generic -> marked, seeded orders: N = 500, 65000 orders 144 -> 43 us, of two bytes a rank 140 -> 38 us; N = 1000, 65000 orders
// 335 -> 102 us.  Orders of small hops only: N = 500, 65000 orders 113 -> 38 us.  An order's entries
// reduced before the next order was looked at: two bytes a rank, N = 300, 200000 orders 75 us, now 56; N = 400, 50000 31.5, now 28.1;
// N = 500, 65000 41.0, now 37.9; N = 700, 60000 72, now 70; N = 1000, 65000 81, now 79; slower where every hop of an order is marked and none
// is the largest (two values and a search's results, N = 500, 65000 orders 92 -> 96, N = 300, 200000 189 -> 202).  All in repeated passes over
// the same orders; a first pass over new ones waits for the stream and gained nothing (N = 500, 65000 orders 65, now 66).
// W consecutive ranks of an order, aligned as a rank is
template <typename RANK, int W>
struct Ranks;
template <>
struct Ranks<uint16_t, 4> {
    typedef unsigned short type __attribute__((ext_vector_type(4), aligned(2)));
};
template <>
struct Ranks<uint16_t, 8> {
    typedef unsigned short type __attribute__((ext_vector_type(8), aligned(2)));
};
template <>
struct Ranks<int32_t, 4> {
    typedef ranks4 type;
};
template <>
struct Ranks<int32_t, 8> {
    struct type {
        ranks4 a, b;
        __device__ __forceinline__ int operator[](int i) const { return i < 4 ? a[i] : b[i - 4]; }
    };
};

// A lane takes the R = ceil(N / 64) ranks from R * lane on, W + SECOND of them at most: W from there and W up to their end, of which
// the last SECOND are looked at (W = 4 up to N = 512, so that 5 .. 8 ranks are 5 .. 8 look-ups; above W = 8).
template <typename RANK, int W, int SECOND>
__global__ __launch_bounds__(1024) void ring_batch_max_marked_kernel(const int32_t* __restrict__ c, int N,
                                                                     const RANK* __restrict__ perms, int64_t B,
                                                                     int64_t* __restrict__ out, int wanted) {
    using Part = typename Ranks<RANK, W>::type;
    constexpr int H = W + SECOND;                                // hops of a lane
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_ring_marks[];
    int* per_wave = (int*)smem_ring_marks;                       // [2][16]: the waves' estimates of T, their maxima
    uint32_t* marks = (uint32_t*)(smem_ring_marks + 128);        // bit e of the flat matrix: bit e & 31 of word e >> 5
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * 16, first_order = (int64_t)blockIdx.x * 16 + wv;
    // 4 * node, to be the byte offset of an entry when multiplied
    auto node = [&](int r) { return (unsigned)(sizeof(RANK) == 4 ? clampi(r, 0, N - 1) : min(r, N - 1)) << 2; };
    const int R = (N + 63) >> 6, start = min(lane * R, N - R);   // the last lanes have ranks of others again
    struct Mine {
        Part a, b;
    };
    auto load = [&](int64_t b) {
        const RANK* pi = perms + b * N + start;
        Mine m;
        m.a = *(const Part*)pi;
        m.b = *(const Part*)(pi + R - W);
        return m;
    };
    Mine next = load(min(first_order, B - 1));
    int v[4];
    {
        // hops of 16 of the orders that this workgroup will look at, one per wave, spread over the batch (of orders from all over the
        // batch, the same in every workgroup: 12 us, now 3)
        const int64_t turns = (B + waves - 1) / waves;
        const Mine m = load(min(first_order + wv % turns * waves, B - 1));
        auto hop = [&](int x, int y) { return max(*(const int32_t*)((const char*)c + (__umul24(node(x), (unsigned)N) + node(y))), 0); };
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = hop(m.a[i + 1], m.a[i]);
        v[3] = hop(m.b[W - 1], m.b[W - 2]);
    }
    const int T = sampled_threshold(v, wanted, per_wave);
    // 2048 entries per wave and pass, all loads in flight; the workgroups start at different places, so that they
    // do not all ask the same L2 channel at once
    int top = 0;
    const int total = N * N, passes = (total + 16 * 2048 - 1) / (16 * 2048);
    const int first = (int)((int64_t)blockIdx.x * passes / gridDim.x);
    for (int i = 0; i < passes; ++i) {
        const int at = ((first + i < passes ? first + i : first + i - passes) * 16 + wv) * 2048;
        if (at + 2048 <= total) {
            // a lane's four entries make four bits (the sign of T - 1 - entry), eight lanes' a word
            ranks4 e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) e[k] = *(const ranks4*)(c + at + 256 * k + 4 * lane);
            uint32_t word = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint32_t bits = 0;
#pragma unroll
                for (int q = 3; q >= 0; --q) bits = __builtin_amdgcn_alignbit(bits, (uint32_t)(T - 1) - (uint32_t)e[k][q], 31);
                top = max(max(top, e[k][0]), max(max(e[k][1], e[k][2]), e[k][3]));
                int v = (int)(bits << (4 * (lane & 7)));
                v |= __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);        // quad_perm 1, 0, 3, 2
                v |= __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);        // quad_perm 2, 3, 0, 1
                v |= __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);       // row_half_mirror
                if ((lane & 7) == k) word = (uint32_t)v;
            }
            marks[(at >> 5) + 8 * (lane & 7) + (lane >> 3)] = word;
        } else if (at < total) {
            uint32_t word = 0;
#pragma unroll 4
            for (int k = 0; k < 32; ++k) {
                const int e = c[min(at + 64 * k + lane, total - 1)];
                const unsigned long long bits = __ballot(e >= T);
                top = max(top, e);
                if ((lane >> 1) == k) word = lane & 1 ? (uint32_t)(bits >> 32) : (uint32_t)bits;
            }
            if (at + 32 * lane < total) marks[(at >> 5) + lane] = word;
        }
    }
    top = wave_max(top);
    if (lane == 0) per_wave[16 + wv] = top;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) top = max(top, per_wave[16 + k]);
    Mine after = load(min(first_order + waves, B - 1));
    const bool known = T >= top;                                 // what a marked entry costs
    const bool whole = lane * R <= N - R;                        // not: the first rank's hop is an earlier lane's
    const bool own = lane * R < N;                               // not: all of them are
    auto entry = [&](unsigned at) { return *(const int32_t*)((const char*)c + at); };
    // the next order's hops: where their entries lie, which of them are marked
    auto test = [&](int64_t b, unsigned (&at)[H], int (&hit)[H], int& any) {
        const Mine now = next;
        next = after;
        after = load(min(b + 2 * waves, B - 1));
        // hop i leads into x[i] from y[i]
        unsigned x[H], y[H];
#pragma unroll
        for (int i = 0; i < W; ++i) {
            x[i] = node(now.a[i]);
            if (i) y[i] = x[i - 1];
        }
#pragma unroll
        for (int i = 0; i < SECOND; ++i) {
            x[W + i] = node(now.b[W - SECOND + i]);
            if (i) y[W + i] = x[W + i - 1];
            else if (SECOND < W) y[W] = node(now.b[SECOND < W ? W - SECOND - 1 : 0]);
            else y[W] = R == 2 * W ? x[W - 1] : x[W - 2];        // its own predecessor, or that of the rank it has again
        }
        y[0] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x[H - 1], w64::kDppWaveRor1, 0xf, 0xf, true);
        any = 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            at[i] = __umul24(x[i], (unsigned)N) + y[i];
            const uint32_t word = *(const uint32_t*)((const char*)marks + ((at[i] >> 5) & ~3u));
            hit[i] = __builtin_amdgcn_sbfe((int)word, at[i] >> 2, 1);                    // -1 where it is marked
        }
        if (!whole) hit[0] = 0;
#pragma unroll
        for (int i = 0; i < H; ++i) any |= hit[i];
        if (!own) any = 0;
    };
    if (known) {
        for (int64_t b = first_order; b < B; b += waves) {
            unsigned at[H];
            int hit[H], any, best = 0;
            test(b, at, hit, any);
            if (__ballot(any != 0)) {
                best = top;
            } else {                                             // an order without a marked hop: all of them
                int value[H];
#pragma unroll
                for (int i = 0; i < H; ++i) value[i] = entry(at[i]);
                if (!whole) value[0] = 0;
#pragma unroll
                for (int i = 0; i < H; ++i) best = max(best, value[i]);
                best = wave_max(best);
            }
            if (lane == 0) out[b] = best;
        }
        return;
    }
    // An order's entries are reduced when the next order's hops have been tested.  They are asked for in every order and at one place in the
    // code: waits count the loads behind, over all ways, and a wait for an order's ranks would otherwise be one for the entries of the
    // order before as well (which costs what reducing them later gains).
    int value[H], counts[H], more = 0;
    auto finish = [&](int64_t b) {
        int best = more;
#pragma unroll
        for (int i = 0; i < H; ++i) best = max(best, value[i] & counts[i]);
        best = wave_max(own ? best : 0);
        if (lane == 0) out[b] = best;
    };
    for (int64_t b = first_order; b < B; b += waves) {
        unsigned at[H];
        int hit[H], any, best = 0;
        test(b, at, hit, any);
        const int hits = __popcll(__ballot(any != 0));           // lanes with one
        if (b != first_order) finish(b - waves);
        if (hits > 32) {                                         // a matrix of few values: until one of the largest is met
#pragma unroll
            for (int i0 = 0; i0 < H; i0 += 4) {
                int some[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) some[i] = i0 + i < H ? entry(own ? at[i0 + i] & (unsigned)hit[i0 + i] : 0u) & hit[i0 + i] : 0;
                best = max(max(best, some[0]), max(max(some[1], some[2]), some[3]));
                if (!own) best = 0;
                if (__ballot(best >= top)) break;
            }
#pragma unroll
            for (int i = 0; i < H; ++i) hit[i] = 0;
        } else if (!hits) {                                      // an order without a marked hop: all of them
#pragma unroll
            for (int i = 0; i < H; ++i) hit[i] = i || whole ? -1 : 0;
        }
        more = best;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            counts[i] = own ? hit[i] : 0;
            value[i] = entry(at[i] & (unsigned)counts[i]);
        }
    }
    if (first_order < B) finish(first_order + (B - 1 - first_order) / waves * waves);
}

template <typename RANK, int W, int SECOND>
static hipError_t ring_max_marked_launch(const int32_t* c, int N, const RANK* perms, int64_t B, int64_t* out,
                                         hipStream_t s) {
    const size_t lds = 128 + sizeof(uint32_t) * (((size_t)N * N + 31) / 32);
    hipError_t e = hipFuncSetAttribute((const void*)ring_batch_max_marked_kernel<RANK, W, SECOND>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int64_t blocks = (B + 63) / 64;
    if (blocks > 256) blocks = 256;                             // one per compute unit: each reads the whole matrix
    const int wanted = (256 * 6 + N / 2) / N;                   // of 256 samples: 6 of N, ln N being 5.6 .. 6.9
    hipLaunchKernelGGL((ring_batch_max_marked_kernel<RANK, W, SECOND>), dim3((int)blocks), dim3(1024), lds, s, c, N, perms, B, out,
                       wanted);
    return hipGetLastError();
}
template <typename RANK>
static hipError_t ring_max_marked(const int32_t* c, int N, const RANK* perms, int64_t B, int64_t* out, hipStream_t s) {
    switch ((N + 63) / 64) {
        case 5: return ring_max_marked_launch<RANK, 4, 1>(c, N, perms, B, out, s);
        case 6: return ring_max_marked_launch<RANK, 4, 2>(c, N, perms, B, out, s);
        case 7: return ring_max_marked_launch<RANK, 4, 3>(c, N, perms, B, out, s);
        case 8: return ring_max_marked_launch<RANK, 4, 4>(c, N, perms, B, out, s);
        case 9:
        case 10: return ring_max_marked_launch<RANK, 8, 2>(c, N, perms, B, out, s);
        case 11:
        case 12: return ring_max_marked_launch<RANK, 8, 4>(c, N, perms, B, out, s);
        case 13:
        case 14: return ring_max_marked_launch<RANK, 8, 6>(c, N, perms, B, out, s);
        default: return ring_max_marked_launch<RANK, 8, 8>(c, N, perms, B, out, s);
    }
}

// The threshold and the marking, once per workgroup, take about as long as the generic kernel takes for 8000 (N = 500) to
// 12000 orders (N = 300; generic / marked: N = 300, 20000 orders 26.7 / 17.1 us; N = 1000, 20000 orders 105 / 66 us).  Orders that
// differ in a few ranks ask for the same few entries, which the caches hold: for them the lines meet later (N = 300, 28000
// orders 21.2 / 19.2 us, of two bytes a rank 17.1 / 18.7; N = 1000, 20000 orders 60 / 62, 28000 orders 89 / 68).
constexpr int64_t kRingMaxMarkedMinOrders = 24576;
static bool ring_max_marked_pays(int N, int64_t B) { return N > kRingRowsMaxN && B >= kRingMaxMarkedMinOrders; }

hipError_t launch_ring_cost_batch(const int32_t* c, int N, bool is_max, const int32_t* perms, int64_t B,
                                  int64_t* out, hipStream_t s) {
    if (B == 0) return hipSuccess;
    const bool aligned = ((uintptr_t)perms & 15u) == 0;
    if (aligned) {
        switch (N) {
            case 8: return ring_lds<8>(c, is_max, perms, B, out, s);
            case 16: return ring_lds<16>(c, is_max, perms, B, out, s);
            case 32: return ring_lds<32>(c, is_max, perms, B, out, s);
            case 64: return ring_lds<64>(c, is_max, perms, B, out, s);
            case 128: return ring_lds<128>(c, is_max, perms, B, out, s);
            default: break;
        }
        // staging 128 KiB per compute unit pays from a few ten thousand orders on
        if (N == 256 && B >= 32768)
            return is_max ? ring_n256_launch<true>(c, perms, B, out, s) : ring_n256_launch<false>(c, perms, B, out, s);
    }
    if (ring_rows_pays(N, B))
        return is_max ? ring_rows_launch<int32_t, true>(c, N, perms, B, out, s)
                      : ring_rows_launch<int32_t, false>(c, N, perms, B, out, s);
    if (is_max && ring_max_marked_pays(N, B)) return ring_max_marked(c, N, perms, B, out, s);
    const int grid = batch_grid(4, B);
    if (is_max)
        hipLaunchKernelGGL((ring_batch_generic_kernel<true>), dim3(grid), dim3(256), 0, s, c, N, perms, B, out);
    else
        hipLaunchKernelGGL((ring_batch_generic_kernel<false>), dim3(grid), dim3(256), 0, s, c, N, perms, B, out);
    return hipGetLastError();
}

template <int N>
static hipError_t ring_u8_lds(const int32_t* c, bool is_max, const uint8_t* perms, int64_t B, int64_t* out,
                              hipStream_t s) {
    constexpr int PPW = 64 / (N / 16);
    const int grid = batch_grid((int64_t)PPW * 2 * 4, B);
    if (is_max)
        hipLaunchKernelGGL((ring_batch_u8_lds_kernel<N, true>), dim3(grid), dim3(256), 0, s, c, (const int4*)perms, B,
                           out);
    else
        hipLaunchKernelGGL((ring_batch_u8_lds_kernel<N, false>), dim3(grid), dim3(256), 0, s, c, (const int4*)perms, B,
                           out);
    return hipGetLastError();
}

hipError_t launch_ring_cost_batch_u8(const int32_t* c, int N, bool is_max, const uint8_t* perms, int64_t B,
                                     int64_t* out, hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (((uintptr_t)perms & 15u) == 0) {
        switch (N) {
            case 16: return ring_u8_lds<16>(c, is_max, perms, B, out, s);
            case 32: return ring_u8_lds<32>(c, is_max, perms, B, out, s);
            case 64: return ring_u8_lds<64>(c, is_max, perms, B, out, s);
            case 128: return ring_u8_lds<128>(c, is_max, perms, B, out, s);
            default: break;
        }
    }
    if (ring_rows_pays(N, B))
        return is_max ? ring_rows_launch<uint8_t, true>(c, N, perms, B, out, s)
                      : ring_rows_launch<uint8_t, false>(c, N, perms, B, out, s);
    const int grid = batch_grid(4, B);
    if (is_max)
        hipLaunchKernelGGL((ring_batch_narrow_generic_kernel<uint8_t, true>), dim3(grid), dim3(256), 0, s, c, N, perms, B,
                           out);
    else
        hipLaunchKernelGGL((ring_batch_narrow_generic_kernel<uint8_t, false>), dim3(grid), dim3(256), 0, s, c, N, perms, B,
                           out);
    return hipGetLastError();
}

hipError_t launch_ring_cost_batch_u16(const int32_t* c, int N, bool is_max, const uint16_t* perms, int64_t B,
                                      int64_t* out, hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (ring_rows_pays(N, B))
        return is_max ? ring_rows_launch<uint16_t, true>(c, N, perms, B, out, s)
                      : ring_rows_launch<uint16_t, false>(c, N, perms, B, out, s);
    if (is_max && ring_max_marked_pays(N, B)) return ring_max_marked(c, N, perms, B, out, s);
    const int grid = batch_grid(4, B);
    if (is_max)
        hipLaunchKernelGGL((ring_batch_narrow_generic_kernel<uint16_t, true>), dim3(grid), dim3(256), 0, s, c, N, perms,
                           B, out);
    else
        hipLaunchKernelGGL((ring_batch_narrow_generic_kernel<uint16_t, false>), dim3(grid), dim3(256), 0, s, c, N, perms,
                           B, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------- halving-doubling rounds
// One wave per order.  The order is parked in the wave's LDS slice so that rank i can look up its
// partner i xor 2^k; NM = ceil(N / 64) ranks per lane.  Matrix in LDS when it fits 16 KiB (N <= 64),
// otherwise gathered through L2.
template <int NM, bool LDS_MATRIX>
__global__ __launch_bounds__(256) void rd_batch_kernel(const int32_t* __restrict__ c, int N,
                                                       const int32_t* __restrict__ weights,
                                                       const int32_t* __restrict__ perms, int64_t B,
                                                       int64_t* __restrict__ out,
                                                       const int32_t* __restrict__ skip_if_small) {
    // enqueued beside the folded-matrix kernel: flags[0] = max(c) decides which of the two does the work
    if (skip_if_small && skip_if_small[0] < (1 << 16)) return;
    extern __shared__ int32_t sm[];
    int32_t* order = sm + (threadIdx.x >> 6) * N;   // this wave's slice
    const int32_t* mat = c;
    if (LDS_MATRIX) {
        int32_t* m = sm + 4 * N;
        for (int e = threadIdx.x; e < N * N; e += 256) m[e] = c[e];
        __syncthreads();
        mat = m;
    }
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t b = wave; b < B; b += nwaves) {
        const int32_t* pi = perms + b * N;
        int a[NM];
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            const int p = lane + 64 * k;
            a[k] = p < N ? clampi(pi[p], 0, N - 1) : 0;
            if (p < N) order[p] = a[k];
        }
        __builtin_amdgcn_wave_barrier();
        long long total = 0;
        int round = 0;
        for (int bit = 1; bit < N; bit <<= 1, ++round) {
            int worst = 0;
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                const int p = lane + 64 * k;
                if (p < N) worst = max(worst, mat[a[k] * N + order[p ^ bit]]);
            }
            const long long w = weights ? (long long)clampi(weights[round], 0, kMaxRoundWeight) : 1ll;
            total += w * wave_max(worst);
        }
        __builtin_amdgcn_wave_barrier();   // all partner look-ups done before the slice is overwritten
        if (lane == 0) out[b] = total;
    }
}

// N = 64 with one order per LANE (orders 16-byte aligned): nothing is reduced across lanes.  A wave takes 64 orders:
// sixteen coalesced 1 KiB loads bring them in (lane l of load i holds four ranks of order 4i + l / 16), every rank
// is packed as the byte 4 * node, the packed words go through a 4.25 KiB LDS tile (17 words per order: writes two
// lanes per bank, reads conflict-free) and come back as the lane's own order, 64 bytes in 16 registers.  With all
// loops unrolled every rank of the order is a register with a constant index, so a matrix entry between the nodes
// at two ranks is { address = byte[x] << 6 | byte[y]; gather }, and the lane writes its own cost: 64 consecutive
// results per wave.
constexpr int kLaneTileStride = 17;                 // words per staged order: 16 of packed ranks, 1 of padding

// node4[p] = 4 * node at rank p of order b0 + lane (the last order again beyond the batch's end)
__device__ __forceinline__ void load_order_per_lane(const int4* __restrict__ perms4, int64_t b0, int64_t B,
                                                    uint32_t* tile, int lane, unsigned (&node4)[64]) {
    constexpr int N = 64;
    const int quarter = lane >> 4, piece = lane & 15;
    uint32_t packed[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        int64_t o = b0 + 4 * i + quarter;
        o = o < B ? o : B - 1;
        const int4 v = perms4[o * 16 + piece];
        packed[i] = (uint32_t)(clampi(v.x, 0, N - 1) << 2) | (uint32_t)(clampi(v.y, 0, N - 1) << 10) |
                    (uint32_t)(clampi(v.z, 0, N - 1) << 18) | (uint32_t)(clampi(v.w, 0, N - 1) << 26);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) tile[(4 * i + quarter) * kLaneTileStride + piece] = packed[i];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const uint32_t word = tile[lane * kLaneTileStride + q];
#pragma unroll
        for (int j = 0; j < 4; ++j) node4[4 * q + j] = (word >> (8 * j)) & 0xffu;
    }
    __builtin_amdgcn_wave_barrier();                               // the tile is free for the next 64 orders
}

// stages the matrix; FOLD: both directed entries of a pair replaced by the larger (an exchange costs the slower way)
template <bool FOLD>
__device__ __forceinline__ void stage_matrix_64(const int32_t* __restrict__ c, int32_t* m) {
    constexpr int N = 64;
    for (int e = threadIdx.x; e < N * N; e += 256) m[e] = clampi(c[e], 0, (1 << 21) - 1);
    __syncthreads();
    if (FOLD) {
        w64::for_each_pair_64((int)threadIdx.x, [&](int lo, int hi) {
            const int both = max(m[lo * N + hi], m[hi * N + lo]);
            m[lo * N + hi] = both;
            m[hi * N + lo] = both;
        });
        __syncthreads();
    }
}

// halving-doubling: the 6 x 32 links of an order, one folded entry each
__global__ __launch_bounds__(256) void rd_batch_lanes64_kernel(const int32_t* __restrict__ c,
                                                               const int32_t* __restrict__ weights,
                                                               const int4* __restrict__ perms4, int64_t B,
                                                               int64_t* __restrict__ out) {
    constexpr int N = 64;
    __shared__ int32_t m[N * N];
    __shared__ uint32_t tile_all[4][N * kLaneTileStride];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    stage_matrix_64<true>(c, m);
    const char* mbytes = (const char*)m;
    long long w[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) w[k] = weights ? (long long)clampi(weights[k], 0, kMaxRoundWeight) : 1ll;
    const int64_t tasks = (B + 63) >> 6;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t task = (int64_t)blockIdx.x * 4 + wv; task < tasks; task += nwaves) {
        const int64_t b0 = task << 6;
        unsigned node4[N];
        load_order_per_lane(perms4, b0, B, tile_all[wv], lane, node4);
        long long total = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            int worst = 0;
#pragma unroll
            for (int li = 0; li < N / 2; ++li) {
                const int lo = ((li >> k) << (k + 1)) | (li & ((1 << k) - 1)), hi = lo | (1 << k);
                worst = max(worst, *(const int32_t*)(mbytes + ((node4[lo] << 6) | node4[hi])));
            }
            total += w[k] * worst;
        }
        if (b0 + lane < B) out[b0 + lane] = total;
    }
}

// BCube, base 4: the four ranks that differ in one base-4 digit exchange pairwise; 3 rounds x 16 groups x 6 pairs,
// one folded entry each
__global__ __launch_bounds__(256) void bcube_b4_lanes64_kernel(const int32_t* __restrict__ c,
                                                               const int32_t* __restrict__ weights,
                                                               const int4* __restrict__ perms4, int64_t B,
                                                               int64_t* __restrict__ out) {
    constexpr int N = 64;
    __shared__ int32_t m[N * N];
    __shared__ uint32_t tile_all[4][N * kLaneTileStride];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    stage_matrix_64<true>(c, m);
    const char* mbytes = (const char*)m;
    long long w[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) w[r] = weights ? (long long)clampi(weights[r], 0, kMaxRoundWeight) : 1ll;
    const int64_t tasks = (B + 63) >> 6;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t task = (int64_t)blockIdx.x * 4 + wv; task < tasks; task += nwaves) {
        const int64_t b0 = task << 6;
        unsigned node4[N];
        load_order_per_lane(perms4, b0, B, tile_all[wv], lane, node4);
        long long total = 0;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            int worst = 0;
#pragma unroll
            for (int g = 0; g < N / 4; ++g) {
                const int p0 = ((g >> (2 * r)) << (2 * r + 2)) | (g & ((1 << (2 * r)) - 1));
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int e = d + 1; e < 4; ++e)
                        worst = max(worst, *(const int32_t*)(mbytes + ((node4[p0 | (d << (2 * r))] << 6) |
                                                                       node4[p0 | (e << (2 * r))])));
            }
            total += w[r] * worst;
        }
        if (b0 + lane < B) out[b0 + lane] = total;
    }
}

// Double binary tree over N ranks in registers: the tree over positions LO .. HI hangs below a parent whose node and path cost are
// given; the costliest root-to-leaf path is the largest path cost met.  SHIFT: tree position p holds rank (p + SHIFT) mod N.  Nodes
// times 4, rows of 64 words.
template <int LO, int HI, int SHIFT, int N>
__device__ __forceinline__ void dbt_walk_64(const char* mbytes, const unsigned (&node4)[N], unsigned parent4, int cost,
                                            bool has_parent, int& worst) {
    if constexpr (LO <= HI) {
        constexpr int M = (LO + HI) / 2;
        const unsigned here = node4[(M + SHIFT) % N];
        const int mine = has_parent ? cost + *(const int32_t*)(mbytes + ((parent4 << 6) | here)) : 0;
        worst = max(worst, mine);
        dbt_walk_64<LO, M - 1, SHIFT, N>(mbytes, node4, here, mine, true, worst);
        dbt_walk_64<M + 1, HI, SHIFT, N>(mbytes, node4, here, mine, true, worst);
    }
}

__global__ __launch_bounds__(256) void dbt_lanes64_kernel(const int32_t* __restrict__ c,
                                                          const int4* __restrict__ perms4, int64_t B,
                                                          int64_t* __restrict__ out) {
    constexpr int N = 64;
    __shared__ int32_t m[N * N];
    __shared__ uint32_t tile_all[4][N * kLaneTileStride];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    stage_matrix_64<false>(c, m);
    const char* mbytes = (const char*)m;
    const int64_t tasks = (B + 63) >> 6;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t task = (int64_t)blockIdx.x * 4 + wv; task < tasks; task += nwaves) {
        const int64_t b0 = task << 6;
        unsigned node4[N];
        load_order_per_lane(perms4, b0, B, tile_all[wv], lane, node4);
        int worst = 0;
        dbt_walk_64<0, N - 1, 0, N>(mbytes, node4, 0u, 0, false, worst);
        dbt_walk_64<0, N - 1, 1, N>(mbytes, node4, 0u, 0, false, worst);
        if (b0 + lane < B) out[b0 + lane] = worst;
    }
}

// N = 64: a round costs the largest of its 32 links and a link costs the larger of its two directed entries, so the
// kernel folds the two entries of every pair into both places while staging (max(c[x][y], c[y][x])) and then scores
// links, not ranks: the 6 x 32 links of an order are three gathers per lane (lanes 0..31 one round, lanes 32..63 the
// next), and the six maxima come from three reductions over half waves.
__global__ __launch_bounds__(256) void rd_batch_links64_kernel(const int32_t* __restrict__ c,
                                                               const int32_t* __restrict__ weights,
                                                               const int32_t* __restrict__ perms, int64_t B,
                                                               int64_t* __restrict__ out) {
    constexpr int N = 64;
    __shared__ int32_t m[N * N];
    __shared__ int32_t order_all[4][N];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    for (int e = threadIdx.x; e < N * N; e += 256) m[e] = clampi(c[e], 0, (1 << 21) - 1);
    __syncthreads();
    w64::for_each_pair_64((int)threadIdx.x, [&](int lo, int hi) {
        const int both = max(m[lo * N + hi], m[hi * N + lo]);
        m[lo * N + hi] = both;
        m[hi * N + lo] = both;
    });
    __syncthreads();
    int32_t* order = order_all[wv];
    const int64_t wave = (int64_t)blockIdx.x * 4 + wv;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    long long w[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) w[k] = weights ? (long long)clampi(weights[k], 0, kMaxRoundWeight) : 1ll;
    // link j of this lane: round k = 2j + (lane >> 5), link index lane & 31 = the lower rank with bit k taken out
    int lower[3], upper[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int k = 2 * j + (lane >> 5), li = lane & 31;
        lower[j] = ((li >> k) << (k + 1)) | (li & ((1 << k) - 1));
        upper[j] = lower[j] | (1 << k);
    }
    int next = wave < B ? perms[wave * N + lane] : 0;
    for (int64_t b = wave; b < B; b += nwaves) {
        order[lane] = clampi(next, 0, N - 1);
        const int64_t bn = b + nwaves;
        next = bn < B ? perms[bn * N + lane] : 0;
        __builtin_amdgcn_wave_barrier();
        int v[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) v[j] = m[order[lower[j]] * N + order[upper[j]]];
        __builtin_amdgcn_wave_barrier();   // all look-ups done before the slice is overwritten
        half_wave_max3(v[0], v[1], v[2]);
        long long total = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j)
            total += w[2 * j] * __builtin_amdgcn_readlane(v[j], 31) + w[2 * j + 1] * __builtin_amdgcn_readlane(v[j], 63);
        if (lane == 0) out[b] = total;
    }
}

template <int NM>
static hipError_t rd_launch(const int32_t* c, int N, const int32_t* weights, const int32_t* perms, int64_t B,
                            int64_t* out, const int32_t* skip_if_small, hipStream_t s) {
    const int grid = batch_grid(4, B);
    if (N <= 64) {
        const size_t lds = sizeof(int32_t) * (size_t)(4 * N + N * N);
        hipLaunchKernelGGL((rd_batch_kernel<NM, true>), dim3(grid), dim3(256), lds, s, c, N, weights, perms, B, out,
                           skip_if_small);
    } else {
        const size_t lds = sizeof(int32_t) * (size_t)(4 * N);
        hipLaunchKernelGGL((rd_batch_kernel<NM, false>), dim3(grid), dim3(256), lds, s, c, N, weights, perms, B, out,
                           skip_if_small);
    }
    return hipGetLastError();
}

// N = 128, 256 (small batches) on a folded 16-bit copy of the matrix, folded[x][y] = max(c[x][y], c[y][x]) (fold_to_u16_kernel): a
// link, the two ranks i and i xor 2^k, is one look-up by one lane instead of one per end, so a round is N / 2
// scattered L2 requests instead of N - and that request rate is what bounds this kernel.  One wave per order, the
// order parked in LDS; every lane first takes the maximum over its links of every round (all gathers independent),
// then the rounds' maxima are reduced over the wave three at a time.  Returns at once when the matrix has an entry
// from 2^16 up (flags[0] = max(c)): the general kernel, enqueued beside it, then does the work.
template <int LOGN>
__global__ __launch_bounds__(256) void rd_batch_folded_kernel(const uint16_t* __restrict__ folded,
                                                              const int32_t* __restrict__ weights,
                                                              const int32_t* __restrict__ perms, int64_t B,
                                                              int64_t* __restrict__ out,
                                                              const int32_t* __restrict__ flags) {
    constexpr int N = 1 << LOGN, NM = N / 64, LM = NM / 2;      // ranks and links per lane
    if (flags[0] >= (1 << 16)) return;
    __shared__ int32_t order_all[4][N];
    int32_t* order = order_all[threadIdx.x >> 6];
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    long long w[LOGN];
#pragma unroll
    for (int k = 0; k < LOGN; ++k) w[k] = weights ? (long long)clampi(weights[k], 0, kMaxRoundWeight) : 1ll;
    for (int64_t b = wave; b < B; b += nwaves) {
        const int32_t* pi = perms + b * N;
#pragma unroll
        for (int k = 0; k < NM; ++k) order[lane + 64 * k] = clampi(pi[lane + 64 * k], 0, N - 1);
        __builtin_amdgcn_wave_barrier();
        int worst[LOGN + 2];
        worst[LOGN] = worst[LOGN + 1] = 0;
#pragma unroll
        for (int k = 0; k < LOGN; ++k) {
            const int bit = 1 << k;
            int v = 0;
#pragma unroll
            for (int u = 0; u < LM; ++u) {
                const int i = lane + 64 * u;                                      // link index
                const int j = ((i >> k) << (k + 1)) | (i & (bit - 1));            // its lower rank
                const unsigned at = ((unsigned)order[j] << (LOGN + 1)) | ((unsigned)order[j | bit] << 1);
                v = max(v, (int)*(const uint16_t*)((const char*)folded + at));
            }
            worst[k] = v;
        }
        __builtin_amdgcn_wave_barrier();   // all look-ups done before the slice is overwritten
#pragma unroll
        for (int k = 0; k < LOGN; k += 3) wave_max3(worst[k], worst[k + 1], worst[k + 2]);
        long long total = 0;
#pragma unroll
        for (int k = 0; k < LOGN; ++k) total += w[k] * worst[k];
        if (lane == 0) out[b] = total;
    }
}

// N = 128, 256 for large batches, matrix in LDS: a 1024-thread workgroup per compute unit stages the matrix as 16-bit
// entries, folds the two directions of every pair into both places (every unordered pair once) and then scores one
// order per wave as rd_batch_folded_kernel / bcube_b4_folded_kernel do, with LDS gathers instead of L2 requests.
// The workgroup finds the matrix maximum while staging; with an entry outside 0 .. 2^16 - 1 its links are scored from
// the caller's matrix through L2 (both directions per link).  BCUBE4: base-4 BCube rounds instead of halving-doubling.
template <int LOGN, bool BCUBE4>
__global__ __launch_bounds__(1024) void links_batch_lds16_kernel(const int32_t* __restrict__ c,
                                                                 const int32_t* __restrict__ weights,
                                                                 const int32_t* __restrict__ perms, int64_t B,
                                                                 int64_t* __restrict__ out) {
    constexpr int N = 1 << LOGN, NM = N / 64, ROUNDS = BCUBE4 ? LOGN / 2 : LOGN;
    static_assert(!BCUBE4 || LOGN % 2 == 0, "base 4 needs an even log2 N");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_links[];
    uint16_t* m16 = (uint16_t*)smem_links;                                  // [N * N]
    int32_t* order_all = (int32_t*)(smem_links + sizeof(uint16_t) * N * N);  // [16][N]
    __shared__ unsigned wave_top[16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    unsigned top = 0;
    for (int e = tid; e < N * N; e += 1024) {
        const unsigned v = (unsigned)c[e];                 // a negative entry counts as too large
        top = max(top, v);
        m16[e] = (uint16_t)v;
    }
    top = (unsigned)wave_max((int)min(top, 0x7fffffffu));
    if (lane == 0) wave_top[wv] = top;
    __syncthreads();
    unsigned all_top = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) all_top = max(all_top, wave_top[k]);
    const bool in_lds = all_top < (1u << 16);
    if (in_lds) {
        // the threads of rank p take the pairs {p, p + j}, j = 1 .. N/2: every unordered pair exactly once
        const int p = tid & (N - 1);
        for (int j = 1 + (tid >> LOGN); j <= N / 2; j += 1024 / N) {
            const int b = (p + j) & (N - 1);
            if (j < N / 2 || p < N / 2) {
                const uint16_t both = max(m16[p * N + b], m16[b * N + p]);
                m16[p * N + b] = both;
                m16[b * N + p] = both;
            }
        }
    }
    __syncthreads();
    auto pair_value = [&](int x, int y) {
        if (in_lds) return (int)*(const uint16_t*)((const char*)m16 + ((x << (LOGN + 1)) | (y << 1)));
        return max(clampi(c[x * N + y], 0, (1 << 21) - 1), clampi(c[y * N + x], 0, (1 << 21) - 1));
    };
    int32_t* order = order_all + wv * N;
    long long w[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) w[r] = weights ? (long long)clampi(weights[r], 0, kMaxRoundWeight) : 1ll;
    const int64_t nwaves = (int64_t)gridDim.x * 16;
    for (int64_t b = (int64_t)blockIdx.x * 16 + wv; b < B; b += nwaves) {
        const int32_t* pi = perms + b * N;
#pragma unroll
        for (int k = 0; k < NM; ++k) order[lane + 64 * k] = clampi(pi[lane + 64 * k], 0, N - 1);
        __builtin_amdgcn_wave_barrier();
        int worst[ROUNDS + 2];
        worst[ROUNDS] = worst[ROUNDS + 1] = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            int v = 0;
            if (BCUBE4) {
#pragma unroll
                for (int u = 0; u < N / 256; ++u) {
                    const int g = lane + 64 * u;                                   // group: the rank without digit r
                    const int p0 = ((g >> (2 * r)) << (2 * r + 2)) | (g & ((1 << (2 * r)) - 1));
                    int node[4];
#pragma unroll
                    for (int d = 0; d < 4; ++d) node[d] = order[p0 | (d << (2 * r))];
#pragma unroll
                    for (int d = 0; d < 3; ++d)
#pragma unroll
                        for (int e = d + 1; e < 4; ++e) v = max(v, pair_value(node[d], node[e]));
                }
            } else {
                const int bit = 1 << r;
#pragma unroll
                for (int u = 0; u < NM / 2; ++u) {
                    const int i = lane + 64 * u;                                   // link index
                    const int j = ((i >> r) << (r + 1)) | (i & (bit - 1));         // its lower rank
                    v = max(v, pair_value(order[j], order[j | bit]));
                }
            }
            worst[r] = v;
        }
        __builtin_amdgcn_wave_barrier();   // all look-ups done before the slice is overwritten
#pragma unroll
        for (int r = 0; r < ROUNDS; r += 3) wave_max3(worst[r], worst[r + 1], worst[r + 2]);
        long long total = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) total += w[r] * worst[r];
        if (lane == 0) out[b] = total;
    }
}

// N = 512, 1024 with a workspace, halving-doubling and (N = 1024) BCube base 4: a round costs its largest link, so only links among the largest entries have to be
// looked up exactly.  mark_links_kernel writes one bit per pair of nodes, "the larger direction costs T or more" (128 KiB
// at N = 1024, which fits LDS; the 16-bit folded matrix, 2 MiB, does not); T is chosen so that about 5 of a
// round's N / 2 links carry the bit, from the same 2048 sampled entries in every workgroup: 4 to 7 of them take the same time
// within 4 %, with fewer the rounds without a marked link, whose links are all looked up, cost more than the exact look-ups
// saved (N = 512, 65536 orders, 2.6 / 4 / 5 / 8 of 256: 93 / 76 / 75 / 80 us).  Any T gives the right result, only the time
// depends on it.  The samples lie apart, so that T does not follow how the nodes are numbered: 256 places of 4 x 4 neighbouring
// pairs held one value sixteen times where the numbers follow the hosts, and five times as many links were marked (pairs that
// cost what their hosts do, 65536 orders: N = 1024 187 us, now 138; N = 512 89, now 75; numbers in no order 137 and 75 either
// way); 4096 places of their own mark no better and take 8 us to read at N = 1024.
// A word holds the pairs of x with the 32 nodes that share their low LOGN - 5 bits with y, the bit of y's high bits h at 31 - h, so that
// a shift by h puts it at the top.  Its byte address takes bits from x and bits from y, all of which mark_word<LOGN> of either
// holds in their places: one v_bfi per look-up.  tops[workgroup] = largest entry seen, tops[kMarkBlocks] = T, for the early end in rd_batch_marked_kernel.
// Behind the marks (N^2 / 8 bytes) the folded entries themselves, 16 bits each, lower triangle with diagonal by rows
// (N (N + 1) bytes, both within the workspace's 2 N^2): an exact look-up is then one request; used when all fit 16 bits.
// Behind those the workgroups' largest entries.  A workgroup per compute unit (64 workgroups: 16.5 us, 256: 15.6).
constexpr int kMarkBlocks = 256;
constexpr size_t mark_tops_offset(size_t N) { return N * N / 8 + N * (N + 1); }

// Of an address in the marks, what x gives: node << 3 or 4, its low bits in the bank's; the others are y's low bits.  y's high bits,
// the shift, are bits 8 .. 12 of its own word.
template <int LOGN>
constexpr unsigned kMarkX = LOGN == 10 ? 0x1ff8u : 0x1ff0u;
template <int LOGN>
__device__ __forceinline__ unsigned mark_word(unsigned node) {
    if (LOGN == 10) return (__umul24(node, 0x2008u) & 0x1fff8u) | ((node >> 2) & 4u);
    return (__umul24(node, 0x2010u) & 0x7ff0u) | (node & 12u);
}

template <int LOGN, int WANTED>
__global__ __launch_bounds__(1024) void mark_links_kernel(const int32_t* __restrict__ c, uint32_t* __restrict__ marks,
                                                          int32_t* __restrict__ tops) {
    constexpr int N = 1 << LOGN;
    constexpr int kRows = N * N / 64 / (16 * kMarkBlocks);                      // rows of 64 entries per wave
    uint16_t* folded = (uint16_t*)(marks + N * N / 32);
    constexpr int kGroupRows = kRows * 16 * 64 / N, kLow = LOGN - 5;            // rows of N entries per workgroup
    __shared__ int per_wave[16], wave_top[16];
    __shared__ uint32_t row_bits[kGroupRows][N / 32];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    auto entry = [&](int x, int y) { return clampi(max(c[x * N + y], c[y * N + x]), 0, (1 << 21) - 1); };
    int v[2];
    {
        // two lanes share a place: the pairs of x, x ^ 16 with y, y ^ 16, two cache lines for both directions of a lane's two
        const uint32_t h = (uint32_t)splitmix64_at(0, (uint64_t)((threadIdx.x >> 1) + 1));
        const int x = (h & (N - 1)) ^ ((lane & 1) << 4), y = (h >> LOGN) & (N - 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) v[i] = entry(x, x == (y ^ (i << 4)) ? x ^ 1 : y ^ (i << 4));
    }
    // a wave takes 64 consecutive x and kRows consecutive y, so both directions come from few cache lines
    const int w = blockIdx.x * 16 + wv, x0 = (w & (N / 64 - 1)) * 64, y0 = (w / (N / 64)) * kRows;
    int e[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) e[k] = entry(x0 + lane, y0 + k);
    const int T = sampled_threshold<5>(v, WANTED, per_wave);
    int top = 0;
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = y0 + k;
        const unsigned long long bits = __ballot(e[k] >= T);
        top = max(top, e[k]);
        if (lane < 2) row_bits[y - kGroupRows * blockIdx.x][(x0 >> 5) + lane] = lane ? (uint32_t)(bits >> 32) : (uint32_t)bits;
        if (x0 + lane <= y) folded[y * (y + 1) / 2 + x0 + lane] = (uint16_t)e[k];
    }
    top = wave_max(top);
    if (lane == 0) wave_top[wv] = top;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 16; ++k) top = max(top, wave_top[k]);
        tops[blockIdx.x] = top;
        if (blockIdx.x == 0) tops[kMarkBlocks] = T;
    }
    // the rows' bits into words of nodes with the same low bits, half a wave per word
#pragma unroll
    for (int i = 0; i < (kGroupRows << kLow) / 32; ++i) {
        const int o = 32 * i + 2 * wv + (lane >> 5), row = o >> kLow, low = o & ((1 << kLow) - 1);
        const int x = low | ((31 - (lane & 31)) << kLow);
        const unsigned long long bits = __ballot((row_bits[row][x >> 5] >> (x & 31)) & 1u);
        const unsigned at = (mark_word<LOGN>(kGroupRows * blockIdx.x + row) & kMarkX<LOGN>) | (mark_word<LOGN>(low) & ~kMarkX<LOGN>);
        if ((lane & 31) == 0) marks[at >> 2] = lane ? (uint32_t)(bits >> 32) : (uint32_t)bits;
    }
}

// The two ends of the links of ranks that differ in lane bit M < 4, or (M = 4, 5) in lane bits 0 and 1, 2 and 3 both, from the registers v[2u] and v[2u + 1]: a lane with the bit clear
// takes the link of the even register, a lane with the bit set that of the odd one, so the 64 lanes hold 64 different links.  One
// instruction per end: the lane's own register or, through DPP, its partner's other one.  A DPP operand must have been written
// two instructions before: one wait for four of them.
#define CC_LANE_ENDS(dpp_x, dpp_y)                                                                                     \
    asm("s_mov_b64 vcc, %12\n\ts_nop 0\n\t"                                                                            \
        "v_cndmask_b32_dpp %0, %5, %4, vcc " dpp_x " row_mask:0xf bank_mask:0xf\n\t"                                   \
        "v_cndmask_b32_dpp %1, %7, %6, vcc " dpp_x " row_mask:0xf bank_mask:0xf\n\t"                                   \
        "v_cndmask_b32_dpp %2, %9, %8, vcc " dpp_x " row_mask:0xf bank_mask:0xf\n\t"                                   \
        "v_cndmask_b32_dpp %3, %11, %10, vcc " dpp_x " row_mask:0xf bank_mask:0xf"                                     \
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])                                                           \
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "s"(~kUpper) : "vcc"); \
    asm("s_mov_b64 vcc, %12\n\ts_nop 0\n\t"                                                                            \
        "v_cndmask_b32_dpp %0, %4, %5, vcc " dpp_y " row_mask:0xf bank_mask:0xf\n\t"                                   \
        "v_cndmask_b32_dpp %1, %6, %7, vcc " dpp_y " row_mask:0xf bank_mask:0xf\n\t"                                   \
        "v_cndmask_b32_dpp %2, %8, %9, vcc " dpp_y " row_mask:0xf bank_mask:0xf\n\t"                                   \
        "v_cndmask_b32_dpp %3, %10, %11, vcc " dpp_y " row_mask:0xf bank_mask:0xf"                                     \
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])                                                           \
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "s"(kUpper) : "vcc")
template <int M>
__device__ __forceinline__ void lane_links(const unsigned* v, unsigned (&x)[4], unsigned (&y)[4]) {
    constexpr unsigned long long kUpper = M == 0 || M == 4 ? 0xaaaaaaaaaaaaaaaaull : M == 1 ? 0xccccccccccccccccull : M == 3 ? 0xff00ff00ff00ff00ull : 0xf0f0f0f0f0f0f0f0ull;
    if constexpr (M == 0) {
        CC_LANE_ENDS("quad_perm:[1,0,3,2]", "quad_perm:[1,0,3,2]");
    } else if constexpr (M == 1) {
        CC_LANE_ENDS("quad_perm:[2,3,0,1]", "quad_perm:[2,3,0,1]");
    } else if constexpr (M == 2) {
        CC_LANE_ENDS("row_ror:4", "row_ror:12");
    } else if constexpr (M == 4) {
        CC_LANE_ENDS("quad_perm:[3,2,1,0]", "quad_perm:[3,2,1,0]");
    } else if constexpr (M == 5) {
        CC_LANE_ENDS("row_ror:12", "row_ror:4");
    } else {
        CC_LANE_ENDS("row_ror:8", "row_ror:8");
    }
}
#undef CC_LANE_ENDS

// One order per wave, its ranks in registers: lane l holds ranks 256 q + 4 l + j (register 4 q + j), so rounds 0, 1 and
// 8, 9 pair registers of a lane and rounds 2 .. 7 pair lanes.  A link is at most one VALU instruction per end to bring the ends together,
// one for the address, one LDS look-up and two to shift its bit into the lane's word of tested links.  The marked ones, about 60 of
// 5120 at N = 1024, are then looked up exactly, each lane its first and its last one at a time, all rounds mixed, their maxima
// formed in LDS.  A round without a marked link is looked up whole; one that has reached the matrix maximum is finished, so a
// matrix of few values ends early, and where T is the maximum nothing is looked up at all.
// What bounds it: N = 1024, 65536 orders keep LDS (6.4 clocks per look-up of 64 random words, two thirds of them bank conflicts) and VALU
// busy for 60 % of the time each at 2.4 GHz, 75 % in a run at 2.0 GHz that took as long (620 instructions per order, 880 before the address was one instruction and
// the bit two); fifteen wavefronts are what fits beside the marks.  Both launches together, seeded orders, before -> now: N = 1024,
// 65536 orders 137 -> 116 us, 1000 orders 22.0 -> 20.9; N = 512, 131072 orders 142 -> 115 us, 65536 75 -> 62 us, 8000 18.4 -> 17.0;
// two values, 16384 orders N = 1024 87 -> 39 us, N = 512 56 -> 20; 16384 orders near a search's result as before (102 -> 101, 52.2
// -> 52.0).  A link's word is asked for twelve links before it is used (eight at a time, waited for together: 121 us).  Through the folded
// 16-bit matrix, bound by L2 requests: 1384 us and 1136.  Orders without any marked link, every link looked up: N = 1024, 65536
// orders 1213 -> 1227 us, N = 512 458 -> 455 us.  So nothing else serves these sizes.
// BCube base 4, N = 1024 (half as many links marked for the rounds are three times as long): 7680 links per order, before from the folded
// matrix through L2 (bcube_b4_folded_kernel): 65536 seeded orders 1964 -> 150 us, of entries from 2^16 up 4939 -> 153, a search's results
// 1979 -> 338; 1000 orders 116 -> 23, one order 90 -> 15.
// BCUBE4: the 4 x 3 / 2 links of a group of four ranks are those of its two rank bits and those of ranks that differ in both.
template <int LOGN, bool BCUBE4>
__global__ __launch_bounds__(LOGN == 10 ? 960 : 1024) void rd_batch_marked_kernel(
    const int32_t* __restrict__ c, const uint32_t* __restrict__ marks, const int32_t* __restrict__ tops,
    const int32_t* __restrict__ weights, const int32_t* __restrict__ perms, int64_t B, int64_t* __restrict__ out) {
    constexpr int N = 1 << LOGN, RK = N / 64, LM = RK / 2, Q = N / 256;         // ranks, links, quads of ranks per lane
    constexpr int WAVES = LOGN == 10 ? 15 : 16, ROUNDS = BCUBE4 ? LOGN / 2 : LOGN;
    constexpr int KINDS = BCUBE4 ? LOGN + LOGN / 2 : LOGN, kLinks = LM * KINDS, WORDS = (kLinks + 31) / 32, kIdle = 32 * WORDS - kLinks;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_marked[];
    uint32_t* lmarks = (uint32_t*)smem_marked;                                              // [N * N / 32], at LDS address 0, which the build checks: the kernel has no other LDS
    uint16_t* order = (uint16_t*)(smem_marked + N * N / 8) + (threadIdx.x >> 6) * N;        // [WAVES][N]
    int* worst = (int*)(smem_marked + N * N / 8 + sizeof(uint16_t) * WAVES * N) + (threadIdx.x >> 6) * 16;  // [WAVES][16]
    // by its place in the order of testing: lower rank of the link but for the lane's part << 0, round << 10, lane bit that counts << 14
    // and whether one does << 19, whether the lanes have changed places << 20, the bits in which the other rank differs << 21
    int* links = (int*)(smem_marked + N * N / 8 + (sizeof(uint16_t) * N + sizeof(int) * 16) * WAVES);       // [kLinks]
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    // links tested nth: of rank bit kind, or of both bits of digit kind - LOGN
    auto kind_of = [](int nth) {
        if (BCUBE4) {
            const int digit = nth < 9 ? nth / 3 : nth < 12 ? 4 : 3;
            return nth % 3 < 2 ? 2 * digit + nth % 3 : LOGN + digit;
        }
        return nth < 6 ? nth : LOGN == 10 ? (nth < 8 ? nth + 2 : nth - 2) : nth == 6 ? 8 : nth - 1;
    };
    auto round_of = [=](int nth) {
        const int kind = kind_of(nth);
        return !BCUBE4 ? kind : kind < LOGN ? kind >> 1 : kind - LOGN;
    };
    auto round_bits = [](int nth) {                                              // in its word of tested links
        const int from = nth * LM, in_word = kLinks - (from & ~31) < 32 ? kLinks - (from & ~31) : 32;
        return ((1u << LM) - 1) << (in_word - (from & 31) - LM);
    };
    if ((int)threadIdx.x < kLinks) {
        const int u = threadIdx.x % LM, nth = threadIdx.x / LM, kind = kind_of(nth);
        const int both = kind >= LOGN, bit = both ? 2 * (kind - LOGN) : kind;                       // the lower one
        const bool in_lane = bit >= 2 && bit < 8, swapped = kind == 7 || (both && bit == 6);
        const int r = bit < 2 ? bit : bit - 6;                                                      // of the register's number
        const int i = in_lane ? 2 * u : ((u >> r) << (r + 1)) | (u & ((1 << r) - 1));               // register
        links[threadIdx.x] = (256 * (i >> 2) + (i & 3)) | round_of(nth) << 10 | (in_lane && !swapped ? (bit - 2) << 14 | 1 << 19 : 0) |
                             (swapped ? 1 << 20 : 0) | (both ? 3 : 1) << (21 + bit);
    }
    const int lane_swapped = (lane >> 5) << 6 | (lane & 15) << 2 | (lane >> 4 & 1);
    for (int e = threadIdx.x; e < N * N / 128; e += 64 * WAVES) ((int4*)lmarks)[e] = ((const int4*)marks)[e];
    int top = 0;
#pragma unroll
    for (int k = 0; k < kMarkBlocks; k += 64) top = max(top, tops[k + lane]);
    top = wave_max(top);
    const bool marked_is_top = tops[kMarkBlocks] >= top;
    const long long weight =
        lane < ROUNDS ? (weights ? (long long)clampi(weights[lane], 0, kMaxRoundWeight) : 1ll) : 0ll;
    __syncthreads();
    const uint16_t* folded = (const uint16_t*)(marks + N * N / 32);
    const bool halves = top < (1 << 16);
    auto exact = [&](int x, int y) {
        if (halves) {
            const int hi = max(x, y), lo = min(x, y);
            return (int)folded[hi * (hi + 1) / 2 + lo];
        }
        return clampi(max(c[x * N + y], c[y * N + x]), 0, (1 << 21) - 1);
    };
    const bool aligned = ((uintptr_t)perms & 15u) == 0;
    auto load = [&](int64_t b, int4 (&v)[Q]) {
        const int32_t* pi = perms + b * N + 4 * lane;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (aligned) v[q] = *(const int4*)(pi + 256 * q);
            else v[q] = make_int4(pi[256 * q], pi[256 * q + 1], pi[256 * q + 2], pi[256 * q + 3]);
        }
    };
    const int64_t nwaves = (int64_t)gridDim.x * WAVES;
    int64_t b = (int64_t)blockIdx.x * WAVES + wv;
    int4 v[Q];
    if (b < B) load(b, v);
    for (; b < B; b += nwaves) {
        unsigned X[RK];                                                          // mark_word of the node
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const unsigned n[4] = {(unsigned)clampi(v[q].x, 0, N - 1), (unsigned)clampi(v[q].y, 0, N - 1), (unsigned)clampi(v[q].z, 0, N - 1),
                                   (unsigned)clampi(v[q].w, 0, N - 1)};
            const uint2 four = make_uint2(n[0] | n[1] << 16, n[2] | n[3] << 16);
            __builtin_memcpy(__builtin_assume_aligned(order + 256 * q + 4 * lane, 8), &four, 8);
#pragma unroll
            for (int j = 0; j < 4; ++j) X[4 * q + j] = mark_word<LOGN>(n[j]);
        }
        if (lane < 16) worst[lane] = -1;
        if (b + nwaves < B) load(b + nwaves, v);
        // a bit per link, LM of each kind, the first one tested on top
        uint32_t hits[WORDS] = {};
        // A link's word is asked for kAhead links before its bit is taken.
        constexpr int kAhead = 12;
        int asked = 0, taken = 0;                                                // constants at every use
        uint32_t word[2 * kAhead];
        unsigned shift[2 * kAhead];
        auto take = [&] {
            uint32_t shifted;
            asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD"
                : "=v"(shifted) : "v"(shift[taken % (2 * kAhead)]), "v"(word[taken % (2 * kAhead)]));
            hits[taken >> 5] = __builtin_amdgcn_alignbit(hits[taken >> 5], shifted, 31);
            ++taken;
        };
        auto test = [&](unsigned x, unsigned y) {
            // written out: the compiler masks both ends and adds a base that is 0
            uint32_t at;
            asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(at) : "s"(kMarkX<LOGN>), "v"(x), "v"(y));
            word[asked % (2 * kAhead)] = *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)at;
            shift[asked % (2 * kAhead)] = y;
            if (++asked % 4 == 0) {
                __builtin_amdgcn_sched_barrier(0);
                while (taken + kAhead < asked) take();
            }
        };
        auto lane_round = [&](auto m) {
#pragma unroll
            for (int u = 0; u < LM; u += 4) {
                unsigned x[4], y[4];
                lane_links<decltype(m)::value>(X + 2 * u, x, y);
#pragma unroll
                for (int i = 0; i < 4; ++i) test(x[i], y[i]);
            }
        };
        auto register_round = [&](auto m) {
            constexpr int bit = decltype(m)::value;
#pragma unroll
            for (int u = 0; u < LM; ++u) {
                const int i = ((u >> bit) << (bit + 1)) | (u & ((1 << bit) - 1));
                test(X[i], X[i | (1 << bit)]);
            }
        };
        // ranks that differ in both register bits from `bit` on
        auto both_round = [&](auto m) {
            constexpr int bit = decltype(m)::value;
#pragma unroll
            for (int u = 0; u < LM; ++u) {
                const int i = ((u >> bit) << (bit + 1)) | (u & ((1 << bit) - 1));
                test(X[i], X[i ^ (3 << bit)]);
            }
        };
        register_round(std::integral_constant<int, 0>{});
        register_round(std::integral_constant<int, 1>{});
        if constexpr (BCUBE4) both_round(std::integral_constant<int, 0>{});
        lane_round(std::integral_constant<int, 0>{});
        lane_round(std::integral_constant<int, 1>{});
        if constexpr (BCUBE4) lane_round(std::integral_constant<int, 4>{});
        lane_round(std::integral_constant<int, 2>{});
        lane_round(std::integral_constant<int, 3>{});
        if constexpr (BCUBE4) lane_round(std::integral_constant<int, 5>{});
        register_round(std::integral_constant<int, 2>{});
        if constexpr (LOGN == 10) register_round(std::integral_constant<int, 3>{});
        if constexpr (BCUBE4) both_round(std::integral_constant<int, 2>{});
        // Lane bits 4 and 5 change places with the lowest bit of the register's number: a swap per two registers, after which they hold
        // the two ends (and rank bit 0 is where bit 6 was, then bit 6 where bit 7 was)
#pragma unroll
        for (int u = 0; u < LM; ++u) {
            const auto r = __builtin_amdgcn_permlane16_swap(X[2 * u], X[2 * u + 1], false, false);
            X[2 * u] = r[0];
            X[2 * u + 1] = r[1];
            test(r[0], r[1]);
        }
#pragma unroll
        for (int u = 0; u < LM; ++u) {
            const auto r = __builtin_amdgcn_permlane32_swap(X[2 * u], X[2 * u + 1], false, false);
            X[2 * u] = r[0];
            X[2 * u + 1] = r[1];
            test(r[0], r[1]);
        }
        if constexpr (BCUBE4) {
#pragma unroll
            for (int u = 0; u < LM; ++u) {
                const auto r = __builtin_amdgcn_permlane32_swap(X[2 * u + 1], X[2 * u + 1], false, false);
                test(X[2 * u], lane < 32 ? r[1] : r[0]);
            }
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) take();
        __builtin_amdgcn_wave_barrier();
        uint32_t finished = 0;
        if (marked_is_top) {
            // a matrix of few values: a marked link is worth the matrix maximum, which ends its round
#pragma unroll
            for (int nth = 0; nth < KINDS; ++nth) finished |= __ballot(hits[nth * LM >> 5] & round_bits(nth)) ? 1u << round_of(nth) : 0u;
            if (lane < ROUNDS && (finished >> lane & 1)) worst[lane] = top;
#pragma unroll
            for (int w = 0; w < WORDS; ++w) hits[w] = 0;
            __builtin_amdgcn_wave_barrier();
        }
        for (;;) {
            uint32_t any = 0;
#pragma unroll
            for (int w = 0; w < WORDS; ++w) any |= hits[w];
            if (__ballot(any != 0) == 0) break;
            // a lane's first and its last link, their look-ups in flight together
            uint32_t first = hits[WORDS - 1], last = hits[0];
            int in_first = WORDS - 1, in_last = 0;
#pragma unroll
            for (int w = 1; w < WORDS; ++w) {
                in_first = hits[WORDS - 1 - w] ? WORDS - 1 - w : in_first;
                first = hits[WORDS - 1 - w] ? hits[WORDS - 1 - w] : first;
                in_last = hits[w] ? w : in_last;
                last = hits[w] ? hits[w] : last;
            }
            const int from_top = __builtin_clz(first | 1u), from_bottom = __builtin_ctz(last | 0x80000000u);
            const uint32_t bit_first = any ? 0x80000000u >> from_top : 0u, bit_last = any ? 1u << from_bottom : 0u;
#pragma unroll
            for (int w = 0; w < WORDS; ++w) hits[w] &= ~((in_first == w ? bit_first : 0u) | (in_last == w ? bit_last : 0u));
            const int at[2] = {32 * in_first + from_top - (in_first == WORDS - 1 ? kIdle : 0),
                               32 * in_last + 31 - from_bottom - (in_last == WORDS - 1 ? kIdle : 0)};
            int k[2], x[2], y[2], value[2];
            if (any) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const unsigned link = (unsigned)links[at[i]];
                    k[i] = (int)(link >> 10 & 15);
                    const int p = (int)(link & 1023) + (link >> 20 & 1 ? lane_swapped : 4 * lane) +
                                  (int)__builtin_amdgcn_ubfe((unsigned)lane, link >> 14 & 31, link >> 19 & 1);
                    x[i] = order[p];
                    y[i] = order[p ^ (int)(link >> 21)];
                }
                if (halves) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const unsigned hi = (unsigned)max(x[i], y[i]), lo = (unsigned)min(x[i], y[i]);
                        value[i] = folded[(__umul24(hi, hi + 1) >> 1) + lo];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i) value[i] = exact(x[i], y[i]);
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) atomicMax(worst + k[i], value[i]);
            }
            __builtin_amdgcn_wave_barrier();
            const uint32_t full = (uint32_t)__ballot(lane < ROUNDS && *(volatile int*)(worst + (lane & 15)) >= top);
            if (full != finished) {
                finished = full;
#pragma unroll
                for (int nth = 0; nth < KINDS; ++nth)
                    if ((full >> round_of(nth)) & 1) hits[nth * LM >> 5] &= ~round_bits(nth);
            }
        }
        int mine = lane < ROUNDS ? *(volatile int*)(worst + (lane & 15)) : 0;
        for (uint32_t missing = (uint32_t)__ballot(mine < 0); missing; missing &= missing - 1) {
            const int k = __builtin_ctz(missing);
            int t = 0;
            for (int j = 0; j < (BCUBE4 ? 3 : 1); ++j) {
                const int bit = BCUBE4 ? 2 * k + (j & 1) : k, other = (j == 2 ? 3 : 1) << bit;
#pragma unroll
                for (int u = 0; u < LM; ++u) {
                    const int i = lane + 64 * u, p = ((i >> bit) << (bit + 1)) | (i & ((1 << bit) - 1));
                    t = max(t, exact(order[p], order[p ^ other]));
                }
            }
            t = wave_max(t);
            if (lane == k) mine = t;
        }
        const long long total = weights ? wave_sum64(weight * mine) : (long long)wave_sum(mine);
        __builtin_amdgcn_wave_barrier();   // all look-ups done before the slices are overwritten
        if (lane == 0) out[b] = total;
    }
}

template <int LOGN, bool BCUBE4 = false>
static hipError_t rd_marked_launch(const int32_t* c, void* room, const int32_t* weights,
                                   const int32_t* perms, int64_t B, int64_t* out, hipStream_t s) {
    constexpr int N = 1 << LOGN, WAVES = LOGN == 10 ? 15 : 16;
    constexpr int kWanted = LOGN == 10 ? BCUBE4 ? 1 : 2 : 3;                    // of 128 samples: 6 or 5 of N / 2, half as many under BCube
    int32_t* tops = (int32_t*)((char*)room + mark_tops_offset(N));
    const size_t lds = N * N / 8 + sizeof(uint16_t) * WAVES * N + sizeof(int) * WAVES * 16 + sizeof(int) * (N / 128 * (BCUBE4 ? LOGN / 2 * 3 : LOGN));
    hipError_t e = hipFuncSetAttribute((const void*)(rd_batch_marked_kernel<LOGN, BCUBE4>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((mark_links_kernel<LOGN, kWanted>), dim3(kMarkBlocks), dim3(1024), 0, s, c, (uint32_t*)room, tops);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    int64_t blocks = (B + WAVES - 1) / WAVES;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL((rd_batch_marked_kernel<LOGN, BCUBE4>), dim3((int)blocks), dim3(64 * WAVES), lds, s, c,
                       (const uint32_t*)room, tops, weights, perms, B, out);
    return hipGetLastError();
}

// N = 4 .. 32, halving-doubling and base-4 BCube (4, 16): one order per LANE.  A lane loads its own order (16 N bytes of
// consecutive cache lines per four lanes at N = 16; all of every line is used), the folded matrix, both directions of a
// pair in one entry, is in LDS, and with all loops unrolled the ends of a link are registers: per link one address, one
// LDS look-up and half a maximum, nothing is reduced across lanes.  Bound by the order stream and the launch.  One wave per
// order, as before, left lanes idle and paid for reductions; 10^6 orders: halving-doubling N = 8 150 -> 8 us, N = 16
// 184 -> 14 us (4.9 TB/s), N = 32 176 -> 26 us (5.3 TB/s), BCube N = 16 295 -> 14 us; 1000 orders the launch's 7.4 us.
template <int LOGN, bool BCUBE4>
__global__ __launch_bounds__(256) void rounds_batch_small_kernel(const int32_t* __restrict__ c,
                                                                 const int32_t* __restrict__ weights,
                                                                 const int32_t* __restrict__ perms, int64_t B,
                                                                 int64_t* __restrict__ out) {
    constexpr int N = 1 << LOGN, ROUNDS = BCUBE4 ? LOGN / 2 : LOGN;
    __shared__ int32_t m[N * N];
    for (int e = threadIdx.x; e < N * N; e += 256) {
        const int x = e >> LOGN, y = e & (N - 1);
        m[e] = max(c[e], c[y * N + x]);
    }
    __syncthreads();
    long long w[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) w[r] = weights ? (long long)clampi(weights[r], 0, kMaxRoundWeight) : 1ll;
    const bool aligned = ((uintptr_t)perms & 15u) == 0;
    for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < B; b += (int64_t)gridDim.x * 256) {
        int t[N];
        const int32_t* pi = perms + b * N;
        if (aligned) {
#pragma unroll
            for (int q = 0; q < N / 4; ++q) {
                const int4 v = ((const int4*)pi)[q];
                t[4 * q] = v.x;
                t[4 * q + 1] = v.y;
                t[4 * q + 2] = v.z;
                t[4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int p = 0; p < N; ++p) t[p] = pi[p];
        }
#pragma unroll
        for (int p = 0; p < N; ++p) t[p] = clampi(t[p], 0, N - 1);
        long long total = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            int worst = 0;
#pragma unroll
            for (int p = 0; p < N; ++p) {
                const int step = BCUBE4 ? 1 << (2 * r) : 1 << r;
#pragma unroll
                for (int d = 1; d < (BCUBE4 ? 4 : 2); ++d)                 // peers above p in digit r
                    if ((p / step) % (BCUBE4 ? 4 : 2) + d < (BCUBE4 ? 4 : 2))
                        worst = max(worst, m[(t[p] << LOGN) | t[p + d * step]]);
            }
            total += w[r] * worst;
        }
        out[b] = total;
    }
}

template <int LOGN, bool BCUBE4>
static hipError_t rounds_small_launch(const int32_t* c, const int32_t* weights, const int32_t* perms, int64_t B,
                                      int64_t* out, hipStream_t s) {
    hipLaunchKernelGGL((rounds_batch_small_kernel<LOGN, BCUBE4>), dim3(batch_grid(256, B)), dim3(256), 0, s, c, weights, perms,
                       B, out);
    return hipGetLastError();
}

constexpr int64_t kLdsBatchMinOrders = 32768;      // staging a matrix per compute unit pays from here on

template <int LOGN, bool BCUBE4>
static hipError_t links_lds16_launch(const int32_t* c, const int32_t* weights, const int32_t* perms, int64_t B,
                                     int64_t* out, hipStream_t s) {
    constexpr int N = 1 << LOGN;
    const size_t lds = sizeof(uint16_t) * N * N + sizeof(int32_t) * 16 * N;
    hipError_t e = hipFuncSetAttribute((const void*)links_batch_lds16_kernel<LOGN, BCUBE4>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int64_t blocks = (B + 15) / 16;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL((links_batch_lds16_kernel<LOGN, BCUBE4>), dim3((int)blocks), dim3(1024), lds, s, c, weights, perms,
                       B, out);
    return hipGetLastError();
}

template <int LOGN>
static hipError_t rd_folded_launch(const uint16_t* folded, const int32_t* weights, const int32_t* perms, int64_t B,
                                   int64_t* out, const int32_t* flags, hipStream_t s) {
    hipLaunchKernelGGL(rd_batch_folded_kernel<LOGN>, dim3(batch_grid(4, B)), dim3(256), 0, s, folded, weights, perms, B,
                       out, flags);
    return hipGetLastError();
}

hipError_t launch_rd_cost_batch(const int32_t* c, int N, const int32_t* weights, const int32_t* perms, int64_t B,
                                int64_t* out, hipStream_t s, int32_t* flags, uint16_t* folded) {
    if (B == 0) return hipSuccess;
    if (N == 64) {
        if (((uintptr_t)perms & 15u) == 0)
            hipLaunchKernelGGL(rd_batch_lanes64_kernel, dim3(batch_grid(4 * 64, B)), dim3(256), 0, s, c, weights,
                               (const int4*)perms, B, out);
        else
            hipLaunchKernelGGL(rd_batch_links64_kernel, dim3(batch_grid(4, B)), dim3(256), 0, s, c, weights, perms, B, out);
        return hipGetLastError();
    }
    if (N == 4) return rounds_small_launch<2, false>(c, weights, perms, B, out, s);
    if (N == 8) return rounds_small_launch<3, false>(c, weights, perms, B, out, s);
    if (N == 16) return rounds_small_launch<4, false>(c, weights, perms, B, out, s);
    if (N == 32) return rounds_small_launch<5, false>(c, weights, perms, B, out, s);
    if (N <= 64) return rd_launch<1>(c, N, weights, perms, B, out, nullptr, s);
    if (B >= kLdsBatchMinOrders) {
        if (N == 128) return links_lds16_launch<7, false>(c, weights, perms, B, out, s);
        if (N == 256) return links_lds16_launch<8, false>(c, weights, perms, B, out, s);
    }
    if (flags && folded && N == 512) return rd_marked_launch<9>(c, folded, weights, perms, B, out, s);
    if (flags && folded && N == 1024) return rd_marked_launch<10>(c, folded, weights, perms, B, out, s);
    const int32_t* skip = nullptr;
    if (flags && folded) {
        // both kernels are enqueued; the matrix maximum, computed on the device, decides which of them works
        hipError_t e = launch_matrix_max(c, N, flags, s);
        if (e == hipSuccess) e = launch_fold_to_u16(c, N, folded, flags, s);
        if (e == hipSuccess)
            e = N == 128 ? rd_folded_launch<7>(folded, weights, perms, B, out, flags, s)
                         : rd_folded_launch<8>(folded, weights, perms, B, out, flags, s);
        if (e != hipSuccess) return e;
        skip = flags;
    }
    if (N == 128) return rd_launch<2>(c, N, weights, perms, B, out, skip, s);
    if (N == 256) return rd_launch<4>(c, N, weights, perms, B, out, skip, s);
    if (N == 512) return rd_launch<8>(c, N, weights, perms, B, out, skip, s);
    return rd_launch<16>(c, N, weights, perms, B, out, skip, s);
}

// ------------------------------------------------------------------------------- BCube cost model
// Section 4.1, equation C_b: round i pairs every rank with the base-1 ranks that differ from it in
// base-`base` digit i only; the round costs its slowest exchange.  Same gather-max-sum shape as the
// halving-doubling kernel with base-1 gathers per rank and round.
template <int NM, bool LDS_MATRIX>
__global__ __launch_bounds__(256) void bcube_batch_kernel(const int32_t* __restrict__ c, int N, int base,
                                                          const int32_t* __restrict__ weights,
                                                          const int32_t* __restrict__ perms, int64_t B,
                                                          int64_t* __restrict__ out,
                                                          const int32_t* __restrict__ skip_if_small) {
    // enqueued beside the folded-matrix kernel: flags[0] = max(c) decides which of the two does the work
    if (skip_if_small && skip_if_small[0] < (1 << 16)) return;
    extern __shared__ int32_t sm[];
    int32_t* order = sm + (threadIdx.x >> 6) * N;
    const int32_t* mat = c;
    if (LDS_MATRIX) {
        int32_t* m = sm + 4 * N;
        for (int e = threadIdx.x; e < N * N; e += 256) m[e] = c[e];
        __syncthreads();
        mat = m;
    }
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t b = wave; b < B; b += nwaves) {
        const int32_t* pi = perms + b * N;
        int a[NM];
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            const int p = lane + 64 * k;
            a[k] = p < N ? clampi(pi[p], 0, N - 1) : 0;
            if (p < N) order[p] = a[k];
        }
        __builtin_amdgcn_wave_barrier();
        long long total = 0;
        int round = 0;
        for (int stride = 1; stride < N; stride *= base, ++round) {
            int worst = 0;
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                const int p = lane + 64 * k;
                if (p < N) {
                    const int digit = (p / stride) % base;
                    const int* row = mat + a[k] * N;
                    int peer_digit = digit;
                    for (int step = 1; step < base; ++step) {
                        peer_digit = peer_digit + 1 == base ? 0 : peer_digit + 1;
                        worst = max(worst, row[order[p + (peer_digit - digit) * stride]]);
                    }
                }
            }
            const long long w = weights ? (long long)clampi(weights[round], 0, kMaxRoundWeight) : 1ll;
            total += w * wave_max(worst);
        }
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) out[b] = total;
    }
}

template <int NM>
static hipError_t bcube_launch(const int32_t* c, int N, int base, const int32_t* weights, const int32_t* perms,
                               int64_t B, int64_t* out, const int32_t* skip_if_small, hipStream_t s) {
    const int grid = batch_grid(4, B);
    if (N <= 64) {
        const size_t lds = sizeof(int32_t) * (size_t)(4 * N + N * N);
        hipLaunchKernelGGL((bcube_batch_kernel<NM, true>), dim3(grid), dim3(256), lds, s, c, N, base, weights, perms, B,
                           out, skip_if_small);
    } else {
        const size_t lds = sizeof(int32_t) * (size_t)(4 * N);
        hipLaunchKernelGGL((bcube_batch_kernel<NM, false>), dim3(grid), dim3(256), lds, s, c, N, base, weights, perms, B,
                           out, skip_if_small);
    }
    return hipGetLastError();
}

// N = 64, base 4 (the paper's BCube setting at the size of the bench's batch): lane = rank, the nine peers of a rank
// (three per round) are fixed lane numbers computed once, the three rounds' maxima are reduced together, the next
// order of the wave is requested while this one is scored.
__global__ __launch_bounds__(256) void bcube_batch_b4n64_kernel(const int32_t* __restrict__ c,
                                                                const int32_t* __restrict__ weights,
                                                                const int32_t* __restrict__ perms, int64_t B,
                                                                int64_t* __restrict__ out) {
    constexpr int N = 64;
    __shared__ int32_t m[N * N];
    __shared__ int32_t order_all[4][N];
    for (int e = threadIdx.x; e < N * N; e += 256) m[e] = c[e];
    __syncthreads();
    const int lane = lane_id();
    int32_t* order = order_all[threadIdx.x >> 6];
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    long long w[3];
    int peer[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        w[r] = weights ? (long long)clampi(weights[r], 0, kMaxRoundWeight) : 1ll;
        const int digit = (lane >> (2 * r)) & 3, rest = lane & ~(3 << (2 * r));
#pragma unroll
        for (int s = 1; s <= 3; ++s) peer[r][s - 1] = rest | (((digit + s) & 3) << (2 * r));
    }
    int next = wave < B ? perms[wave * N + lane] : 0;
    for (int64_t b = wave; b < B; b += nwaves) {
        const int a = clampi(next, 0, N - 1);
        const int64_t bn = b + nwaves;
        next = bn < B ? perms[bn * N + lane] : 0;
        order[lane] = a;
        __builtin_amdgcn_wave_barrier();
        int v[3];
#pragma unroll
        for (int r = 0; r < 3; ++r)
            v[r] = max(m[a * N + order[peer[r][0]]], max(m[a * N + order[peer[r][1]]], m[a * N + order[peer[r][2]]]));
        __builtin_amdgcn_wave_barrier();   // all look-ups done before the slice is overwritten
        wave_max3(v[0], v[1], v[2]);
        if (lane == 0) out[b] = w[0] * v[0] + w[1] * v[1] + w[2] * v[2];
    }
}

// Base 4 at N = 256, small batches, on the folded 16-bit copy of the matrix (as rd_batch_folded_kernel): the four ranks that
// differ in one base-4 digit exchange pairwise, and both directions of a pair are one folded entry, so a round is the
// maximum over N / 4 groups of six entries - 1.5 N look-ups instead of 3 N.  A lane takes whole groups: four order
// look-ups in LDS, six gathers.  Returns at once when flags[0] = max(c) is 2^16 or more.
template <int ROUNDS>
__global__ __launch_bounds__(256) void bcube_b4_folded_kernel(const uint16_t* __restrict__ folded,
                                                              const int32_t* __restrict__ weights,
                                                              const int32_t* __restrict__ perms, int64_t B,
                                                              int64_t* __restrict__ out,
                                                              const int32_t* __restrict__ flags) {
    constexpr int LOGN = 2 * ROUNDS, N = 1 << LOGN, NM = N / 64, GM = N / 256;      // ranks and groups per lane
    if (flags[0] >= (1 << 16)) return;
    __shared__ int32_t order_all[4][N];
    int32_t* order = order_all[threadIdx.x >> 6];
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    long long w[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) w[r] = weights ? (long long)clampi(weights[r], 0, kMaxRoundWeight) : 1ll;
    for (int64_t b = wave; b < B; b += nwaves) {
        const int32_t* pi = perms + b * N;
#pragma unroll
        for (int k = 0; k < NM; ++k) order[lane + 64 * k] = clampi(pi[lane + 64 * k], 0, N - 1);
        __builtin_amdgcn_wave_barrier();
        int worst[ROUNDS + 2];
        worst[ROUNDS] = worst[ROUNDS + 1] = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            int v = 0;
#pragma unroll
            for (int u = 0; u < GM; ++u) {
                const int g = lane + 64 * u;                                       // group: the rank without digit r
                const int p0 = ((g >> (2 * r)) << (2 * r + 2)) | (g & ((1 << (2 * r)) - 1));
                unsigned node[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) node[d] = (unsigned)order[p0 | (d << (2 * r))];
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int e = d + 1; e < 4; ++e)
                        v = max(v, (int)*(const uint16_t*)((const char*)folded +
                                                            ((node[d] << (LOGN + 1)) | (node[e] << 1))));
            }
            worst[r] = v;
        }
        __builtin_amdgcn_wave_barrier();   // all look-ups done before the slice is overwritten
#pragma unroll
        for (int r = 0; r < ROUNDS; r += 3) wave_max3(worst[r], worst[r + 1], worst[r + 2]);
        long long total = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) total += w[r] * worst[r];
        if (lane == 0) out[b] = total;
    }
}

hipError_t launch_bcube_cost_batch(const int32_t* c, int N, int base, const int32_t* weights, const int32_t* perms,
                                   int64_t B, int64_t* out, hipStream_t s, int32_t* flags, uint16_t* folded) {
    if (B == 0) return hipSuccess;
    if (base == 2) return launch_rd_cost_batch(c, N, weights, perms, B, out, s, flags, folded);
    if (N == 64 && base == 4) {
        if (((uintptr_t)perms & 15u) == 0)
            hipLaunchKernelGGL(bcube_b4_lanes64_kernel, dim3(batch_grid(4 * 64, B)), dim3(256), 0, s, c, weights,
                               (const int4*)perms, B, out);
        else
            hipLaunchKernelGGL(bcube_batch_b4n64_kernel, dim3(batch_grid(4, B)), dim3(256), 0, s, c, weights, perms, B, out);
        return hipGetLastError();
    }
    if (base == 4 && N == 4) return rounds_small_launch<2, true>(c, weights, perms, B, out, s);
    if (base == 4 && N == 16) return rounds_small_launch<4, true>(c, weights, perms, B, out, s);
    if (base == 4 && N == 256 && B >= kLdsBatchMinOrders) return links_lds16_launch<8, true>(c, weights, perms, B, out, s);
    if (flags && folded && base == 4 && N == 1024) return rd_marked_launch<10, true>(c, folded, weights, perms, B, out, s);
    const int32_t* skip = nullptr;
    if (flags && folded && base == 4 && N == 256) {
        // both kernels are enqueued; the matrix maximum, computed on the device, decides which of them works
        hipError_t e = launch_matrix_max(c, N, flags, s);
        if (e == hipSuccess) e = launch_fold_to_u16(c, N, folded, flags, s);
        if (e != hipSuccess) return e;
        const int grid = batch_grid(4, B);
        hipLaunchKernelGGL(bcube_b4_folded_kernel<4>, dim3(grid), dim3(256), 0, s, folded, weights, perms, B, out, flags);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        skip = flags;
    }
    if (N <= 64) return bcube_launch<1>(c, N, base, weights, perms, B, out, skip, s);
    if (N <= 128) return bcube_launch<2>(c, N, base, weights, perms, B, out, skip, s);
    if (N <= 256) return bcube_launch<4>(c, N, base, weights, perms, B, out, skip, s);
    if (N <= 512) return bcube_launch<8>(c, N, base, weights, perms, B, out, skip, s);
    return bcube_launch<16>(c, N, base, weights, perms, B, out, skip, s);
}

// --------------------------------------------------------------------- double-binary-tree cost model
// Section 4.1, equation C_dbt: the ranks form an in-order binary tree whose subtree roots are the middle
// ranks of their ranges; a tree costs its most expensive root-to-leaf path; the second tree has the same
// shape one position further along the order; the result is the larger of the two.
//
// Any N, one wave per order, entries through L2: each half wave takes one tree, each lane the path to one of the 32 subtrees
// below the fifth level and then that subtree, REST levels below its root (N < 2^(6 + REST)).  Which ranks these are does not
// depend on the order: their places in LDS are found once.  (5 + 2^(REST + 1) - 1) look-ups per lane for 2 (N - 1) edges; what
// bounds it is the rate of scattered requests to the L2 (about 3e11 a second).  Every rank walking its whole path -> this kernel: N = 1000,
// 65000 orders 851 -> 544 us, 1000 orders 72 -> 13 us; N = 1024 (242 registers, two waves per SIMD) 909 -> 600 and 76 -> 15 us; N = 500,
// 65000 orders 338 -> 244 us; N = 300, 16000 orders 51 -> 38 us.
// `order`: N + N / 32 + 1 words for this wave, number `wave` of nwaves.
template <int REST>
__device__ __forceinline__ void dbt_wave_per_order(const int32_t* __restrict__ c, int N, const int32_t* __restrict__ perms, int64_t B,
                                                   int64_t* __restrict__ out, int32_t* order, int64_t wave, int64_t nwaves) {
    constexpr int SUB = (2 << REST) - 1;                   // places of a subtree, heap order: 0; 1, 2; 3 .. 6; ..
    constexpr int CHUNKS = REST < 5 ? 1 << REST : 16;      // 64 ranks each
    const int lane = lane_id(), shift = lane >> 5;
    // one word left out behind every 32: the places of a level lie N / 32 ranks apart
    auto place = [](int rank) { return rank + (rank >> 5); };
    auto rank_at = [&](int position) { return position + shift >= N ? position + shift - N : position + shift; };
    int path[6], sub[SUB];
    bool on_path[6], in_sub[SUB];
    int first[SUB], last[SUB];
    {
        int lo = 0, hi = N - 1;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int mid = (lo + hi) >> 1;
            on_path[k] = lo <= hi;
            path[k] = place(rank_at(on_path[k] ? mid : 0));
            if (k == 5) {
                first[0] = lo;
                last[0] = hi;
            } else {
                const bool right = (lane >> (4 - k)) & 1;
                lo = right ? mid + 1 : lo;
                hi = right ? hi : mid - 1;
            }
        }
#pragma unroll
        for (int h = 0; h < SUB; ++h) {
            if (h) {
                const int up = (h - 1) >> 1, mid = (first[up] + last[up]) >> 1;
                const bool there = first[up] <= last[up];
                first[h] = there ? ((h & 1) ? first[up] : mid + 1) : 1;
                last[h] = there ? ((h & 1) ? mid - 1 : last[up]) : 0;
            }
            in_sub[h] = first[h] <= last[h];
            sub[h] = place(rank_at(in_sub[h] ? (first[h] + last[h]) >> 1 : 0));
        }
    }
    int next[CHUNKS];
    auto request = [&](int64_t b) {
        const int32_t* pi = perms + (b < B ? b : B - 1) * N;
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) next[u] = pi[min(lane + 64 * u, N - 1)];
    };
    request(wave);
    for (int64_t b = wave; b < B; b += nwaves) {
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u)
            if (lane + 64 * u < N) order[place(lane + 64 * u)] = clampi(next[u], 0, N - 1);
        request(b + nwaves);
        __builtin_amdgcn_wave_barrier();
        int node[6], below[SUB], cost[SUB];
        int way = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) node[k] = order[path[k]];
#pragma unroll
        for (int h = 1; h < SUB; ++h) below[h] = order[sub[h]];
        below[0] = node[5];
        int edge[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) edge[k] = c[REST > 0 || on_path[k + 1] ? (unsigned)(node[k] * N + node[k + 1]) : 0u];
        // every level but the last is full; where a place is empty all lanes ask for the same entry
#pragma unroll
        for (int h = 1; h < SUB; ++h)
            cost[h] = c[h < (SUB >> 1) || in_sub[h] ? (unsigned)(below[(h - 1) >> 1] * N + below[h]) : 0u];
#pragma unroll
        for (int k = 0; k < 5; ++k) way += REST > 0 || on_path[k + 1] ? edge[k] : 0;
        cost[0] = way;
        int worst = way;
#pragma unroll
        for (int h = 1; h < SUB; ++h) {
            cost[h] = cost[(h - 1) >> 1] + (h < (SUB >> 1) || in_sub[h] ? cost[h] : 0);
            worst = max(worst, cost[h]);
        }
        const int total = wave_max(worst);
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) out[b] = total;
    }
}

template <int REST>
__global__ __launch_bounds__(256) void dbt_batch_kernel(const int32_t* __restrict__ c, int N,
                                                        const int32_t* __restrict__ perms, int64_t B,
                                                        int64_t* __restrict__ out) {
    extern __shared__ int32_t sm[];
    dbt_wave_per_order<REST>(c, N, perms, B, out, sm + (threadIdx.x >> 6) * (N + N / 32 + 1),
                             (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), (int64_t)gridDim.x * 4);
}

template <int REST>
static hipError_t dbt_launch(const int32_t* c, int N, const int32_t* perms, int64_t B, int64_t* out, hipStream_t s) {
    const size_t lds = sizeof(int32_t) * 4 * (size_t)(N + N / 32 + 1);
    hipLaunchKernelGGL(dbt_batch_kernel<REST>, dim3(batch_grid(4, B)), dim3(256), lds, s, c, N, perms, B, out);
    return hipGetLastError();
}

// Large batches of 8 <= N <= 255: one order per lane, the matrix in LDS, 64 orders at a time as bytes beside it
// (a tile: by rank, so that the lanes of a wave read one rank of all orders from consecutive bytes).  All lanes walk
// the tree together: where a rank range begins and ends is scalar arithmetic, and every edge is looked up once per tree.  A tile belongs
// to as many waves as make eight bottom subtrees each (K of them in all): every wave stages its part of the orders and walks
// its part of both trees, the next tile's ranks on their way meanwhile.  The bottom subtrees are of two or three ranks
// (AT_MOST 3: N >= 3 K) or of one or two: three or two look-ups per tree, of which the one that not every subtree has is masked.
// What bounds it: LDS look-ups (two bytes and two entries per rank) and, up to some 100000 orders, the latency of one or two tiles per
// wave.  Level by level with sixteen lanes per order, top levels nearly empty -> here: N = 100, 100000 orders 33.3 -> 18.5 us, 300000
// orders 80 -> 38 us; N = 50, 10^6 orders 120 -> 58 us; N = 8, 10^6 orders 78 -> 10 us; N = 255 (few waves beside the
// matrix), 100000 orders 212 -> 40 us; N = 200, 300000 orders 202 -> 73 us.  Matrices with hardly an
// entry below 65535, N >= 186: through L2 there is nothing to gain from this walk, so such a workgroup's waves take an order each (level
// by level / this walk / now: N = 200, 8000 orders 22.5 / 23.0 / 18.0 us, 30000 52 / 56 / 49, 100000 148 / 175 / 156; N = 254, 8000 orders
// 19.7 / 27.7 / 23.2, 100000 261 / 205 / 203).  One wave per tile: N = 255,
// 100000 orders 127 us; two workgroups of eight waves per unit: N = 100, 50000 orders 11.2 instead of 9.4 us.
constexpr int kDbtRow = 68;                     // bytes per rank: 64 orders, and a bank further from rank to rank

// MIXED: the staged entry 0xffff stands for one in the caller's matrix
template <typename ENTRY, bool MIXED>
struct DbtTile {
    const ENTRY* mat;
    const int32_t* callers;
    const unsigned char* tile;                  // byte `lane` of rank 0 is this lane's
    int N, lane;
    __device__ __forceinline__ unsigned node(int rank) const { return tile[rank * kDbtRow + lane]; }
    // of the second tree's positions the last one holds rank 0
    __device__ __forceinline__ unsigned next_node(int rank) const { return node(rank >= N ? rank - N : rank); }
    // rows in bytes
    __device__ __forceinline__ unsigned row_of(unsigned x) const { return __umul24(x, (unsigned)(sizeof(ENTRY) * N)); }
    __device__ __forceinline__ int edge(unsigned from_row, unsigned to) const {
        const unsigned at = from_row + (unsigned)sizeof(ENTRY) * to;
        const int entry = *(const ENTRY*)((const char*)mat + at);
        if (!MIXED) return entry;
        const bool large = entry == 0xffff;
        const int callers_entry = callers[large ? at / (unsigned)sizeof(ENTRY) : 0u];
        return large ? callers_entry : entry;
    }
};

// A bottom subtree: of three ranks the middle one is the root, of two the lower.  nodes[]: (AT_MOST 3) its lowest rank, then
// for either the root and the two ranks above it.
template <int AT_MOST>
struct DbtBottom {
    unsigned lowest, nodes[3];
    int more;                                   // 1: as many ranks as there may be
    int edges[AT_MOST == 3 ? 6 : 4];

    template <class TILE>
    __device__ __forceinline__ void read_nodes(const TILE& t, int lo, int hi) {
        more = hi - lo - (AT_MOST - 2);
        const int root = AT_MOST == 3 ? lo + more : lo;
        lowest = AT_MOST == 3 ? t.node(lo) : 0;
        nodes[0] = t.node(root);
        nodes[1] = AT_MOST == 3 ? t.node(root + 1) : t.next_node(root + 1);
        nodes[2] = t.next_node(root + 2);
    }
    // p0, p1: rows of the node above in either tree
    template <class TILE>
    __device__ __forceinline__ void read_edges(const TILE& t, unsigned p0, unsigned p1) {
        const unsigned r0 = t.row_of(nodes[0]), r1 = t.row_of(nodes[1]);
        edges[0] = t.edge(p0, nodes[0]);
        edges[1] = t.edge(p1, nodes[1]);
        edges[2] = t.edge(r0, nodes[1]);
        edges[3] = t.edge(r1, nodes[2]);
        if constexpr (AT_MOST == 3) {
            edges[4] = t.edge(r0, lowest);
            edges[5] = t.edge(r1, nodes[0]);
        }
    }
    __device__ __forceinline__ int costliest(int k0, int k1) const {
        if constexpr (AT_MOST == 3)
            return max(k0 + edges[0] + max(edges[2], edges[4] & -more), k1 + edges[1] + max(edges[3], edges[5] & -more));
        else
            return max(k0 + edges[0] + (edges[2] & -more), k1 + edges[1] + (edges[3] & -more));
    }
};

// The tree of positions lo .. hi, LEFT levels above the bottom subtrees, below the node of row p0 (p1 in the second tree; root:
// below none).  Two levels above the bottom ones it is read as a whole, all nodes and then all entries in flight together.
template <int LEFT, int AT_MOST, class TILE>
__device__ __forceinline__ void dbt_descend(TILE& t, int lo, int hi, bool root, unsigned p0, unsigned p1, int k0, int k1, int& worst) {
    const int mid = (lo + hi) >> 1;
    const unsigned x0 = t.node(mid), x1 = t.node(mid + 1), x0_row = t.row_of(x0), x1_row = t.row_of(x1);
    if constexpr (LEFT > 2) {
        k0 += root ? 0 : t.edge(p0, x0);
        k1 += root ? 0 : t.edge(p1, x1);
        dbt_descend<LEFT - 1, AT_MOST>(t, lo, mid - 1, false, x0_row, x1_row, k0, k1, worst);
        dbt_descend<LEFT - 1, AT_MOST>(t, mid + 1, hi, false, x0_row, x1_row, k0, k1, worst);
    } else {
        unsigned y0[2], y1[2];
        DbtBottom<AT_MOST> bottom[4];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int from = side ? mid + 1 : lo, to = side ? hi : mid - 1, m = (from + to) >> 1;
            y0[side] = t.node(m);
            y1[side] = t.node(m + 1);
            bottom[2 * side].read_nodes(t, from, m - 1);
            bottom[2 * side + 1].read_nodes(t, m + 1, to);
        }
        const int e0 = root ? 0 : t.edge(p0, x0), e1 = root ? 0 : t.edge(p1, x1);
        int f0[2], f1[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            f0[side] = t.edge(x0_row, y0[side]);
            f1[side] = t.edge(x1_row, y1[side]);
            const unsigned y0_row = t.row_of(y0[side]), y1_row = t.row_of(y1[side]);
            bottom[2 * side].read_edges(t, y0_row, y1_row);
            bottom[2 * side + 1].read_edges(t, y0_row, y1_row);
        }
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int m0 = k0 + e0 + f0[side], m1 = k1 + e1 + f1[side];
            worst = max(worst, max(bottom[2 * side].costliest(m0, m1), bottom[2 * side + 1].costliest(m0, m1)));
        }
        // the next look-ups wait for this group's: the compiler would have all of them in flight and spill
        asm volatile("" : "+v"(t.lane), "+v"(worst));
    }
}

// PARTS: waves per tile
__host__ __device__ constexpr int dbt_parts(int K) { return K <= 8 ? 1 : K / 8; }

// ENTRY: 32 bits where the matrix has room as such, 16 above
template <int K, int AT_MOST, bool QUADS, typename ENTRY>
__global__ __launch_bounds__(1024) void dbt_batch_lanes_kernel(const int32_t* __restrict__ c, int N, int tiles,
                                                               const int32_t* __restrict__ perms, int64_t B,
                                                               int64_t* __restrict__ out) {
    constexpr int PARTS = dbt_parts(K), LEVELS = 31 - __builtin_clz((unsigned)K), SPLIT = 31 - __builtin_clz((unsigned)PARTS);
    constexpr int U = K / PARTS;                                        // loads of a wave for a tile: N <= 4 K - 1
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_lanes[];
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = wv % PARTS, slot = wv / PARTS;
    unsigned* wave_top = (unsigned*)smem_lanes;                         // [16]
    int* costliest = (int*)(smem_lanes + 64) + 64 * slot;               // [tiles][64]
    ENTRY* staged = (ENTRY*)(smem_lanes + 64 + 256 * tiles);            // [N * N]
    unsigned char* tile = (unsigned char*)(staged + ((N * N + 7) & ~7)) + slot * N * kDbtRow;
    const int64_t elements = B * N, stride = (int64_t)gridDim.x * tiles;
    ranks4 v[U];
    // this wave's part of 64 orders, which lie one after the other; past the batch's end whatever is there
    auto request = [&](int64_t task) {
        const int64_t first = task * 64 * N + 256 * part + 4 * lane;
        if (QUADS || (task + 1) * 64 <= B) {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *(const ranks4*)(perms + min(first + 256 * PARTS * u, elements - 4));
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[u][j] = perms[min(first + 256 * PARTS * u + j, elements - 1)];
        }
    };
    if (slot < tiles) request((int64_t)blockIdx.x * tiles + slot);
    unsigned top = 0;
    int done = 0;
    if constexpr (sizeof(ENTRY) == 2) {
        // The first 32768 of at least 34596 entries (N >= 186).  Where nearly all of the first half are 65535 or more, most look-ups would go
        // through L2, and a wave per order is the faster (share of such entries, N = 193, 100000 orders, this walk / a wave per order: 0.9
        // 156 / 150 us, 1.0 171 / 150; N = 254 187 / 203, 205 / 203); the second half is on its way while the waves agree.
        constexpr int U = 16, kHalf = U * 1024;
        unsigned v[2][U];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < U; ++u) v[h][u] = (unsigned)c[h * kHalf + u * 1024 + (int)threadIdx.x];
        int* large = (int*)(staged + ((N * N + 7) & ~7));               // [16], where the tiles come
        int mine = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) mine += __popcll(__ballot(v[0][u] >= 0xffffu));
        if (lane == 0) large[wv] = mine;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            top = max(top, v[0][u]);
            staged[u * 1024 + threadIdx.x] = (ENTRY)min(v[0][u], 0xffffu);
        }
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) all += large[k];
        if (__builtin_amdgcn_readfirstlane(all) > kHalf / 16 * 15) {
            dbt_wave_per_order<2>(c, N, perms, B, out, (int32_t*)staged + wv * (N + N / 32 + 1), (int64_t)blockIdx.x * 16 + wv,
                                  (int64_t)gridDim.x * 16);
            return;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            top = max(top, v[1][u]);
            staged[kHalf + u * 1024 + threadIdx.x] = (ENTRY)min(v[1][u], 0xffffu);
        }
        done = 2 * kHalf;
    }
    top = max(top, stage_matrix(c + done, N * N - done, staged + done));
    top = (unsigned)wave_max((int)min(top, 0x7fffffffu));
    if (lane == 0) wave_top[wv] = top;
    if (PARTS > 1 && part == 0 && slot < tiles) costliest[lane] = 0;
    __syncthreads();
    if (slot >= tiles) return;                                          // they staged only; later barriers wait for the others
    for (int k = 0; k < (int)blockDim.x >> 6; ++k) top = max(top, wave_top[k]);
    // where this wave's first four ranks are (order and rank), and how far on those of its next load
    const int first = 256 * part + 4 * lane, first_o = first / N, first_p = first - first_o * N;
    const int step_o = 256 * PARTS / N, step_p = 256 * PARTS - step_o * N;
    auto score = [&](auto mixed) {
        for (int64_t base = (int64_t)blockIdx.x * tiles; base * 64 < B; base += stride) {
            const int64_t task = base + slot;
            int p = first_p, o = first_o;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (4 * (u * PARTS + part) < N) {
                    // the four's first byte, and, where the next order begins among them, what the later ones are counted from;
                    // past the 64 orders (the last load, N no multiple of 4): the byte behind a rank's 64
                    int to = p * kDbtRow + o, to_next = to - N * kDbtRow + 1;
                    if (!QUADS) {
                        to = o < 64 ? to : 64;
                        to_next = o < 63 ? to_next : 64;
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        tile[(QUADS || p + j < N ? to : to_next) + j * kDbtRow] = (unsigned char)clampi(v[u][j], 0, N - 1);
                    p += step_p;
                    o += step_o;
                    if (p >= N) {
                        p -= N;
                        ++o;
                    }
                }
            }
            if (PARTS > 1) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
            request(task + stride);
            // ---- both trees of every lane's order; new to the compiler in every round: it would keep the addresses of all ranks in
            // registers, more than there are
            DbtTile<ENTRY, decltype(mixed)::value> t{staged, c, tile, N, lane};
            int worst = 0, lo = 0, hi = N - 1, k0 = 0, k1 = 0;
            unsigned p0 = 0, p1 = 0;
            asm volatile("" : "+v"(t.lane), "+s"(hi));
#pragma unroll
            for (int k = 0; k < SPLIT; ++k) {
                const int mid = (lo + hi) >> 1;
                const unsigned x0 = t.node(mid), x1 = t.node(mid + 1);
                if (k) {
                    k0 += t.edge(p0, x0);
                    k1 += t.edge(p1, x1);
                }
                p0 = t.row_of(x0);
                p1 = t.row_of(x1);
                const bool right = (part >> (SPLIT - 1 - k)) & 1;
                lo = right ? mid + 1 : lo;
                hi = right ? hi : mid - 1;
            }
            dbt_descend<LEVELS - SPLIT, AT_MOST>(t, lo, hi, SPLIT == 0, p0, p1, k0, k1, worst);
            const int64_t b = task * 64 + lane;
            if (PARTS > 1) {
                atomicMax(&costliest[lane], worst);
                __syncthreads();
                if (part == 0) {
                    if (b < B) out[b] = costliest[lane];
                    costliest[lane] = 0;
                }
            } else {
                if (b < B) out[b] = worst;
                __builtin_amdgcn_wave_barrier();
            }
        }
    };
    if (sizeof(ENTRY) == 4 || __builtin_amdgcn_readfirstlane(top) < 0xffffu) score(std::false_type{});
    else score(std::true_type{});
}

// N < 8: one order per lane in registers, the matrix in LDS.  10^6 orders of N = 7: 7.7 us (a wave per order 130, sixteen lanes 65).
template <int N>
__global__ __launch_bounds__(256) void dbt_batch_tiny_kernel(const int32_t* __restrict__ c, const int32_t* __restrict__ perms,
                                                             int64_t B, int64_t* __restrict__ out) {
    __shared__ int32_t m[N * 64];
    for (int e = threadIdx.x; e < N * N; e += 256) m[e / N * 64 + e % N] = c[e];
    __syncthreads();
    for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < B; b += (int64_t)gridDim.x * 256) {
        unsigned node4[N];
#pragma unroll
        for (int p = 0; p < N; ++p) node4[p] = (unsigned)clampi(perms[b * N + p], 0, N - 1) << 2;
        int worst = 0;
        dbt_walk_64<0, N - 1, 0, N>((const char*)m, node4, 0u, 0, false, worst);
        dbt_walk_64<0, N - 1, 1, N>((const char*)m, node4, 0u, 0, false, worst);
        out[b] = worst;
    }
}

template <int N>
static hipError_t dbt_tiny_launch(const int32_t* c, const int32_t* perms, int64_t B, int64_t* out, hipStream_t s) {
    hipLaunchKernelGGL(dbt_batch_tiny_kernel<N>, dim3(batch_grid(256, B)), dim3(256), 0, s, c, perms, B, out);
    return hipGetLastError();
}

static size_t dbt_lanes_bytes(int N, int entry, int tiles) {
    return 64 + 256 * (size_t)tiles + (size_t)entry * ((N * N + 7) & ~7) + (size_t)tiles * N * kDbtRow;
}

template <int K, int AT_MOST>
static hipError_t dbt_lanes_launch(const int32_t* c, int N, const int32_t* perms, int64_t B, int64_t* out, hipStream_t s) {
    constexpr size_t kLds = 160 * 1024;
    const int64_t tasks = (B + 63) / 64;
    int64_t tiles = 16 / dbt_parts(K);
    const int entry = dbt_lanes_bytes(N, 4, (int)tiles) <= kLds ? 4 : 2;
    while (tiles > 1 && dbt_lanes_bytes(N, entry, (int)tiles) > kLds) --tiles;
    const int64_t per_round = 256 * tiles;
    // few orders: on as many compute units as there are; many: as many at a time as make the rounds equally long
    const int64_t rounds = (tasks + per_round - 1) / per_round;
    if (rounds == 1 && tasks < 256 * tiles) tiles = (tasks + 255) / 256;
    const bool quads = (N & 3) == 0 && ((uintptr_t)perms & 15u) == 0;
    auto kernel = quads ? dbt_batch_lanes_kernel<K, AT_MOST, true, int32_t> : dbt_batch_lanes_kernel<K, AT_MOST, false, int32_t>;
    if constexpr (K == 64)
        if (entry == 2) kernel = quads ? dbt_batch_lanes_kernel<K, AT_MOST, true, uint16_t> : dbt_batch_lanes_kernel<K, AT_MOST, false, uint16_t>;
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (e != hipSuccess) return e;
    const int64_t blocks = (tasks + tiles * rounds - 1) / (tiles * rounds);
    hipLaunchKernelGGL(kernel, dim3((int)blocks), dim3(1024), dbt_lanes_bytes(N, entry, (int)tiles), s, c, N, (int)tiles, perms, B, out);
    return hipGetLastError();
}

static hipError_t dbt_lanes(const int32_t* c, int N, const int32_t* perms, int64_t B, int64_t* out, hipStream_t s) {
    if (N < 12) return dbt_lanes_launch<4, 2>(c, N, perms, B, out, s);
    if (N < 16) return dbt_lanes_launch<4, 3>(c, N, perms, B, out, s);
    if (N < 24) return dbt_lanes_launch<8, 2>(c, N, perms, B, out, s);
    if (N < 32) return dbt_lanes_launch<8, 3>(c, N, perms, B, out, s);
    if (N < 48) return dbt_lanes_launch<16, 2>(c, N, perms, B, out, s);
    if (N < 64) return dbt_lanes_launch<16, 3>(c, N, perms, B, out, s);
    if (N < 96) return dbt_lanes_launch<32, 2>(c, N, perms, B, out, s);
    if (N < 128) return dbt_lanes_launch<32, 3>(c, N, perms, B, out, s);
    if (N < 192) return dbt_lanes_launch<64, 2>(c, N, perms, B, out, s);
    return dbt_lanes_launch<64, 3>(c, N, perms, B, out, s);
}

// One order per wave is the faster until its waves take several orders each or the L2 has enough requests to bound it; the matrix in
// LDS has its staging to bring in (through L2 / from LDS: N = 8, 32000 orders 7.4 / 7.4 us, 65000 orders 10.7 / 7.2; N = 50, 16000
// orders 7.0 / 7.2, 32000 8.3 / 7.4; N = 100, 8000 orders 6.9 / 7.0, 16000 8.3 / 7.0; N = 150, 4000 orders 6.7 / 9.0, 8000 9.9 / 8.6;
// N = 255, 4000 orders 10.3 / 12.7, 8000 17.4 / 12.0).
static bool dbt_lanes_pay(int N, int64_t B) {
    return N < 256 && (B >= 40000 || B * N >= (N > 192 ? 5 << 18 : 1 << 20));
}

hipError_t launch_dbt_cost_batch(const int32_t* c, int N, const int32_t* perms, int64_t B, int64_t* out,
                                 hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (N == 64 && ((uintptr_t)perms & 15u) == 0) {
        hipLaunchKernelGGL(dbt_lanes64_kernel, dim3(batch_grid(4 * 64, B)), dim3(256), 0, s, c, (const int4*)perms, B, out);
    } else if (N < 8) {
        switch (N) {
            case 2: return dbt_tiny_launch<2>(c, perms, B, out, s);
            case 3: return dbt_tiny_launch<3>(c, perms, B, out, s);
            case 4: return dbt_tiny_launch<4>(c, perms, B, out, s);
            case 5: return dbt_tiny_launch<5>(c, perms, B, out, s);
            case 6: return dbt_tiny_launch<6>(c, perms, B, out, s);
            default: return dbt_tiny_launch<7>(c, perms, B, out, s);
        }
    } else if (dbt_lanes_pay(N, B)) {
        return dbt_lanes(c, N, perms, B, out, s);
    } else {
        if (N < 64) return dbt_launch<0>(c, N, perms, B, out, s);
        if (N < 128) return dbt_launch<1>(c, N, perms, B, out, s);
        if (N < 256) return dbt_launch<2>(c, N, perms, B, out, s);
        if (N < 512) return dbt_launch<3>(c, N, perms, B, out, s);
        if (N < 1024) return dbt_launch<4>(c, N, perms, B, out, s);
        return dbt_launch<5>(c, N, perms, B, out, s);
    }
    return hipGetLastError();
}

// --------------------------------------------------------------------------------- initial orders
// One wave per order.  N <= 64: no serial chain - lane v follows node v through the shuffle: at step k (k = N-1 .. 1)
// ranks k and j_k swap, so a node sitting at rank k moves to j_k and a node sitting at j_k moves to k, where it
// stays (later steps only touch ranks below k); the partners j_k are drawn in parallel, one per lane, and read
// step by step; each lane finally stores its node at the rank where it ended.  N <= 256: the same with up to four
// nodes per lane and the partners read from LDS (one broadcast read per step).  Larger N: the partners are drawn in
// parallel, lane 0 replays the swaps in order in LDS, all lanes store the result coalesced.
__global__ __launch_bounds__(256) void init_tours_kernel(int N, int64_t first, int64_t count, uint64_t seed,
                                                         int32_t* __restrict__ tours) {
    extern __shared__ int32_t sm[];
    int32_t* t = sm + (threadIdx.x >> 6) * 2 * N;
    int32_t* partner = t + N;
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t w = wave; w < count; w += nwaves) {
        const uint32_t r = (uint32_t)(first + w);
        if (N <= kWave) {
            const int mine = (lane > 0 && lane < N) ? shuffle_partner(seed, r, lane) : 0;
            int pos = lane;
            for (int k = N - 1; k >= 1; --k) {
                const int j = __builtin_amdgcn_readlane(mine, k);
                const int moved = (pos == k) ? j : pos;
                pos = (pos == j) ? k : moved;
            }
            if (lane < N) tours[w * N + pos] = lane;
            continue;
        }
        for (int k = lane; k < N; k += kWave) {
            t[k] = k;
            partner[k] = k ? shuffle_partner(seed, r, k) : 0;
        }
        __builtin_amdgcn_wave_barrier();
        if (N <= 4 * kWave) {
            int pos[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pos[i] = lane + kWave * i;       // node ids; those >= N never match a rank
            for (int k = N - 1; k >= 1; --k) {
                const int j = partner[k];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int moved = (pos[i] == k) ? j : pos[i];
                    pos[i] = (pos[i] == j) ? k : moved;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (lane + kWave * i < N) tours[w * N + pos[i]] = lane + kWave * i;
            __builtin_amdgcn_wave_barrier();
            continue;
        }
        if (lane == 0) {
            for (int k = N - 1; k >= 1; --k) {
                const int j = partner[k];
                const int tk = t[k], tj = t[j];
                t[k] = tj;
                t[j] = tk;
            }
        }
        __builtin_amdgcn_wave_barrier();
        for (int k = lane; k < N; k += kWave) tours[w * N + k] = t[k];
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t launch_init_tours(int N, int64_t first, int64_t count, uint64_t seed, int32_t* tours, hipStream_t s) {
    if (count == 0) return hipSuccess;
    const int grid = batch_grid(4, count);
    hipLaunchKernelGGL(init_tours_kernel, dim3(grid), dim3(256), sizeof(int32_t) * 8 * (size_t)N, s, N, first, count,
                       seed, tours);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------ matrix contract
// flags[0] bit 0: an entry outside [0, 2^21 - 1]; bit 1: c[a][b] != c[b][a] somewhere.
__global__ __launch_bounds__(256) void validate_kernel(const int32_t* __restrict__ c, int N, int require_symmetric,
                                                       int32_t* __restrict__ flags) {
    int bad = 0;
    const int64_t total = (int64_t)N * N;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int v = c[e];
        if (v < 0 || v > (1 << 21) - 1) bad |= 1;
        if (require_symmetric) {
            const int a = (int)(e / N), b = (int)(e % N);
            if (c[(int64_t)b * N + a] != v) bad |= 2;
        }
    }
    if (bad) atomicOr(flags, bad);
}

hipError_t launch_validate(const int32_t* c, int N, bool require_symmetric, int32_t* flags, hipStream_t s) {
    const int64_t total = (int64_t)N * N;
    int grid = (int)((total + 255) / 256);
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(validate_kernel, dim3(grid), dim3(256), 0, s, c, N, require_symmetric ? 1 : 0, flags);
    return hipGetLastError();
}

}  // namespace cc
