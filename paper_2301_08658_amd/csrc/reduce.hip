// Partial-sum reduction (the arithmetic of the grouped all-reduce of a
// Partial(SUM) output, Sec. 3.1 / 3.2) with fused bias, GeLU and GeLU'
// epilogues, and the bias-gradient column sum (Sec. 4.2).
//
// The reduction is HBM-bound: per output element it streams nparts fp32
// (or bf16: the 16-bit partials variant, Sec. 5) values in and one
// bf16/fp32 value out.  Each thread owns 8 consecutive columns of one row:
// two 16-byte non-temporal loads per fp32 part (one per bf16 part), all
// parts of a group of 8 issued before the first add so up to 16 loads are
// in flight per thread; parts are then summed in fp32 in group order
// 0..d-1, so the result is bit-identical on every member of the group.
// Rows of a chunk are contiguous, so a launch is one linear sweep of
// [rows x ncols].
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "epilogue_math.h"
#include "kernels.h"

namespace atp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int RT = 256;        // threads per block
constexpr int PGROUP = 8;      // parts loaded before summing

using epi::bf16_to_f32;
using epi::f32_to_bf16_rne;
using epi::gelu_f;
using epi::gelu_grad_f;

__device__ __forceinline__ void unpack8(const u32x4& w, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = bf16_to_f32(w[i] & 0xffffu);
        f[2 * i + 1] = bf16_to_f32(w[i] >> 16);
    }
}

__device__ __forceinline__ u32x4 pack8(const float* f) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = f32_to_bf16_rne(f[2 * i]) | (f32_to_bf16_rne(f[2 * i + 1]) << 16);
    return w;
}

template <int EPI, bool OUT_BF16, bool PART_BF16>
__global__ __launch_bounds__(RT) void reduce_kernel(ReduceProblem p) {
    const int64_t cols8 = p.ncols >> 3;
    const int64_t total = p.rows * cols8;
    const int64_t g = (int64_t)blockIdx.x * RT + threadIdx.x;
    if (g >= total) return;
    const int64_t r = g / cols8;
    const int64_t c = (g - r * cols8) << 3;
    const int64_t row = p.row0 + r;
    const int64_t off = row * p.ldp + c;

    float s[8];
    for (int j0 = 0; j0 < p.nparts; j0 += PGROUP) {
        f32x4 lo[PGROUP], hi[PGROUP];
        u32x4 hw[PGROUP];   // eight bf16 parts
#pragma unroll
        for (int u = 0; u < PGROUP; ++u) {
            if (j0 + u < p.nparts) {
                if constexpr (PART_BF16) {
                    hw[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(
                        static_cast<const uint16_t*>(p.parts[j0 + u]) + off));
                } else {
                    const f32x4* q = reinterpret_cast<const f32x4*>(
                        static_cast<const float*>(p.parts[j0 + u]) + off);
                    lo[u] = __builtin_nontemporal_load(q);
                    hi[u] = __builtin_nontemporal_load(q + 1);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < PGROUP; ++u) {
            if (j0 + u < p.nparts) {
                if constexpr (PART_BF16) {
                    float f[8];
                    unpack8(hw[u], f);
#pragma unroll
                    for (int e = 0; e < 4; ++e) { lo[u][e] = f[e]; hi[u][e] = f[4 + e]; }
                }
                if (j0 + u == 0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) { s[e] = lo[u][e]; s[4 + e] = hi[u][e]; }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) { s[e] += lo[u][e]; s[4 + e] += hi[u][e]; }
                }
            }
        }
    }

    const int64_t oo = row * p.ldo + c;
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) {
        float b[8];
        unpack8(*reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(p.bias) + c), b);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += b[e];
    }
    if constexpr (EPI == EPI_BIAS_GELU) {
        if (p.pre_out) {
            const u32x4 w = pack8(s);
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(
                                               static_cast<uint16_t*>(p.pre_out) + oo));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = gelu_f(s[e]);
    }
    if constexpr (EPI == EPI_GELU_BWD) {
        float x[8];
        unpack8(*reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(p.pre_in) + oo), x);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] *= gelu_grad_f(x[e]);
    }
    if constexpr (OUT_BF16) {
        __builtin_nontemporal_store(pack8(s),
                                    reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.out) + oo));
    } else {
        f32x4* q = reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + oo);
        __builtin_nontemporal_store(f32x4{s[0], s[1], s[2], s[3]}, q);
        __builtin_nontemporal_store(f32x4{s[4], s[5], s[6], s[7]}, q + 1);
    }
}

template <int EPI, bool OUT_BF16, bool PART_BF16>
hipError_t launch_r(const ReduceProblem& p, hipStream_t s) {
    const int64_t total = p.rows * (p.ncols >> 3);
    if (total == 0) return hipSuccess;
    const int64_t blocks = (total + RT - 1) / RT;
    hipLaunchKernelGGL((reduce_kernel<EPI, OUT_BF16, PART_BF16>), dim3((unsigned)blocks), dim3(RT),
                       0, s, p);
    return hipGetLastError();
}

// Column sums in one fixed order, the same on every path (so db has the
// same bits whether or not it is formed during dY's transpose):
//   db[c] = (((0 + S_0) + S_1) + ...),  S_b over the 64-row block b,
//   S_b = (((0 + G_b0) + G_b1) + ...)   over its 8-row groups inside [0, T),
//   G_bg = (((0 + x_r) + x_r+1) + ...)  over the group's rows inside [0, T).
// A block owns 8 CL columns (CL column lanes, one 16-byte load per row each)
// x CS_T / CL row lanes; a row lane forms the G of one 8-row group (eight
// loads in flight), a round of CS_T / CL / 8 row blocks at a time.  Through
// LDS every thread then forms the S_b of one (row block, column) and the first
// 8 CL threads fold the round's S_b into their columns' sums in ascending b.
// The next round's rows are on their way while a round is folded.
// Bound by the rows in flight: 8192 x 6144 25.6 us (3.9 TB/s; 39.9 with 16
// columns a block and no row ahead), 2048 x 4096 7 (25.6 with one row lane per
// 64-row block, 64 loads in sequence, which took 30.4 for 8192 x 6144).
// Blocks are renumbered so neighbouring column groups run on the same XCD.
constexpr int CS_T = 1024;               // threads per block

// A workgroup barrier over LDS accesses only: __syncthreads() would also wait
// for the loads in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int CL>
__global__ __launch_bounds__(CS_T) void colsum_kernel(const uint16_t* __restrict__ dy, int64_t ld,
                                                      int64_t T, int64_t N, float* __restrict__ db) {
    constexpr int COLS = CL * 8;           // columns per block
    constexpr int GL = CS_T / CL;          // row lanes: 8-row groups per round
    constexpr int RB = GL / 8;             // row blocks per round
    static_assert(RB * COLS == CS_T, "one (row block, column) per thread");
    __shared__ float gsum[GL][COLS + 1];
    __shared__ float bsum[RB][COLS + 1];
    const int tx = threadIdx.x % CL;
    const int ty = threadIdx.x / CL;
    const int G = gridDim.x, xcd = blockIdx.x % 8, idx = blockIdx.x / 8;
    const int per = G / 8, rem = G % 8;
    const int64_t blk = (xcd < rem) ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    const int64_t c = blk * COLS + tx * 8;
    const int64_t nb = (T + 63) / 64;
    const int sb = threadIdx.x / COLS, sc = threadIdx.x % COLS;
    float acc = 0.0f;                      // column blk * COLS + threadIdx.x (first COLS threads)
    u32x4 w[8];                            // this lane's rows of the round
    auto load = [&](int64_t r0) {
        if (c < N && r0 < T) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = *reinterpret_cast<const u32x4*>(dy + min(r0 + i, T - 1) * ld + c);
        }
    };
    load((int64_t)ty * 8);
    for (int64_t b0 = 0; b0 < nb; b0 += RB) {
        const int64_t r0 = b0 * 64 + ty * 8;
        float gs[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) gs[e] = 0.0f;
        if (c < N) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (r0 + i < T) {
                    float f[8];
                    unpack8(w[i], f);
#pragma unroll
                    for (int e = 0; e < 8; ++e) gs[e] += f[e];
                }
        }
        load(r0 + RB * 64);                // in flight while this round is folded
#pragma unroll
        for (int e = 0; e < 8; ++e) gsum[ty][tx * 8 + e] = gs[e];
        lds_barrier();
        // the groups of row block b0 + sb inside [0, T)
        const int64_t left = T - (b0 + sb) * 64;
        const int ng = left <= 0 ? 0 : left >= 64 ? 8 : (int)((left + 7) / 8);
        float s = 0.0f;
#pragma unroll
        for (int g = 0; g < 8; ++g)
            if (g < ng) s += gsum[sb * 8 + g][sc];
        bsum[sb][sc] = s;
        lds_barrier();
        if (threadIdx.x < COLS) {
            const int nr = nb - b0 < RB ? (int)(nb - b0) : RB;
#pragma unroll 8
            for (int r = 0; r < nr; ++r) acc += bsum[r][threadIdx.x];
        }
    }
    if (threadIdx.x < COLS) {
        const int64_t col = blk * COLS + threadIdx.x;
        if (col < N) db[col] = acc;
    }
}

// db[c] = (((0 + part_0[c]) + part_1[c]) + ...) over nb row-block partials.
// The loads of 32 partials are issued before their sums, so a thread waits
// for memory once per 32 blocks instead of once per block; the additions
// keep the block order.
__global__ __launch_bounds__(256) void colsum_finish_kernel(const float* __restrict__ part,
                                                            int64_t ldp, int64_t nb, int64_t N,
                                                            float* __restrict__ db) {
    constexpr int U = 32;
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= N) return;
    float acc = 0.0f;
    int64_t b = 0;
    for (; b + U <= nb; b += U) {
        float v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) v[i] = part[(b + i) * ldp + c];
#pragma unroll
        for (int i = 0; i < U; ++i) acc += v[i];
    }
    for (; b < nb; ++b) acc += part[b * ldp + c];
    db[c] = acc;
}

template <bool PART_BF16>
hipError_t launch_reduce_parts(const ReduceProblem& p, hipStream_t s) {
    const bool b = p.out_bf16;
    switch (p.epi) {
    case EPI_NONE:
        return b ? launch_r<EPI_NONE, true, PART_BF16>(p, s)
                 : launch_r<EPI_NONE, false, PART_BF16>(p, s);
    case EPI_BIAS:
        return b ? launch_r<EPI_BIAS, true, PART_BF16>(p, s)
                 : launch_r<EPI_BIAS, false, PART_BF16>(p, s);
    case EPI_BIAS_GELU:
        return b ? launch_r<EPI_BIAS_GELU, true, PART_BF16>(p, s)
                 : launch_r<EPI_BIAS_GELU, false, PART_BF16>(p, s);
    case EPI_GELU_BWD:
        return b ? launch_r<EPI_GELU_BWD, true, PART_BF16>(p, s)
                 : launch_r<EPI_GELU_BWD, false, PART_BF16>(p, s);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_reduce(const ReduceProblem& p, hipStream_t s) {
    return p.parts_bf16 ? launch_reduce_parts<true>(p, s) : launch_reduce_parts<false>(p, s);
}

hipError_t launch_split_sum(const float* ws, int S, int64_t stride, int64_t ld, int64_t rows,
                            int64_t cols, void* out, int64_t ldo, bool out_bf16, hipStream_t s) {
    if (S < 1 || S > kMaxParts || (cols & 7) || (ld & 3) || (ldo & (out_bf16 ? 7 : 3)))
        return hipErrorInvalidValue;
    ReduceProblem p{};
    p.nparts = S;
    for (int i = 0; i < S; ++i) p.parts[i] = ws + i * stride;
    p.ldp = ld;
    p.row0 = 0;
    p.rows = rows;
    p.ncols = cols;
    p.epi = EPI_NONE;
    p.out = out;
    p.ldo = ldo;
    p.out_bf16 = out_bf16;
    return launch_reduce(p, s);
}

hipError_t launch_colsum_finish(const float* part, int64_t ldp, int64_t nb, int64_t N, float* db,
                                hipStream_t s) {
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(colsum_finish_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s,
                       part, ldp, nb, N, db);
    return hipGetLastError();
}

hipError_t launch_colsum(const void* dy, int64_t ld, int64_t T, int64_t N, float* db,
                         hipStream_t s) {
    if (N <= 0) return hipSuccess;
    const uint16_t* y = static_cast<const uint16_t*>(dy);
    // Column lanes: 2 while one block per CU covers the columns (its 32-byte row
    // segments cost more than they give in a second round), else the one of 4 and
    // 8 with the least work in its rounds of 256 blocks; few rows don't pay the
    // launch of more than 256 blocks.  8192 rows (us for 2, 4, 8): 3072 columns 20
    // 23 27, 6144 34 26 29, 10240 39 46 34, 20480 89 71 86; 64 rows of 20480: 9 7 6.
    auto rounds = [&](int w) { return (N + 256 * 8 * w - 1) / (256 * 8 * w) * w; };
    const int cl = N <= 256 * 16                                           ? 2
                   : rounds(4) < rounds(8) && (N <= 256 * 32 || T >= 1000) ? 4
                                                                           : 8;
    const dim3 blocks((unsigned)((N + 8 * cl - 1) / (8 * cl)));
    if (cl == 8) hipLaunchKernelGGL((colsum_kernel<8>), blocks, dim3(CS_T), 0, s, y, ld, T, N, db);
    else if (cl == 4) hipLaunchKernelGGL((colsum_kernel<4>), blocks, dim3(CS_T), 0, s, y, ld, T, N, db);
    else hipLaunchKernelGGL((colsum_kernel<2>), blocks, dim3(CS_T), 0, s, y, ld, T, N, db);
    return hipGetLastError();
}

}  // namespace atp
