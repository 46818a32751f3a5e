// Pieces shared by the compute-bound GEMM kernels (int8-MFMA kernel in gemm_prefill.hip, FP6-MFMA
// kernel in gemm_f6.hip): hand-placed waits, LDS-DMA loads, the transposing epilogue, launch helpers.
#pragma once

#include "sr_common.h"
#include "gemm_rules.h"

#include <hip/hip_fp16.h>

#include <type_traits>

namespace sr {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------
// The DMA loads, their waits and the barrier are inline assembly on purpose: the compiler
// would order every LDS read behind ALL outstanding LDS-DMA loads (vmcnt(0)) and put a full
// fence on every barrier, which serialises the pipeline.  Hazards are handled by hand:
// wait_vmcnt<n>() lets the n youngest loads stay in flight (loads complete in order), and the
// "memory" clobbers keep the compiler from moving LDS accesses across these statements.
// ------------------------------------------------------------------------------------------
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void barrier_nofence() { asm volatile("s_barrier" ::: "memory"); }

// 64 lanes x 16 bytes: global (base + per-lane 32-bit offset) -> LDS bytes [lds, lds + 1024)
__device__ __forceinline__ void dma16(const uint8_t *base, uint32_t lane_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(lane_off), "s"(base)
                 : "memory", "m0");
}

// f(0), .. f(N - 1) with constants
template <int N, typename F> __device__ __forceinline__ void static_for(F f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// 32 packed codes -> the operands of two 16x16x64 int8 products
__device__ __forceinline__ void unpack16(const u32x4 w, v4i &a0, v4i &a1)
{
    constexpr unsigned HM = 0xF0F0F0F0u;     // nibble kept in the high half of its byte = code * 16
    a0[0] = (int)((w.x << 4) & HM); a0[1] = (int)(w.x & HM);
    a0[2] = (int)((w.y << 4) & HM); a0[3] = (int)(w.y & HM);
    a1[0] = (int)((w.z << 4) & HM); a1[1] = (int)(w.z & HM);
    a1[2] = (int)((w.w << 4) & HM); a1[3] = (int)(w.w & HM);
}

// fp16 of a * b, rounded once, or to fp32 first.  Spelled out in the kernels for up to 16 tokens, because the calls in one launch
// reproduce the outputs of the kernel that they replace bit for bit: from __float2half_rn(a * b) the compiler makes the first where
// one value is stored at a time and the second where it converts pairs.
__device__ __forceinline__ __half rounded_once(float a, float b)
{
    uint32_t h;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(a), "v"(b));
    return __ushort_as_half((unsigned short)h);
}
__device__ __forceinline__ __half rounded_twice(float a, float b)
{
    float p = a * b;
    asm("" : "+v"(p));
    return __float2half_rn(p);
}

// ------------------------------------------------------------------------------------------
// Epilogue for 32 x 32 MFMA tiles: dequantise, then transpose the wave's WM x WN tile through LDS,
// 32 tokens at a time, so that global memory is written in whole rows of the tile (16 bytes per
// lane, WN * 2 contiguous bytes per token) instead of 8-byte pieces scattered over 32 rows per
// instruction.  In the accumulator layout a lane owns token (l & 31) and, per quad q, the four
// output channels 8q + 4 (l >> 5) .. + 3 of each tile.  `stage` is this wave's private LDS area of
// 32 * (WN * 2 + 16) bytes; the caller has made sure nobody else touches it.  sx[j] is the token
// scale / 256 of this lane's token in row block j, sw[i][q] the four channel scales of quad q of
// column block i (fetched by the caller; unused for the raw int32 output).
// The accumulators are either int32 holding 256 x the sum (int8 MFMA on codes x 16) or fp32
// holding the sum / 64 exactly (FP6 MFMA on codes / 8); sx carries the matching factor.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float acc_f32(int a) { return (float)a; }
__device__ __forceinline__ float acc_f32(float a) { return a; }
__device__ __forceinline__ int acc_i32(int a) { return a >> 8; }
__device__ __forceinline__ int acc_i32(float a) { return (int)(a * 64.f); }

// CG = MFMA column tiles staged at a time (FN by default; fewer where the staging area is small): the rows
// written to memory are then CG * 64 bytes long.
template <int FM, int FN, int CG = FN, typename V16>
__device__ __forceinline__ void store_wave_tile(const V16 (&acc)[FN][FM], uint8_t *stage, int lane, int m_base, int n_base,
                                                int M, int N, const float (&sx)[FM], const float4 (&sw)[FN][4],
                                                void *__restrict__ Yv, int64_t ldy, int out_i32)
{
    constexpr int WN = FN * 32;
    const int fr = lane & 31, fg = lane >> 5;
    if (out_i32) {                                          // raw accumulators: a debugging / test output, stored directly
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int m = m_base + j * 32 + fr, n = n_base + i * 32 + q * 8 + fg * 4;
                    if (m < M && n < N)
                        *reinterpret_cast<int4 *>(static_cast<int32_t *>(Yv) + (int64_t)m * ldy + n) =
                            make_int4(acc_i32(acc[i][j][4 * q]), acc_i32(acc[i][j][4 * q + 1]), acc_i32(acc[i][j][4 * q + 2]),
                                      acc_i32(acc[i][j][4 * q + 3]));
                }
    } else {
        constexpr int GW = CG * 32;                          // channels per staged group
        constexpr int RS = GW * 2 + 16;
        constexpr int CPR = GW * 2 / 16;
        constexpr int RPI = 64 / CPR;
        const int c = lane % CPR, r0 = lane / CPR;
#pragma unroll
        for (int j = 0; j < FM; ++j) {
#pragma unroll
            for (int i0 = 0; i0 < FN; i0 += CG) {
#pragma unroll
                for (int i = i0; i < i0 + CG && i < FN; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int nl = (i - i0) * 32 + q * 8 + fg * 4;
                        union { __half h[4]; uint2 u; } o;
                        o.h[0] = __float2half_rn(acc_f32(acc[i][j][4 * q]) * sx[j] * sw[i][q].x);
                        o.h[1] = __float2half_rn(acc_f32(acc[i][j][4 * q + 1]) * sx[j] * sw[i][q].y);
                        o.h[2] = __float2half_rn(acc_f32(acc[i][j][4 * q + 2]) * sx[j] * sw[i][q].z);
                        o.h[3] = __float2half_rn(acc_f32(acc[i][j][4 * q + 3]) * sx[j] * sw[i][q].w);
                        *reinterpret_cast<uint2 *>(stage + fr * RS + nl * 2) = o.u;
                    }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
                for (int r = r0; r < 32; r += RPI) {
                    const int m = m_base + j * 32 + r, nloc = i0 * 32 + c * 8, n = n_base + nloc;
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(stage + r * RS + c * 16);
                    // streamed once, never read back by this kernel: keep it from displacing operand panels in L2
                    if (lane < RPI * CPR && nloc < WN && m < M && n < N)
                        __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(static_cast<__half *>(Yv) + (int64_t)m * ldy + n));
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            }
        }
    }
}

}  // namespace
}  // namespace sr
