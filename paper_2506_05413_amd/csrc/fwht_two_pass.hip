// Rotation + quantiser for rows of 2048, 4096, 8192 and 14336 values: one row per workgroup, two passes over the row.
// (Paper: online exact Hadamard before the projection, section "Methodology"; quantiser Eq. (1).)
//
// Pass 1 covers the index bits 0..5 of the row, straight from the global load: four in registers (a thread holds 16
// contiguous values), two across neighbouring lanes by DPP.  Pass 2 covers the rest: registers take the bits 6..9 (or,
// for 14336 = 28 * 512, the Paley factor H_28), the lane bits 0.. the 1, 2 or 3 bits that are left.  So the row goes
// through LDS twice (pass 1 -> pass 2, pass 2 -> quantiser), whatever its length, where passes of four bits in registers
// alone (fwht_quant_kernel) take one round trip and one barrier more for every four bits, and a whole one for a single
// bit left over.  A single wave of this chip issues a vector instruction every ~5 cycles however independent its
// instructions are, and two waves per SIMD double that: with few rows what counts is the chain of one row, which is
// spread over K / 16 threads here (14336: 896, of which 512 do the second pass, while every row has a CU to itself; 512
// beyond, two rows per CU).
//
// Bound by: the chain of one row with few rows; vector-ALU issue with many (K = 14336 gated, 16384 rows: 1.12 GB in 258 us,
// 4.3 TB/s).  Measured against fwht_quant_kernel, which these rows took before (graph-timed, us, tiles; rows 1 / 128 / 2048 /
// 16384):  14336 gated 6.2 / 8.4 / 45.4 / 297 -> 5.8 / 7.2 / 38.1 / 260;  14336 5.3 / 6.8 / 33.9 / 219 -> 4.9 / 6.1 / 28.8 /
// 193;  8192 gated, factors 4.9 / 6.2 / 25.3 / 164 -> 4.2 / 5.4 / 21.6 / 150;  8192 4.6 / 5.7 / 21.0 / 133 -> 3.8 / 4.9 /
// 17.2 / 112;  2048 3.3 / 3.6 / 6.9 / 33.5 -> 3.0 / 3.2 / 6.2 / 30.2;  4096 gated 3.8 / 4.9 / 13.9 / 82.3 -> 3.5 / 4.5 /
// 12.9 / 80.5.  Nibble output gains the same or a little more.  Every level is the same addition of the same two values as
// there (index bits in rising order), so codes and scales did not change.  Tiles show the sign of a zero (field 32 is -0):
// a value that is exactly zero gets the field 0, as without flips; only where all of a row is zero with negative zeros among
// them, and for the zeros that H_28 negates (K = 14336), the general kernel wrote 32.  (Ending the flips in front of H_28
// keeps those too: 16384 gated rows 256 -> 261 us, for the same numbers; dropped.)
// Measured and dropped for 14336: 896 threads with two rows per CU (14 waves each: 1024 rows 21.1 -> 27.4 us); workgroups
// that walk over rows, the next row requested after pass 1 (it helped the three-pass kernel: 264 -> 243 us; here 193 against
// 192 us without a gate, spills and 375 against 258 us with one); for 4096 two, four or eight rows per workgroup one after
// the other, all loads issued up front (9.7 / 10.8 / 13.8 against 9.0 us at 2048 rows).
#include "two_pass_row.h"

namespace sr {
namespace {

// MASKED: head-wise transform -- only the index bits set in had_mask are butterflied (uniform branches; powers of two).
template <int K, int THREADS, bool HAS_PRE, bool F6, bool GATE, bool MASKED>
__global__ __launch_bounds__((TwoPass<K, THREADS>::NT)) void fwht_two_pass_kernel(const __half *__restrict__ X, int64_t ldx, int64_t rows,
                                                                      const float *__restrict__ pre, float clip, float post_scale,
                                                                      uint8_t *__restrict__ Q, float *__restrict__ scale_out,
                                                                      const __half *__restrict__ gate, int64_t ldg,
                                                                      const uint32_t *__restrict__ warm, int64_t warm_lines,
                                                                      uint32_t had_mask)
{
    using S = TwoPass<K, THREADS>;
    static_assert(!MASKED || (!GATE && !F6 && !S::KRON), "head-wise: powers of two without a gate row, nibbles");
    constexpr int NT = S::NT;
    const uint32_t mask = MASKED ? had_mask : 0xFFFFFFFFu;
    extern __shared__ __attribute__((aligned(16))) float row[];
    __shared__ float red[NT / 64];
    const int t = threadIdx.x;
    int64_t m = blockIdx.x;
    if constexpr (F6) {
        // the eight rows of a tile block from the same XCD: workgroup w = 8 a + x (XCD x) takes row a % 8 of
        // block 8 (a / 8) + x
        const int64_t w = blockIdx.x, x = w & 7, a = w >> 3;
        m = 8 * (8 * (a >> 3) + x) + (a & 7);
    }
    if (m >= rows) {                                     // the whole workgroup: no barrier is left behind
        if constexpr (F6) zero_f6_padding_row<K, NT>(Q, (rows + 7) >> 3, m, t);
        return;
    }

    // ---- pass 1: index bits 0..5 ------------------------------------------------------------------
    RowLoad<K, NT> ld;
    row_load<K, NT, false, GATE, HAS_PRE ? 5 : 1>(X + m * ldx, pre, t, ld, GATE ? gate + m * ldg : nullptr);
    uint32_t warm_acc = 0;
    float o[S::R];
    const float amax = two_pass_rotate<S, K, HAS_PRE, GATE, MASKED, false>(ld, row, red, t, mask, o, [&]() {
        // warming the memory-side cache for the kernel that follows (see fwht4096_wave_kernel): one word of every
        // 128-byte line of the region, shared among the threads of the launch, ordinary loads, never looked at
        if (warm) {
            const int64_t nthreads = (int64_t)gridDim.x * NT;
            for (int64_t l = (int64_t)blockIdx.x * NT + t; l < warm_lines; l += nthreads) warm_acc ^= warm[l * 32];
        }
    });
    // Delta = clip * absmax / 7 (1 for an all-zero row), Eq. (1) with the signed range
    const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
    const float inv_delta = 1.f / delta;
    if (t == 0) scale_out[m] = (amax == 0.f) ? 1.f : delta * post_scale;

    // ---- quantise ----------------------------------------------------------------------------------
    if constexpr (F6) {
        if (t < K / 32) {
            const float lo = S::flipped(2 * t, mask) ? -inv_delta : inv_delta, hi = S::flipped(2 * t + 1, mask) ? -inv_delta : inv_delta;
            // exact zeros become the field 0 (plain rows of 4096, which have always come from this kernel, write 32 where the
            // sign is flipped)
            quant_store_f6_piece<GATE || K != 4096>(row + S::pos(32 * t), lo, hi, Q, (rows + 7) >> 3, m, t);
        }
    } else {
        quantise_row_nibbles<S, K>(row, inv_delta, mask, Q + m * (int64_t)(K / 2), t);
    }
    asm volatile("" ::"v"(warm_acc));                    // keeps the warming loads; they returned long ago
}

template <int K, int THREADS, bool HAS_PRE, bool F6, bool GATE, bool MASKED = false>
hipError_t launch(const __half *X, int64_t rows, int64_t ldx, const float *pre, float clip, float post_scale, uint8_t *Q,
                  float *scale_out, const __half *gate, int64_t ldg, hipStream_t st, const void *warm, size_t warm_bytes,
                  uint32_t had_mask = 0xFFFFFFFFu)
{
    using S = TwoPass<K, THREADS>;
    constexpr size_t lds = S::LEN * sizeof(float);
    constexpr auto kern = fwht_two_pass_kernel<K, THREADS, HAS_PRE, F6, GATE, MASKED>;
    if constexpr (lds > 40 * 1024)
        if (hipError_t e = allow_dynamic_lds<kern>((int)lds); e != hipSuccess) return e;
    const int64_t blocks = F6 ? (rows + 63) / 64 * 64 : rows;
    // the hint is honoured from 256 workgroups on (a launch of a few rows cannot move megabytes on the side)
    const bool warms = warm && warm_bytes >= 128 && blocks >= 256;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(S::NT), lds, st, X, ldx, rows, pre, clip, post_scale, Q, scale_out, gate,
                       ldg, warms ? static_cast<const uint32_t *>(warm) : nullptr, (int64_t)(warm_bytes / 128), had_mask);
    return hipGetLastError();
}

template <int K, int THREADS = 0>
hipError_t launch_k(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip, float post_scale, uint8_t *Q,
                    float *scale_out, const __half *gate, int64_t ldg, hipStream_t st, bool f6, const void *warm, size_t warm_bytes)
{
    const __half *x = static_cast<const __half *>(X);
#define SR_LAUNCH(P, F, G) launch<K, THREADS, P, F, G>(x, rows, ldx, pre, clip, post_scale, Q, scale_out, gate, ldg, st, warm, warm_bytes)
    if (gate) return pre ? (f6 ? SR_LAUNCH(true, true, true) : SR_LAUNCH(true, false, true))
                         : (f6 ? SR_LAUNCH(false, true, true) : SR_LAUNCH(false, false, true));
    return pre ? (f6 ? SR_LAUNCH(true, true, false) : SR_LAUNCH(true, false, false))
               : (f6 ? SR_LAUNCH(false, true, false) : SR_LAUNCH(false, false, false));
#undef SR_LAUNCH
}

template <int K>
hipError_t launch_masked(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip, float post_scale, uint8_t *Q,
                         float *scale_out, uint32_t had_mask, hipStream_t st)
{
    const __half *x = static_cast<const __half *>(X);
#define SR_LAUNCH(P) launch<K, 0, P, false, false, true>(x, rows, ldx, pre, clip, post_scale, Q, scale_out, nullptr, 0, st, nullptr, 0, had_mask)
    return pre ? SR_LAUNCH(true) : SR_LAUNCH(false);
#undef SR_LAUNCH
}

}  // namespace

hipError_t launch_fwht_two_pass_heads(const void *X, int64_t rows, int64_t K, int64_t ldx, const float *pre, float clip,
                                      float post_scale, uint8_t *Q, float *scale_out, uint32_t had_mask, hipStream_t st)
{
    switch (K) {
        case 2048: return launch_masked<2048>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, had_mask, st);
        case 4096: return launch_masked<4096>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, had_mask, st);
        case 8192: return launch_masked<8192>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, had_mask, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fwht_two_pass(const void *X, int64_t rows, int64_t K, int64_t ldx, const float *pre, float clip,
                                float post_scale, uint8_t *Q, float *scale_out, const __half *gate, int64_t ldg,
                                hipStream_t st, bool f6, const void *warm, size_t warm_bytes)
{
#define SR_ARGS X, rows, ldx, pre, clip, post_scale, Q, scale_out, gate, ldg, st, f6, warm, warm_bytes
    switch (K) {
        case 2048: return launch_k<2048>(SR_ARGS);
        case 4096: return launch_k<4096>(SR_ARGS);
        case 8192: return launch_k<8192>(SR_ARGS);
        case 14336: {
            // 896 threads shorten pass 1 (one set of 16 values per thread instead of two) while every row has a CU to
            // itself: gated, one row 6.0 -> 5.8 us, 256 rows 8.9 -> 8.5; with two rows per CU they lose (see above)
            bool wide = rows <= compute_units();
            if (int64_t f; tuned(kTuneFwhtStream, f)) wide = f != 0;
            return wide ? launch_k<14336, 896>(SR_ARGS) : launch_k<14336>(SR_ARGS);
        }
        default: return hipErrorInvalidValue;
    }
#undef SR_ARGS
}

}  // namespace sr
