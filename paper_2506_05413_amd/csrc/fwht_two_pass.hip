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
//
// A butterfly across lanes is ONE instruction per value, v <- v + c * v[partner] (v_fmac_f32 with a DPP source, c = +1
// in the lane whose bit is clear, -1 in the other): the lane with the bit clear gets a + b, the other b - a -- the
// difference with its sign flipped.  The flip is not undone on the spot: every later step is linear and pairs only
// values with equal flips, so a value simply carries the sign (-1)^(number of set bits among the lane bits used so
// far); row maxima ignore it, and the quantiser multiplies by 1/Delta anyway, so it multiplies by -1/Delta where the
// sign is -1 (exact).
//
// LDS layout: element i at i + 4 (i >> 5) + a few floats per block of the lane bits of pass 2, so that the 16-byte
// writes of pass 1, the 4-byte accesses of pass 2 (a half-wave covers all 32 banks) and the 16-byte reads of the
// quantiser are free of bank conflicts.
#include "fwht_row.h"
#include "gemm_common.h"      // fence-free barrier

namespace sr {
namespace {

// ---- butterflies across lanes ---------------------------------------------------------------------------
// v[e] += c * v[e] of the partner lane, for N values: LEVEL 0 lane ^ 1, 1 lane ^ 2, 2 lane ^ 7.
// (Inline assembly: the two wait states a DPP read needs after a vector write of the same register are given
// by the s_nop in front; inside the block no instruction reads what its predecessor wrote.)
#define SR_DPP_FMAC(i, ctrl) "v_fmac_f32_dpp %" #i ", %" #i ", %[c] " ctrl " row_mask:0xf bank_mask:0xf\n\t"
#define SR_DPP_14(ctrl)                                                                                                   \
    SR_DPP_FMAC(0, ctrl) SR_DPP_FMAC(1, ctrl) SR_DPP_FMAC(2, ctrl) SR_DPP_FMAC(3, ctrl) SR_DPP_FMAC(4, ctrl)              \
    SR_DPP_FMAC(5, ctrl) SR_DPP_FMAC(6, ctrl) SR_DPP_FMAC(7, ctrl) SR_DPP_FMAC(8, ctrl) SR_DPP_FMAC(9, ctrl)              \
    SR_DPP_FMAC(10, ctrl) SR_DPP_FMAC(11, ctrl) SR_DPP_FMAC(12, ctrl) SR_DPP_FMAC(13, ctrl)
#define SR_DPP_16(ctrl) SR_DPP_14(ctrl) SR_DPP_FMAC(14, ctrl) SR_DPP_FMAC(15, ctrl)
#define SR_OPS_14(v)                                                                                                      \
    "+v"((v)[0]), "+v"((v)[1]), "+v"((v)[2]), "+v"((v)[3]), "+v"((v)[4]), "+v"((v)[5]), "+v"((v)[6]), "+v"((v)[7]),       \
        "+v"((v)[8]), "+v"((v)[9]), "+v"((v)[10]), "+v"((v)[11]), "+v"((v)[12]), "+v"((v)[13])
#define SR_LANE_BUTTERFLY(ctrl)                                                                                           \
    if constexpr (N == 16) {                                                                                              \
        asm("s_nop 1\n\t" SR_DPP_16(ctrl) : SR_OPS_14(v), "+v"(v[14]), "+v"(v[15]) : [c] "v"(c));                         \
    } else {                                                                                                              \
        asm("s_nop 1\n\t" SR_DPP_14(ctrl) : SR_OPS_14(v) : [c] "v"(c));                                                   \
        asm("s_nop 1\n\t" SR_DPP_14(ctrl) : SR_OPS_14(v + 14) : [c] "v"(c));                                              \
    }
template <int LEVEL, int N>
__device__ __forceinline__ void lane_butterfly(float (&v)[N], float c)
{
    static_assert(N == 16 || N == 28, "register sets of pass 1 and pass 2");
    if constexpr (LEVEL == 0) { SR_LANE_BUTTERFLY("quad_perm:[1,0,3,2]") }
    else if constexpr (LEVEL == 1) { SR_LANE_BUTTERFLY("quad_perm:[2,3,0,1]") }
    else { SR_LANE_BUTTERFLY("row_half_mirror") }
}

// ---- shape of a row -----------------------------------------------------------------------------------
template <int K, int THREADS = 0>
struct TwoPass {
    static constexpr bool KRON = !is_pow2(K);            // 28 * 512
    static constexpr int R = KRON ? 28 : 16;             // values per thread in pass 2
    static constexpr int Q = KRON ? 3 : ilog2(K) - 10;   // index bits across lanes in pass 2
    static constexpr int Q0 = KRON ? 6 : 10;             // the lowest of them
    static constexpr int RSTRIDE = KRON ? 512 : 64;      // elements between a thread's values in pass 2
    static constexpr int COLS = KRON ? 512 : K / 16;     // sets of values in pass 2
    static constexpr int NT = THREADS ? THREADS : COLS;  // threads (a multiple of 64)
    static constexpr int NG = (K / 16 + NT - 1) / NT;    // sets of 16 contiguous values per thread in pass 1
    // Bank of a lane's access in pass 2: the element's 1 << Q0 is a multiple of 32 banks for the powers of two (8 banks
    // for 14336, where 64 floats come with 8 of padding), so EXTRA floats of padding per 1 << XSH elements spread the
    // lane bits over the banks that the 5 - Q low bits of the index leave free.  A multiple of 4: 16-byte accesses.
    static constexpr int XSH = KRON ? 8 : 10;
    static constexpr int EXTRA = KRON ? 4 : 32 >> Q;
    static constexpr int LEN = K + K / 32 * 4 + (K >> XSH) * EXTRA;
    static_assert(NT % 64 == 0 && NT >= COLS);
    static_assert(Q >= 1 && Q <= 3 && (KRON ? K == 14336 : true), "two passes of 6 and 4 + Q bits");
    __device__ static __forceinline__ constexpr int pos(int i) { return i + ((i >> 5) << 2) + (i >> XSH) * EXTRA; }
    static constexpr int RPOS = RSTRIDE + RSTRIDE / 32 * 4 + (KRON ? (RSTRIDE >> XSH) * EXTRA : 0);
    // sign that the 16 values of set g = i >> 4 carry into the quantiser: the lane bits of pass 1 were g & 3, those of
    // pass 2 the index bits Q0 .. Q0 + Q - 1
    // (bits that `mask` leaves out are not transformed and flip nothing)
    __device__ static __forceinline__ bool flipped(int g, uint32_t mask = 0xFFFFFFFFu)
    {
        const int i = (int)((uint32_t)(16 * g) & mask);
        return __builtin_popcount(((i >> 4) & 3) | (((i >> Q0) & ((1 << Q) - 1)) << 2)) & 1;
    }
};

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
    constexpr int NT = S::NT, NW = NT / 64;
    const uint32_t mask = MASKED ? had_mask : 0xFFFFFFFFu;
    extern __shared__ __attribute__((aligned(16))) float row[];
    __shared__ float red[NW];
    const int t = threadIdx.x, lane = t & 63;
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
    const float c0 = (lane & 1) ? -1.f : 1.f, c1 = (lane & 2) ? -1.f : 1.f;
#pragma unroll
    for (int i = 0; i < S::NG; ++i) {
        const int g = t + i * NT;
        if (K / 16 % NT == 0 || g < K / 16) {            // whole waves (K / 16 is a multiple of 64)
            float v[16];
            if constexpr (MASKED) {
                union { uint4 u[2]; half2v h[8]; } raw;
                raw.u[0] = ld.u[i][0];
                raw.u[1] = ld.u[i][1];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 f = HAS_PRE ? ld.p[i][q] : make_float4(1.f, 1.f, 1.f, 1.f);
                    v[4 * q] = __builtin_fmaf((float)raw.h[2 * q][0], f.x, 0.f);
                    v[4 * q + 1] = __builtin_fmaf((float)raw.h[2 * q][1], f.y, 0.f);
                    v[4 * q + 2] = __builtin_fmaf((float)raw.h[2 * q + 1][0], f.z, 0.f);
                    v[4 * q + 3] = __builtin_fmaf((float)raw.h[2 * q + 1][1], f.w, 0.f);
                }
                butterflies_masked<4>(v, mask & 15u);
            } else {
                first_level16<GATE>(ld.u[i], ld.gu[i], ld.p[i], HAS_PRE, v);
                butterflies_from<4, 2>(v);
            }
            if (mask & 16u) lane_butterfly<0>(v, c0);
            if (mask & 32u) lane_butterfly<1>(v, c1);
            float *d = row + S::pos(16 * g);
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<float4 *>(d + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        }
    }
    // (barriers without the fence of __syncthreads: that would also wait for the warming loads below)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_nofence();
    // warming the memory-side cache for the kernel that follows (see fwht4096_wave_kernel): one word of every
    // 128-byte line of the region, shared among the threads of the launch, ordinary loads, never looked at
    uint32_t warm_acc = 0;
    if (warm) {
        const int64_t nthreads = (int64_t)gridDim.x * NT;
        for (int64_t l = (int64_t)blockIdx.x * NT + t; l < warm_lines; l += nthreads) warm_acc ^= warm[l * 32];
    }

    // ---- pass 2: the other bits -------------------------------------------------------------------
    // Lane ^ 7 is the partner of the third level, so the bits that index the row are those of a ^ (a >> 2): each of the
    // partners lane ^ 1, ^ 2, ^ 7 then differs in one of them.
    float amax = 0.f;
    if (NT == S::COLS || t < S::COLS) {                  // whole waves
        const int a = lane & ((1 << S::Q) - 1);
        const int q = S::Q == 3 ? a ^ ((a >> 2) * 3) : a;
        float *col = row + S::pos((t >> S::Q) + (q << S::Q0));
        float v[S::R], o[S::R];
#pragma unroll
        for (int r = 0; r < S::R; ++r) v[r] = col[S::RPOS * r];
        auto across_lanes = [&]() {
            if (mask & (1u << S::Q0)) lane_butterfly<0>(v, (q & 1) ? -1.f : 1.f);
            if constexpr (S::Q >= 2) if (mask & (2u << S::Q0)) lane_butterfly<1>(v, (q & 2) ? -1.f : 1.f);
            if constexpr (S::Q >= 3) if (mask & (4u << S::Q0)) lane_butterfly<2>(v, (q & 4) ? -1.f : 1.f);
        };
        if constexpr (S::KRON) {
            across_lanes();
            h28_program(v, o);
        } else {
            if constexpr (MASKED) butterflies_masked<4>(v, (mask >> 6) & 15u);
            else butterflies<4>(v);
            across_lanes();
#pragma unroll
            for (int r = 0; r < S::R; ++r) o[r] = v[r];
        }
#pragma unroll
        for (int r = 0; r < S::R; r += 2) amax = fmaxf(fmaxf(amax, fabsf(o[r])), fabsf(o[r + 1]));
#pragma unroll
        for (int r = 0; r < S::R; ++r) col[S::RPOS * r] = o[r];    // the same thread read these: nothing to wait for
    }
    amax = max_of_wave(amax);
    if (lane == 0) red[t >> 6] = amax;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_nofence();
    amax = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) amax = fmaxf(amax, red[w]);
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
        uint32_t *q = reinterpret_cast<uint32_t *>(Q + m * (int64_t)(K / 2));
#pragma unroll
        for (int i = 0; i < S::NG; ++i) {
            const int g = t + i * NT;
            if (K / 16 % NT == 0 || g < K / 16) {
                const float *s16 = row + S::pos(16 * g);
                const float sd = S::flipped(g, mask) ? -inv_delta : inv_delta;
                uint32_t w2[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 a = *reinterpret_cast<const float4 *>(s16 + 8 * h);
                    const float4 b = *reinterpret_cast<const float4 *>(s16 + 8 * h + 4);
                    const float y[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                    w2[h] = quant_pack8(y, sd);
                }
                *reinterpret_cast<uint2 *>(q + 2 * g) = make_uint2(w2[0], w2[1]);
            }
        }
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
