// Device code shared by the kernels that rotate a row on chip (T(v) = v H) and quantise it:
// the compile-time Paley matrix of order 28, register butterflies, the padded LDS row layout,
// the passes over it, and the INT4 quantise-and-pack step.
// (Paper: online exact Hadamard, section "Methodology"; quantiser Eq. (1).)
#pragma once

#include "sr_common.h"
#include "h28_program.h"

#include <hip/hip_fp16.h>
#include <utility>

namespace sr {
namespace {

// ---- Paley type-I Hadamard matrix of order 28, built at compile time -------------
// GF(27) = GF(3)[x] / (x^3 + 2x + 1); element c0 + c1 x + c2 x^2 has index c0 + 3 c1 + 9 c2.
constexpr int gf27_sub(int a, int b)
{
    int r = 0, w = 1;
    for (int d = 0; d < 3; ++d) {
        r += ((a % 3 - b % 3 + 3) % 3) * w;
        a /= 3; b /= 3; w *= 3;
    }
    return r;
}
constexpr int gf27_mul(int a, int b)
{
    int ca[3] = {a % 3, a / 3 % 3, a / 9}, cb[3] = {b % 3, b / 3 % 3, b / 9};
    int p[5] = {0, 0, 0, 0, 0};
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) p[i + j] += ca[i] * cb[j];
    // x^3 = x + 2 and x^4 = x^2 + 2x over GF(3)
    p[1] += 2 * p[4]; p[2] += p[4];
    p[0] += 2 * p[3]; p[1] += p[3];
    return p[0] % 3 + 3 * (p[1] % 3) + 9 * (p[2] % 3);
}
constexpr bool gf27_is_square(int e)
{
    for (int r = 1; r < 27; ++r)
        if (gf27_mul(r, r) == e) return true;
    return false;
}
// sign of H28[i][j]: first row +1, rest of first column -1, else chi(e_i - e_j) + identity
constexpr int h28_sign(int i, int j)
{
    if (i == 0) return 1;
    if (j == 0) return -1;
    if (i == j) return 1;
    return gf27_is_square(gf27_sub(i - 1, j - 1)) ? 1 : -1;
}
// The product itself is the generated straight-line program of h28_program.h (235 additions with shared partial
// sums; "row sum minus twice the negative terms" took 419).  It must reproduce the matrix built above: checked
// here on the 28 unit vectors, in integers, at compile time.
constexpr bool h28_program_matches()
{
    for (int i = 0; i < 28; ++i) {
        int e[28] = {}, o[28] = {};
        e[i] = 1;
        h28_program(e, o);
        for (int j = 0; j < 28; ++j)
            if (o[j] != h28_sign(i, j)) return false;
    }
    return true;
}
static_assert(h28_program_matches(), "h28_program.h does not compute the Paley matrix of this file");

// ---- radix-2 butterflies on 2^B register values -----------------------------------
template <int B>
__device__ __forceinline__ void butterflies(float (&v)[1 << B])
{
#pragma unroll
    for (int h = 1; h < (1 << B); h <<= 1) {
#pragma unroll
        for (int i = 0; i < (1 << B); ++i) {
            if (!(i & h)) {
                float a = v[i], b = v[i | h];
                v[i] = a + b;
                v[i | h] = a - b;
            }
        }
    }
}

// the same, index bit 0 (.., log2 H0 - 1) already done
template <int B, int H0>
__device__ __forceinline__ void butterflies_from(float (&v)[1 << B])
{
#pragma unroll
    for (int h = H0; h < (1 << B); h <<= 1) {
#pragma unroll
        for (int i = 0; i < (1 << B); ++i) {
            if (!(i & h)) {
                float a = v[i], b = v[i | h];
                v[i] = a + b;
                v[i | h] = a - b;
            }
        }
    }
}

// ---- first butterfly level straight from a dword of two halves ------------------------------
// A product of a half with a float written as an FMA compiles to one mixed-precision FMA that reads the half
// in place (lower or upper half of the dword selected in the instruction); a plain conversion or product
// costs an instruction more per value.  For a pair (a, b) with factors (fa, fb):
//     b' = b fb,   a fa + b',   a fa - b'          three instructions for two values
// and without factors a * 1 + b, a * 1 - b (exact) with the 1 kept from the optimiser in a scalar register,
// which would otherwise turn the FMA back into conversions and an addition: two instructions.
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void pair_level(half2v h, float fa, float fb, float &sum, float &dif)
{
    const float b = __builtin_fmaf((float)h[1], fb, 0.f);
    sum = __builtin_fmaf((float)h[0], fa, b);
    dif = __builtin_fmaf((float)h[0], fa, -b);
}
__device__ __forceinline__ void pair_level(half2v h, float &sum, float &dif)
{
    float one;
    asm("s_mov_b32 %0, 1.0" : "=s"(one));
    sum = __builtin_fmaf((float)h[0], one, (float)h[1]);
    dif = __builtin_fmaf((float)h[0], one, -(float)h[1]);
}

__device__ __forceinline__ int pad(int i) { return i + ((i >> 6) << 2); }
constexpr int padded_len(int K) { return K + (K >> 6) * 4; }
// pad(g + i * P) - pad(g): a compile-time constant where P is a multiple of 64 (one base register and immediate
// offsets for a column of values P apart; written out, the compiler spends four integer instructions per access)
template <int P>
__device__ __forceinline__ int strided(int g, int i)
{
    if constexpr (P % 64 == 0) return i * (P + P / 16);
    else return pad(g + i * P) - pad(g);
}

constexpr int ilog2(int64_t v) { int l = 0; while ((int64_t(1) << (l + 1)) <= v) ++l; return l; }

// In-LDS pass over index bits [LO, LO+B).
// Where a thread has at least ~3.4 groups of 2^B values to do, it takes four groups that are neighbours in the low
// index bits at once: 16-byte LDS accesses instead of 4-byte ones (a quarter of the LDS instructions, four
// independent butterfly sets in flight; measured inside the K = 14336 kernel: this pass 1.8 -> 1.0 us of a
// workgroup's 7 us).  Lanes then read 4 q + 272 b floats apart (q = 0..3, b = block of 256): every bank once.
template <int K, int NT, int LO, int B, bool TRACK>
__device__ __forceinline__ void lds_pass(float *row, int t, float &amax)
{
    constexpr int E = 1 << B;
    if constexpr (LO >= 2 && ((K >> B) * 5 >= NT * 17) && (K >> B) % 4 == 0) {
        for (int g = t; g < (K >> B) / 4; g += NT) {
            const int g_low = g & ((1 << (LO - 2)) - 1);
            const int base = ((g >> (LO - 2)) << (LO + B)) | (g_low << 2);
            float4 q[E];
#pragma unroll
            for (int e = 0; e < E; ++e) q[e] = *reinterpret_cast<const float4 *>(row + pad(base + (e << LO)));
            float v[4][E];
#pragma unroll
            for (int e = 0; e < E; ++e) { v[0][e] = q[e].x; v[1][e] = q[e].y; v[2][e] = q[e].z; v[3][e] = q[e].w; }
#pragma unroll
            for (int c = 0; c < 4; ++c) butterflies<B>(v[c]);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                *reinterpret_cast<float4 *>(row + pad(base + (e << LO))) = make_float4(v[0][e], v[1][e], v[2][e], v[3][e]);
                if (TRACK) amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v[0][e]), fabsf(v[1][e]))), fmaxf(fabsf(v[2][e]), fabsf(v[3][e])));
            }
        }
        return;
    }
    for (int g = t; g < (K >> B); g += NT) {
        const int g_low = g & ((1 << LO) - 1);
        const int base = ((g >> LO) << (LO + B)) | g_low;
        float v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = row[pad(base + (e << LO))];
        butterflies<B>(v);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            row[pad(base + (e << LO))] = v[e];
            if (TRACK) amax = fmaxf(amax, fabsf(v[e]));
        }
    }
}

// All remaining power-of-two passes from bit LO up to LOGP.
template <int K, int NT, int LO, int LOGP, bool TRACK_LAST>
__device__ __forceinline__ void lds_passes(float *row, int t, float &amax)
{
    if constexpr (LO < LOGP) {
        constexpr int B = (LOGP - LO) >= 4 ? 4 : (LOGP - LO);
        constexpr bool last = (LO + B == LOGP);
        lds_pass<K, NT, LO, B, last && TRACK_LAST>(row, t, amax);
        __syncthreads();
        lds_passes<K, NT, LO + B, LOGP, TRACK_LAST>(row, t, amax);
    }
}

// ---- the same passes with a run-time choice of index bits (head-wise transforms) ---------------
// Bit b of `mask` set <=> the 2 x 2 factor on index bit b is applied; a clear bit leaves the
// identity there.  The branches are uniform over the workgroup.
template <int B>
__device__ __forceinline__ void butterflies_masked(float (&v)[1 << B], uint32_t mask)
{
#pragma unroll
    for (int h = 1; h < (1 << B); h <<= 1) {
        if (mask & (uint32_t)h) {
#pragma unroll
            for (int i = 0; i < (1 << B); ++i) {
                if (!(i & h)) {
                    float a = v[i], b = v[i | h];
                    v[i] = a + b;
                    v[i | h] = a - b;
                }
            }
        }
    }
}

template <int K, int NT, int LO, int LOGP>
__device__ __forceinline__ void lds_passes_masked(float *row, int t, uint32_t mask)
{
    if constexpr (LO < LOGP) {
        constexpr int B = (LOGP - LO) >= 4 ? 4 : (LOGP - LO);
        constexpr int E = 1 << B;
        const uint32_t mb = (mask >> LO) & (uint32_t)(E - 1);
        if (mb) {                                           // a pass with no selected bit is skipped whole
            for (int g = t; g < (K >> B); g += NT) {
                const int g_low = g & ((1 << LO) - 1);
                const int base = ((g >> LO) << (LO + B)) | g_low;
                float v[E];
#pragma unroll
                for (int e = 0; e < E; ++e) v[e] = row[pad(base + (e << LO))];
                butterflies_masked<B>(v, mb);
#pragma unroll
                for (int e = 0; e < E; ++e) row[pad(base + (e << LO))] = v[e];
            }
            __syncthreads();
        }
        lds_passes_masked<K, NT, LO + B, LOGP>(row, t, mask);
    }
}

// ---- quantise + pack eight values (shared by all kernels) ---------------------------------
// t = fma(y, 1/Delta, 1.5 * 2^23) rounds y/Delta to the nearest-even integer in the low mantissa
// bits (one rounding); the clamp to [-8, 7] is an integer median on those bits; the eight clamped
// words are packed by shift-adds modulo 2^32, the constant part subtracted once, and the
// offset-binary nibbles become two's complement by XOR 0x88888888.
constexpr uint32_t kMagicBits = 0x4B400000u;             // bit pattern of 1.5 * 2^23
constexpr uint32_t pack_bias()
{
    uint32_t c = 0;
    for (int e = 0; e < 8; ++e) c += (kMagicBits - 8u) << (4 * e);
    return c;
}
__device__ __forceinline__ uint32_t quant_pack8(const float (&y)[8], float inv_delta)
{
    const float magic = __uint_as_float(kMagicBits);
    uint32_t word = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        int bits = (int)__float_as_uint(fmaf(y[e], inv_delta, magic));
        bits = min(max(bits, (int)kMagicBits - 8), (int)kMagicBits + 7);
        word += (uint32_t)bits << (4 * e);
    }
    return (word - pack_bias()) ^ 0x88888888u;
}

// a rotated row in the padded layout -> packed nibbles at `out`
template <int K, int NT>
__device__ __forceinline__ void quantise_padded_row_nibbles(const float *row, const float inv_delta, uint8_t *out, const int t)
{
    uint32_t *q = reinterpret_cast<uint32_t *>(out);
    for (int c = t; c < K / 8; c += NT) {
        const float *src = row + pad(8 * c);
        const float4 a = *reinterpret_cast<const float4 *>(src);
        const float4 b = *reinterpret_cast<const float4 *>(src + 4);
        const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        q[c] = quant_pack8(v, inv_delta);
    }
}

// ---- the same quantiser writing "f6 tiles" (operand layout of the FP6-MFMA GEMM, see gemm_f6.hip) ----------
// A code c becomes the 6-bit sign-magnitude field (c < 0 ? 32 : 0) | |c| (the E2M3 pattern of c / 8).  The E2M3
// grid is uniform (steps of 1/8) up to 1.875, so the hardware conversion of (y / Delta) / 8, which rounds to
// nearest-even, yields exactly the field of rint(y / Delta); only the one-sided clamp (+7, -8) is done here.  A
// negative value that rounds to 0 becomes the field 32 (-0), which multiplies like 0.
// v_cvt_scalef32_2xpk16_fp6_f32 takes the even values of 32 consecutive ones in its first operand and the odd
// ones in its second, divides by its scale operand (a power of two) and returns the 32 fields in order, 6 bits
// each (checked value by value on the device: every code, every tie, both zeros, values beyond the clamp).
//
// One thread quantises the 32 consecutive values at s32 (16-byte aligned) = piece p of row m (k = 32 p ..
// 32 p + 31) and stores its 24 bytes: the first 16 and the last 8 go to different places of the tile block.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v6u __attribute__((ext_vector_type(6)));
__device__ __forceinline__ void store_f6_piece(const v6u f, uint8_t *__restrict__ T6, int64_t row_blocks, int64_t m, int p)
{
    const int C = p >> 2, t = (p >> 1) & 1, g = p & 1;
    const int64_t R = m >> 3;
    const int r = (int)(m & 7), swz = (int)(R & 1);
    uint8_t *blk = T6 + ((int64_t)C * row_blocks + R) * 768;
    *reinterpret_cast<uint4 *>(blk + 256 * t + 128 * (g ^ swz) + 16 * r) = make_uint4(f[0], f[1], f[2], f[3]);
    *reinterpret_cast<uint2 *>(blk + 512 + 128 * (g ^ swz) + 16 * r + 8 * t) = make_uint2(f[4], f[5]);
}
// thread t of NT: zero codes into row m if it pads the last block of 8 (rows <= m < 8 row_blocks)
template <int K, int NT>
__device__ __forceinline__ void zero_f6_padding_row(uint8_t *__restrict__ T6, int64_t row_blocks, int64_t m, int t)
{
    if (m >= 8 * row_blocks) return;
    for (int p = t; p < K / 32; p += NT) store_f6_piece(v6u{0u, 0u, 0u, 0u, 0u, 0u}, T6, row_blocks, m, p);
}
// (inv_lo for the first 16 values, inv_hi for the last 16: callers whose values carry a sign per group of 16
// pass +-1/Delta; the others the same factor twice.  PLUS_ZERO: a value that is exactly zero gets the field 0 although its
// factor is negative: + 0 inside the multiply-add turns -0 into +0.)
template <bool PLUS_ZERO = false>
__device__ __forceinline__ void quant_store_f6_piece(const float *s32, float inv_lo, float inv_hi, uint8_t *__restrict__ T6,
                                                     int64_t row_blocks, int64_t m, int p)
{
    v16f ev, od;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float4 q = *reinterpret_cast<const float4 *>(s32 + 4 * k);
        const float inv_delta = k < 4 ? inv_lo : inv_hi;
        auto scaled = [&](float y) { return __builtin_amdgcn_fmed3f(PLUS_ZERO ? __builtin_fmaf(y, inv_delta, 0.f) : y * inv_delta, -8.f, 7.f); };
        ev[2 * k] = scaled(q.x);
        od[2 * k] = scaled(q.y);
        ev[2 * k + 1] = scaled(q.z);
        od[2 * k + 1] = scaled(q.w);
    }
    store_f6_piece(__builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(ev, od, 8.f), T6, row_blocks, m, p);
}
__device__ __forceinline__ void quant_store_f6_piece(const float *s32, float inv_delta, uint8_t *__restrict__ T6,
                                                     int64_t row_blocks, int64_t m, int p)
{
    quant_store_f6_piece(s32, inv_delta, inv_delta, T6, row_blocks, m, p);
}

// ---- rotation of one row by a whole workgroup -----------------------------------------------
// x (fp16, optionally times pre) -> T(x) in `row` (fp32, padded layout, LDS) and the row's
// absolute maximum, returned to every thread.  NT threads, t = thread index, red = NT / 64 floats
// of LDS.  Ends with the row complete and visible to all threads.
// The first pass (index bits 0..3, 16 contiguous values per group) is split into its global
// loads and the rest, so that a caller can put other loads between the two.
template <int K, int NT>
struct RowLoad {
    static constexpr int NG = (K / 16 + NT - 1) / NT;      // groups of 16 values per thread
    uint4 u[NG][2];
    float4 p[NG][4];                                       // the matching 16 values of `pre`, if any
    uint4 gu[NG][2];                                       // the matching 16 values of the gate row, if any
};

// ALWAYS: threads beyond the row load group 0 instead of nothing, so that the loads sit in straight-line code
// (for a caller that issues further loads behind these and wants the compiler to count them in its waits).
// PARTS: 1 = the row (and its gate row), 2 = the values of `pre` if there is one, 4 = of a `pre` that is known to be there
// (no branch between the loads)
template <int K, int NT, bool ALWAYS = false, bool GATE = false, int PARTS = 3>
__device__ __forceinline__ void row_load(const __half *__restrict__ x, const float *__restrict__ pre, const int t,
                                         RowLoad<K, NT> &ld, const __half *__restrict__ gate = nullptr)
{
#pragma unroll
    for (int i = 0; i < RowLoad<K, NT>::NG; ++i) {
        int g = t + i * NT;
        if (ALWAYS) g = g < K / 16 ? g : 0;
        if (K / 16 % NT == 0 || g < K / 16) {
            if constexpr (PARTS & 1) {
                ld.u[i][0] = *reinterpret_cast<const uint4 *>(x + 16 * g);
                ld.u[i][1] = *reinterpret_cast<const uint4 *>(x + 16 * g + 8);
                if constexpr (GATE) {
                    ld.gu[i][0] = *reinterpret_cast<const uint4 *>(gate + 16 * g);
                    ld.gu[i][1] = *reinterpret_cast<const uint4 *>(gate + 16 * g + 8);
                }
            }
            if constexpr (PARTS & 6) {
                if ((PARTS & 4) || pre) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) ld.p[i][q] = *reinterpret_cast<const float4 *>(pre + 16 * g + 4 * q);
                }
            }
        }
    }
}

// The 16 loaded values of a thread, times silu(gate) and / or the factors, after the butterfly level of index bit 0.
// ROUNDED: both products of a pair are rounded before they are added (pair_level rounds one of them).
template <bool GATE, bool ROUNDED = false>
__device__ __forceinline__ void first_level16(const uint4 (&u)[2], const uint4 (&gu)[2], const float4 (&p)[4],
                                              const bool has_pre, float (&v)[16])
{
    union { uint4 u[2]; half2v h[8]; } raw;
    raw.u[0] = u[0];
    raw.u[1] = u[1];
    float f[16];                                       // per-element factor: silu(gate) and / or 1 / s
    if constexpr (GATE) {
        union { uint4 u[2]; half2v h[8]; } graw;
        graw.u[0] = gu[0];
        graw.u[1] = gu[1];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            // silu(g) = g / (1 + exp(-g)); exp(-g) = inf for very negative g gives g * 0 = 0
            const _Float16 gh = graw.h[e >> 1][e & 1];
            const float sig = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(__builtin_fmaf((float)gh, -1.44269504088896341f, 0.f)));
            f[e] = __builtin_fmaf((float)gh, sig, 0.f);
        }
    }
    if (GATE || has_pre) {
        if (has_pre) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 sc = p[q];
                if constexpr (GATE) { f[4 * q] *= sc.x; f[4 * q + 1] *= sc.y; f[4 * q + 2] *= sc.z; f[4 * q + 3] *= sc.w; }
                else { f[4 * q] = sc.x; f[4 * q + 1] = sc.y; f[4 * q + 2] = sc.z; f[4 * q + 3] = sc.w; }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (ROUNDED) {
                const float a = __builtin_fmaf((float)raw.h[e][0], f[2 * e], 0.f), b = __builtin_fmaf((float)raw.h[e][1], f[2 * e + 1], 0.f);
                v[2 * e] = a + b;
                v[2 * e + 1] = a - b;
            } else {
                pair_level(raw.h[e], f[2 * e], f[2 * e + 1], v[2 * e], v[2 * e + 1]);
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) pair_level(raw.h[e], v[2 * e], v[2 * e + 1]);
    }
}

// GATE: x = silu(gate) * x in fp32 before the smoothing factors (the down-projection input of a gated FFN,
// paper Fig. 2: sigma(gate) (.) up, then 1/s, Hadamard, quantiser).
struct NoHook { __device__ __forceinline__ void operator()() const {} };

// after_pass1: called once the loaded values have been consumed (for loads that should travel during the rest of the
// row's work).
template <int K, int NT, bool GATE = false, bool ROUNDED = false, typename Hook = NoHook>
__device__ __forceinline__ float rotate_loaded_row_absmax(const RowLoad<K, NT> &ld, const float *__restrict__ pre,
                                                          float *row, float *red, const int t, Hook after_pass1 = Hook{})
{
    constexpr bool KRON = !is_pow2(K);
    constexpr int P2 = KRON ? K / 28 : K;       // power-of-two factor
    constexpr int LOGP = ilog2(P2);
    static_assert(LOGP >= 4 && K % 16 == 0, "first pass needs 16 contiguous values");

    // ---- pass 1: bits 0..3 on the loaded values ------------------------------------------
#pragma unroll
    for (int i = 0; i < RowLoad<K, NT>::NG; ++i) {
        const int g = t + i * NT;
        if (K / 16 % NT == 0 || g < K / 16) {
            float v[16];
            first_level16<GATE, ROUNDED>(ld.u[i], ld.gu[i], ld.p[i], pre != nullptr, v);
            butterflies_from<4, 2>(v);
            float *dst = row + pad(16 * g);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4 *>(dst + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        }
    }
    after_pass1();
    __syncthreads();

    // ---- remaining power-of-two bits ---------------------------------------------------
    float amax = 0.f;
    if constexpr (LOGP == 4 && !KRON) {
        // K = 16 cannot occur (K >= 64); kept for completeness of the template
    }
    // a single leftover bit of the power-of-two part is folded into the Paley pass (56 values per group)
    // (with more than 256 threads per row the merged pass would leave most of them idle: 28 values per thread then)
    constexpr bool MERGE = KRON && ((LOGP - 4) % 4 == 1) && NT <= 256;
    lds_passes<K, NT, 4, MERGE ? LOGP - 1 : LOGP, !KRON>(row, t, amax);

    // ---- Paley factor: 28 values at stride P2 per group ---------------------------------
    if constexpr (MERGE) {
        constexpr int HALF = P2 / 2;
        for (int g = t; g < HALF; g += NT) {
            float a[28], b[28], o[28];
            float *lo_p = row + pad(g), *hi_p = row + pad(g + HALF);
#pragma unroll
            for (int i = 0; i < 28; ++i) {
                const float lo = lo_p[strided<P2>(g, i)], hi = hi_p[strided<P2>(g + HALF, i)];
                a[i] = lo + hi;
                b[i] = lo - hi;
            }
            h28_program(a, o);
#pragma unroll
            for (int j = 0; j < 28; ++j) {
                lo_p[strided<P2>(g, j)] = o[j];
                amax = fmaxf(amax, fabsf(o[j]));
            }
            h28_program(b, o);
#pragma unroll
            for (int j = 0; j < 28; ++j) {
                hi_p[strided<P2>(g + HALF, j)] = o[j];
                amax = fmaxf(amax, fabsf(o[j]));
            }
        }
        __syncthreads();
    } else if constexpr (KRON) {
        for (int g = t; g < P2; g += NT) {
            float v[28], o[28];
            float *col = row + pad(g);
#pragma unroll
            for (int i = 0; i < 28; ++i) v[i] = col[strided<P2>(g, i)];
            h28_program(v, o);
#pragma unroll
            for (int j = 0; j < 28; ++j) {
                col[strided<P2>(g, j)] = o[j];
                amax = fmaxf(amax, fabsf(o[j]));
            }
        }
        __syncthreads();
    }

    // ---- row absmax ----------------------------------------------------------------------
    amax = max_of_wave(amax);
    if ((t & 63) == 0) red[t >> 6] = amax;
    __syncthreads();
    amax = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) amax = fmaxf(amax, red[w]);

    return amax;
}

template <int K, int NT, bool ROUNDED>
__device__ __forceinline__ float rotate_row_absmax(const __half *__restrict__ x, const float *__restrict__ pre,
                                                   float *row, float *red, const int t)
{
    RowLoad<K, NT> ld;
    row_load<K, NT>(x, pre, t, ld);
    return rotate_loaded_row_absmax<K, NT, false, ROUNDED>(ld, pre, row, red, t);
}

}  // namespace
}  // namespace sr
