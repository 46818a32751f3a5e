// Rotation of one row by a workgroup in two passes over it: device code shared by the token quantiser (fwht_two_pass.hip) and
// the weight fold with clip search (fold_search.hip).
//
// Pass 1 covers the index bits 0..5 of the row, straight from the global load: four in registers (a thread holds 16
// contiguous values), two across neighbouring lanes by DPP.  Pass 2 covers the rest: registers take the bits 6..9 (or, for
// 14336 = 28 * 512, the Paley factor H_28), the lane bits 0.. the 1, 2 or 3 bits that are left.  Every level is the same
// addition of the same two values as in the general kernels (fwht_row.h).
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
#pragma once

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
    // first value of thread t in pass 2.  Lane ^ 7 is the partner of the third level, so the bits that index the row are those
    // of a ^ (a >> 2): each of the partners lane ^ 1, ^ 2, ^ 7 then differs in one of them.
    __device__ static __forceinline__ int lane_bits(int t)
    {
        const int a = t & ((1 << Q) - 1);
        return Q == 3 ? a ^ ((a >> 2) * 3) : a;
    }
    __device__ static __forceinline__ int first(int t) { return (t >> Q) + (lane_bits(t) << Q0); }
    // sign that the 16 values of set g = i >> 4 carry into the quantiser: the lane bits of pass 1 were g & 3, those of
    // pass 2 the index bits Q0 .. Q0 + Q - 1
    // (bits that `mask` leaves out are not transformed and flip nothing)
    __device__ static __forceinline__ bool flipped(int g, uint32_t mask = 0xFFFFFFFFu)
    {
        const int i = (int)((uint32_t)(16 * g) & mask);
        return __builtin_popcount(((i >> 4) & 3) | (((i >> Q0) & ((1 << Q) - 1)) << 2)) & 1;
    }
};

// The loaded row -> its rotation: in `row` (LDS, at S::pos, every value with the sign of S::flipped) and in the registers o of
// the threads t < S::COLS (values S::first(t) + S::RSTRIDE r, the same sign); returns the row's absolute maximum to every
// thread, for which all of `row` is then visible.  red: NT / 64 floats of LDS.  between() runs after pass 1.
// MASKED: only the index bits set in `mask` are butterflied (uniform branches; powers of two).  ROUNDED: see first_level16.
template <class S, int K, bool HAS_PRE, bool GATE, bool MASKED, bool ROUNDED, typename Hook>
__device__ __forceinline__ float two_pass_rotate(const RowLoad<K, S::NT> &ld, float *row, float *red, const int t,
                                                 const uint32_t mask, float (&o)[S::R], Hook between)
{
    constexpr int NT = S::NT, NW = NT / 64;
    const int lane = t & 63;
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
                first_level16<GATE, ROUNDED>(ld.u[i], ld.gu[i], ld.p[i], HAS_PRE, v);
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
    between();

    // ---- pass 2: the other bits -------------------------------------------------------------------
    float amax = 0.f;
    if (NT == S::COLS || t < S::COLS) {                  // whole waves
        const int q = S::lane_bits(t);
        float *col = row + S::pos(S::first(t));
        float v[S::R];
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
    return amax;
}

// The rotated row -> packed nibbles at `out`
template <class S, int K>
__device__ __forceinline__ void quantise_row_nibbles(const float *row, const float inv_delta, const uint32_t mask, uint8_t *out, const int t)
{
    uint32_t *q = reinterpret_cast<uint32_t *>(out);
#pragma unroll
    for (int i = 0; i < S::NG; ++i) {
        const int g = t + i * S::NT;
        if (K / 16 % S::NT == 0 || g < K / 16) {
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

}  // namespace
}  // namespace sr
