// Choice of a row's clipping ratio by the squared quantisation error (paper, "Quantization" settings for the weights): device
// code of the searched weight folds (fwht_quant.hip, fold_search.hip).
#pragma once

#include "fwht_row.h"

namespace sr {
namespace {

// ------------------------------------------------------------------------------------------
// Clipping-ratio search over a rotated row in LDS (read(g, a, b): its values 8 g .. 8 g + 7; maximum `amax` > 0), by a
// workgroup of NT threads:
//     err_i = sum_j (y_j - Delta_i * code_i(y_j))^2,   Delta_i = grid[i] * amax / 7
// for every ratio; returns the ratio with the smallest error (first minimum in grid order) to every thread.
//
// Bound by vector-ALU issue: what counts is the number and kind of instructions per value and ratio.  On this chip
// fp32 add / mul / fma with VGPR operands issue in ~2.7 cycles, rint / min / max / med3, conversions, and anything with
// an SGPR or DPP operand in ~4.6 (measured per instruction).  So
//  * a LANE owns a ratio (Delta_i, 1/Delta_i in its registers) and the values come by broadcast LDS reads: no scalar
//    operands, and no reduction over lanes per ratio.  64 / n subsets of lanes (8 at most) take different groups of 8
//    values (21 ratios: 3 subsets, 63 lanes at work);
//  * a value costs five of the cheap instructions: clamp to [0, 1] of (y / Delta + 8) / 15 (the clamp is an output
//    modifier of the fma), times 15 plus 1.5 * 2^23 (rounds to an integer), minus 1.5 * 2^23 + 8 (the code), residual,
//    square-accumulate.  The scaling by 15 moves a rounding boundary by less than 1e-6 code units, where both codes
//    give the same error; the codes themselves are taken from the chosen ratio by the usual quantiser.
// Eight terms are summed in fp32, those sums in fp64.  4096 x 14336, 21 ratios, whole kernel: 288 -> 190 us (five
// instructions of 4.6 cycles per value and a six-step lane reduction per ratio before).  `err_w` is as small as it can be, so that two
// rows of 16384 fit a CU (4 subsets of 32 ratios each: 2048 channels, 21 ratios, 121 us a call against 95).
// ------------------------------------------------------------------------------------------
constexpr int search_scratch(int NT) { return NT; }      // doubles of err_w: one per unit and ratio, at most one per lane
template <int K, int NT, typename Read8>
__device__ __forceinline__ float search_ratio(Read8 read, const float amax, const float *grid, const int n, const int t, double *err_w)
{
    constexpr int NW = NT / 64, G = K / 8, MAX_SUB = 8;
    __shared__ float ratios[kMaxClipGrid];
    if (t == 0) {
#pragma unroll
        for (int i = 0; i < kMaxClipGrid; ++i) ratios[i] = grid[i];
    }
    __syncthreads();
    const int lane = t & 63, subs = 64 / n < MAX_SUB ? 64 / n : MAX_SUB;
    const int sub = lane / n, i = lane - sub * n;        // lanes of subset `subs` and above idle along with subset 0
    const int units = NW * subs, unit = (t >> 6) * subs + (sub < subs ? sub : 0);
    const float d = (ratios[i] * amax) / 7.f, inv15 = 1.f / (15.f * d);
    constexpr float magic = 12582912.f;                  // 1.5 * 2^23
    double acc = 0.0;
    auto add_group = [&](const float4 &a, const float4 &b) {
        const float y[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        float u[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = __builtin_amdgcn_fmed3f(fmaf(y[e], inv15, 8.f / 15.f), 0.f, 1.f);
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = fmaf(u[e], 15.f, magic);
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = fmaf(-d, u[e] - (magic + 8.f), y[e]);
        float even = 0.f, odd = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            even = fmaf(u[e], u[e], even);
            odd = fmaf(u[e + 1], u[e + 1], odd);
        }
        acc += (double)(even + odd);
    };
    float4 a0, b0, a1, b1;
    int g = unit;                                        // a unit's groups: unit, unit + units, ..
    read(g < G ? g : 0, a0, b0);
    for (; g + units < G; g += 2 * units) {              // the group after the one at work is on its way
        read(g + units, a1, b1);
        add_group(a0, b0);
        read(g + 2 * units < G ? g + 2 * units : 0, a0, b0);
        add_group(a1, b1);
    }
    if (g < G) add_group(a0, b0);
    if (sub < subs) err_w[unit * n + i] = acc;
    __syncthreads();
    if (t < n) {
        double e = err_w[t];
        for (int u = 1; u < units; ++u) e += err_w[u * n + t];
        err_w[t] = e;
    }
    __syncthreads();
    double best = err_w[0];
    int best_i = 0;
    for (int k = 1; k < n; ++k) {                        // every thread takes the same decision
        const double e = err_w[k];
        if (e < best) { best = e; best_i = k; }
    }
    return ratios[best_i];
}

// ------------------------------------------------------------------------------------------
// The same choice from ONE pass over the row, for ratios that are multiples of 1 / q (21 ratios from 1 to 0.5: q = 40).
// With u = |y| / amax, Delta_i = a_i / (7 q) and c the magnitude of the code,
//     err_i = sum u^2 - 2 Delta_i sum u c + Delta_i^2 sum c^2,
//     sum u c = sum over j of the sum of u above the j-th rounding boundary,  sum c^2 = sum over j of (2 j - 1) times their number,
// j = 1 .. 7 (8 where y < 0), and the j-th boundary of ratio i is (2 j - 1) a_i / (14 q): a multiple of 1 / (14 q) whatever
// the row.  So the values are counted and summed in cells of width 1 / (14 q), one 64-bit LDS atomic per value (number in the
// upper 16 bits, sum of u * 2^30 in the lower 48: integers, exact in any order), negative and positive ones apart, a prefix
// sum over the cells gives every boundary's number and sum, and err_i without the common first term is 8 terms in fp64.
//
// The result is that of search_ratio, ratio for ratio.  Both errors are rounded: search_ratio's by fp32 terms and a boundary moved by
// 1e-6 code units where values sit on it, these by the fp32 cell index (a value next to a boundary in the wrong cell, where both codes
// give the same error) and by sums of u cut at 2^-30.  Bounds for the worst row do not add up to a proof: with err_0 <= K / 196 (no
// value is further from its code than half a step of 1 / 7) the first alone may reach 1.2e-5 K / 196 for each of two ratios.  Emulated
// in these precisions, on normal, long-tailed, sparse, spiked and tied rows and rows of rounding boundaries, the difference to the
// smallest error never differed by more than 0.6 of 2^-16 K / 196, and by 0.01 of it for ratios that come close.  So where only one
// ratio is within 2^-16 K / 196 of the smallest error it is taken; else (about 2 % of normal rows) the caller runs search_ratio.
//
// Bound by the LDS atomics (a wave's 64 cells fall on random banks); search_ratio needs 105 vector instructions per value for
// 21 ratios, this 9.  4096 x 14336, 21 ratios, whole kernel: 190 -> 92 us (85 with the rotation of fold_search.hip).
// ------------------------------------------------------------------------------------------
// 14 q + 1 cells for either sign, dealt to the threads in runs.  LDS for them: whole runs, so that no thread need know where the
// cells end, or (from 8192 on, where the rows leave little) the cells alone: 14336 values and q = 56 .. 70 then run in two
// workgroups per CU instead of one, 174 us against 124.  Not runs of 8 or 16 cells, with which a wave's reads fall on one bank in 16
// or 32 (6 ratios 1 / 70 apart: 4096 x 2048 73 -> 38 us a call, 4096 x 4096 59 -> 45), nor, from 8192 on, of any even number.
constexpr int histogram_cells(int q) { return 2 * (14 * q + 1); }
constexpr bool histogram_trimmed(int K) { return K >= 8192; }
constexpr int histogram_run(int K, int NT, int q)
{
    const int run = (histogram_cells(q) + NT - 1) / NT;
    return histogram_trimmed(K) ? run | 1 : run % 8 ? run : run + 1;
}
constexpr int histogram_words(int K, int NT, int q) { return histogram_trimmed(K) ? histogram_cells(q) : histogram_run(K, NT, q) * NT; }
template <int K, int NT> __device__ __forceinline__ void clear_cells(uint64_t *cells, const int q, const int t)
{
    if constexpr (histogram_trimmed(K)) {
        for (int c = t; c < histogram_cells(q); c += NT) cells[c] = 0;
    } else {
        for (int e = 0; e < histogram_run(K, NT, q); ++e) cells[t + e * NT] = 0;
    }
}

// q where the ratios of a fold may be taken from the count, 0 where not
inline int counted_fraction(const RowExtras &ex)
{
    if (int64_t f; tuned(kTuneClipSearch, f) && f == 1) return 0;
    return clip_grid_denominator(ex.grid, ex.n_grid);
}

template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint64_t add_shifted(uint64_t v)   // v + the permuted lane's v (0 where there is none)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROW_MASK, 0xF, false);
    return v + ((uint64_t)hi << 32 | lo);
}
template <int CTRL> __device__ __forceinline__ double add_partner(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)lane_perm<CTRL>((int)(uint32_t)b), hi = (uint32_t)lane_perm<CTRL>((int)(uint32_t)(b >> 32));
    return v + __longlong_as_double((int64_t)((uint64_t)hi << 32 | lo));
}

// Words of the cells: cell c of the negative values is word top - c, of the others word 2 top + 1 - c (top = 14 q):
// descending, so that a prefix sum up to a cell is the sum of what lies above its lower boundary.  |y| <= amax: c <= top.
struct CellScale {
    float to_cell, to_fixed;
    __device__ __forceinline__ CellScale(int q, float amax) : to_cell((float)(14 * q) / amax), to_fixed(1073741824.f / amax) {}
};
// (neg, pos: words of cell 0 for the two signs, swapped by a caller whose value carries a flipped sign; LOWEST: cells below
// `lowest` are left out)
template <bool LOWEST> __device__ __forceinline__ void count_value(uint64_t *cells, const CellScale &s, int neg, int pos, float y, int lowest = 0)
{
    const int cell = (int)(uint32_t)(fabsf(y) * s.to_cell);
    if (LOWEST && cell < lowest) return;
    const uint64_t one = (uint64_t)1 << 48 | (uint32_t)(fabsf(y) * s.to_fixed);
    __hip_atomic_fetch_add(cells + (y < 0.f ? neg : pos) - cell, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Few large values among small ones (weights of one sign, of equal size, ..): at most half of the waves have a value of amax / 19
// (red: their maxima).  The small values meet in a few cells, and hardly one of them decides between the ratios.  So
//  * values below every boundary of every ratio are not counted in such a row (in others the comparison is not worth it);
//  * a row whose large value does not decide either (undecided_signs; any row of K = 28 2^p, where 28 large values come together)
//    goes to search_ratio at once: the count would leave nearly every one open.
// us a call, weights between -0.05 and 0, 21 ratios, 4096 channels of 2048, 4096, 8192, 14336: 75, 103, 192, 358 counted like other
// rows, 59, 80, 146, 257 this way (50, 70, 131, 255 in fwht_quant_search_kernel, whose workgroups have no cells); 11 ratios: 36, 48, 91,
// 192 -> 33, 39, 67, 198.
// The line: rows of one value among normally distributed ones, 21 ratios 0.025 apart, leave two ratios or more up to a standard
// deviation of 0.014 .. 0.016 amax, where a wave's largest value is 0.048 .. 0.055 amax, and one ratio beyond.
template <int NT> __device__ __forceinline__ bool spiked(const float *red, const float amax)
{
    int reach = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) reach += red[w] >= amax * (1.f / 19.f);
    return 2 * reach <= NT / 64;
}
// note_sign: 1 for a positive, 2 for a negative value of magnitude amax (see undecided_signs).
__device__ __forceinline__ int lowest_boundary(float smallest_ratio, int q) { return (int)(smallest_ratio * (float)q + 0.5f); }
__device__ __forceinline__ void note_sign(int *signs, float y, float amax, bool flipped)
{
    if (fabsf(y) == amax) __hip_atomic_fetch_or(signs, (y < 0.f) != flipped ? 2 : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// `cells`: histogram_words(K, NT, q) words in which a row of K values has been counted (visible to the workgroup).  Returns
// the index of the ratio, or -1 where more than one comes into question, to every thread.
template <int K, int NT>
__device__ __forceinline__ int ratio_of_cells(const float *grid, const int n, const int q, uint64_t *cells, const int t)
{
    constexpr int NW = NT / 64;
    static_assert(K <= 32768, "16 bits of number and 48 of sum");
    __shared__ uint64_t wave_sum[NW];
    __shared__ double err[kMaxClipGrid];
    __shared__ int choice;
    const int lane = t & 63, top = 14 * q;

    // ---- inclusive prefix sums over all words
    const int run = histogram_run(K, NT, q);
    int from = 0, to = run;                              // of its run: known to be the same for all threads where it is not trimmed
    uint64_t *own = cells + t * run;
    if constexpr (histogram_trimmed(K)) {
        own = cells;
        from = t * run;
        to = from + run < histogram_cells(q) ? from + run : histogram_cells(q);
    }
    uint64_t sum = 0;
    for (int c = from; c < to; ++c) sum += own[c];
    uint64_t upto = add_shifted<0x111, 0xF>(sum);        // row_shr 1, 2, 4, 8, then the rows before
    upto = add_shifted<0x112, 0xF>(upto);
    upto = add_shifted<0x114, 0xF>(upto);
    upto = add_shifted<0x118, 0xF>(upto);
    upto = add_shifted<0x142, 0xA>(upto);
    upto = add_shifted<0x143, 0xC>(upto);
    if (lane == 63) wave_sum[t >> 6] = upto;
    __syncthreads();
    {
        uint64_t acc = upto - sum;
        for (int w = 0; w < NW; ++w) acc += w < (t >> 6) ? wave_sum[w] : 0;
        for (int c = from; c < to; ++c) {
            acc += own[c];
            own[c] = acc;
        }
    }
    __syncthreads();

    // ---- one lane per ratio and boundary
    for (int x = t; x < 8 * n; x += NT) {                // whole groups of 8 lanes
        const int i = x >> 3, j = (x & 7) + 1;
        const int a = (int)(grid[i] * (float)q + 0.5f), c = (2 * j - 1) * a;
        uint64_t above = 0;
        if (c <= top) above = cells[top - c] + (j < 8 ? cells[2 * top + 1 - c] - cells[top] : 0);
        const double d = (double)a / (7.0 * q), s = (double)(above & (((uint64_t)1 << 48) - 1)) * 0x1p-30;
        double e = d * (d * (double)((2 * j - 1) * (int)(above >> 48)) - 2.0 * s);
        e = add_partner<0xB1>(e);
        e = add_partner<0x4E>(e);
        e = add_partner<0x141>(e);
        if (j == 1) err[i] = e;
    }
    __syncthreads();
    if (t < 64) {
        const double e = err[lane < n ? lane : 0];
        double best = e;
        for (int h = 16; h >= 1; h >>= 1) best = fmin(best, __shfl_xor(best, h));   // the ratios are in lanes 0 .. 31
        const uint64_t near = __ballot(lane < n && e <= best + K * (0x1p-16 / 196.0));
        if (t == 0) choice = __popcll(near) == 1 ? __builtin_ctzll(near) : -1;
    }
    __syncthreads();
    return choice;
}

}  // namespace
}  // namespace sr
