// Weight fold with clip search for rows of 2048, 4096, 8192 and 14336 values, full transform, ratios that are multiples of a
// common 1 / q: one workgroup per output channel, rotation in two passes (two_pass_row.h), the ratio from one pass over the
// values (clip_search.h), quantiser.  (Paper, section "Methodology": weights rotated offline; Eq. (1).)
//
// The values of pass 2 are counted straight from the registers that hold them.  Against the general rotation with the values
// read back from LDS (4096 x 14336, 21 ratios): 92 -> 85 us.  The products with the smoothing factors are rounded as in
// fwht_quant_ex_kernel, so codes, scales and ratios are bit for bit those of the other searched folds.
#include "two_pass_row.h"
#include "clip_search.h"

namespace sr {
namespace {

template <int K>
__global__ __launch_bounds__((TwoPass<K>::NT)) void fold_search_kernel(const __half *__restrict__ Wt, int64_t ldw,
                                                                       const float *__restrict__ s, float post_scale,
                                                                       uint8_t *__restrict__ Q, float *__restrict__ scale_out,
                                                                       const RowExtras ex, const int q, const int undecided)
{
    using S = TwoPass<K>;
    constexpr int NT = S::NT;
    constexpr uint32_t ALL = 0xFFFFFFFFu;
    static_assert(NT == S::COLS, "every thread holds values after the rotation");
    extern __shared__ __attribute__((aligned(16))) float row[];
    __shared__ float red[NT / 64];
    __shared__ int signs;                                // of the values of magnitude amax
    void *const scratch = row + S::LEN;                  // the cells, or partial errors of search_ratio
    uint64_t *const cells = static_cast<uint64_t *>(scratch);
    const int t = threadIdx.x;
    const int64_t m = blockIdx.x;
    RowLoad<K, NT> ld;
    row_load<K, NT, false, false, 5>(Wt + m * ldw, s, t, ld);
    clear_cells<K, NT>(cells, q, t);                     // visible after the rotation's barriers
    if (t == 0) signs = 0;
    float o[S::R];
    const float amax = two_pass_rotate<S, K, true, false, false, true>(ld, row, red, t, ALL, o, NoHook{});
    if (!(amax > 0.f && amax < __builtin_inff())) {
        // nothing to search: zeros, or infinities and NaNs, whose signs (code 7 or -8) depend on the signs that values carry
        // on the way -- rotated again as the other kernels do
        __syncthreads();
        const float a = rotate_row_absmax<K, NT, true>(Wt + m * ldw, s, row, red, t);
        const float delta = a == 0.f ? 1.f : (ex.grid[0] * a) / 7.f;
        if (ex.ratio_out && t == 0) ex.ratio_out[m] = ex.grid[0];
        if (t == 0) scale_out[m] = a == 0.f ? 1.f : delta * post_scale;
        quantise_padded_row_nibbles<K, NT>(row, 1.f / delta, Q + m * (int64_t)(K / 2), t);
        return;
    }
    const bool f = S::flipped(S::first(t) >> 4);         // the sign that all values of a thread carry
    // (beyond this range the scaled values would not stay inside fp32)
    bool count = amax > 0x1p-90f && amax < 0x1p90f;
    const bool spikes = spiked<NT>(red, amax);
    if constexpr (!is_pow2(K)) {
        count = count && !spikes;
    } else if (count && spikes && undecided) {
        if (undecided != 3) {
#pragma unroll
            for (int r = 0; r < S::R; ++r) note_sign(&signs, o[r], amax, f);
            __syncthreads();
        }
        count = undecided != 3 && (signs & undecided) == 0;
    }
    int i = -1;
    if (count) {
        const CellScale scale(q, amax);
        const int neg = f ? 28 * q + 1 : 14 * q, pos = f ? 14 * q : 28 * q + 1;
        if (is_pow2(K) && spikes) {
            const int lowest = lowest_boundary(ex.grid[ex.n_grid - 1], q);
#pragma unroll
            for (int r = 0; r < S::R; ++r) count_value<true>(cells, scale, neg, pos, o[r], lowest);
        } else {
#pragma unroll
            for (int r = 0; r < S::R; ++r) count_value<false>(cells, scale, neg, pos, o[r]);
        }
        __syncthreads();
        i = ratio_of_cells<K, NT>(ex.grid, ex.n_grid, q, cells, t);
    }
    float clip;
    uint32_t flips = ALL;
    if (i >= 0) {
        clip = ex.grid[i];
    } else {
        // the signs are put right once (undone at every read they cost the search a quarter more instructions)
#pragma unroll
        for (int e = 0; e < S::NG; ++e) {
            const int g = t + e * NT;
            if ((K / 16 % NT == 0 || g < K / 16) && S::flipped(g)) {
                float4 *v = reinterpret_cast<float4 *>(row + S::pos(16 * g));
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = make_float4(-v[c].x, -v[c].y, -v[c].z, -v[c].w);
            }
        }
        flips = 0;
        __syncthreads();
        auto read8 = [&](int g, float4 &a, float4 &b) {
            const float *src = row + S::pos(8 * g);
            a = *reinterpret_cast<const float4 *>(src);
            b = *reinterpret_cast<const float4 *>(src + 4);
        };
        clip = search_ratio<K, NT>(read8, amax, ex.grid, ex.n_grid, t, static_cast<double *>(scratch));
    }
    if (ex.ratio_out && t == 0) ex.ratio_out[m] = clip;
    const float delta = (clip * amax) / 7.f;
    if (t == 0) scale_out[m] = delta * post_scale;
    quantise_row_nibbles<S, K>(row, 1.f / delta, flips, Q + m * (int64_t)(K / 2), t);
}

template <int K>
hipError_t launch(const void *Wt, int64_t rows, int64_t ldw, const float *s, float post_scale, uint8_t *Q, float *scale_out,
                  const RowExtras &ex, int q, hipStream_t st)
{
    using S = TwoPass<K>;
    constexpr auto kern = fold_search_kernel<K>;
    constexpr int row_bytes = S::LEN * (int)sizeof(float), search = search_scratch(S::NT) * 8;
    constexpr int most = histogram_words(K, S::NT, kMaxClipDenominator) * 8;
    static_assert(most >= search && row_bytes + most + 1024 <= 160 * 1024, "LDS");
    if constexpr (row_bytes + most > 40 * 1024)
        if (hipError_t e = allow_dynamic_lds<kern>(row_bytes + most); e != hipSuccess) return e;
    const int cells = histogram_words(K, S::NT, q) * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3(S::NT), row_bytes + (cells > search ? cells : search), st,
                       static_cast<const __half *>(Wt), ldw, s, post_scale, Q, scale_out, ex, q, undecided_signs(ex.grid, ex.n_grid, K));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fold_search(const void *Wt, int64_t rows, int64_t K, int64_t ldw, const float *s, float post_scale,
                              uint8_t *Q, float *scale_out, const RowExtras &ex, hipStream_t st, bool &taken)
{
    const int q = counted_fraction(ex);
    // Fine fractions: the cells take the LDS of other rows, and a sum for each of a few ratios is done sooner (us a call, 4096 channels,
    // sums against counts: 2048, 11 ratios 0.01 apart 39 / 42, 16 42 / 42; 4096, 2 48 / 49; 14336, 2 165 / 177, 8 168 / 177, 10 184 /
    // 177; but 8192, 2 113 / 84; q = 70: 2048, 6 36 / 36, 14336, 6 166 / 127)
    const int sums_up_to = q <= 70 ? 0 : K == 2048 ? 11 : K == 4096 ? 3 : K == 14336 ? 8 : 0;
    taken = q > 0 && s && ex.n_grid > sums_up_to;
    if (!taken) return hipSuccess;
    switch (K) {
        case 2048: return launch<2048>(Wt, rows, ldw, s, post_scale, Q, scale_out, ex, q, st);
        case 4096: return launch<4096>(Wt, rows, ldw, s, post_scale, Q, scale_out, ex, q, st);
        case 8192: return launch<8192>(Wt, rows, ldw, s, post_scale, Q, scale_out, ex, q, st);
        case 14336: return launch<14336>(Wt, rows, ldw, s, post_scale, Q, scale_out, ex, q, st);
        default: taken = false; return hipSuccess;
    }
}

}  // namespace sr
