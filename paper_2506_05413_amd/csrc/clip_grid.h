// What the ratios of a clip search allow (see clip_search.h).  Plain C++ (no HIP), so that it can be compiled and checked on its own.
#pragma once

namespace sr {

constexpr int kMaxClipGrid = 32;                         // ratios of a search
constexpr int kMaxClipDenominator = 100;

// The smallest q <= kMaxClipDenominator of which every ratio is a multiple of 1 / q, to the last bit of a float, and each a smaller
// one than the ratio before; 0: none.  (Equal ratios have equal errors, every row would be left open: 5 ratios of 1, 4096 x 8192,
// 166 us a call against 112.)
inline int clip_grid_denominator(const float *grid, int n)
{
    for (int q = 1; q <= kMaxClipDenominator; ++q) {
        bool all = true;
        long long before = (1ll << 62);
        for (int i = 0; i < n && all; ++i) {
            const double a = (double)grid[i] * q, r = (double)(long long)(a + 0.5);
            all = r >= 1.0 && a - r <= q * 0x1p-24 && r - a <= q * 0x1p-24 && (long long)r < before;
            before = (long long)r;
        }
        if (all) return q;
    }
    return 0;
}

// The signs of a row's one large value among zeros (1: positive, 2: negative) with which it does not decide between the ratios:
// the errors it has itself (code 7 at most, -8 at least), more than one of them within the margin of ratio_of_cells.
inline int undecided_signs(const float *grid, int n, int K)
{
    int signs = 0;
    for (int negative = 0; negative < 2; ++negative) {
        double err[kMaxClipGrid], best = 1.0;
        for (int i = 0; i < n; ++i) {
            const double step = grid[i] / 7.0, code = (double)(int)(1.0 / step + 0.5), most = 7 + negative;
            const double r = 1.0 - step * (code < most ? code : most);
            err[i] = r * r;
            if (err[i] < best) best = err[i];
        }
        int near = 0;
        for (int i = 0; i < n; ++i) near += err[i] <= best + K * (0x1p-16 / 196.0);
        signs |= (near > 1) << negative;
    }
    return signs;
}

}  // namespace sr
