// INT4 x INT4 GEMM on the FP6 matrix pipe for few token rows: the operands go from memory straight into the
// registers that the matrix instruction reads.
//
//   acc[m][n] = sum_k cX[m][k] * cW[n][k],   Y = fp16(acc * dx[m] * dw[n])
//
// (Paper: the quantised forward pass of the linear layer; dequantisation per Eq. (1).  Same sums, operands and
// outputs as the tile kernel of gemm_f6.hip, whose header has the f6-tile layout and why FP6 holds INT4 exactly.)
//
// Why: with up to a few hundred rows the product is bound by fetching W once, and the tile kernel (256 x 128
// outputs per workgroup) then leaves most CUs without a tile and multiplies padding rows.  Here a workgroup owns
// FM * 16 rows x FN * 16 channels (at least 16 channels, so that N = 4096 still gives 256 workgroups) and its NW
// waves split K: wave w takes the 128-code chunks w, w + NW, ..  Every wave reads each byte of its chunks once, so
// nothing is shared through LDS and the loop has no barrier; the waves' sums (exact in fp32, any order) meet in
// LDS at the end.  What bounds it: the ~90 GB/s at which a CU takes operands from L2 (64 x 64 outputs, K = 14336:
// 0.13 us per 12 KB stage), so near-square tiles win once N / 16 column tiles fill the chip (gemm_rules.h picks).
// Measured against the 256 x 128 tile kernel, weights in the memory-side cache: 37 x 6144 x 4096 15.8 -> 6.1 us,
// 37 x 4096 x 14336 40.5 -> 10.4, 128 x 4096 x 14336 40.8 -> 14.8, 256 x 4096 x 4096 17.2 -> 8.6; the 18.9 MB of the
// first take 3.6 us to read.  Non-temporal loads of W: 5 % faster from HBM, 5 - 20 % slower out of that cache; dropped.
//
// A fragment of v_mfma_scale_f32_16x16x128_f8f6f4 wants lane l to hold the 32 codes 32 q .. 32 q + 31 (q = l >> 4)
// of row l & 15: exactly piece (r = l & 7, t = q >> 1, g = q & 1) of block l >> 3 & 1 of two neighbouring 768-byte
// blocks.  The 16-byte heads of a fragment are two runs of 512 contiguous bytes, its 8-byte tails two of 256 (fetched for
// two fragments at a time where that pays, see launch_st).
#include "sr_common.h"
#include "gemm_common.h"

#include <type_traits>

namespace sr {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_dword __attribute__((ext_vector_type(4), aligned(4)));     // the channel scales: 4-byte aligned only
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int BLK = 768;     // bytes of one block (8 rows x 128 codes x 6 bits)

// D = chunks a wave keeps in flight; TPP = 16 x 16 tiles whose partial sums are in LDS at a time.
template <int FM, int FN, int NW, int D, bool PAIRS>
__global__ __launch_bounds__(NW * 64) void gemm_f6_stream_kernel(
    const uint8_t *__restrict__ X6, const float *__restrict__ xs, const uint8_t *__restrict__ W6,
    const float *__restrict__ ws, int M, int N, int K, void *__restrict__ Yv, int64_t ldy, int out_i32,
    int tiles_m, int tiles_n)
{
    constexpr int TILES = FM * FN, TPP = TILES <= 8 ? TILES : TILES % 8 == 0 ? 8 : 6;
    __shared__ __attribute__((aligned(16))) v4f red[NW][TPP][64];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups are dealt round-robin to the 8 XCDs: XCD x takes an eighth of the tiles in a row, row tiles fastest
    // (the row tiles of a column tile share its weights in that L2, neighbouring column tiles share lines of Y)
    const int total = tiles_m * tiles_n, xcd = blockIdx.x & 7, first = (int)((int64_t)xcd * total >> 3);
    const int v = first + (blockIdx.x >> 3);
    if (v >= (int)((int64_t)(xcd + 1) * total >> 3)) return;
    const int tm = v % tiles_m, tn = v / tiles_m;
    const int m0 = tm * FM * 16, n0 = tn * FN * 16;
    const int nc = K >> 7;
    const uint32_t xb = (uint32_t)((M + 7) >> 3), wb = (uint32_t)((N + 7) >> 3);     // 8-row blocks of a chunk
    const uint32_t cx_bytes = xb * BLK, cw_bytes = wb * BLK;

    // lane offsets of a fragment inside its pair of blocks; rows past the end re-read the last block
    const int half = (lane >> 3) & 1, q = lane >> 4;
    const uint32_t head = 256 * (q >> 1) + 128 * ((q & 1) ^ half) + 16 * (lane & 7);
    const uint32_t tail = 512 + 128 * ((q & 1) ^ half) + 16 * (lane & 7) + 8 * (q >> 1);
    uint32_t xo[FM], wo[FN];                             // byte offset of the lane's block inside a chunk
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        uint32_t b = (uint32_t)(m0 >> 3) + 2 * f + half;
        // an odd last block has no partner: both halves read it (the parity of its rows decides the swizzle, so the
        // lanes of the missing half fetch wrong codes of rows that are never stored)
        xo[f] = (b < xb ? b : xb - 1) * BLK;
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        uint32_t b = (uint32_t)(n0 >> 3) + 2 * f + half;
        wo[f] = (b < wb ? b : wb - 1) * BLK;
    }

    // Tails: the two steps of a (row, k half) share a 16-byte slot, so lanes 0 .. 31 fetch the slots of one fragment and lanes
    // 32 .. 63 those of the next (lane bits: row, block, k half), whole lines; exchanging the halves of the wave then leaves
    // every lane the 8 bytes of its step for either fragment.  (8 bytes per lane and fragment look every 64-byte piece up twice:
    // 16 of the 64 lookups of two fragments less.)
    // An odd last fragment, and all of them without PAIRS, are fetched 8 bytes a lane.
    constexpr int XP = PAIRS ? FM / 2 : 0, WP = PAIRS ? FN / 2 : 0;
    constexpr int XL = FM - 2 * XP, WL = FN - 2 * WP;
    const uint32_t slot = 512 + 128 * ((q & 1) ^ half) + 16 * (lane & 7);
    uint32_t xp[XP + 1], wp[WP + 1];
#pragma unroll
    for (int f = 0; f < XP; ++f) {
        const uint32_t b = (uint32_t)(m0 >> 3) + 4 * f + 2 * (lane >> 5) + half;
        xp[f] = (b < xb ? b : xb - 1) * BLK + slot;
    }
#pragma unroll
    for (int f = 0; f < WP; ++f) {
        const uint32_t b = (uint32_t)(n0 >> 3) + 4 * f + 2 * (lane >> 5) + half;
        wp[f] = (b < wb ? b : wb - 1) * BLK + slot;
    }

    u32x4 xh[D][FM], wh[D][FN];                          // chunk d in flight: heads and tails of its fragments
    u32x4 xt[D][XP + 1], wt[D][WP + 1];
    u32x2 xl[D][XL + 1], wl[D][WL + 1];
    auto load = [&](auto DC, int s) {
        constexpr int d = decltype(DC)::value;
        const uint8_t *w = W6 + (int64_t)s * cw_bytes, *x = X6 + (int64_t)s * cx_bytes;
#pragma unroll
        for (int f = 0; f < FN; ++f) {
            wh[d][f] = *reinterpret_cast<const u32x4 *>(w + wo[f] + head);
            if (f >= 2 * WP) wl[d][f - 2 * WP] = *reinterpret_cast<const u32x2 *>(w + wo[f] + tail);
        }
#pragma unroll
        for (int f = 0; f < WP; ++f) wt[d][f] = *reinterpret_cast<const u32x4 *>(w + wp[f]);
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            xh[d][f] = *reinterpret_cast<const u32x4 *>(x + xo[f] + head);
            if (f >= 2 * XP) xl[d][f - 2 * XP] = *reinterpret_cast<const u32x2 *>(x + xo[f] + tail);
        }
#pragma unroll
        for (int f = 0; f < XP; ++f) xt[d][f] = *reinterpret_cast<const u32x4 *>(x + xp[f]);
    };
    // the tails of fragments 2 f and 2 f + 1 from the slots of both
    auto split_tails = [](const u32x4 t, u32x2 &a, u32x2 &b) {
        const auto lo = __builtin_amdgcn_permlane32_swap(t.x, t.z, false, false), hi = __builtin_amdgcn_permlane32_swap(t.y, t.w, false, false);
        a = u32x2{lo[0], hi[0]};
        b = u32x2{lo[1], hi[1]};
    };
    // Output o of pass p0 / TPP of the reduction = lane o & 63 of tile p0 + (o >> 6): four channels of one token.  Its
    // dequantisation factors are fetched ahead of the operands and used last (fetched after the reduction, their
    // latency would end every workgroup); the raw int32 output has readable stand-ins and ignores them.
    constexpr int PASSES = TILES / TPP, OPT = (TPP * 64 + NW * 64 - 1) / (NW * 64);     // outputs per thread and pass
    static_assert(TILES % TPP == 0 && OPT == 1, "one output per thread and pass");
    float fx[PASSES];
    v4f_dword fw[PASSES];
    int om[PASSES], on[PASSES];
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int p = k * TPP + (wave < TPP ? wave : 0);
        om[k] = m0 + 16 * (p % FM) + (lane & 15);
        on[k] = n0 + 16 * (p / FM) + 4 * q;
        fx[k] = xs[om[k] < M ? om[k] : M - 1];
        fw[k] = *reinterpret_cast<const v4f_dword *>(ws + (on[k] < N ? on[k] : N - 4));
    }
    v4f acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int f = 0; f < FM; ++f) acc[i][f] = v4f{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](auto DC) {
        constexpr int d = decltype(DC)::value;
        u32x2 xe[FM], we[FN];
#pragma unroll
        for (int f = 0; f < XP; ++f) split_tails(xt[d][f], xe[2 * f], xe[2 * f + 1]);
#pragma unroll
        for (int f = 0; f < XL; ++f) xe[2 * XP + f] = xl[d][f];
#pragma unroll
        for (int f = 0; f < WP; ++f) split_tails(wt[d][f], we[2 * f], we[2 * f + 1]);
#pragma unroll
        for (int f = 0; f < WL; ++f) we[2 * WP + f] = wl[d][f];
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const v8i w = {(int)wh[d][i].x, (int)wh[d][i].y, (int)wh[d][i].z, (int)wh[d][i].w, (int)we[i].x, (int)we[i].y, 0, 0};
#pragma unroll
            for (int f = 0; f < FM; ++f) {
                const v8i x = {(int)xh[d][f].x, (int)xh[d][f].y, (int)xh[d][f].z, (int)xh[d][f].w, (int)xe[f].x, (int)xe[f].y, 0, 0};
                acc[i][f] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w, x, acc[i][f], 2, 2, 0, 0, 0, 0);
            }
        }
    };

    // chunk i of this wave is chunk wave + NW i of K; n of them
    const int n = nc > wave ? (nc - wave + NW - 1) / NW : 0;
    auto at = [&](int i) { return wave + NW * i; };
    if (n > 0) {
        static_for<D>([&](auto DC) { load(DC, at(DC < n ? (int)DC : n - 1)); });
        __builtin_amdgcn_sched_barrier(0);
        int i = 0;
        for (; i + 2 * D <= n; i += D) {
            static_for<D>([&](auto DC) {
                multiply(DC);
                __builtin_amdgcn_sched_barrier(0);
                load(DC, at(i + D + DC));
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        // the last D .. 2 D - 1 chunks (fewer where the wave has fewer in all)
        static_for<D>([&](auto DC) {
            if (i + DC < n) multiply(DC);
            if (i + D + DC < n) load(DC, at(i + D + DC));
        });
        static_for<D - 1>([&](auto DC) {
            if (i + D + DC < n) multiply(DC);
        });
    }

    // ---- the waves' sums, TPP tiles at a time: lane l of tile (i, f) holds token l & 15, channels 4 (l >> 4) .. + 3
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        if (k) __syncthreads();
#pragma unroll
        for (int p = 0; p < TPP; ++p) red[wave][p][lane] = acc[(k * TPP + p) / FM][(k * TPP + p) % FM];
        __syncthreads();
        if (wave < TPP && om[k] < M && on[k] < N) {
            v4f s = red[0][wave][lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) s += red[w][wave][lane];
            if (out_i32) {
                *reinterpret_cast<int4 *>(static_cast<int32_t *>(Yv) + (int64_t)om[k] * ldy + on[k]) =
                    make_int4((int)(s[0] * 64.f), (int)(s[1] * 64.f), (int)(s[2] * 64.f), (int)(s[3] * 64.f));
            } else {
                const float f = fx[k] * 64.f;               // both operands carried a factor 1/8
                union { __half h[4]; uint2 u; } y;
                y.h[0] = __float2half_rn(s[0] * f * fw[k].x);
                y.h[1] = __float2half_rn(s[1] * f * fw[k].y);
                y.h[2] = __float2half_rn(s[2] * f * fw[k].z);
                y.h[3] = __float2half_rn(s[3] * f * fw[k].w);
                *reinterpret_cast<uint2 *>(static_cast<__half *>(Yv) + (int64_t)om[k] * ldy + on[k]) = y.u;
            }
        }
    }
}

template <int FM, int FN, int NW, int D>
hipError_t launch_st(const uint8_t *X6, const float *xs, const uint8_t *W6, const float *ws, int64_t M, int64_t N,
                     int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st)
{
    const int tiles_m = (int)((M + FM * 16 - 1) / (FM * 16)), tiles_n = (int)((N + FN * 16 - 1) / (FN * 16));
    constexpr bool CAN_PAIR = FM > 1 || FN > 1;
    const bool pairs = CAN_PAIR && f6_pairs_tails(tiles_m, tiles_n, FM, FN, compute_units());
    const auto kern = pairs ? gemm_f6_stream_kernel<FM, FN, NW, D, CAN_PAIR> : gemm_f6_stream_kernel<FM, FN, NW, D, false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)((tiles_m * tiles_n + 7) / 8 * 8)), dim3(NW * 64), 0, st,
                       X6, xs, W6, ws, (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f6_stream(const uint8_t *X6, const float *xs, const uint8_t *W6, const float *ws, int64_t M,
                                 int64_t N, int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st, int bm, int bn)
{
    if (out_i32) {                   // the scales may be NULL then: readable stand-ins (see launch_f6 in gemm_f6.hip)
        xs = reinterpret_cast<const float *>(X6);
        ws = reinterpret_cast<const float *>(W6);
    }
#define SR_STREAM(FM, FN, D) \
    if (bm == 16 * FM && bn == 16 * FN) return launch_st<FM, FN, 8, D>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st)
    SR_STREAM(1, 1, 4); SR_STREAM(1, 2, 2); SR_STREAM(2, 2, 2); SR_STREAM(2, 4, 2); SR_STREAM(3, 2, 2); SR_STREAM(3, 4, 2); SR_STREAM(4, 4, 2);
#undef SR_STREAM
    return hipErrorInvalidValue;
}

}  // namespace sr
