// INT4 x INT4 GEMM for few and medium row counts on packed nibbles (M > 16): the operands go from memory straight into
// registers, as in gemm_f6_stream.hip, and are widened there for the int8 matrix instruction.
//
//   acc[m][n] = sum_k cX[m][k] * cW[n][k]  (exact INT32),   Y = fp16(acc * dx[m] * dw[n])
//
// (Paper: the quantised forward pass of the linear layer; dequantisation per Eq. (1).  Same sums and outputs as the tile
// kernel of gemm_prefill.hip, whose header explains the widening to code * 16.)
//
// A workgroup owns FM * 16 rows x FN * 16 channels and its NW waves split K in chunks of 256 codes -- one 128-byte line
// of every row, which eight neighbouring lanes fetch whole.  A wave brings each 16-row fragment into operand order through
// two small buffers of its own LDS (no barrier: a wave's LDS accesses execute in order); each 16-byte piece then widens to
// the operands of two v_mfma_i32_16x16x64_i8 (the order of k inside a dot product is free and X and W are widened alike).
// No barrier until the waves' partial sums meet at the end.
//
// Loading the operand order directly (neighbouring lanes on 16 different rows) cost a lookup of the L1 per lane, 60 for a
// load of 1 KB where whole lines take 16 (TCP_TOTAL_CACHE_ACCESSES): that bounded the kernel.  Weights in the memory-side
// cache, us: 60 x 4096 x 4096 6.2 -> 4.8, 29 x 4096 x 14336 11.6 -> 8.1, 128 x 4096 x 8192 13.9 -> 10.1, 353 x 2096 x 8192
// 19.0 -> 12.2 (from HBM 18.9 -> 12.6).  What bounds it now: the L1 still (16 KB per chunk of 64 x 64 outputs at 64 B per
// clock), the widening and its matrix instructions, which do not overlap, and the trip through LDS, about equally.
#include "sr_common.h"
#include "gemm_common.h"

#include <type_traits>

namespace sr {
namespace {

typedef float v4f_dword __attribute__((ext_vector_type(4), aligned(4)));

// D = chunks a wave keeps in flight; TPP = 16 x 16 tiles whose partial sums are in LDS at a time.
template <int FM, int FN, int NW, int D>
__global__ __launch_bounds__(NW * 64) void gemm_w4a4_stream_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ xs, const uint8_t *__restrict__ Wq,
    const float *__restrict__ ws, int M, int N, int K, void *__restrict__ Yv, int64_t ldy, int out_i32,
    int tiles_m, int tiles_n)
{
    constexpr int TILES = FM * FN, TPP = TILES <= 8 ? TILES : TILES % 8 == 0 ? 8 : 6;
    // a wave's partial sums; before that, two fragments on their way from load order to operand order
    constexpr int ROW = 144, FRAG = 16 * ROW, OWN = TPP * 1024 > 2 * FRAG ? TPP * 1024 : 2 * FRAG;
    __shared__ __attribute__((aligned(16))) uint8_t lds[NW][OWN];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups are dealt round-robin to the 8 XCDs: XCD x takes an eighth of the tiles in a row, row tiles fastest
    // (the row tiles of a column tile share its weights in that L2, neighbouring column tiles share lines of Y)
    const int total = tiles_m * tiles_n, xcd = blockIdx.x & 7, first = (int)((int64_t)xcd * total >> 3);
    const int v = first + (blockIdx.x >> 3);
    if (v >= (int)((int64_t)(xcd + 1) * total >> 3)) return;
    const int tm = v % tiles_m, tn = v / tiles_m;
    const int m0 = tm * FM * 16, n0 = tn * FN * 16;
    const int nc = K >> 8, Kb = K >> 1, q = lane >> 4;

    // Load order: eight neighbouring lanes fetch a 128-byte line, load j of a fragment its rows 8 j .. 8 j + 7.  Rows past the
    // end re-read the last.
    uint32_t xo[FM][2], wo[FN][2];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + 16 * f + 8 * j + (lane >> 3);
            xo[f][j] = (uint32_t)(m < M ? m : M - 1) * (uint32_t)Kb + 16 * (lane & 7);
        }
#pragma unroll
    for (int f = 0; f < FN; ++f)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + 16 * f + 8 * j + (lane >> 3);
            wo[f][j] = (uint32_t)(n < N ? n : N - 1) * (uint32_t)Kb + 16 * (lane & 7);
        }

    u32x4 x[D][FM][2], w[D][FN][2];                      // chunk d in flight, in load order
    auto load = [&](auto DC, int s) {
        constexpr int d = decltype(DC)::value;
        const uint8_t *wp = Wq + (int64_t)s * 128, *xp = Xq + (int64_t)s * 128;
#pragma unroll
        for (int f = 0; f < FN; ++f)
#pragma unroll
            for (int j = 0; j < 2; ++j) w[d][f][j] = *reinterpret_cast<const u32x4 *>(wp + wo[f][j]);
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int j = 0; j < 2; ++j) x[d][f][j] = *reinterpret_cast<const u32x4 *>(xp + xo[f][j]);
    };
    // Load order -> operand order (lane (i = l & 15, g = l >> 4): bytes 16 g .. + 15 and 64 + 16 g .. + 15 of row i) through the
    // wave's own LDS; its accesses execute in order.  Rows 144 bytes apart: free of bank conflicts both ways.
    uint8_t *const put = &lds[wave][0] + (lane >> 3) * ROW + (lane & 7) * 16;
    const uint8_t *const get = &lds[wave][0] + (lane & 15) * ROW + q * 16;
    auto operands = [&](const u32x4 (&p)[2], int buffer, u32x4 (&h)[2]) {
        *reinterpret_cast<u32x4 *>(put + buffer * FRAG) = p[0];
        *reinterpret_cast<u32x4 *>(put + buffer * FRAG + 8 * ROW) = p[1];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        h[0] = *reinterpret_cast<const u32x4 *>(get + buffer * FRAG);
        h[1] = *reinterpret_cast<const u32x4 *>(get + buffer * FRAG + 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // Output o of pass k of the reduction = lane o & 63 of tile k TPP + (o >> 6): four channels of one token.  Its
    // dequantisation factors are fetched ahead of the operands and used last (see gemm_f6_stream.hip).
    constexpr int PASSES = TILES / TPP;
    static_assert(TILES % TPP == 0 && TPP <= NW, "one output per thread and pass");
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
    v4i acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int f = 0; f < FM; ++f) acc[i][f] = v4i{0, 0, 0, 0};
    auto multiply = [&](auto DC) {
        constexpr int d = decltype(DC)::value;
        v4i xa[FM][2][2];
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            u32x4 h[2];
            operands(x[d][f], f & 1, h);
            unpack16(h[0], xa[f][0][0], xa[f][0][1]);
            unpack16(h[1], xa[f][1][0], xa[f][1][1]);
        }
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            u32x4 h[2];
            operands(w[d][i], (FM + i) & 1, h);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                v4i wa[2];
                unpack16(h[k], wa[0], wa[1]);
#pragma unroll
                for (int f = 0; f < FM; ++f) {
                    acc[i][f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[0], xa[f][k][0], acc[i][f], 0, 0, 0);
                    acc[i][f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[1], xa[f][k][1], acc[i][f], 0, 0, 0);
                }
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
    auto sums = [&](int from, int tile) -> v4i & { return *reinterpret_cast<v4i *>(&lds[from][(tile * 64 + lane) * 16]); };
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        if (k) __syncthreads();
#pragma unroll
        for (int p = 0; p < TPP; ++p) sums(wave, p) = acc[(k * TPP + p) / FM][(k * TPP + p) % FM];
        __syncthreads();
        if (wave < TPP && om[k] < M && on[k] < N) {
            v4i s = sums(0, wave);
#pragma unroll
            for (int u = 1; u < NW; ++u) s += sums(u, wave);
            s >>= 8;                                        // both operands carried a factor 16
            if (out_i32) {
                *reinterpret_cast<v4i *>(static_cast<int32_t *>(Yv) + (int64_t)om[k] * ldy + on[k]) = s;
            } else {
                union { __half h[4]; uint2 u; } y;
                y.h[0] = __float2half_rn((float)s[0] * fx[k] * fw[k].x);
                y.h[1] = __float2half_rn((float)s[1] * fx[k] * fw[k].y);
                y.h[2] = __float2half_rn((float)s[2] * fx[k] * fw[k].z);
                y.h[3] = __float2half_rn((float)s[3] * fx[k] * fw[k].w);
                *reinterpret_cast<uint2 *>(static_cast<__half *>(Yv) + (int64_t)om[k] * ldy + on[k]) = y.u;
            }
        }
    }
}

template <int FM, int FN, int NW, int D>
hipError_t launch_st(const uint8_t *Xq, const float *xs, const uint8_t *Wq, const float *ws, int64_t M, int64_t N,
                     int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st)
{
    const int tiles_m = (int)((M + FM * 16 - 1) / (FM * 16)), tiles_n = (int)((N + FN * 16 - 1) / (FN * 16));
    hipLaunchKernelGGL((gemm_w4a4_stream_kernel<FM, FN, NW, D>), dim3((unsigned)((tiles_m * tiles_n + 7) / 8 * 8)), dim3(NW * 64),
                       0, st, Xq, xs, Wq, ws, (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_w4a4_stream(const uint8_t *Xq, const float *xs, const uint8_t *Wq, const float *ws, int64_t M,
                                   int64_t N, int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st, int bm, int bn)
{
    if (out_i32) {                   // the scales may be NULL then: readable stand-ins (see launch_tile in gemm_prefill.hip)
        xs = reinterpret_cast<const float *>(Xq);
        ws = reinterpret_cast<const float *>(Wq);
    }
#define SR_STREAM(FM, FN, D) \
    if (bm == 16 * FM && bn == 16 * FN) return launch_st<FM, FN, 8, D>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st)
    SR_STREAM(2, 1, 2); SR_STREAM(2, 2, 2); SR_STREAM(2, 4, 2); SR_STREAM(3, 2, 2); SR_STREAM(3, 4, 1); SR_STREAM(4, 4, 1);
#undef SR_STREAM
    return hipErrorInvalidValue;
}

}  // namespace sr
