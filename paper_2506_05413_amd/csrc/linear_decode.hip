// Whole online path of the W4A4 linear layer for a decode step behind one entry point; for up to four tokens and
// K = 2048 / 4096 in ONE launch:
//     x^ = quantise((x * inv_s) H),   Y = dequantise(x^ W^)
// (Paper: online Hadamard + per-token INT4 of the activations in front of the quantised
// projection, section "Methodology" and Eq. (1); this is the decode step, where a launch and a
// round trip through memory cost as much as the arithmetic.)
//
// One token (several: see linear_decode_rows_kernel): a workgroup owns 8 G output channels over
// all of K.  It first ISSUES the loads of its token row and smoothing factors, then of all its weights (they stay in flight in registers), then rotates
// and quantises the row in LDS while the weights travel, and finally multiplies packed codes with
// v_dot8_i32_i4 straight from the registers against the codes in LDS.  Every workgroup repeats
// the rotation, so the grid is kept near one workgroup per CU; and only power-of-two K up to 8192
// is offered, because the rotation of a longer or a 28 * 2^p row takes one workgroup longer than
// the weights take to arrive.  Loads return in order per wave: whatever the rotation needs has to
// be issued BEFORE the weights.  Lane (r = l >> 3, c = l & 7) holds the 16-byte chunk c of a
// 128-byte slab of row r of an 8-row group, so every load instruction reads whole lines; wave w
// takes slabs w, w + 8, ...
#include "two_pass_row.h"

#include <type_traits>

namespace sr {
namespace {

constexpr int LD_NT = 512;                 // threads per workgroup
constexpr int LD_NW = LD_NT / 64;
constexpr int LD_MT = 1;                   // tokens per call

template <int K, int G>
__global__ __launch_bounds__(LD_NT) void linear_decode_kernel(const __half *__restrict__ X, int M, int64_t ldx,
                                                              const float *__restrict__ pre, float clip,
                                                              const uint8_t *__restrict__ Wq,
                                                              const float *__restrict__ ws, int N,
                                                              __half *__restrict__ Y, int64_t ldy,
                                                              uint8_t *__restrict__ Xq_out, float *__restrict__ xs_out)
{
    constexpr int Kb = K / 2;
    constexpr int NSLAB = (Kb + 127) / 128;
    constexpr int U = (NSLAB + LD_NW - 1) / LD_NW;
    static_assert(G * U <= 16, "weights in flight must fit the register file");

    // padded_len(K) floats, then the codes; aligned for the 16-byte accesses (4096 -> 14336: 8.2 -> 7.1 us)
    extern __shared__ __attribute__((aligned(16))) float row[];
    uint32_t *xq = reinterpret_cast<uint32_t *>(row + padded_len(K));   // [LD_MT][K / 8] packed codes
    __shared__ float red[LD_NW];
    __shared__ float sx[LD_MT];

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int r = lane >> 3, c = lane & 7;
    const int n0 = blockIdx.x * (8 * G);

    // ---- the first token row's loads go first (they are what the rotation waits for) ...
    RowLoad<K, LD_NT> xld;
    row_load<K, LD_NT, true>(X, pre, t, xld);

    // ---- ... the channel scale of this thread's output (fetched now, used last: a load after the reduction would
    // put one more memory latency at the end of the kernel) ...
    static_assert(8 * G <= LD_NT, "one output per thread");
    const float w_scale = (t < 8 * G && n0 + t < N) ? ws[n0 + t] : 0.f;

    // ---- ... then all weight loads of this workgroup, up front, every one unconditional: a load under a
    // branch would make the compiler wait for ALL outstanding loads before the rotation may touch the row, and the
    // rotation would then start when the last weight has arrived instead of running while they travel
    static_assert(NSLAB % LD_NW == 0 && Kb % 128 == 0, "every wave owns whole slabs");
    u32x4 w[G][U];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        // register slot g holds row group (g + workgroup index) mod G: at any moment the workgroups of the
        // chip then ask for different offsets inside their 8 G rows, not all for the same memory channels
        int n = n0 + 8 * ((g + (int)blockIdx.x) % G) + r;
        n = n < N ? n : N - 1;                                          // ragged last workgroup: re-read the last row
        const uint8_t *wp = Wq + (int64_t)n * Kb + c * 16;
#pragma unroll
        for (int u = 0; u < U; ++u)
            w[g][u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(wp + (wave + LD_NW * u) * 128));
    }

    // nothing of the rotation may be scheduled ahead of the weight loads (its first instructions wait for the row)
    __builtin_amdgcn_sched_barrier(0);

    // ---- rotate + quantise the token row into LDS (M = 1: the host rejects more) ----------------
    {
        constexpr int m = 0;
        const float amax = rotate_loaded_row_absmax<K, LD_NT>(xld, pre, row, red, t);
        const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
        const float inv_delta = 1.f / delta;
        if (t == 0) {
            sx[m] = delta;
            if (xs_out && blockIdx.x == 0) xs_out[m] = delta;
        }
        uint32_t *q = xq + m * (K / 8);
        for (int i = t; i < K / 8; i += LD_NT) {
            const float *src = row + pad(8 * i);
            const float4 a = *reinterpret_cast<const float4 *>(src);
            const float4 b = *reinterpret_cast<const float4 *>(src + 4);
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            const uint32_t code = quant_pack8(v, inv_delta);
            q[i] = code;
            if (Xq_out && blockIdx.x == 0) reinterpret_cast<uint32_t *>(Xq_out + (int64_t)m * Kb)[i] = code;
        }
        __syncthreads();                                               // row is free again, codes are visible
    }

    // ---- dot products: registers (weights) x LDS (activation codes) ---------------------------
    int acc[G][LD_MT];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int m = 0; m < LD_MT; ++m) acc[g][m] = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int off = (wave + LD_NW * u) * 128 + c * 16;             // byte offset inside a row of codes
        {
#pragma unroll
            for (int m = 0; m < LD_MT; ++m) {
                {
                    const u32x4 x = *reinterpret_cast<const u32x4 *>(xq + m * (K / 8) + off / 4);
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        int a = acc[g][m];
                        a = __builtin_amdgcn_sdot8((int)w[g][u].x, (int)x.x, a, false);
                        a = __builtin_amdgcn_sdot8((int)w[g][u].y, (int)x.y, a, false);
                        a = __builtin_amdgcn_sdot8((int)w[g][u].z, (int)x.z, a, false);
                        a = __builtin_amdgcn_sdot8((int)w[g][u].w, (int)x.w, a, false);
                        acc[g][m] = a;
                    }
                }
            }
        }
    }
    // the 8 lanes of a row, then the waves (through the now idle row buffer)
    int *part = reinterpret_cast<int *>(row);                          // [LD_NW][LD_MT][8 G]
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int m = 0; m < LD_MT; ++m) {
            int v = acc[g][m];
            v = sum_of_8_lanes(v);
            if (c == 0) part[(wave * LD_MT + m) * (8 * G) + ((g + (int)blockIdx.x) % G) * 8 + r] = v;
        }
    __syncthreads();
    if (t < 8 * G && n0 + t < N) {                                      // M = 1: output t of the workgroup
        int sum = 0;
#pragma unroll
        for (int wv = 0; wv < LD_NW; ++wv) sum += part[wv * LD_MT * (8 * G) + t];
        Y[n0 + t] = rounded_once((float)sum * sx[0], w_scale);
    }
}

template <int K, int G>
hipError_t launch_ld(const void *X, int64_t M, int64_t ldx, const float *pre, float clip, const uint8_t *Wq,
                     const float *ws, int64_t N, void *Y, int64_t ldy, uint8_t *Xq_out, float *xs_out, hipStream_t st)
{
    constexpr auto kern = linear_decode_kernel<K, G>;
    constexpr int lds = (int)(sizeof(float) * padded_len(K)) + LD_MT * (K / 2);
    static_assert(lds + 64 <= 160 * 1024, "LDS");
    if (lds > 40 * 1024) {
        hipError_t e = allow_dynamic_lds<kern>(lds);
        if (e != hipSuccess) return e;
    }
    const unsigned blocks = (unsigned)((N + 8 * G - 1) / (8 * G));
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(LD_NT), lds, st, static_cast<const __half *>(X), (int)M, ldx, pre, clip,
                       Wq, ws, (int)N, static_cast<__half *>(Y), ldy, Xq_out, xs_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Two to four tokens in ONE launch, K = 2048 and 4096: every workgroup rotates and quantises all token rows itself while its
// weights travel, then multiplies as gemm_decode_stream_kernel does.
//
// A workgroup of K / 256 waves takes UPW units of 8 channels.  It issues the loads of the token rows and factors, then those
// of its weights, rotates four rows at a time (K / 16 threads each, two passes, two_pass_row.h: the additions, and so the
// codes, of the token quantiser) and leaves codes and scales in LDS; wave w then multiplies slab w of 256 codes: activation
// fragments straight from the codes in LDS, widened once, two units of weights at a time through the wave's staging buffers
// as one operand of v_mfma_i32_16x16x64_i8.  Partial sums are added through LDS, over the idle rows.
//
// Bound by the rotation that every CU repeats (vector-ALU issue, about 0.6 us per row of 4096) plus start-up while the weights
// of a workgroup take less than that, by their arrival beyond.  Against the two launches (us a call, passes one behind the
// other, same box; 2 / 4 tokens; outputs bit for bit the same): 2048 x 4096 6.8 / 6.8 -> 6.0 / 6.0, 2048 x 28672 9.0 / 9.2 ->
// 8.2 / 8.1, 4096 x 4096 6.6 / 7.2 -> 6.5 / 6.6, 4096 x 14336 9.7 / 9.5 -> 8.7 / 8.6, 4096 x 28672 13.3 / 14.1 -> 13.9 / 13.8; with
// a slower host, which takes 4 us for a launch, 2048 x 1024 8.3 -> 5.7, 4096 x 4096 8.3 / 9.4 -> 7.0 / 7.2.  A second batch of
// four tokens adds 2.4 us, as much as the launch it saves: 6 tokens 2048 x 1024 6.7 -> 8.3, 4096 x 14336 10.2 -> 11.4; K = 8192
// (two rows at a time, two passes over the weights) lost beyond two tokens.
// ------------------------------------------------------------------------------------------
template <int LO, int HI, typename F> __device__ __forceinline__ void units_from_to(F f)
{
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>{});
        units_from_to<LO + 1, HI>(f);
    }
}

template <int K> struct DecodeRows {
    using S = TwoPass<K>;
    static constexpr int NW = K / 256;                   // waves, one slab of 256 codes each
    static constexpr int ROWS = NW * 64 / S::NT;         // rows rotated side by side
    static constexpr int CROW = K / 2 + 16;              // bytes from one row of codes to the next
    static constexpr int WROW = 144;                     // from one staged row of weights to the next
    static constexpr int ROW_BYTES = ROWS * S::LEN * 4, STAGE = NW * 2 * 8 * WROW;
    static_assert(S::NT == S::COLS && ROWS == 4, "one thread per 16 values of a row");
    static constexpr int sum_bytes(int upw) { return NW * ((upw + 1) / 2) * 64 * 16; }
    static constexpr int front(int upw) { return ROW_BYTES > sum_bytes(upw) ? ROW_BYTES : sum_bytes(upw); }
    static constexpr int lds(int upw) { return front(upw) + STAGE + ROWS * CROW; }
};

// once: outputs are rounded to fp16 once (see gemm_decode_streams)
template <int K, int UPW>
__global__ __launch_bounds__(DecodeRows<K>::NW * 64, 4) void linear_decode_rows_kernel(
    const __half *__restrict__ X, int M, int64_t ldx, const float *__restrict__ pre, float clip, const uint8_t *__restrict__ Wq,
    const float *__restrict__ ws, int N, __half *__restrict__ Y, int64_t ldy, uint8_t *__restrict__ Xq_out, float *__restrict__ xs_out,
    const bool once)
{
    using D = DecodeRows<K>;
    using S = typename D::S;
    constexpr int NW = D::NW, ROWS = D::ROWS, Kb = K / 2, PAIRS = (UPW + 1) / 2, WROW = D::WROW;
    static_assert(PAIRS <= NW, "one wave per pair adds the sums");
    constexpr uint32_t ALL = 0xFFFFFFFFu;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    __shared__ float red[NW], scale[ROWS];
    v4i *const sums = reinterpret_cast<v4i *>(smem);
    uint8_t *const stage = smem + D::front(UPW), *const codes = stage + D::STAGE;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = threadIdx.x % S::NT, m = threadIdx.x / S::NT;            // thread of a row, row

    // ---- loads: token rows and factors, then the first weights; every one unconditional (see above)
    RowLoad<K, S::NT> ld;
    {
        const __half *x = X + (int64_t)(m < M ? m : 0) * ldx + 16 * t;
        ld.u[0][0] = *reinterpret_cast<const uint4 *>(x);
        ld.u[0][1] = *reinterpret_cast<const uint4 *>(x + 8);
        // without factors 16 other readable floats (of the weights), replaced by ones below
        const float *p = pre ? pre + 16 * t : reinterpret_cast<const float *>(Wq);
#pragma unroll
        for (int q = 0; q < 4; ++q) ld.p[0][q] = *reinterpret_cast<const float4 *>(p + 4 * q);
    }
    // (left to itself the scheduler puts the factors behind the weights, and the rotation waits for all of them)
    __builtin_amdgcn_sched_barrier(0);

    const int units = N >> 3, xcd = blockIdx.x & 7, wg = blockIdx.x >> 3, WGX = gridDim.x >> 3;
    auto unit_of = [xcd](int e) { return ((e >> 3) * 8 + xcd) * 8 + (e & 7); };   // lines of Y go to the XCDs in turn
    const int r8 = lane >> 3, chunk = (lane & 7) * 16;   // load order: row of the unit, byte offset inside a slab
    u32x4 w[PAIRS * 2];
    auto load_unit = [&](auto J) {
        constexpr int j = decltype(J)::value;
        if constexpr (j < UPW) {
            const int un = unit_of(wg + j * WGX);        // a missing unit re-reads the last row; its sums are dropped
            w[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(Wq + (int64_t)(un < units ? 8 * un + r8 : N - 1) * Kb + chunk + wave * 128));
        } else {
            w[j] = u32x4{0u, 0u, 0u, 0u};
        }
    };
    // output of a thread: lane l of wave q < PAIRS owns token l & 15 and channels 4 ((l >> 4) & 1) .. + 3 of unit 2 q + (l >> 5)
    const int om = lane & 15, oj = 2 * wave + (lane >> 5), ou = unit_of(wg + oj * WGX);
    const bool stores = wave < PAIRS && oj < UPW && om < M && ou < units;
    const int on = stores ? 8 * ou + 4 * ((lane >> 4) & 1) : 0;
    const float4 fw = *reinterpret_cast<const float4 *>(ws + on);
    // A CU takes loads only as fast as earlier ones return: a wave that issued all of its weights at once would come to the
    // rotation when most of them have arrived (4096 x 14336, four tokens: 10.2 us a call against 8.7).  So three units go
    // out before it, the others behind its two passes.
    constexpr int FIRST = PAIRS * 2 < 3 ? PAIRS * 2 : 3, SECOND = PAIRS * 2 < 5 ? PAIRS * 2 : 5;
    units_from_to<0, FIRST>(load_unit);
    __builtin_amdgcn_sched_barrier(0);

    // ---- rotate + quantise
    if (!pre) {
#pragma unroll
        for (int q = 0; q < 4; ++q) ld.p[0][q] = make_float4(1.f, 1.f, 1.f, 1.f);
    }
    {
        float *const row = reinterpret_cast<float *>(smem) + m * S::LEN;
        float o[S::R];
        const float amax = two_pass_rotate<S, K, true, false, false, false>(ld, row, red + m * (S::NT / 64), t, ALL, o, [&]() {
            units_from_to<FIRST, SECOND>(load_unit);
            __builtin_amdgcn_sched_barrier(0);
        });
        units_from_to<SECOND, PAIRS * 2>(load_unit);
        __builtin_amdgcn_sched_barrier(0);
        const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
        const float inv_delta = 1.f / delta;
        quantise_row_nibbles<S, K>(row, inv_delta, ALL, codes + m * D::CROW, t);
        if (t == 0) scale[m] = delta;
        if (blockIdx.x == 0 && m < M) {
            if (xs_out && t == 0) xs_out[m] = delta;
            if (Xq_out) quantise_row_nibbles<S, K>(row, inv_delta, ALL, Xq_out + (int64_t)m * Kb, t);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_nofence();                                   // codes and scales are visible, the rows free

    // ---- multiply (tokens beyond the rows repeat them and are not stored)
    v4i xa[2][2];
    {
        const uint8_t *c = codes + (lane & (ROWS - 1)) * D::CROW + wave * 128 + (lane >> 4) * 16;
        unpack16(*reinterpret_cast<const u32x4 *>(c), xa[0][0], xa[0][1]);
        unpack16(*reinterpret_cast<const u32x4 *>(c + 64), xa[1][0], xa[1][1]);
    }
    const float fx = scale[om & (ROWS - 1)];
    uint8_t *const st_put = stage + wave * (2 * 8 * WROW) + r8 * WROW + chunk;
    const uint8_t *const st_get = stage + wave * (2 * 8 * WROW) + ((lane >> 3) & 1) * (8 * WROW) + (lane & 7) * WROW + (lane >> 4) * 16;
    v4i acc[PAIRS];
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) {
        // two units in load order -> one operand in fragment order (a wave's LDS accesses execute in order)
        *reinterpret_cast<u32x4 *>(st_put) = w[2 * q];
        *reinterpret_cast<u32x4 *>(st_put + 8 * WROW) = w[2 * q + 1];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const u32x4 h0 = *reinterpret_cast<const u32x4 *>(st_get);
        const u32x4 h1 = *reinterpret_cast<const u32x4 *>(st_get + 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        v4i a0, a1;
        unpack16(h0, a0, a1);
        acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, xa[0][0], v4i{0, 0, 0, 0}, 0, 0, 0);
        acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, xa[0][1], acc[q], 0, 0, 0);
        unpack16(h1, a0, a1);
        acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, xa[1][0], acc[q], 0, 0, 0);
        acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, xa[1][1], acc[q], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) sums[(wave * PAIRS + q) * 64 + lane] = acc[q];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_nofence();
    if (stores) {
        v4i sum = sums[wave * 64 + lane];
#pragma unroll
        for (int v = 1; v < NW; ++v) sum += sums[(v * PAIRS + wave) * 64 + lane];
        sum >>= 8;                                       // both operands carried the factor 16
        union { __half h[4]; uint2 u; } y;
        y.h[0] = once ? rounded_once((float)sum[0] * fx, fw.x) : rounded_twice((float)sum[0] * fx, fw.x);
        y.h[1] = once ? rounded_once((float)sum[1] * fx, fw.y) : rounded_twice((float)sum[1] * fx, fw.y);
        y.h[2] = once ? rounded_once((float)sum[2] * fx, fw.z) : rounded_twice((float)sum[2] * fx, fw.z);
        y.h[3] = once ? rounded_once((float)sum[3] * fx, fw.w) : rounded_twice((float)sum[3] * fx, fw.w);
        *reinterpret_cast<uint2 *>(Y + (int64_t)om * ldy + on) = y.u;
    }
}

template <int K, int UPW>
hipError_t launch_rows(const void *X, int64_t M, int64_t ldx, const float *pre, float clip, const uint8_t *Wq, const float *ws,
                       int64_t N, void *Y, int64_t ldy, uint8_t *Xq_out, float *xs_out, int wgx, hipStream_t st)
{
    using D = DecodeRows<K>;
    constexpr auto kern = linear_decode_rows_kernel<K, UPW>;
    constexpr int lds = D::lds(UPW);
    static_assert((lds + 256) * (16 / D::NW) <= 160 * 1024, "LDS");
    hipError_t e = allow_dynamic_lds<kern>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(8 * wgx), dim3(D::NW * 64), lds, st, static_cast<const __half *>(X), (int)M, ldx, pre, clip, Wq,
                       ws, (int)N, static_cast<__half *>(Y), ldy, Xq_out, xs_out, !gemm_decode_streams(M, N, K));
    return hipGetLastError();
}

// one workgroup of 16 waves per CU, two of 8; the units of 8 channels that each takes
template <int K> int rows_wgx() { return (compute_units() >= 8 ? compute_units() / 8 : 1) * (16 / DecodeRows<K>::NW); }
template <int K> int64_t rows_units(int64_t N)
{
    const int64_t lines = (N / 8 + 7) / 8, per_xcd = 8 * ((lines + 7) / 8);
    return (per_xcd + rows_wgx<K>() - 1) / rows_wgx<K>();
}
constexpr int kMaxUnits2048 = 8, kMaxUnits4096 = 14, kMaxUnits4096TwoTokens = 10;      // (14: all that the LDS holds)

template <int K>
hipError_t launch_rows_units(const void *X, int64_t M, int64_t ldx, const float *pre, float clip, const uint8_t *Wq, const float *ws,
                             int64_t N, void *Y, int64_t ldy, uint8_t *Xq_out, float *xs_out, hipStream_t st)
{
#define SR_ROWS(U) case U: return launch_rows<K, U>(X, M, ldx, pre, clip, Wq, ws, N, Y, ldy, Xq_out, xs_out, rows_wgx<K>(), st)
    switch (rows_units<K>(N)) {
        SR_ROWS(1); SR_ROWS(2); SR_ROWS(3); SR_ROWS(4); SR_ROWS(5); SR_ROWS(6); SR_ROWS(7); SR_ROWS(8);
        default: break;
    }
    if constexpr (K == 4096) {
        switch (rows_units<K>(N)) {
            SR_ROWS(9); SR_ROWS(10); SR_ROWS(11); SR_ROWS(12); SR_ROWS(13); SR_ROWS(14);
            default: break;
        }
    }
#undef SR_ROWS
    return hipErrorInvalidValue;
}

// Whether the call goes through linear_decode_rows_kernel: 2 .. 4 tokens, as many channels as its registers hold at once -- for
// two tokens fewer, because the dot-product kernel behind the token quantiser is ahead there (24576 channels 12.1 against
// 12.5 us; 20480 the same).
//
// Captured calls, which cost the host nothing when they run, with two tokens or K = 2048 only from 40 M weights on: below, the
// GPU is done sooner with two small launches (graph of calls, 2 / 4 tokens: 2048 x 6144 5.4 / 5.7 against 6.1 / 6.1 us, 4096 x
// 4096 6.5 / 6.6 against 6.9 / 6.6; but 2048 x 28672 8.9 / 9.3 against 8.2 / 8.1, 4096 x 14336 9.6 / 9.6 against 9.3 / 9.1; the
// linears of a layer, 4 tokens, 54.5 against 54.2).
// In a stream the launches follow each other as fast as the host makes them: 3.2 - 3.9 us a call with one, 4.9 - 6.5 with two from a
// C program, 6 and 9 from Python.  So small calls wait for the host: 1024 .. 4096 channels of 2048, C 6.4 -> 5.5 .. 5.8 us a call for
// two tokens, 6.6 -> 5.5 .. 5.8 for four, Python 8.7 -> 5.9; of 4096, C 6.5 .. 6.7 -> 6.0 .. 6.3 and 7.1 .. 7.4 -> 6.1 .. 6.4.  Behind
// a stream that is never empty three and four tokens win or lose nothing (2048 x 4096, weights cached, 5.5 -> 5.7, from HBM 6.2 ->
// 5.8; 4096 x 4096 6.9 -> 6.2 and 7.2 -> 6.7); two tokens lose with cached weights of up to 8192 channels of 2048 and 5120 of 4096
// (5.2 -> 5.7 and 5.7 -> 6.2 at worst); with weights from HBM they take from 5 % longer (4096 x 3072) to 11 % less.
//
// Not where an output overlaps the token rows, which other workgroups may still be reading.
bool rows_path(const void *X, int64_t M, int64_t K, int64_t ldx, int64_t N, const void *Y, int64_t ldy, const void *Xq_out, const void *xs_out,
               hipStream_t st)
{
    if (M < 2 || M > 4 || (K != 2048 && K != 4096)) return false;
    const int64_t units = K == 2048 ? rows_units<2048>(N) : rows_units<4096>(N);
    if (units > (K == 2048 ? kMaxUnits2048 : M == 2 ? kMaxUnits4096TwoTokens : kMaxUnits4096)) return false;
    if (int64_t f; tuned(kTuneDecodeKernel, f)) {
        if (f != 4) return false;
    } else if ((M == 2 || K == 2048) && N * K < 40000000 && st) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone) return false;
    }
    const uintptr_t x = reinterpret_cast<uintptr_t>(X), x_end = x + (size_t)((M - 1) * ldx + K) * 2;
    auto overlaps = [&](const void *p, int64_t bytes) { const uintptr_t a = reinterpret_cast<uintptr_t>(p); return p && a < x_end && x < a + (size_t)bytes; };
    return !overlaps(Y, ((M - 1) * ldy + N) * 2) && !overlaps(Xq_out, M * (K / 2)) && !overlaps(xs_out, M * 4);
}

constexpr int LD_WS_SCALES = 256, LD_WS_CODES = 512;      // workspace of the two-launch path: scales [16], codes [M][K / 2]

// Row groups of 8 channels per workgroup: every workgroup repeats the rotation, so few large workgroups are
// cheaper, but the chip should be filled in whole rounds -- the G <= gmax with the least (rounds x G), ties to
// the larger G (14336 channels on 256 CUs: G = 7 gives exactly 256 workgroups, G = 8 would leave 32 CUs idle).
inline int pick_g(int64_t N, int gmax)
{
    const int64_t cus = compute_units();
    int best = 1;
    int64_t best_cost = -1;
    for (int g = 1; g <= gmax; ++g) {
        const int64_t blocks = (N + 8 * g - 1) / (8 * g);
        const int64_t cost = ((blocks + cus - 1) / cus) * g;
        if (best_cost < 0 || cost <= best_cost) { best = g; best_cost = cost; }
    }
    return best;
}

}  // namespace

bool linear_decode_supported(int64_t K) { return K == 2048 || K == 4096 || K == 8192 || K == 14336; }

// one token and a power-of-two order up to 4096: ONE launch in which every workgroup rotates the row itself
// (4096 -> 14336, weights from HBM: 7.3 against 9.0 us for two launches; 4096 -> 4096: 5.0 against 6.5 us; K = 8192: 11.3 us
// either way, so it takes the general path)
static bool redundant_rotation_path(int64_t M, int64_t K) { return M == 1 && (K == 2048 || K == 4096); }

size_t linear_decode_workspace_bytes(int64_t M, int64_t K)
{
    if (M < 1 || M > 16 || !linear_decode_supported(K) || redundant_rotation_path(M, K)) return 0;
    return (size_t)LD_WS_CODES + (size_t)M * (size_t)(K / 2);
}

hipError_t launch_linear_decode(const void *X, int64_t M, int64_t K, int64_t ldx, const float *pre, float clip,
                                const uint8_t *Wq, const float *ws, int64_t N, void *Y, int64_t ldy,
                                uint8_t *Xq_out, float *xs_out, void *workspace, hipStream_t st)
{
    if (redundant_rotation_path(M, K)) {
#define SR_LD(KK, GG) case GG: return launch_ld<KK, GG>(X, M, ldx, pre, clip, Wq, ws, N, Y, ldy, Xq_out, xs_out, st)
        switch (K) {
            case 2048: switch (pick_g(N, 8)) { SR_LD(2048, 1); SR_LD(2048, 2); SR_LD(2048, 3); SR_LD(2048, 4); SR_LD(2048, 5); SR_LD(2048, 6); SR_LD(2048, 7); SR_LD(2048, 8); default: break; } break;
            case 4096: switch (pick_g(N, 8)) { SR_LD(4096, 1); SR_LD(4096, 2); SR_LD(4096, 3); SR_LD(4096, 4); SR_LD(4096, 5); SR_LD(4096, 6); SR_LD(4096, 7); SR_LD(4096, 8); default: break; } break;
            default: break;
        }
        return hipErrorInvalidValue;
#undef SR_LD
    }
    if (rows_path(X, M, K, ldx, N, Y, ldy, Xq_out, xs_out, st)) {
        if (K == 2048) return launch_rows_units<2048>(X, M, ldx, pre, clip, Wq, ws, N, Y, ldy, Xq_out, xs_out, st);
        return launch_rows_units<4096>(X, M, ldx, pre, clip, Wq, ws, N, Y, ldy, Xq_out, xs_out, st);
    }
    // Everything else -- more tokens, K = 8192 where the two are level, K = 14336 = 28 * 512 -- runs as two launches
    // behind the one entry point: the rotation + quantiser of the M rows, then the M <= 16 GEMM; codes and scales go
    // through the workspace (or straight into the caller's optional outputs).  One-launch variants for these shapes
    // were built and measured against exactly this pair (4096 -> 14336 / 14336 -> 4096, 20 rotating weight copies):
    //  - every workgroup rotating the row(s) itself: 13.4 us against 11.9 us at K = 14336, one token (the rotation
    //    of such a row takes a 512-thread workgroup longer than its weights take to arrive);
    //  - rows rotated once by M extra workgroups and handed to the others through memory (agent-scope release,
    //    relaxed polling, coherent loads of the codes): 11.9 - 12.3 us against 11.9 us at K = 14336 for one token,
    //    13.4 - 15.5 against 12.1 - 12.5 us for 2 - 4 tokens, 12.2 against 10.1 us at K = 4096 for two tokens -- the
    //    producers' own loads queue behind 29 MB of weight requests (rotation done 7.6 us into the kernel instead
    //    of 5.2 us), and dot products on packed nibbles for several tokens lose to the matrix-pipe GEMM;
    //  - the pair with the quantiser launch also pulling the weights into the memory-side cache: 13.5 against
    //    12.1 us (a GEMM that is bound by HBM gains nothing from reading the weights twice).
    uint8_t *wsp = static_cast<uint8_t *>(workspace);
    uint8_t *xq = Xq_out ? Xq_out : wsp + LD_WS_CODES;
    float *xs = xs_out ? xs_out : reinterpret_cast<float *>(wsp + LD_WS_SCALES);
    hipError_t e = launch_fwht_quant(X, M, K, ldx, pre, clip, 1.0f, xq, xs, st);
    if (e != hipSuccess) return e;
    return launch_gemm_decode(xq, xs, Wq, ws, M, N, K, Y, ldy, 0, st);
}

}  // namespace sr
