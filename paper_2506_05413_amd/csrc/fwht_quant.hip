// Online Hadamard rotation fused with per-row symmetric INT4 quantisation.
//
// One workgroup owns one row (a token of X, or an output channel of the transposed,
// smoothed weight during the fold).  The row is converted to fp32, rotated by
// T(v) = v H on chip and quantised; only the packed codes and one scale per row go
// back to memory.  (Paper: online exact Hadamard before the projection, section
// "Methodology"; quantiser Eq. (1) with per-token / per-channel symmetric scales.)
//
// Rotation schedule.  H = (x) of 2x2 Sylvester factors (and H_28 for K = 28 * 2^p);
// Kronecker factors commute, so the butterflies are grouped into passes of up to four
// index bits that a thread can do entirely in registers on 16 values:
//   pass 1   bits 0-3, straight from the global load (16 contiguous fp16 per group)
//   pass 2.. bits 4-7, 8-11, ... gathered from / scattered to an fp32 row in LDS
//   H_28     28 values at stride 2^p per group, as  y_j = S - 2 * sum_{H[i][j]=-1} v_i
// The LDS row is padded by 4 floats per 64 so that every access pattern above is
// bank-conflict free for K = 4096.
#include "fwht_row.h"
#include "clip_search.h"
#include "gemm_common.h"      // LDS-DMA load, hand-placed waits, fence-free barrier

#include <type_traits>

namespace sr {
namespace {

// F6: Q receives f6 tiles (operands of the FP6-MFMA GEMM) instead of packed nibbles; K % 128 == 0 then.
template <int K, int NT, bool F6, bool GATE = false>
__global__ __launch_bounds__(NT) void fwht_quant_kernel(const __half *__restrict__ X, int64_t ldx, int64_t rows,
                                                        const float *__restrict__ pre, float clip,
                                                        float post_scale, uint8_t *__restrict__ Q,
                                                        float *__restrict__ scale_out,
                                                        const __half *__restrict__ gate, int64_t ldg,
                                                        const uint32_t *__restrict__ warm, int64_t warm_lines)
{
    // The alignment is part of the layout: without it the row starts where the static LDS of the kernel happens to end
    // (8 bytes in with two waves), and every 16-byte access splits -- K = 2048, 16384 rows: 44.5 -> 33.7 us, K = 1024,
    // 4096 rows: 12.5 -> 6.1 us.
    extern __shared__ __attribute__((aligned(16))) float row[];
    __shared__ float red[NT / 64];

    const int t = threadIdx.x;
    // warming the memory-side cache for the kernel that follows (see fwht4096_wave_kernel): the threads of the
    // launch share the lines and read one word of each once the workgroup's first row has left its load registers
    uint32_t warm_acc = 0;
    auto warm_lines_now = [&]() {
        if (warm) {
            const int64_t gt = (int64_t)blockIdx.x * NT + t, nt = (int64_t)gridDim.x * NT;
            for (int64_t l = gt; l < warm_lines; l += nt) warm_acc ^= warm[l * 32];
        }
    };
    // F6: the eight rows of a tile block (768 contiguous bytes per 128 codes) should be written from ONE XCD at
    // about the same time, so that its L2 assembles whole lines: workgroups are dealt round-robin to the 8
    // XCDs, so (virtual) workgroup w = 8 a + x (XCD x) takes row r = a % 8 of row block 8 (a / 8) + x.
    int64_t m = blockIdx.x;
    if constexpr (F6) {
        const int64_t w = blockIdx.x, x = w & 7, a = w >> 3;
        m = 64 * (a >> 3) + 8 * x + (a & 7);
        if (m >= rows) {                                 // the grid is rounded up to a multiple of 64
            zero_f6_padding_row<K, NT>(Q, (rows + 7) >> 3, m, t);
            return;
        }
    }
    RowLoad<K, NT> ld;
    row_load<K, NT, false, GATE>(X + m * ldx, pre, t, ld, GATE ? gate + m * ldg : nullptr);
    const float amax = rotate_loaded_row_absmax<K, NT, GATE>(ld, pre, row, red, t, warm_lines_now);

    // Delta = clip * absmax / 7 (1 for an all-zero row), Eq. (1) with the signed range
    const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
    const float inv_delta = 1.f / delta;
    if (t == 0) scale_out[m] = (amax == 0.f) ? 1.f : delta * post_scale;

    if constexpr (F6) {
        // ---- 32 contiguous values -> one 24-byte piece of a tile (the padding of 4 floats per 64 keeps the
        // 16-byte reads of 16 neighbouring threads on distinct banks) -----------------------------------------
        const int64_t row_blocks = (rows + 7) >> 3;
        for (int p = t; p < K / 32; p += NT) quant_store_f6_piece(row + pad(32 * p), inv_delta, Q, row_blocks, m, p);
    } else {
        // ---- quantise 8 contiguous values -> one packed dword ---------------------------------------------
        uint32_t *q = reinterpret_cast<uint32_t *>(Q + m * (int64_t)(K / 2));
        for (int c = t; c < K / 8; c += NT) {
            const float *src = row + pad(8 * c);
            const float4 a = *reinterpret_cast<const float4 *>(src);
            const float4 b = *reinterpret_cast<const float4 *>(src + 4);
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            q[c] = quant_pack8(v, inv_delta);
        }
    }
    asm volatile("" ::"v"(warm_acc));                    // keeps the warming loads; they returned long ago
}

// search_ratio's view of a row in the padded layout
struct RowRead8 {
    const float *row;
    __device__ __forceinline__ void operator()(int g, float4 &a, float4 &b) const
    {
        const float *src = row + pad(8 * g);
        a = *reinterpret_cast<const float4 *>(src);
        b = *reinterpret_cast<const float4 *>(src + 4);
    }
};

// The fold of a weight with the search, full transform: one workgroup per output channel.  The products with the smoothing
// factors are rounded as in fwht_quant_ex_kernel, which folds the other searched weights and folded these before: left
// unrounded in the first level, scales moved by an ulp and three codes of 16.8 million by one (4096 x 4096).
// HIST: the ratio from one pass over the row where that decides it (q: see ratio_of_cells).
template <int K, int NT, bool HIST>
__global__ __launch_bounds__(NT) void fwht_quant_search_kernel(const __half *__restrict__ X, int64_t ldx,
                                                               const float *__restrict__ pre, float post_scale,
                                                               uint8_t *__restrict__ Q, float *__restrict__ scale_out,
                                                               const RowExtras ex, const int q, const int undecided)
{
    extern __shared__ __attribute__((aligned(16))) float row[];
    __shared__ float red[NT / 64];
    __shared__ int signs;                                // of the values of magnitude amax
    void *const scratch = row + padded_len(K);           // the cells, or partial errors of search_ratio
    const int t = threadIdx.x;
    const int64_t m = blockIdx.x;
    if constexpr (HIST) {                                // visible after the rotation's barriers
        clear_cells<K, NT>(static_cast<uint64_t *>(scratch), q, t);
        if (t == 0) signs = 0;
    }
    const float amax = rotate_row_absmax<K, NT, true>(X + m * ldx, pre, row, red, t);
    const RowRead8 read8{row};
    float clip = ex.grid[0];
    if (amax != 0.f) {
        int i = -1;
        if constexpr (HIST) {
            // (beyond this range the scaled values would not stay inside fp32; the largest being finite, all values are)
            bool count = amax > 0x1p-90f && amax < 0x1p90f;
            const bool spikes = spiked<NT>(red, amax);
            if constexpr (!is_pow2(K)) {
                count = count && !spikes;
            } else if (count && spikes && undecided) {
                if (undecided != 3) {
                    for (int c = t; c < K; c += NT) note_sign(&signs, row[pad(c)], amax, false);
                    __syncthreads();
                }
                count = undecided != 3 && (signs & undecided) == 0;
            }
            if (count) {
                uint64_t *const cells = static_cast<uint64_t *>(scratch);
                const CellScale scale(q, amax);
                auto count_row = [&](auto some, int lowest) {
                    for (int c = t; c < K / 4; c += NT) {
                        const float4 v = *reinterpret_cast<const float4 *>(row + pad(4 * c));
                        count_value<some.value>(cells, scale, 14 * q, 28 * q + 1, v.x, lowest);
                        count_value<some.value>(cells, scale, 14 * q, 28 * q + 1, v.y, lowest);
                        count_value<some.value>(cells, scale, 14 * q, 28 * q + 1, v.z, lowest);
                        count_value<some.value>(cells, scale, 14 * q, 28 * q + 1, v.w, lowest);
                    }
                };
                if (is_pow2(K) && spikes) count_row(std::true_type{}, lowest_boundary(ex.grid[ex.n_grid - 1], q));
                else count_row(std::false_type{}, 0);
                __syncthreads();
                i = ratio_of_cells<K, NT>(ex.grid, ex.n_grid, q, cells, t);
            }
        }
        if (i >= 0) clip = ex.grid[i];
        else clip = search_ratio<K, NT>(read8, amax, ex.grid, ex.n_grid, t, static_cast<double *>(scratch));
    }
    if (ex.ratio_out && t == 0) ex.ratio_out[m] = clip;
    const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
    const float inv_delta = 1.f / delta;
    if (t == 0) scale_out[m] = (amax == 0.f) ? 1.f : delta * post_scale;
    quantise_padded_row_nibbles<K, NT>(row, inv_delta, Q + m * (int64_t)(K / 2), t);
}

// ------------------------------------------------------------------------------------------
// Extended row kernel: the same rotation + quantiser with three optional extras
//   gate       x = silu(gate) * X in fp32 before smoothing (the down-projection input of the gated
//              FFN, paper Fig. 2: sigma(gate) (.) up, then 1/s, Hadamard, quantiser)
//   had_mask   head-wise Hadamard: only the selected index bits are transformed (power-of-two K)
//   grid       per-row clipping ratio by linear search over the squared quantisation error
//              (paper, "Quantization" settings for the weights), first minimum in grid order
// Kept apart from the plain kernel so that the hot path carries none of these branches.
// ------------------------------------------------------------------------------------------
template <int K, int NT, bool F6>
__global__ __launch_bounds__(NT) void fwht_quant_ex_kernel(const __half *__restrict__ X, int64_t ldx, int64_t rows,
                                                           const float *__restrict__ pre, float clip,
                                                           float post_scale, uint8_t *__restrict__ Q,
                                                           float *__restrict__ scale_out, const RowExtras ex)
{
    constexpr bool KRON = !is_pow2(K);
    constexpr int P2 = KRON ? K / 28 : K;
    constexpr int LOGP = ilog2(P2);
    constexpr int NW = NT / 64;

    extern __shared__ __attribute__((aligned(16))) float row[];
    __shared__ float red[NW];

    const int t = threadIdx.x;
    int64_t m = blockIdx.x;
    if constexpr (F6) {                                  // rows of a tile block from one XCD (see fwht_quant_kernel)
        const int64_t w = blockIdx.x, x8 = w & 7, a = w >> 3;
        m = 64 * (a >> 3) + 8 * x8 + (a & 7);
        if (m >= rows) {
            zero_f6_padding_row<K, NT>(Q, (rows + 7) >> 3, m, t);
            return;
        }
    }
    const __half *x = X + m * ldx;
    const __half *gt = ex.gate ? ex.gate + m * ex.ldg : nullptr;
    const uint32_t mask = KRON ? 0xFFFFFFFFu : ex.had_mask;

    // ---- pass 1: bits 0..3 from global ------------------------------------------------
    for (int g = t; g < K / 16; g += NT) {
        union { uint4 u[2]; __half h[16]; } raw, graw;
        raw.u[0] = *reinterpret_cast<const uint4 *>(x + 16 * g);
        raw.u[1] = *reinterpret_cast<const uint4 *>(x + 16 * g + 8);
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = __half2float(raw.h[e]);
        if (gt) {
            graw.u[0] = *reinterpret_cast<const uint4 *>(gt + 16 * g);
            graw.u[1] = *reinterpret_cast<const uint4 *>(gt + 16 * g + 8);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float gv = __half2float(graw.h[e]);
                // silu(g) = g / (1 + exp(-g)); exp(-g) = inf for very negative g gives g * 0 = -0
                v[e] *= gv * __builtin_amdgcn_rcpf(1.f + __expf(-gv));
            }
        }
        if (pre) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 s = *reinterpret_cast<const float4 *>(pre + 16 * g + 4 * q);
                v[4 * q + 0] *= s.x; v[4 * q + 1] *= s.y; v[4 * q + 2] *= s.z; v[4 * q + 3] *= s.w;
            }
        }
        butterflies_masked<4>(v, mask & 15u);
        float *dst = row + pad(16 * g);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(dst + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    }
    __syncthreads();

    lds_passes_masked<K, NT, 4, LOGP>(row, t, mask);

    if constexpr (KRON) {
        for (int g = t; g < P2; g += NT) {
            float v[28], o[28];
            float *col = row + pad(g);
#pragma unroll
            for (int i = 0; i < 28; ++i) v[i] = col[strided<P2>(g, i)];
            h28_program(v, o);
#pragma unroll
            for (int j = 0; j < 28; ++j) col[strided<P2>(g, j)] = o[j];
        }
        __syncthreads();
    }

    // ---- row absmax (own sweep: the last transforming pass depends on the mask) -----------------
    float amax = 0.f;
    for (int c = t; c < K / 8; c += NT) {
        const float *src = row + pad(8 * c);
        const float4 a = *reinterpret_cast<const float4 *>(src);
        const float4 b = *reinterpret_cast<const float4 *>(src + 4);
        amax = fmaxf(amax, fmaxf(fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))),
                                 fmaxf(fmaxf(fabsf(b.x), fabsf(b.y)), fmaxf(fabsf(b.z), fabsf(b.w)))));
    }
    amax = max_of_wave(amax);
    if ((t & 63) == 0) red[t >> 6] = amax;
    __syncthreads();
    amax = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) amax = fmaxf(amax, red[w]);

    if constexpr (!F6) {                                 // (the search belongs to the weight fold, which writes nibbles)
        __shared__ double err_w[search_scratch(NT)];
        if (ex.n_grid > 0) clip = amax != 0.f ? search_ratio<K, NT>(RowRead8{row}, amax, ex.grid, ex.n_grid, t, err_w) : ex.grid[0];
    }
    if (ex.ratio_out && t == 0) ex.ratio_out[m] = clip;

    const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
    const float inv_delta = 1.f / delta;
    if (t == 0) scale_out[m] = (amax == 0.f) ? 1.f : delta * post_scale;

    if constexpr (F6) {
        for (int p = t; p < K / 32; p += NT) quant_store_f6_piece(row + pad(32 * p), inv_delta, Q, (rows + 7) >> 3, m, p);
    } else {
        uint32_t *q = reinterpret_cast<uint32_t *>(Q + m * (int64_t)(K / 2));
        for (int c = t; c < K / 8; c += NT) {
            const float *src = row + pad(8 * c);
            const float4 a = *reinterpret_cast<const float4 *>(src);
            const float4 b = *reinterpret_cast<const float4 *>(src + 4);
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            q[c] = quant_pack8(v, inv_delta);
        }
    }
}

// ------------------------------------------------------------------------------------------
// K = 4096: one WAVE per row, no workgroup barriers.  A lane holds 64 fp32 values, so six index
// bits are butterflied in registers at a time and only one transposition separates the two
// halves of the transform:
//   phase 1  lane l loads the 16-byte chunks l, l+64, ..: registers = index bits {0,1,2,9,10,11}
//   LDS      wave-private transposition (row padded by 8 floats per 512: conflict-free both ways)
//   phase 2  lane (e = l & 7, j = l >> 3) holds elements 512 j + 8 r + e: registers = bits 3..8
//   row absmax by a wave reduction, Delta, then back through LDS to the natural order, where a
//   lane quantises 8 consecutive values into one packed dword.
// ------------------------------------------------------------------------------------------

// STAGED (with factors, full transform): the 16 KB of smoothing factors reach the four waves of a workgroup through
// LDS -- ONE copy per workgroup by LDS-DMA instead of 16 vector loads per wave, a quarter of the traffic on the
// CU's vector-memory path, which every row load of the launch has to share.  The copies are inline assembly with a
// hand-counted wait, so that the order (factors, then the row) and the wait (factors have landed while the row is
// still in flight) are what is written here, not what the compiler's scheduler makes of them.
// MASKED: head-wise transform -- only the index bits set in had_mask are butterflied (uniform branches).
template <bool HAS_PRE, bool F6, bool STAGED = false, bool MASKED = false>
__global__ __launch_bounds__(256) void fwht4096_wave_kernel(const __half *__restrict__ X, int64_t ldx, int64_t rows,
                                                            const float *__restrict__ pre, float clip, float post_scale,
                                                            uint8_t *__restrict__ Q, float *__restrict__ scale_out,
                                                            const uint32_t *__restrict__ warm,
                                                            int64_t warm_lines, uint32_t had_mask)
{
    constexpr int K = 4096, ROWF = F6 ? K + 576 : K + 64;   // floats per wave-private row incl. padding
    extern __shared__ __attribute__((aligned(16))) float smem_rows[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t m = (int64_t)blockIdx.x * 4 + wave;
    if constexpr (F6) {
        // both halves of a tile block (8 rows) from the same XCD: workgroup w = 8 a + x (XCD x) takes half
        // a % 2 of row block 8 (a / 2) + x (see the workgroup-per-row kernel)
        const int64_t w = blockIdx.x, x = w & 7, a = w >> 3;
        m = 8 * (8 * (a >> 1) + x) + 4 * (a & 1) + wave;
    }
    static_assert(!STAGED || (HAS_PRE && !MASKED), "the staged variant is the plain transform with factors");
    static_assert(!MASKED || !F6, "head-wise rows are written as nibbles");
    if constexpr (!STAGED) {
        if (m >= rows) {                                 // no barrier below: waves are independent
            if constexpr (F6) zero_f6_padding_row<K, 64>(Q, (rows + 7) >> 3, m, lane);
            return;
        }
    }
    float *buf = smem_rows + wave * ROWF;
    const __half *x = X + m * ldx;

    // ---- phase 1 --------------------------------------------------------------------------
    // every load of the row first (the scheduling barrier keeps the compiler from sinking each load to its use,
    // which serialised the memory round trips), then the arithmetic, chunk by chunk as the data arrives
    uint4 rx[8];
    u32x4 rxa[8];                                        // STAGED: the row as loaded by inline assembly
    float4 rs[8][2];
    if constexpr (STAGED) {
        const bool active = m < rows;                    // a wave past the last row still helps with the factors
        // wave w copies KB 4 w .. 4 w + 3 of the factors into the staging area, which overlays the row buffers
        // (nobody writes those before the second barrier).  KB q = half h = q & 1 of the 512 factors j = q >> 1:
        // lane l fetches the four factors 512 j + 8 l + 4 h .., so that the reads below are contiguous per lane.
        const uint32_t stage = (uint32_t)(uintptr_t)smem_rows;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = __builtin_amdgcn_readfirstlane(4 * wave + i);
            dma16(reinterpret_cast<const uint8_t *>(pre), (uint32_t)((512 * (q >> 1) + 8 * lane + 4 * (q & 1)) * 4),
                  (uint32_t)__builtin_amdgcn_readfirstlane((int)(stage + q * 1024)));
        }
        // The row's loads are inline assembly too: ordinary loads from a read-only argument float freely in the
        // compiler's schedule (it sank them below both barriers, past the wait that counts on them).  The compiler
        // takes rxa[] for defined where the statement stands; every use goes through the wait statements below.
        const uint64_t xa = (uint64_t)(uintptr_t)(active ? x : X);          // wave-uniform: into scalar registers
        const uint32_t xlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)xa);
        const uint32_t xhi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(xa >> 32));
        const __half *xr = reinterpret_cast<const __half *>((uint64_t)xlo | ((uint64_t)xhi << 32));
#pragma unroll
        for (int j = 0; j < 8; ++j)
            asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(rxa[j]) : "v"((uint32_t)((512 * j + 8 * lane) * 2)), "s"(xr) : "memory");
        wait_vmcnt<8>();
        barrier_nofence();                               // all 16 KB of factors are in LDS
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            rs[j][0] = *reinterpret_cast<const float4 *>(reinterpret_cast<const uint8_t *>(smem_rows) + (2 * j) * 1024 + lane * 16);
            rs[j][1] = *reinterpret_cast<const float4 *>(reinterpret_cast<const uint8_t *>(smem_rows) + (2 * j + 1) * 1024 + lane * 16);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier_nofence();                               // every wave holds its factors: the row buffers are free
        if (!active) {
            wait_vmcnt<0>();                             // (its loads read row 0; nothing may be in flight at the end)
            if constexpr (F6) zero_f6_padding_row<K, 64>(Q, (rows + 7) >> 3, m, lane);
            return;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            rx[j] = *reinterpret_cast<const uint4 *>(x + 512 * j + 8 * lane);
            if (HAS_PRE) {
                rs[j][0] = *reinterpret_cast<const float4 *>(pre + 512 * j + 8 * lane);
                rs[j][1] = *reinterpret_cast<const float4 *>(pre + 512 * j + 8 * lane + 4);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    float v[64];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if constexpr (STAGED) {
            // chunk j has landed once at most 7 - j younger loads are outstanding (loads complete in order)
            if (j == 0) asm volatile("s_waitcnt vmcnt(7)" : "+v"(rxa[0]));
            if (j == 1) asm volatile("s_waitcnt vmcnt(6)" : "+v"(rxa[1]));
            if (j == 2) asm volatile("s_waitcnt vmcnt(5)" : "+v"(rxa[2]));
            if (j == 3) asm volatile("s_waitcnt vmcnt(4)" : "+v"(rxa[3]));
            if (j == 4) asm volatile("s_waitcnt vmcnt(3)" : "+v"(rxa[4]));
            if (j == 5) asm volatile("s_waitcnt vmcnt(2)" : "+v"(rxa[5]));
            if (j == 6) asm volatile("s_waitcnt vmcnt(1)" : "+v"(rxa[6]));
            if (j == 7) asm volatile("s_waitcnt vmcnt(0)" : "+v"(rxa[7]));
            rx[j] = make_uint4(rxa[j][0], rxa[j][1], rxa[j][2], rxa[j][3]);
        }
        union { uint4 u; half2v h[4]; } raw;
        raw.u = rx[j];
        float f[8];
        if (HAS_PRE) {
            const float4 s0 = rs[j][0], s1 = rs[j][1];
            f[0] = s0.x; f[1] = s0.y; f[2] = s0.z; f[3] = s0.w;
            f[4] = s1.x; f[5] = s1.y; f[6] = s1.z; f[7] = s1.w;
        }
        if constexpr (MASKED) {                          // index bit 0 may be unselected: values as they are
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[8 * j + e] = (float)raw.h[e >> 1][e & 1];
                if (HAS_PRE) v[8 * j + e] *= f[e];
            }
        } else {                                         // conversion, factor and index bit 0 in one go
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (HAS_PRE) pair_level(raw.h[e], f[2 * e], f[2 * e + 1], v[8 * j + 2 * e], v[8 * j + 2 * e + 1]);
                else pair_level(raw.h[e], v[8 * j + 2 * e], v[8 * j + 2 * e + 1]);
            }
        }
        // (STAGED: keeps the arithmetic of chunk j between the waits for chunks j and j + 1 -- the compiler
        // otherwise gathers the eight waits in front of all of it)
        if constexpr (STAGED) {
            float *vj = v + 8 * j;
            float blk[8] = {vj[0], vj[1], vj[2], vj[3], vj[4], vj[5], vj[6], vj[7]};
            butterflies_from<3, 2>(blk);                 // index bits 1, 2 inside the chunk, as soon as it is there
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                vj[e] = blk[e];
                asm volatile("" : "+v"(vj[e]));          // pins the arithmetic here (it would be sunk to its first use)
            }
        }
    }
    // register bits = index bits 0, 1, 2, 9, 10, 11
    if constexpr (MASKED) butterflies_masked<6>(v, (had_mask & 7u) | (((had_mask >> 9) & 7u) << 3));
    else if constexpr (STAGED) butterflies_from<6, 8>(v);   // bits 1, 2 were done chunk by chunk
    else butterflies_from<6, 2>(v);
    // Warming the memory-side cache for the kernel that follows (its weights): the waves of the launch share the
    // 128-byte lines of [warm, warm + 128 warm_lines) and read one word of each -- with ordinary loads, so that the
    // lines are allocated -- now that the row's own loads have returned; the words are never looked at.
    uint32_t warm_acc = 0;
    if (warm) {
        const int64_t gw = (int64_t)blockIdx.x * 4 + wave, nw = (int64_t)gridDim.x * 4;
        for (int64_t l = gw * 64 + lane; l < warm_lines; l += nw * 64) warm_acc ^= warm[l * 32];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float *d = buf + 520 * j + 8 * lane;             // element 512 j + 8 l + e lives at 520 j + 8 l + e
        *reinterpret_cast<float4 *>(d) = make_float4(v[8 * j], v[8 * j + 1], v[8 * j + 2], v[8 * j + 3]);
        *reinterpret_cast<float4 *>(d + 4) = make_float4(v[8 * j + 4], v[8 * j + 5], v[8 * j + 6], v[8 * j + 7]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

    // ---- phase 2 --------------------------------------------------------------------------
    const float *src = buf + 520 * (lane >> 3) + (lane & 7);
#pragma unroll
    for (int r = 0; r < 64; ++r) v[r] = src[8 * r];
    if constexpr (MASKED) butterflies_masked<6>(v, (had_mask >> 3) & 63u);      // index bits 3..8
    else butterflies<6>(v);
    float amax = 0.f;
#pragma unroll
    for (int r = 0; r < 64; r += 2) amax = fmaxf(fmaxf(amax, fabsf(v[r])), fabsf(v[r + 1]));
    amax = max_of_wave(amax);
    const float delta = (amax == 0.f) ? 1.f : (clip * amax) / 7.f;
    const float inv_delta = 1.f / delta;
    if (lane == 0) scale_out[m] = (amax == 0.f) ? 1.f : delta * post_scale;

    if constexpr (F6) {
        // ---- f6 tiles: every lane converts two pieces of 32 consecutive values (quant_store_f6_piece) -----------
        // Back through LDS with 4 floats of padding per 32 and 8 per 512 (element i at i + 4 (i >> 5) + 8 (i >> 9)):
        // the scattered writes below and the 16-byte reads of 32 values per lane are both free of bank conflicts.
        float *dst = buf + 584 * (lane >> 3) + (lane & 7);
#pragma unroll
        for (int r = 0; r < 64; ++r) dst[8 * r + 4 * (r >> 2)] = v[r];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        const int64_t row_blocks = (rows + 7) >> 3;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int p = lane + 64 * pass;                  // piece p of the row: k = 32 p .. 32 p + 31
            quant_store_f6_piece(buf + 36 * p + 8 * (p >> 4), inv_delta, Q, row_blocks, m, p);
        }
    } else {
        float *dst = buf + 520 * (lane >> 3) + (lane & 7);
#pragma unroll
        for (int r = 0; r < 64; ++r) dst[8 * r] = v[r];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

        // ---- quantise: 8 consecutive values -> one dword ---------------------------------------
        uint32_t *q = reinterpret_cast<uint32_t *>(Q + m * (int64_t)(K / 2));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float *s8 = buf + 520 * j + 8 * lane;
            const float4 a = *reinterpret_cast<const float4 *>(s8);
            const float4 b = *reinterpret_cast<const float4 *>(s8 + 4);
            const float y[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            q[64 * j + lane] = quant_pack8(y, inv_delta);
        }
    }
    asm volatile("" ::"v"(warm_acc));                    // keeps the warming loads; they returned long ago
}

__global__ __launch_bounds__(256) void fill_f32_kernel(float *__restrict__ dst, int64_t n, float value)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = value;
}

// One workgroup per row.
template <int K, int NT, bool F6, bool GATE>
hipError_t launch_row_kernel(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip, float post_scale,
                             uint8_t *Q, float *scale_out, const __half *gate, int64_t ldg, hipStream_t st,
                             const void *warm = nullptr, size_t warm_bytes = 0)
{
    constexpr size_t lds = sizeof(float) * padded_len(K);
    const int64_t grid = F6 ? (rows + 63) / 64 * 64 : rows;
    constexpr auto kern = fwht_quant_kernel<K, NT, F6, GATE>;
    if (lds > 48 * 1024) {
        hipError_t e = allow_dynamic_lds<kern>((int)lds);
        if (e != hipSuccess) return e;
    }
    // the hint is honoured from 256 workgroups on (a launch of a few rows cannot move megabytes on the side)
    const bool warms = warm && warm_bytes >= 128 && grid >= 256;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NT), lds, st,
                       static_cast<const __half *>(X), ldx, rows, pre, clip, post_scale, Q, scale_out, gate, ldg,
                       warms ? static_cast<const uint32_t *>(warm) : nullptr, (int64_t)(warm_bytes / 128));
    return hipGetLastError();
}

template <int K, bool F6 = false, int NT_FORCE = 0>
hipError_t launch_one(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip,
                      float post_scale, uint8_t *Q, float *scale_out, hipStream_t st,
                      const void *warm = nullptr, size_t warm_bytes = 0)
{
    constexpr int groups = K / 16;
    constexpr int NT = NT_FORCE ? NT_FORCE : (groups >= 256 ? 256 : (groups >= 128 ? 128 : 64));
    // Long rows: more threads per row where they pay (measured, one row / 2048 rows, 256 threads against the
    // choice below).  K = 16384: 9.0 -> 6.0 / 46.6 -> 34.4; 28672 (one workgroup per CU whatever its size): 23.5 ->
    // 9.7 / 257 -> 87; 32768: 24.9 -> 19.9 / 276 -> 222.  K = 7168 only while every row still has a CU to itself (two
    // small workgroups per CU overlap better than one large one).
    if constexpr (NT_FORCE == 0) {
        if constexpr (K == 16384 || K == 28672 || K == 32768)
            return launch_one<K, F6, 1024>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st);
        if constexpr (K == 7168) {
            if (rows <= 512) return launch_one<K, F6, 512>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st);
        }
    }
    return launch_row_kernel<K, NT, F6, false>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, nullptr, 0, st, warm, warm_bytes);
}

// silu(gate) * x in front of the plain kernel (no head mask, no clip search)
template <int K, bool F6 = false, int NT_FORCE = 0>
hipError_t launch_one_gated(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip, float post_scale,
                            uint8_t *Q, float *scale_out, const __half *gate, int64_t ldg, hipStream_t st)
{
    constexpr int groups = K / 16;
    constexpr int NT = NT_FORCE ? NT_FORCE : (groups >= 256 ? 256 : (groups >= 128 ? 128 : 64));
    if constexpr (NT_FORCE == 0) {                          // threads per row as in launch_one
        if constexpr (K == 16384 || K == 28672)
            return launch_one_gated<K, F6, 1024>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, gate, ldg, st);
        if constexpr (K == 7168) {
            if (rows <= 512) return launch_one_gated<K, F6, 512>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, gate, ldg, st);
        }
    }
    return launch_row_kernel<K, NT, F6, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, gate, ldg, st);
}

template <int K, int NT, bool HIST>
hipError_t launch_search(const void *X, int64_t rows, int64_t ldx, const float *pre, float post_scale, uint8_t *Q, float *scale_out,
                         const RowExtras &ex, int q, hipStream_t st)
{
    constexpr auto kern = fwht_quant_search_kernel<K, NT, HIST>;
    constexpr int row_bytes = (int)sizeof(float) * padded_len(K), most = HIST ? histogram_words(K, NT, kMaxClipDenominator) * 8 : 0;
    constexpr int scratch = search_scratch(NT) * 8, lds_most = row_bytes + (most > scratch ? most : scratch);
    static_assert(lds_most + 1024 <= 160 * 1024, "LDS");
    const int cells = HIST ? histogram_words(K, NT, q) * 8 : 0;
    if (lds_most > 40 * 1024) {
        hipError_t e = allow_dynamic_lds<kern>(lds_most);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)rows), dim3(NT), row_bytes + (cells > scratch ? cells : scratch), st,
                       static_cast<const __half *>(X), ldx, pre, post_scale, Q, scale_out, ex, q, HIST ? undecided_signs(ex.grid, ex.n_grid, K) : 0);
    return hipGetLastError();
}

template <int K, bool F6 = false>
hipError_t launch_one_ex(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip,
                         float post_scale, uint8_t *Q, float *scale_out, const RowExtras &ex, hipStream_t st)
{
    constexpr int groups = K / 16;
    constexpr int NT = groups >= 256 ? 256 : (groups >= 128 ? 128 : 64);
    constexpr size_t lds = sizeof(float) * padded_len(K);
    if constexpr (!F6) {
        if (ex.n_grid > 0 && !ex.gate && (ex.had_mask == 0xFFFFFFFFu || !is_pow2(K))) {
            // threads per row as in launch_one (many rows); K = 2048 x 4096 channels, 21 ratios: 34 us with 256 threads
            // against 39 with 128 (1024: 24 against 19 with 64, 512: 17 against 13)
            constexpr int NTS = K == 8192 ? 512 : (K == 16384 || K == 28672 || K == 32768) ? 1024 : K == 2048 ? 256 : NT;
            // The one-pass search, us a call, 21 ratios, without / with it: 7168 x 4096 115 / 80 (2 ratios 0.01 apart 75 / 76, weights of
            // one sign 112 / 125).  2048, 4096, 8192 and 14336 have a kernel of their own (fold_search.hip).  Not 3584, where few or
            // fine ratios lose (72 / 54, but 2 ratios 0.01 apart 47 / 55), nor shorter rows, for which the cells are too many (1792 42 /
            // 45, 1024 30 / 32, 512 34 / 38; 11 ratios 0.01 apart 35 / 54, 26 / 44, 29 / 63).  K = 32768 leaves no LDS beside the row.
            if constexpr (K == 7168 || K == 16384 || K == 28672) {
                if (const int q = counted_fraction(ex); q > 0)
                    return launch_search<K, NTS, true>(X, rows, ldx, pre, post_scale, Q, scale_out, ex, q, st);
            }
            return launch_search<K, NTS, false>(X, rows, ldx, pre, post_scale, Q, scale_out, ex, 0, st);
        }
    }
    constexpr auto kern = fwht_quant_ex_kernel<K, NT, F6>;
    if (lds > 40 * 1024) {
        hipError_t e = allow_dynamic_lds<kern>((int)lds);
        if (e != hipSuccess) return e;
    }
    const unsigned grid = F6 ? (unsigned)((rows + 63) / 64 * 64) : (unsigned)rows;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, st,
                       static_cast<const __half *>(X), ldx, rows, pre, clip, post_scale, Q, scale_out, ex);
    return hipGetLastError();
}

}  // namespace

// K = 4096: the two-pass workgroup-per-row kernel up to here, a wave per row beyond (see launch_fwht_quant)
constexpr int64_t kTwoPassMaxRows4096 = 3072;
constexpr int64_t kTwoPassMaxRows4096Heads = 1024;       // head-wise transform (see launch_fwht_quant_ex)

template <bool HAS_PRE, bool F6, bool STAGED = false, bool MASKED = false>
hipError_t launch_wave4096(const void *X, int64_t rows, int64_t ldx, const float *pre, float clip, float post_scale,
                           uint8_t *Q, float *scale_out, hipStream_t st,
                           const void *warm = nullptr, size_t warm_bytes = 0, uint32_t had_mask = 0xFFFFFFFFu)
{
    constexpr size_t lds = 4 * (4096 + (F6 ? 576 : 64)) * sizeof(float);
    const unsigned blocks = F6 ? (unsigned)((rows + 63) / 64 * 16) : (unsigned)((rows + 3) / 4);
    constexpr auto kern = fwht4096_wave_kernel<HAS_PRE, F6, STAGED, MASKED>;
    hipError_t e = allow_dynamic_lds<kern>((int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, st, static_cast<const __half *>(X), ldx, rows, pre, clip,
                       post_scale, Q, scale_out, warm_bytes >= 128 ? static_cast<const uint32_t *>(warm) : nullptr,
                       (int64_t)(warm_bytes / 128), had_mask);
    return hipGetLastError();
}

hipError_t launch_fwht_quant(const void *X, int64_t rows, int64_t K, int64_t ldx, const float *pre,
                             float clip, float post_scale, uint8_t *Q, float *scale_out, hipStream_t st, bool f6,
                             const void *warm, size_t warm_bytes)
{
    int pick = 0;
    if (int64_t f; tuned(kTuneFwht4096, f)) pick = (int)f;
    // One workgroup per row in two passes: at every row count for 2048, 8192 and 14336 (see fwht_two_pass.hip), for 4096
    // up to kTwoPassMaxRows4096 (every row count measured from 1 to 3072: 3.1 / 3.4 / 4.7 / 6.1 / 9.0 / 12.5 us for 1 /
    // 64 / 512 / 1024 / 2048 / 3072 rows against 3.5 / 3.7 / 5.3 / 6.8 / 9.5 / 13.4 for the general workgroup-per-row
    // kernel and 4.4 / 5.4 / 6.3 / 7.2 / 9.4 / 14.0 for a wave per row); a wave per row beyond (16384 rows: 52 against 57 us)
    if (K == 2048 || K == 8192 || K == 14336 || (K == 4096 && (pick == 5 || (pick == 0 && rows <= kTwoPassMaxRows4096))))
        return launch_fwht_two_pass(X, rows, K, ldx, pre, clip, post_scale, Q, scale_out, nullptr, 0, st, f6, warm, warm_bytes);
    if (K == 4096 && (pick == 0 || pick == 1 || pick == 3 || pick == 4)) {
        // factors through LDS (one copy per workgroup) unless the knob asks for per-wave vector loads (4)
        if (pre && pick != 4 && (reinterpret_cast<uintptr_t>(pre) & 15u) == 0 && ldx * 2 * rows < (int64_t)1 << 40)
            return f6 ? launch_wave4096<true, true, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes)
                      : launch_wave4096<true, false, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes);
        if (pre) return f6 ? launch_wave4096<true, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes)
                           : launch_wave4096<true, false>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes);
        return f6 ? launch_wave4096<false, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes)
                  : launch_wave4096<false, false>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes);
    }
    if (f6) {
#define SR_CASE(KK) case KK: return launch_one<KK, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, warm, warm_bytes);
        switch (K) {                                    // K % 128 == 0
            SR_CASE(128) SR_CASE(256) SR_CASE(512) SR_CASE(1024)
            SR_CASE(4096) SR_CASE(16384) SR_CASE(32768)
            SR_CASE(896) SR_CASE(1792) SR_CASE(3584) SR_CASE(7168) SR_CASE(28672)
            default: return hipErrorInvalidValue;
        }
#undef SR_CASE
    }
#define SR_CASE(KK) case KK: return launch_one<KK>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st);
    switch (K) {
        SR_CASE(64) SR_CASE(128) SR_CASE(256) SR_CASE(512) SR_CASE(1024)
        SR_CASE(4096) SR_CASE(16384) SR_CASE(32768)
        SR_CASE(448) SR_CASE(896) SR_CASE(1792) SR_CASE(3584) SR_CASE(7168) SR_CASE(28672)
        default: return hipErrorInvalidValue;
    }
#undef SR_CASE
}

hipError_t launch_fwht_quant_ex(const void *X, int64_t rows, int64_t K, int64_t ldx, const float *pre,
                                float clip, float post_scale, uint8_t *Q, float *scale_out,
                                const RowExtras &ex, hipStream_t st, bool f6)
{
    // head-wise transform: two passes with the unselected butterflies skipped (817 rows of 8192, 32 heads, across / within:
    // 12.9 / 11.5 -> 9.3 / 10.0 us against the general kernel, 1500 rows of 2048 9.8 -> 6.4); more than 1024 rows of 4096
    // by a wave per row.  There two passes would be faster too (2048 rows 9.6 / 10.0 -> 9.0 / 9.4 us, 8000 rows across
    // 26.2 -> 21.8), but add the values in another order (index bits 0..11 in turn; a wave per row does 0, 1, 2, 9, 10, 11
    // before 3..8): about one code in a million, on a rounding boundary, comes out one off.
    if (!ex.gate && !f6 && ex.n_grid == 0 && (K == 2048 || K == 4096 || K == 8192)) {
        // no search: the ratio "chosen" for every row is the fixed one (the kernel does not report it)
        if (ex.ratio_out) {
            hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st, ex.ratio_out, rows, clip);
            if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        }
        if (K == 4096 && rows > kTwoPassMaxRows4096Heads)
            return pre ? launch_wave4096<true, false, false, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, nullptr, 0, ex.had_mask)
                       : launch_wave4096<false, false, false, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, st, nullptr, 0, ex.had_mask);
        return launch_fwht_two_pass_heads(X, rows, K, ldx, pre, clip, post_scale, Q, scale_out, ex.had_mask, st);
    }
    if (ex.n_grid > 0 && !ex.gate && !f6 && (ex.had_mask == 0xFFFFFFFFu || !is_pow2(K))) {
        bool taken = false;
        const hipError_t e = launch_fold_search(X, rows, K, ldx, pre, post_scale, Q, scale_out, ex, st, taken);
        if (taken || e != hipSuccess) return e;
    }
    // the gate alone (the FFN down-projection input) goes through the plain kernels: fewer passes over the row
    // than the general kernel below (K = 14336, 2048 rows: 38 against 68 us)
    if (ex.gate && ex.n_grid == 0 && (ex.had_mask == 0xFFFFFFFFu || !is_pow2(K))) {
#define SR_CASE(KK)                                                                                                      \
    case KK:                                                                                                             \
        return f6 ? launch_one_gated<KK, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, ex.gate, ex.ldg, st)  \
                  : launch_one_gated<KK, false>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, ex.gate, ex.ldg, st);
        switch (K) {                                    // the FFN widths; other K take the general kernel
            case 2048: case 4096: case 8192: case 14336:
                return launch_fwht_two_pass(X, rows, K, ldx, pre, clip, post_scale, Q, scale_out, ex.gate, ex.ldg, st, f6, nullptr, 0);
            SR_CASE(1024) SR_CASE(16384)
            SR_CASE(3584) SR_CASE(7168) SR_CASE(28672)
            default: break;
        }
#undef SR_CASE
    }
    if (f6) {                                            // a gate row of the other K; nothing else asks for tiles
        if (!ex.gate || ex.n_grid > 0) return hipErrorInvalidValue;
#define SR_CASE(KK) case KK: return launch_one_ex<KK, true>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, ex, st);
        switch (K) {                                    // K % 128 == 0
            SR_CASE(128) SR_CASE(256) SR_CASE(512) SR_CASE(32768) SR_CASE(896) SR_CASE(1792)
            default: return hipErrorInvalidValue;
        }
#undef SR_CASE
    }
#define SR_CASE(KK) case KK: return launch_one_ex<KK>(X, rows, ldx, pre, clip, post_scale, Q, scale_out, ex, st);
    switch (K) {
        SR_CASE(64) SR_CASE(128) SR_CASE(256) SR_CASE(512) SR_CASE(1024) SR_CASE(2048)
        SR_CASE(4096) SR_CASE(8192) SR_CASE(16384) SR_CASE(32768)
        SR_CASE(448) SR_CASE(896) SR_CASE(1792) SR_CASE(3584) SR_CASE(7168) SR_CASE(14336) SR_CASE(28672)
        default: return hipErrorInvalidValue;
    }
#undef SR_CASE
}

}  // namespace sr
