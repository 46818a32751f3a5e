// INT4 x INT4 GEMM on the FP6 matrix pipe, compute-bound shapes.
//
//   acc[m][n] = sum_k cX[m][k] * cW[n][k],   Y = fp16(acc * dx[m] * dw[n])
//
// (Paper: the quantised forward pass of the linear layer; dequantisation per Eq. (1).)
//
// gfx950 has no 4-bit integer matrix instruction, and its int8 MFMA sustains ~3.5 POP/s on this
// chip (power).  The scaled-float MFMA family runs 6-bit floats at twice the int8 rate, and the
// 6-bit format E2M3 (sign, 2 exponent bits, 3 mantissa bits, bias 1) holds every INT4 code
// exactly: its first sixteen magnitudes -- the subnormals m/8 and the first binade 1 + m/8 --
// are the linear sequence 0, 1/8, ..., 15/8, so a code c is the 6-bit pattern
//     f6(c) = (c < 0 ? 32 : 0) | |c|            (value c / 8)
// and needs no arithmetic to build.  Products c_x c_w / 64 and their sums are integers / 64 below
// 2^24 / 64 for K < 262144, so the fp32 accumulation is exact in any order; measured on MI355X:
// v_mfma_f32_32x32x64_f8f6f4 reproduces the integer sums bit for bit (K = 14336, random codes and
// the all -8 worst case) and issues at 5.4 - 6.2 POP/s where the int8 MFMA reaches 3.3 - 3.7.
//
// The operands arrive already packed as 6-bit fields in the layout the MFMA wants ("f6 tiles",
// written by sr_pack_f6_tiles and by the activation quantiser), so the main loop has no vector-ALU
// work at all: LDS-DMA loads, LDS reads, MFMAs.
//
// f6 tiles of a code matrix [rows, K], K % 128 == 0, rows padded to a multiple of 8:
//   block (R, C) = rows 8R .. 8R+7 x codes 128C .. 128C+127, 768 bytes at ((C * rows/8) + R) * 768
//   (chunk-major: the blocks of all rows for one 128-code chunk are contiguous, so one stage of a tile is
//   two contiguous runs -- BM * 96 bytes of X and BN * 96 bytes of W -- copied by whole-KB LDS-DMA loads).
//   Inside a block, piece (r, t, g) = the 32 codes k = 128C + 64t + 32g + j (j = 0..31) of row
//   8R + r, code j in bits [6j, 6j+6) of a 24-byte little-endian string -- exactly the operand
//   of lane (row, k half g) of MFMA step t.  Its first 16 bytes live at
//       256 t + 128 (g ^ (R & 1)) + 16 r
//   and its last 8 bytes at
//       512 + 128 (g ^ (R & 1)) + 16 r + 8 t
//   i.e. the tails of the two steps share one 16-byte slot of the same (g, r) pattern as the first parts; a
//   32-row fragment (four blocks) then touches every LDS bank once per read.  The compiler reads each step's
//   half of the slot with 8-byte reads paired over two fragments (ds_read2st64_b64).  Measured in one process
//   against the first layout (tails in separate, XOR-swizzled 8-byte slots): M = 2048, N = 14336, K = 4096
//   69.8 -> 65.8 us, 4096 x 4096 x 14336 116.7 -> 108.1 us; forcing whole 16-byte tail reads (ds_read_b128,
//   the other half kept in registers for the next step) was 1 - 5 % slower than leaving the split to the compiler.
//   (The 12-byte form of the LDS-DMA load leaves a 4-byte hole after every lane's data in LDS -- measured -- so
//   stages are copied with the 16-byte form, 1 KB per instruction.)
//
// Kernel structure: persistent workgroups, tile BM x BN, ring of SLOTS stages of 128 codes, one
// barrier per stage, two MFMA steps (64 codes) per stage with the fragment reads of the next
// step issued under the MFMAs of the current one; transposing epilogue shared with the int8
// kernel; scales of a tile fetched by LDS-DMA at the start of the tile.
#include "sr_common.h"
#include "gemm_common.h"
#include "gemm_rules.h"

#include <type_traits>

namespace sr {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int BLK = 768;     // bytes of one block (8 rows x 128 codes x 6 bits)

// 64 lanes x 4 bytes -> LDS bytes [lds, lds + 256)
__device__ __forceinline__ void dma4(const void *base, uint32_t lane_off, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(lane_off), "s"(base)
                 : "memory", "m0");
}

// The work of one workgroup: tiles v0, v0 + vstep, ... of the tile grid tiles_m x tiles_n.  CG = MFMA column tiles staged at a time by the epilogue.
// WARM: the workgroup has one wave more than the tile needs.  That wave computes nothing: it reads one word of
// every 128-byte line of the workgroup's share of [warm, warm + 128 warm_lines), a few lines per K stage, so that
// the memory-side cache holds that region when the next kernel asks for it -- the matrix waves are short of L2
// delivery and LDS bandwidth, not of HBM bandwidth, and cannot issue such loads themselves (a wave's loads
// complete in order: a slow load from HBM between the LDS-DMA loads would hold up their counted completion).
// The extra wave joins every barrier of the workgroup, so its loop mirrors the barrier count of the tile loop.
// (Also built and measured for the 256 x 256 configuration, which has no registers for a ninth wave: the
// workgroups that run out of tiles before the last round reading the region instead.  With the 12.6 MB of the
// benchmark's N = 4096 weights behind its N = 14336 launch the step got 2 % slower, not faster; dropped.)
// LIVE < BM / WGM / 32 or SPLIT: a tile has only its first row_step <= BM rows (a multiple of 16), and this wave multiplies only
// LIVE of its fragments of 32 rows (see gemm_f6_rows_kernel).
template <int BM, int BN, int WGM, int WGN, int SLOTS, int CG, bool WARM = false, bool SPLIT = false, int LIVE = BM / WGM / 32>
__device__ __forceinline__ void f6_tiles(
    const uint8_t *__restrict__ X6, const float *__restrict__ xs, const uint8_t *__restrict__ W6,
    const float *__restrict__ ws, const int M, const int N, const int K, void *__restrict__ Yv, const int64_t ldy,
    const int out_i32, const int tiles_m, const int tiles_n, const int xcd_m, const int v0,
    const int vstep, const int row_step, const uint32_t *__restrict__ warm = nullptr, const int64_t warm_lines = 0)
{
    constexpr int NWAVE = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;      // wave tile
    constexpr int FM = LIVE, FN = WN / 32;           // 32 x 32 MFMA tiles per wave
    constexpr int X_BYTES = BM / 8 * BLK, STAGE_BYTES = (BM + BN) / 8 * BLK;
    // 1 KB LDS-DMA instructions per stage: NXI for the X run, NWI for the W run; every wave issues XI + WI of
    // them -- where the count does not divide by the waves, the last ones wrap around and copy a KB a second
    // time (same data to the same place), so that all waves keep the same number of loads in flight
    constexpr int NXI = X_BYTES / 1024, NWI = (STAGE_BYTES - X_BYTES) / 1024;
    constexpr int XI = (NXI + NWAVE - 1) / NWAVE, WI = (NWI + NWAVE - 1) / NWAVE;
    constexpr int RPW = XI + WI;
    constexpr int SCALE_OFF = SLOTS * STAGE_BYTES;   // two areas of BM + BN floats behind the ring
    constexpr int NSC = (BM + BN) / 64;              // scale DMA instructions per tile
    static_assert(X_BYTES % 1024 == 0 && STAGE_BYTES % 1024 == 0 && WM % 32 == 0 && WN % 32 == 0 && BM % 64 == 0 &&
                      BN % 64 == 0 && SLOTS >= 2 && SLOTS * RPW < 64, "tile");

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // SPLIT: the two waves of a SIMD (w, w + 4) share its row of fewer fragments
    const int wm = SPLIT ? wave / WGN : wave % WGM, wn = SPLIT ? wave % WGN : wave / WGM;
    const int nc = K >> 7;                           // 128-code chunks per row = stages
    if constexpr (WARM) {
        if (wave == NWAVE) {
            // load instruction j of this wave touches lines (j * vstep + v0) * 64 + lane: the workgroups of the
            // launch sweep the region front to back together
            const int64_t per_wg = (warm_lines + (int64_t)vstep * 64 - 1) / ((int64_t)vstep * 64);   // instructions of this wave
            int my_tiles = 0;
            while (tile_exists(v0 + my_tiles * vstep, tiles_m, tiles_n, xcd_m)) ++my_tiles;
            if (my_tiles == 0) return;
            // spread evenly over the K stages of this workgroup's tiles (measured inside the benchmark's step, 44 MB
            // behind the M = 2048, N = 4096 GEMM: all loads up front costs the step 2.5 % against one per stage;
            // non-temporal loads are not kept by the memory-side cache; the scope bits make no difference)
            const int per_stage = (int)((per_wg + (int64_t)my_tiles * nc - 1) / ((int64_t)my_tiles * nc));
            int64_t l = (int64_t)v0 * 64 + lane;
            uint32_t word = 0;
            for (int tile = 0; tile < my_tiles; ++tile) {
                barrier_nofence();
                for (int s = 0; s < nc; ++s) {
                    for (int i = 0; i < per_stage; ++i) {
                        if (l < warm_lines) asm volatile("global_load_dword %0, %1, off" : "=v"(word) : "v"(warm + l * 32) : "memory");
                        l += (int64_t)vstep * 64;
                    }
                    barrier_nofence();
                }
                barrier_nofence();
                if (tile + 1 < my_tiles) barrier_nofence();
            }
            wait_vmcnt<0>();
            asm volatile("" ::"v"(word));
            return;
        }
    }
    const uint32_t cx_bytes = (uint32_t)((M + 7) >> 3) * BLK, cw_bytes = (uint32_t)((N + 7) >> 3) * BLK;   // one chunk of X / W

    // ---- DMA sources: X instruction q copies bytes [1024 q, 1024 q + 1024) of the stage's X run, W instruction q
    // of its W run; a lane past the end of the operand re-reads the last 16 bytes
    uint32_t goff[RPW], ldst[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i)
        ldst[i] = i < XI ? (uint32_t)((wave + NWAVE * i) % NXI) * 1024 : X_BYTES + (uint32_t)((wave + NWAVE * (i - XI)) % NWI) * 1024;
    auto set_sources = [&](int m0, int n0) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            uint32_t off;
            if (i < XI) { off = (uint32_t)(m0 >> 3) * BLK + ldst[i] + lane * 16; off = off < cx_bytes ? off : cx_bytes - 16; }
            else { off = (uint32_t)(n0 >> 3) * BLK + (ldst[i] - X_BYTES) + lane * 16; off = off < cw_bytes ? off : cw_bytes - 16; }
            goff[i] = off;
        }
    };
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    auto dma_one = [&](int idx, int s, int slot) {   // instruction idx of this wave, stage s -> ring slot
        dma16((idx < XI ? X6 + (int64_t)s * cx_bytes : W6 + (int64_t)s * cw_bytes), goff[idx],
              smem_base + (uint32_t)slot * STAGE_BYTES + ldst[idx]);
    };
    auto issue = [&](int s, int slot) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) dma_one(i, s, slot);
    };
    // scales of a tile: floats [0, BM) = token scales, [BM, BM + BN) = channel scales, 64 per instruction
    auto issue_scales = [&](int m0, int n0, int area) {
#pragma unroll
        for (int k = 0; k < (NSC + NWAVE - 1) / NWAVE; ++k) {
            const int idx = wave + k * NWAVE;        // wave-uniform
            if (idx < NSC) {
                const int f = idx * 64 + lane;
                const bool is_x = idx < BM / 64;
                int e = is_x ? m0 + f : n0 + f - BM;
                const int last = is_x ? M - 1 : N - 1;
                e = e < last ? e : last;
                const uint32_t dst = smem_base + SCALE_OFF + (uint32_t)area * (BM + BN) * 4 + (uint32_t)idx * 256;
                dma4(is_x ? xs : ws, (uint32_t)e * 4u, (uint32_t)__builtin_amdgcn_readfirstlane((int)dst));
            }
        }
    };

    // ---- fragment addresses: lane (r = l & 31, g = l >> 5) reads row r of a 32-row fragment, k half g
    const int fr = lane & 31, fg = lane >> 5;
    const int rq = fr >> 3;                          // block of the fragment (= R & 3: fragments start at multiples of 32 rows)
    const uint32_t a16 = rq * BLK + ((fg ^ (rq & 1)) << 7) + ((fr & 7) << 4);   // step 0; step 1 at + 256; tails at + 512
    const uint32_t xfrag = (wm * WM / 8) * BLK, wfrag = X_BYTES + (wn * WN / 8) * BLK;

    struct Frags { v8i x[FM]; v8i w[FN]; };
    uint2 tail1[FM + FN];                            // tails of step 1, read together with those of step 0
    // fragment q of a stage, step t: step 0 also fetches the 16 bytes holding both tails.  The W fragments come
    // first and the MFMAs below walk the X fragments in the outer loop, so that the fragments read last in a step
    // are the ones the next step needs last (with X first, the first MFMA of a step waited for the last read).
    auto read_q = [&](Frags &f, int q, uint32_t sbase, int t) {
        const uint32_t base = sbase + (q < FN ? wfrag + q * 4 * BLK : xfrag + (q - FN) * 4 * BLK) + a16;
        v8i &d = q < FN ? f.w[q < FN ? q : 0] : f.x[q < FN ? 0 : q - FN];
        const uint4 lo = *reinterpret_cast<const uint4 *>(smem + base + t * 256);
        d[0] = (int)lo.x; d[1] = (int)lo.y; d[2] = (int)lo.z; d[3] = (int)lo.w;
        if (t == 0) {
            const uint4 tl = *reinterpret_cast<const uint4 *>(smem + base + 512);
            d[4] = (int)tl.x; d[5] = (int)tl.y;
            tail1[q] = make_uint2(tl.z, tl.w);
        } else {
            d[4] = (int)tail1[q].x; d[5] = (int)tail1[q].y;
        }
    };

    v16f acc[FN][FM];

    // ---- one MFMA step (64 codes): the FM * FN MFMAs on `cur`, the reads of the next step's FM + FN fragments
    // into `nxt` and a share of the DMA of a later stage, cut into regions of [2 fragment reads, a slice of the
    // MFMAs, some DMA instructions] so that no memory instruction queue sees a burst.
    // regions per step: fragments read in pairs -- measured against 1, 2 and FM + FN regions (M = 2048, N = 14336,
    // K = 4096: 68.9, 63.1, 65.7 us against 62.0 us)
    constexpr int NREG = (FM + FN + 1) / 2;
    constexpr int FPRG = (FM + FN + NREG - 1) / NREG;   // fragments read per region
    constexpr int NM = FM * FN;                      // MFMAs per step
    // (Tried: the two waves of a SIMD issuing their DMA in different steps, so that they are not held up at the
    // same moments -- 1 - 2 % slower.)
    constexpr int HALF = SLOTS == 2 ? RPW : (RPW + 1) / 2;      // DMA instructions issued in the step after the barrier
    auto step = [&](auto PART, const Frags &cur, Frags &nxt, uint32_t rbase, int t, int dstage, int dslot) {
        constexpr int part = decltype(PART)::value;             // 0: step after the barrier, 1: step before it
        constexpr int dlo = part == 0 ? 0 : HALF, dhi = part == 0 ? HALF : RPW;
        constexpr int DPR = (dhi - dlo + NREG - 1) / NREG;
#pragma unroll
        for (int r = 0; r < NREG; ++r) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = r * FPRG; q < (r + 1) * FPRG && q < FM + FN; ++q) read_q(nxt, q, rbase, t);
            const int mlo = r * NM / NREG, mhi = (r + 1) * NM / NREG;
#pragma unroll
            for (int m = mlo; m < mhi; ++m) {
                const int j = m / FN, i = m % FN;
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cur.w[i], cur.x[j], acc[i][j], 2, 2, 0, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int idx = dlo + r * DPR; idx < dlo + (r + 1) * DPR && idx < dhi; ++idx) dma_one(idx, dstage, dslot);
        }
    };
    constexpr std::integral_constant<int, 0> AFTER{};
    constexpr std::integral_constant<int, 1> BEFORE{};

    // epilogue staging: one piece = 32 tokens x CG * 32 channels of fp16 per wave, in the last ring slot
    constexpr int PIECE = 32 * (CG * 64 + 16);
    static_assert(NWAVE * PIECE <= STAGE_BYTES, "epilogue staging must fit one ring slot");

    int v = v0;
    int m0, n0;
    if (!tile_exists(v, tiles_m, tiles_n, xcd_m)) return;      // the whole workgroup
    tile_origin(v, tiles_m, tiles_n, xcd_m, SPLIT ? row_step : BM, BN, m0, n0);
    set_sources(m0, n0);
    // order of a wave's loads at the start of every tile: stage 0, scales, stages 1 .. SLOTS-2, first part of
    // stage SLOTS-1 (its second part is issued by the first step of the loop)
    int area = 0;
    issue(0, 0);
    issue_scales(m0, n0, area);
#pragma unroll
    for (int q = 1; q < SLOTS - 1; ++q) issue(q < nc ? q : nc - 1, q);
#pragma unroll
    for (int i = 0; i < HALF; ++i) dma_one(i, SLOTS - 1 < nc ? SLOTS - 1 : nc - 1, SLOTS - 1);
    for (;;) {
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

        // Stage 0 (and the scales) have landed once at most (SLOTS-2) RPW + HALF of this wave's memory operations
        // are outstanding: loads complete in order among themselves and that many loads are younger, so an
        // unfinished older load would leave more outstanding -- however many stores of the previous tile are
        // still on their way (stores and loads may overtake each other).
        wait_vmcnt<(SLOTS - 2) * RPW + HALF>();
        barrier_nofence();
        Frags fa, fb;                                // fragments of step 0 / step 1 of a stage
#pragma unroll
        for (int q = 0; q < FM + FN; ++q) read_q(fa, q, 0, 0);
        int slot = 0;
        // Every stage runs the same branch-free body.  Past the end of K the pipeline keeps reading (stale,
        // in-bounds) LDS and re-fetching the last stage; those fragments are never multiplied.
        for (int s = 0; s < nc; ++s) {
            const int nslot = slot == SLOTS - 1 ? 0 : slot + 1, pslot = slot == 0 ? SLOTS - 1 : slot - 1;
            const int sa = s + SLOTS - 1 < nc ? s + SLOTS - 1 : nc - 1, sb = s + SLOTS < nc ? s + SLOTS : nc - 1;
            // step 0 of stage s; reads step 1; second part of the DMA of stage s+SLOTS-1 -> slot of stage s-1
            step(BEFORE, fa, fb, (uint32_t)slot * STAGE_BYTES, 1, sa, pslot);
            // stage s+1 must have landed (the SLOTS-2 younger stages may stay in flight), and every wave's
            // reads of stage s must have returned: its slot takes stage s+SLOTS from here on
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((SLOTS - 2) * RPW) : "memory");
            barrier_nofence();
            // step 1 of stage s; reads step 0 of stage s+1; first part of the DMA of stage s+SLOTS
            step(AFTER, fb, fa, (uint32_t)nslot * STAGE_BYTES, 0, sb, slot);
            slot = nslot;
        }

        // ---- tile boundary
        const int vn = v + vstep;
        const bool more = tile_exists(vn, tiles_m, tiles_n, xcd_m);
        wait_vmcnt<0>();                             // no LDS-DMA write is in flight any more ...
        barrier_nofence();                           // ... and all waves are done reading fragments
        int m1 = 0, n1 = 0;
        if (more) {                                  // the next tile's first stages fly during the epilogue
            tile_origin(vn, tiles_m, tiles_n, xcd_m, SPLIT ? row_step : BM, BN, m1, n1);
            set_sources(m1, n1);
            issue(0, 0);
            issue_scales(m1, n1, area ^ 1);
#pragma unroll
            for (int q = 1; q < SLOTS - 1; ++q) issue(q < nc ? q : nc - 1, q);
        }
        {
            const float *sc = reinterpret_cast<const float *>(smem + SCALE_OFF) + area * (BM + BN);
            float sx[FM];
            float4 sw[FN][4];
#pragma unroll
            for (int j = 0; j < FM; ++j) sx[j] = sc[wm * WM + j * 32 + fr] * 64.f;      // both operands carried a factor 1/8
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    sw[i][q] = *reinterpret_cast<const float4 *>(sc + BM + wn * WN + i * 32 + q * 8 + fg * 4);
            // (rows past row_step belong to the next tile)
            const int end = SPLIT && m0 + row_step < M ? m0 + row_step : M;
            store_wave_tile<FM, FN, CG>(acc, smem + (SLOTS - 1) * STAGE_BYTES + wave * PIECE, lane, m0 + wm * WM, n0 + wn * WN,
                                    end, N, sx, sw, Yv, ldy, out_i32);
        }
        if (!more) break;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier_nofence();                           // every wave has read its staging back: the last slot is free
#pragma unroll
        for (int i = 0; i < HALF; ++i) dma_one(i, SLOTS - 1 < nc ? SLOTS - 1 : nc - 1, SLOTS - 1);
        v = vn;
        m0 = m1;
        n0 = n1;
        area ^= 1;
    }
    wait_vmcnt<0>();
}

constexpr int f6_lds_bytes(int BM, int BN, int SLOTS) { return SLOTS * (BM + BN) / 8 * BLK + 2 * (BM + BN) * 4 + 256; }   // ring, two scale areas, slack

// MFMA column tiles the epilogue stages at a time: a wave's whole width where the staging of all waves fits one slot
constexpr int f6_staged_columns(int BM, int BN, int waves, int WGN)
{
    return waves * 32 * (BN / WGN * 2 + 16) <= (BM + BN) / 8 * BLK ? BN / WGN / 32 : 1;
}

template <int BM, int BN, int WGM, int WGN, int SLOTS, int WG_PER_CU>
__global__ __launch_bounds__(WGM * WGN * 64, WGM * WGN * WG_PER_CU / 4) void gemm_f6_kernel(
    const uint8_t *__restrict__ X6, const float *__restrict__ xs, const uint8_t *__restrict__ W6,
    const float *__restrict__ ws, int M, int N, int K, void *__restrict__ Yv, int64_t ldy, int out_i32,
    int tiles_m, int tiles_n, int xcd_m)
{
    f6_tiles<BM, BN, WGM, WGN, SLOTS, f6_staged_columns(BM, BN, WGM * WGN, WGN)>(X6, xs, W6, ws, M, N, K, Yv, ldy, out_i32, tiles_m, tiles_n, xcd_m,
                                                     (int)blockIdx.x, (int)gridDim.x, BM);
}

// The same with a ninth wave that warms the memory-side cache (one workgroup per CU: three waves then share the
// first SIMD, which the register budget of the 64 x 64 wave tile allows and that of the 128 x 64 one does not).
template <int BM, int BN, int WGM, int WGN, int SLOTS>
__global__ __launch_bounds__((WGM * WGN + 1) * 64) void gemm_f6_warm_kernel(
    const uint8_t *__restrict__ X6, const float *__restrict__ xs, const uint8_t *__restrict__ W6,
    const float *__restrict__ ws, int M, int N, int K, void *__restrict__ Yv, int64_t ldy, int out_i32,
    int tiles_m, int tiles_n, int xcd_m, const uint32_t *__restrict__ warm, int64_t warm_lines)
{
    f6_tiles<BM, BN, WGM, WGN, SLOTS, BN / WGN / 32, true>(X6, xs, W6, ws, M, N, K, Yv, ldy, out_i32, tiles_m, tiles_n, xcd_m,
                                                           (int)blockIdx.x, (int)gridDim.x, BM, warm, warm_lines);
}

// The same for row counts that leave the last row of tiles short: all rows of tiles get row_step rows, and the second row of
// waves multiplies the fragments of 32 rows that are there (LIVE, one copy of the loop per count; the barriers are the same).
// Its waves share their SIMDs with those of the first row, so every SIMD has the fewer products, and the LDS delivers fewer
// fragments (a stage of 256 x 256 tiles moves 196 KB through it: with 128 B per clock that bounds a launch of one round).
// Against padding the last row of tiles: 520 x 14336 x 4096 (six of eight fragments) 24.9 -> 22.9 us, 777 x 14336 x 4096 (seven)
// 30.3 -> 29.3, 616 x 26992 x 4096 58.1 -> 54.2.
template <int BM, int BN, int WGN, int SLOTS>
__global__ __launch_bounds__(2 * WGN * 64, WGN / 2) void gemm_f6_rows_kernel(
    const uint8_t *__restrict__ X6, const float *__restrict__ xs, const uint8_t *__restrict__ W6,
    const float *__restrict__ ws, int M, int N, int K, void *__restrict__ Yv, int64_t ldy, int out_i32,
    int tiles_m, int tiles_n, int xcd_m, int row_step)
{
    static_assert(WGN == 4, "waves w and w + 4 share a SIMD");
    constexpr int WM = BM / 2, CG = f6_staged_columns(BM, BN, 2 * WGN, WGN);
#define SR_ROWS(L)                                                                                                            \
    f6_tiles<BM, BN, 2, WGN, SLOTS, CG, false, true, L>(X6, xs, W6, ws, M, N, K, Yv, ldy, out_i32, tiles_m, tiles_n, xcd_m,    \
                                                        (int)blockIdx.x, (int)gridDim.x, row_step)
    constexpr int FULL = WM / 32, THREE = FULL < 3 ? FULL : 3, TWO = FULL < 2 ? FULL : 2;
    const bool second = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) >= WGN;
    const int live = second ? (row_step - WM + 31) / 32 : FULL;
    if (live >= FULL) SR_ROWS(FULL);
    else if (live == THREE) SR_ROWS(THREE);
    else if (live == TWO) SR_ROWS(TWO);
    else SR_ROWS(1);
#undef SR_ROWS
}

template <int BM, int BN, int WGM, int WGN, int SLOTS, int WG_PER_CU, bool CAN_WARM = false>
hipError_t launch_f6(const uint8_t *X6, const float *xs, const uint8_t *W6, const float *ws, int64_t M, int64_t N,
                     int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st, const void *warm = nullptr,
                     size_t warm_bytes = 0)
{
    constexpr auto kern = gemm_f6_kernel<BM, BN, WGM, WGN, SLOTS, WG_PER_CU>;
    constexpr int lds = f6_lds_bytes(BM, BN, SLOTS);
    static_assert(lds * WG_PER_CU <= 160 * 1024, "LDS");
    if (lds > 48 * 1024) {
        hipError_t e = allow_dynamic_lds<kern>(lds);
        if (e != hipSuccess) return e;
    }
    bool warms = false;
    if constexpr (CAN_WARM) {
        static_assert(WG_PER_CU == 1, "the extra wave is budgeted for one workgroup per CU");
        warms = warm && warm_bytes >= 128;
        if (int64_t w; tuned(kTuneGemmWarm, w) && w == 0) warms = false;
        if (warms && lds > 48 * 1024) {
            hipError_t e = allow_dynamic_lds<gemm_f6_warm_kernel<BM, BN, WGM, WGN, SLOTS>>(lds);
            if (e != hipSuccess) return e;
        }
    }
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((N + BN - 1) / BN);
    const int row_step = WGM == 2 && WGN == 4 ? f6_row_step(M, BM) : BM;
    int xcd_m = choose_xcd_split(tiles_m, tiles_n, row_step, BN);
    // (128 x 64 tiles: the plain order is 2 - 5 % ahead of the runs, 749 x 1984 x 8192 18.0 against 18.5 us)
    if (BN == 64 && xcd_m == kXcdRuns) xcd_m = 0;
    if (int64_t f; tuned(kTuneGemmXcdM, f)) {                         // force the split (0 = none)
        if (f == 0 || ((f == 1 || f == 2 || f == 4 || f == 8) && tiles_m % f == 0 && tiles_n % (8 / f) == 0)) xcd_m = (int)f;
    }
    int64_t grid = (int64_t)compute_units() * WG_PER_CU;
    if (int64_t g; tuned(kTuneGemmGrid, g) && g > 0) grid = g / 8 * 8;
    if (grid < 8) grid = 8;
    grid = tile_workgroups(grid, (int64_t)tiles_m * tiles_n, xcd_m);
    // the raw int32 output takes no scales (they may be NULL): the kernel still fetches M and N floats it then
    // ignores, from the start of the operand arrays (at least 96 M and 96 N bytes, 16-byte aligned)
    if (out_i32) {
        xs = reinterpret_cast<const float *>(X6);
        ws = reinterpret_cast<const float *>(W6);
    }
    if constexpr (CAN_WARM) {
        if (warms) {
            hipLaunchKernelGGL((gemm_f6_warm_kernel<BM, BN, WGM, WGN, SLOTS>), dim3((unsigned)grid), dim3((WGM * WGN + 1) * 64),
                               lds, st, X6, xs, W6, ws, (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n, xcd_m,
                               static_cast<const uint32_t *>(warm), (int64_t)(warm_bytes / 128));
            return hipGetLastError();
        }
    }
    if constexpr (WGM == 2 && WGN == 4) {
        if (row_step < BM) {
            static_assert(lds > 48 * 1024 && WG_PER_CU == 1);
            hipError_t e = allow_dynamic_lds<gemm_f6_rows_kernel<BM, BN, WGN, SLOTS>>(lds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((gemm_f6_rows_kernel<BM, BN, WGN, SLOTS>), dim3((unsigned)grid), dim3(2 * WGN * 64), lds, st, X6, xs,
                               W6, ws, (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n, xcd_m, row_step);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WGM * WGN * 64), lds, st, X6, xs, W6, ws,
                       (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n, xcd_m);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Repacking of canonical INT4 codes (two per byte along K) into f6 tiles.  One thread per piece
// (row, 128-code chunk, step t, half g): 16 bytes in, 24 bytes out.  Rows >= rows (padding of
// the last block) are written as zeros.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_f6_kernel(const uint8_t *__restrict__ Q4, int rows, int K,
                                                      uint8_t *__restrict__ T6, int64_t pieces)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= pieces) return;
    // piece index: [C][R][t][g][r] with r fastest, so that the 16-byte parts of neighbouring threads are neighbours
    const int r = (int)(p & 7), g = (int)((p >> 3) & 1), t = (int)((p >> 4) & 1);
    const int64_t bc = p >> 5;                      // C * row_blocks + R = index of the block in memory
    const int64_t rb = ((int64_t)rows + 7) >> 3;
    const int C = (int)(bc / rb);
    const int64_t R = bc % rb;
    const int64_t row = R * 8 + r;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if (row < rows) {
        const uint4 q = *reinterpret_cast<const uint4 *>(Q4 + row * (int64_t)(K >> 1) + C * 64 + t * 32 + g * 16);
        w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
    }
    uint32_t o[6] = {0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const uint32_t nib = (w[j >> 3] >> ((j & 7) * 4)) & 15u;
        const uint32_t f = nib < 8u ? nib : (32u | (16u - nib));          // sign-magnitude 6-bit field
        const int bit = 6 * j;
        o[bit >> 5] |= f << (bit & 31);
        if ((bit & 31) > 26) o[(bit >> 5) + 1] |= f >> (32 - (bit & 31));
    }
    uint8_t *blk = T6 + bc * BLK;
    const int Rl = (int)(R & 3);
    *reinterpret_cast<uint4 *>(blk + 256 * t + 128 * (g ^ (Rl & 1)) + 16 * r) = make_uint4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<uint2 *>(blk + 512 + 128 * (g ^ (Rl & 1)) + 16 * r + 8 * t) = make_uint2(o[4], o[5]);
}

}  // namespace

hipError_t launch_pack_f6(const uint8_t *Q4, int64_t rows, int64_t K, uint8_t *T6, hipStream_t st)
{
    const int64_t pieces = ((rows + 7) / 8) * 8 * (K / 128) * 4;
    hipLaunchKernelGGL(pack_f6_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, Q4, (int)rows, (int)K, T6,
                       pieces);
    return hipGetLastError();
}

hipError_t launch_gemm_f6(const uint8_t *X6, const float *xs, const uint8_t *W6, const float *ws, int64_t M, int64_t N,
                          int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st, const void *warm, size_t warm_bytes)
{
    const GemmShape shape = f6_shape(M, N, K, compute_units());
    const GemmConfig *best = f6_config(shape), *hinted = &kF6Configs[2];
    int id = best->id;
    // the hint is worth several microseconds to the next launch (44 MB read ahead save it 4 us of 67)
    if (warm && warm_bytes >= ((size_t)1 << 20) && gemm_cost(*hinted, shape) <= 1.15f * gemm_cost(*best, shape)) id = hinted->id;
    // the tile knob selects a configuration by number; not set or unknown = the rule above
    if (int64_t t; tuned(kTuneGemmTile, t)) {
        for (const GemmConfig &c : kF6Configs)
            if (c.id == t) id = (int)t;
    }
    switch (id) {
        case 61: return launch_f6<256, 256, 2, 4, 3, 1>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st);
        case 65: return launch_f6<256, 128, 4, 2, 4, 1, true>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st, warm, warm_bytes);
        case 67: return launch_f6<128, 128, 2, 2, 3, 2>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st);
        case 68: return launch_f6<128, 256, 2, 4, 4, 1>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st);
        case 69: return launch_f6<128, 64, 2, 2, 4, 2>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st);
        case 72: return launch_f6<192, 256, 2, 4, 3, 1>(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st);
        default: return launch_gemm_f6_stream(X6, xs, W6, ws, M, N, K, Y, ldy, out_i32, st, id / 1000, id % 1000);
    }
}

}  // namespace sr
