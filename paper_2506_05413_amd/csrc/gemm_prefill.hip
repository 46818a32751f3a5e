// INT4 x INT4 GEMM, INT32 accumulation, dequantising epilogue -- compute-bound shapes (M > 16).
//
//   acc[m][n] = sum_k cX[m][k] * cW[n][k],   Y = fp16(acc * dx[m] * dw[n])
//
// (Paper: the quantised forward pass of the linear layer; dequantisation per Eq. (1).)
//
// gfx950 has no 4-bit matrix instruction, so the packed codes are widened to int8 in
// registers and fed to the int8 MFMA.  A nibble is sign-extended for free by leaving it in
// the HIGH half of its byte:
//     lo = (w << 4) & 0xF0F0F0F0      (codes 0,2,4,6 of the dword, each x16)
//     hi =  w       & 0xF0F0F0F0      (codes 1,3,5,7 of the dword, each x16)
// Both operands carry the factor 16, so the accumulator holds 256 * acc exactly
// (256 * 64 * K < 2^31 for K < 131072); the factor leaves by an arithmetic shift (int32
// output) or inside the row scale (fp16 output).  A dot product does not care in which
// order k is visited: X and W only have to permute k identically, and they do because both
// are widened by the same three instructions from the same byte offsets.
//
// What the main kernel is built around (all measured on MI355X):
//  * v_mfma_i32_32x32x32_i8 (8 passes, 32 cycles of the matrix pipe) lets vector-ALU instructions
//    of the same wave issue underneath it; v_mfma_i32_16x16x64_i8 (4 passes) does not.  The
//    widening (4.5 - 6 ALU instructions per MFMA) therefore costs little MFMA time.
//  * Memory instructions hold up the wave that issues them (an LDS-DMA load ~50 cycles, a
//    ds_read_b128 ~25), and with one wave per SIMD a held-up wave idles the matrix pipe: timed
//    per stage, DMA and fragment reads ADD to the MFMA time instead of hiding under it.  Hence
//    (a) two waves per SIMD -- eight waves on a 256 x 128 tile, or two four-wave workgroups of
//    128 x 128 per CU -- and (b) no bursts: a 64-code sub-step is cut into regions of
//    [2 fragment reads, 4-5 MFMAs with the widening of 2 fragments underneath, 1-2 DMA
//    instructions], the DMA of a stage being spread over the sub-steps after the barrier that
//    frees its ring slot.
//  * Both operands stay packed (4 bit) all the way into LDS, and every global access fetches
//    whole 128-byte lines (256 codes per row per stage) -- half-line fetches were re-fetched
//    from L2 each time, an int8 copy of X doubled its traffic and was slower.
//  * Global -> LDS copies use the LDS-DMA form of the global load (no staging registers) into a
//    ring of stages of 256 codes (two; four where two sets of waves share a tile, KS = 2); one
//    barrier per stage; per 64 codes a register-level software pipeline (LDS reads for t+2,
//    widening for t+1, MFMAs for t).
//  * The epilogue transposes each wave tile through the idle LDS ring and stores whole rows:
//    8-byte stores scattered over 32 rows per instruction cost 14 us per tile, this costs ~5.
//  * LDS rows are XOR-swizzled in 16-byte chunks (applied on the global side of the DMA,
//    which fills LDS linearly): ds_read_b128 of a fragment runs at the full LDS rate
//    (240 B/clk/CU measured with eight waves; one wave alone reaches 33 B/clk).
//  * MFMA operand roles are swapped (A = weight rows, B = token rows): a lane then owns 4
//    consecutive output channels of one token per accumulator quad = one 8-byte store.
//  * Tried and dropped: three ring slots for 256 x 128 tiles and for two workgroups of 128 x 128
//    per CU (weights in the memory-side cache: their latency is hidden by two slots), dedicated DMA-issuing waves (1, 2 or 4 per workgroup: slower, a wave issues DMA too slowly).
//
// K % 256 != 0 (and any K % 64 == 0) runs on a simpler register-staged kernel further down.
#include "sr_common.h"
#include "gemm_common.h"
#include "gemm_rules.h"

#include <hip/hip_fp16.h>
#include <type_traits>

namespace sr {
namespace {

constexpr unsigned HM = 0xF0F0F0F0u;

constexpr int ROWB = 128;  // packed bytes per row per stage (256 codes = one 128-byte line)

// Persistent workgroups: a workgroup walks over tiles v = blockIdx.x, blockIdx.x + gridDim.x, ... and keeps the
// memory pipeline going across the tile boundary -- the first stage of the next tile is in flight while the
// finished tile is dequantised, transposed and stored, and the stores (fire and forget) drain under the next
// tile's MFMAs (KS = 2: the first two stages, while slots 2 and 3 hold the sums that change hands).  One launch of <= (CUs x workgroups per CU) workgroups instead of one workgroup per tile.
//
// KS = 2: two sets of waves share a tile, each multiplying half of every stage (the 64-code sub-steps 2 kw, 2 kw + 1),
// and add their sums through LDS at the end, each finishing half of the channels.
//
// RUNS: the grid of tiles is cut into runs (kXcdRuns), of which the kernel for grids that divide knows nothing: one kernel for
// both took registers and start-up from the latter (600 x 6144 x 4096 18.0 -> 18.2 us).
template <int BM, int BN, int WGM, int WGN, int KS, bool RUNS>
__global__ __launch_bounds__(WGM * WGN * KS * 64) void gemm_w4a4_kernel(
    const uint8_t *__restrict__ Xq, const float *__restrict__ xs, const uint8_t *__restrict__ Wq,
    const float *__restrict__ ws, int M, int N, int K, void *__restrict__ Yv, int64_t ldy, int out_i32,
    int tiles_m, int tiles_n, int xcd_split)
{
    const int xcd_m = RUNS ? kXcdRuns : xcd_split;
    if constexpr (!RUNS) __builtin_assume(xcd_m != kXcdRuns);
    static_assert(KS == 1 || KS == 2, "waves per tile position");
    constexpr int NWAVE = WGM * WGN * KS;
    constexpr int SLOTS = KS == 2 ? 4 : 2;           // ring stages of LDS
    constexpr int WM = BM / WGM, WN = BN / WGN;      // wave tile
    constexpr int FM = WM / 32, FN = WN / 32;        // 32 x 32 MFMA tiles per wave
    constexpr int REGIONS = (BM + BN) / 8;           // 1 KB DMA regions (8 rows x 128 B) per stage
    constexpr int RPW = REGIONS / NWAVE;             // DMA instructions per wave per stage
    constexpr int X_BYTES = BM * ROWB, STAGE_BYTES = (BM + BN) * ROWB;
    static_assert(REGIONS % NWAVE == 0 && NWAVE % 2 == 0 && WM % 32 == 0 && WN % 32 == 0 && 3 * RPW + 4 * FM < 64,
                  "tile");

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM % WGN, kw = wave / (WGM * WGN);
    const int total = tiles_m * tiles_n;

    // workgroups are dealt round-robin to the 8 XCDs; with the XCD split on, the grid size is a multiple of 8,
    // so a workgroup's later tiles stay in its XCD's rectangle
    auto tile_origin = [&](int v, int &m0, int &n0) { sr::tile_origin(v, tiles_m, tiles_n, xcd_m, BM, BN, m0, n0); };
    const int Kb = K >> 1;
    const int ns = K / 256;                          // stages

    // ---- DMA sources.  Region q = wave + NWAVE * i holds rows 8q .. 8q+7 of the combined
    // [X rows ; W rows] tile.  Lane l lands in row l >> 3, physical chunk l & 7, and therefore
    // fetches logical chunk (l & 7) ^ swz(row), swz(row) = (row >> 1) & 7 (q and wave have
    // the same parity because NWAVE is even).
    const int dchunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
    constexpr int XI = BM / 8 / NWAVE;               // the first XI regions of a wave are X rows, the rest W rows
    static_assert((BM / 8) % NWAVE == 0, "X regions must split evenly over the waves");
    uint32_t goff[RPW];
    auto set_sources = [&](int m0, int n0) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int trow = (wave + NWAVE * i) * 8 + (lane >> 3);
            int r;
            if (i < XI) { r = m0 + trow; r = r < M ? r : M - 1; }
            else { r = n0 + trow - BM; r = r < N ? r : N - 1; }
            goff[i] = (uint32_t)r * (uint32_t)Kb + (dchunk << 4);
        }
    };
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    auto issue = [&](int s, int slot) {              // all of stage s of K -> ring slot
        const uint32_t sb = smem_base + (uint32_t)slot * STAGE_BYTES + wave * 1024;
        const uint8_t *xsrc = Xq + (int64_t)s * ROWB;
        const uint8_t *wsrc = Wq + (int64_t)s * ROWB;
#pragma unroll
        for (int i = 0; i < RPW; ++i) dma16(i < XI ? xsrc : wsrc, goff[i], sb + NWAVE * i * 1024);
    };

    // ---- fragment addresses: lane (r = l & 31, g = l >> 5).  Sub-step p (64 codes) of a stage is
    // chunks 2p, 2p+1 of the row; lane group g takes chunk 2p + g, whose two 8-byte halves are the
    // operands of two consecutive MFMAs (K = 32 each).
    const int fr = lane & 31, fg = lane >> 5;
    const int fz = (fr >> 1) & 7;
    const int xrow = (wm * WM + fr) * ROWB, wrow = X_BYTES + (wn * WN + fr) * ROWB;

    struct Frag { uint4 x[FM]; uint4 w[FN]; };              // packed, as read from LDS
    struct Ops { v4i x[FM][2]; v4i w[FN][2]; };              // widened MFMA operands of one sub-step
    auto load_frags = [&](Frag &f, int slot, int p) {
        const uint8_t *st = smem + slot * STAGE_BYTES + (((2 * p + fg) ^ fz) << 4);
#pragma unroll
        for (int j = 0; j < FM; ++j) f.x[j] = *reinterpret_cast<const uint4 *>(st + xrow + j * 32 * ROWB);
#pragma unroll
        for (int i = 0; i < FN; ++i) f.w[i] = *reinterpret_cast<const uint4 *>(st + wrow + i * 32 * ROWB);
    };

    v16i acc[FN][FM];

    auto widen = [](const uint4 w, v4i &a0, v4i &a1) {
        a0 = v4i{(int)((w.x << 4) & HM), (int)(w.x & HM), (int)((w.y << 4) & HM), (int)(w.y & HM)};
        a1 = v4i{(int)((w.z << 4) & HM), (int)(w.z & HM), (int)((w.w << 4) & HM), (int)(w.w & HM)};
    };
    auto widen_all = [&](const Frag &f, Ops &o) {
#pragma unroll
        for (int j = 0; j < FM; ++j) widen(f.x[j], o.x[j][0], o.x[j][1]);
#pragma unroll
        for (int i = 0; i < FN; ++i) widen(f.w[i], o.w[i][0], o.w[i][1]);
    };

    // ---- smooth issue: memory instructions block the issuing wave while their queue is full, and a blocked
    // wave idles the matrix pipe unless the SIMD's other wave has MFMAs to issue.  So nothing is issued in
    // bursts: a sub-step (64 codes) is cut into NREG regions of [FPR fragment reads, ~NM/NREG MFMAs with the
    // widening of FPR fragments underneath, DPR DMA instructions].  Three things are in flight per sub-step t
    // (a register-level software pipeline): the LDS reads of the packed fragments of sub-step t+2 (rd), the
    // widening of the fragments of sub-step t+1 (wd -> nxt), and the MFMAs of sub-step t (cur).  The DMA of a
    // stage is spread over the two sub-steps after the barrier that frees its ring slot.
    static_assert((FM + FN) % 2 == 0, "smooth schedule");
    constexpr int FPR = 2;                       // fragments per region
    constexpr int NREG = (FM + FN) / FPR;        // regions per sub-step
    constexpr int NR = 2 * NREG;                 // regions a stage's DMA is spread over
    constexpr int DPR = (RPW + NR - 1) / NR;     // DMA instructions per region
    constexpr int NM = 2 * FM * FN;              // MFMAs per sub-step
    auto region = [&](auto RC, auto PARTC, const Ops &cur, Ops &nxt, const Frag &wd, Frag &rd, int rslot, int p,
                      int dstage, int dslot) {
        constexpr int r = decltype(RC)::value, part = decltype(PARTC)::value;
        constexpr int mlo = r * NM / NREG, mhi = (r + 1) * NM / NREG;
        constexpr int per = (12 * FPR + (mhi - mlo) - 1) / (mhi - mlo);
        __builtin_amdgcn_sched_barrier(0);
        const uint8_t *st = smem + rslot * STAGE_BYTES + (((2 * p + fg) ^ fz) << 4);
#pragma unroll
        for (int q = r * FPR; q < (r + 1) * FPR; ++q) {
            if (q < FM) rd.x[q < FM ? q : 0] = *reinterpret_cast<const uint4 *>(st + xrow + q * 32 * ROWB);
            else rd.w[q < FM ? 0 : q - FM] = *reinterpret_cast<const uint4 *>(st + wrow + (q - FM) * 32 * ROWB);
        }
#pragma unroll
        for (int m = mlo; m < mhi; ++m) {
            const int h = m / (FM * FN), i = (m % (FM * FN)) / FM, j = m % FM;
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(cur.w[i][h], cur.x[j][h], acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int q = r * FPR; q < (r + 1) * FPR; ++q) {
            if (q < FM) widen(wd.x[q < FM ? q : 0], nxt.x[q < FM ? q : 0][0], nxt.x[q < FM ? q : 0][1]);
            else widen(wd.w[q < FM ? 0 : q - FM], nxt.w[q < FM ? 0 : q - FM][0], nxt.w[q < FM ? 0 : q - FM][1]);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, FPR, 0);
#pragma unroll
        for (int k = mlo; k < mhi; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, per, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        constexpr int g = part * NREG + r;       // ordinal of this region among those that issue DMA
        if constexpr (g < NR) {
#pragma unroll
            for (int idx = g * DPR; idx < (g + 1) * DPR && idx < RPW; ++idx)
                dma16((idx < XI ? Xq : Wq) + (int64_t)dstage * ROWB, goff[idx],
                      smem_base + (uint32_t)dslot * STAGE_BYTES + wave * 1024 + NWAVE * idx * 1024);
        }
    };
    auto ssub = [&](auto PARTC, const Ops &cur, Ops &nxt, const Frag &wd, Frag &rd, int rslot, int p, int dstage,
                    int dslot) {
        region(std::integral_constant<int, 0>{}, PARTC, cur, nxt, wd, rd, rslot, p, dstage, dslot);
        if constexpr (NREG >= 2) region(std::integral_constant<int, 1>{}, PARTC, cur, nxt, wd, rd, rslot, p, dstage, dslot);
        if constexpr (NREG >= 3) region(std::integral_constant<int, 2>{}, PARTC, cur, nxt, wd, rd, rslot, p, dstage, dslot);
        if constexpr (NREG >= 4) region(std::integral_constant<int, 3>{}, PARTC, cur, nxt, wd, rd, rslot, p, dstage, dslot);
        static_assert(NREG <= 4, "regions");
    };
    constexpr std::integral_constant<int, 0> P0{};   // first / second sub-step after the barrier: issue DMA
    constexpr std::integral_constant<int, 1> P1{};
    constexpr std::integral_constant<int, 2> P2{};   // the two sub-steps before the barrier: no DMA
    constexpr std::integral_constant<int, 3> P3{};

    // epilogue staging: one piece = 32 tokens x WN channels of fp16 per wave, in ring slot 1
    // (KS = 2: of WN / 2 channels, in the exchange area)
    constexpr int EN = FN / KS;                      // 32-channel tiles a wave finishes
    constexpr int PIECE = 32 * (EN * 64 + 16);
    static_assert(FN % KS == 0 && NWAVE * PIECE <= STAGE_BYTES, "epilogue staging must fit one ring slot");

    // Token and channel scales of the tile's epilogue are fetched at the start of the tile (10 loads per lane for
    // a 64 x 64 wave tile) -- fetched at the tile boundary, their latency was exposed on every tile.
    float sx[FM];
    float4 sw[EN][4];
    // (With the raw int32 output the host passes readable stand-ins for the two scale vectors, so the loads
    // need no branch -- a branch made the compiler wait for them at once; the values are then not used.)
    auto load_scales = [&](int m0, int n0) {
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const int m = m0 + wm * WM + j * 32 + fr;
            sx[j] = xs[m < M ? m : M - 1];
        }
#pragma unroll
        for (int i = 0; i < EN; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + wn * WN + (kw * EN + i) * 32 + q * 8 + fg * 4;
                sw[i][q] = *reinterpret_cast<const float4 *>(ws + (n < N ? n : N - 4));
            }
    };

    int v = blockIdx.x;
    int m0, n0;
    if constexpr (RUNS)                              // (a divided grid has a tile for every workgroup)
        if (!tile_exists(v, tiles_m, tiles_n, xcd_m)) return;      // the whole workgroup
    tile_origin(v, m0, n0);
    set_sources(m0, n0);
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) issue(i < ns ? i : ns - 1, i);
    for (;;) {
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

        // Stage 0 has landed once at most RPW of this wave's memory operations are still outstanding: loads
        // complete in order among themselves and the RPW loads of stage 1 are the youngest, so an unfinished
        // older load would leave more than RPW outstanding -- however many stores of the previous tile are
        // still on their way (stores and loads may overtake each other).
        // (KS = 2: the same with the three stages behind stage 0.)
        wait_vmcnt<(SLOTS - 1) * RPW>();
        barrier_nofence();
        load_scales(m0, n0);                         // used after the K loop, whose first wait covers them
        Ops o0, o1;
        Frag fa, fb;                                 // fragments of even / odd sub-steps
        load_frags(fa, 0, 2 * kw);
        load_frags(fb, 0, 2 * kw + 1);
        widen_all(fa, o0);
        int slot = 0;
        // Every stage runs the same branch-free body.  Past the end of K the pipeline keeps reading (stale,
        // in-bounds) LDS and re-fetching the last stage; those fragments are widened but never multiplied.
        if constexpr (KS == 2) {
            for (int s = 0; s < ns; ++s) {
                const int nslot = (slot + 1) & (SLOTS - 1);
                const int st4 = s + SLOTS < ns ? s + SLOTS : ns - 1;
                // stage s + 1 has landed (at most the two behind it are on their way), and every wave's reads of stage s
                // have returned: its slot takes stage s + 4
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((SLOTS - 2) * RPW) : "memory");
                barrier_nofence();
                ssub(P0, o0, o1, fb, fa, nslot, 2 * kw, st4, slot);
                ssub(P1, o1, o0, fa, fb, nslot, 2 * kw + 1, st4, slot);
                slot = nslot;
            }
        }
        for (int s = 0; KS == 1 && s < ns; ++s) {
            const int nslot = slot ^ 1;
            const int st2 = s + 2 < ns ? s + 2 : ns - 1;
            ssub(P2, o0, o1, fb, fa, slot, 2, st2, nslot);
            ssub(P3, o1, o0, fa, fb, slot, 3, st2, nslot);
            // stage s+1 must have landed, and every wave's reads of stage s must have returned: its slot takes
            // stage s+2 from here on
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            barrier_nofence();
            ssub(P0, o0, o1, fb, fa, nslot, 0, st2, slot);
            ssub(P1, o1, o0, fa, fb, nslot, 1, st2, slot);
            slot = nslot;
        }

        // ---- tile boundary
        const int vn = v + (int)gridDim.x;
        const bool more = RUNS ? tile_exists(vn, tiles_m, tiles_n, xcd_m) : vn < total;
        wait_vmcnt<0>();                             // no LDS-DMA write is in flight any more ...
        // (the scales arrived long ago; naming them here keeps the compiler's own wait for them at this point
        // and not behind the loads issued next)
#pragma unroll
        for (int j = 0; j < FM; ++j) asm volatile("" : "+v"(sx[j]));
#pragma unroll
        for (int i = 0; i < EN; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                asm volatile("" : "+v"(sw[i][q].x), "+v"(sw[i][q].y), "+v"(sw[i][q].z), "+v"(sw[i][q].w));
        barrier_nofence();                           // ... and all waves are done reading fragments
        int m1 = 0, n1 = 0;
        if (more) {                                  // first stage of the next tile flies during the epilogue
            tile_origin(vn, m1, n1);
            set_sources(m1, n1);
            issue(0, 0);
            if constexpr (KS == 2) issue(ns > 1 ? 1 : 0, 1);
        }
#pragma unroll
        for (int j = 0; j < FM; ++j) sx[j] *= 1.f / 256.f;      // both operands carried a factor 16
        if constexpr (KS == 2) {
            // the sums of the other half of the channels go to the wave that finishes them (ring slots 2 and 3)
            constexpr int PART = EN * FM * 16 * 256;             // bytes a wave hands over
            static_assert(NWAVE * PART <= 2 * STAGE_BYTES && PIECE <= PART, "exchange area");
            uint8_t *mine = smem + 2 * STAGE_BYTES + wave * PART + lane * 16;
            uint8_t *other = smem + 2 * STAGE_BYTES + (wave ^ (WGM * WGN)) * PART;
            v16i fin[EN][FM];
#pragma unroll
            for (int i = 0; i < EN; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j) {
                    v16i give;
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        fin[i][j][e] = kw ? acc[EN + i][j][e] : acc[i][j][e];
                        give[e] = kw ? acc[i][j][e] : acc[EN + i][j][e];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<v4i *>(mine + ((i * FM + j) * 4 + q) * 1024) = v4i{give[4 * q], give[4 * q + 1], give[4 * q + 2], give[4 * q + 3]};
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            barrier_nofence();
#pragma unroll
            for (int i = 0; i < EN; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const v4i o = *reinterpret_cast<const v4i *>(other + lane * 16 + ((i * FM + j) * 4 + q) * 1024);
#pragma unroll
                        for (int e = 0; e < 4; ++e) fin[i][j][4 * q + e] += o[e];
                    }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            // (only this wave reads `other`: its staging may follow there)
            store_wave_tile<FM, EN>(fin, other, lane, m0 + wm * WM, n0 + wn * WN + kw * EN * 32, M, N, sx, sw, Yv, ldy, out_i32);
        } else {
            store_wave_tile<FM, EN>(acc, smem + STAGE_BYTES + wave * PIECE, lane, m0 + wm * WM, n0 + wn * WN, M, N, sx, sw,
                                    Yv, ldy, out_i32);
        }
        if (!more) break;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier_nofence();                           // every wave has read its staging back: slot 1 (KS = 2: 2, 3) is free
#pragma unroll
        for (int i = SLOTS / 2; i < SLOTS; ++i) issue(i < ns ? i : ns - 1, i);
        v = vn;
        m0 = m1;
        n0 = n1;
    }
    wait_vmcnt<0>();
}

template <int BM, int BN, int WGM, int WGN, int WG_PER_CU, int KS = 1>
hipError_t launch_tile(const uint8_t *Xq, const float *xs, const uint8_t *Wq, const float *ws, int64_t M, int64_t N,
                       int64_t K, void *Y, int64_t ldy, int out_i32, hipStream_t st)
{
    constexpr auto divided = gemm_w4a4_kernel<BM, BN, WGM, WGN, KS, false>, runs = gemm_w4a4_kernel<BM, BN, WGM, WGN, KS, true>;
    constexpr int lds = 2 * KS * (BM + BN) * ROWB;
    static_assert(lds * WG_PER_CU <= 160 * 1024, "LDS");
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((N + BN - 1) / BN);
    const int xcd_m = choose_xcd_split(tiles_m, tiles_n, BM, BN);
    const auto kern = xcd_m == kXcdRuns ? runs : divided;
    if (lds > 48 * 1024) {
        hipError_t e = xcd_m == kXcdRuns ? allow_dynamic_lds<runs>(lds) : allow_dynamic_lds<divided>(lds);
        if (e != hipSuccess) return e;
    }
    // persistent grid: as many workgroups as the chip holds at once (a multiple of 8, as the XCD map needs)
    int64_t grid = (int64_t)compute_units() * WG_PER_CU;
    if (int64_t g; tuned(kTuneGemmGrid, g) && g > 0) grid = g / 8 * 8;
    if (grid < 8) grid = 8;
    grid = tile_workgroups(grid, (int64_t)tiles_m * tiles_n, xcd_m);
    // the raw int32 output takes no scales (they may be NULL): the kernel still fetches M and N floats it
    // then ignores, from the start of the code arrays (M * K / 2 >= 4 M bytes, 16-byte aligned)
    if (out_i32) {
        xs = reinterpret_cast<const float *>(Xq);
        ws = reinterpret_cast<const float *>(Wq);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WGM * WGN * KS * 64), lds, st, Xq, xs, Wq, ws,
                       (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n, xcd_m);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Generic kernel (any K % 64 == 0): 128 x 128 tile, K step of 128 codes, global -> registers
// -> LDS double buffering, v_mfma_i32_16x16x64_i8; a K tail of 64 codes is zero-filled.
// ------------------------------------------------------------------------------------------
constexpr int KB = 64;   // packed bytes of one K step per row (128 codes)

__device__ __forceinline__ int swz_off(int row, int chunk)
{
    return row * KB + ((chunk ^ ((row >> 2) & 3)) << 4);
}

__device__ __forceinline__ void unpack16(const uint4 w, v4i &a0, v4i &a1)
{
        a0[0] = (int)((w.x << 4) & HM); a0[1] = (int)(w.x & HM);
    a0[2] = (int)((w.y << 4) & HM); a0[3] = (int)(w.y & HM);
    a1[0] = (int)((w.z << 4) & HM); a1[1] = (int)(w.z & HM);
    a1[2] = (int)((w.w << 4) & HM); a1[3] = (int)(w.w & HM);
}

template <int BM, int BN>
__global__ __launch_bounds__(256) void gemm_w4a4_generic_kernel(const uint8_t *__restrict__ Xq, const float *__restrict__ xs,
                                                        const uint8_t *__restrict__ Wq, const float *__restrict__ ws,
                                                        int M, int N, int K, void *__restrict__ Yv, int64_t ldy,
                                                        int out_i32, int tiles_m, int tiles_n)
{
    constexpr int WM = BM / 2, WN = BN / 2;          // wave tile
    constexpr int FM = WM / 16, FN = WN / 16;        // MFMA tiles per wave
    constexpr int LX = BM * 4 / 256, LW = BN * 4 / 256;   // 16-byte loads per thread per K step
    static_assert(BM % 64 == 0 && BN % 64 == 0, "tile");

    __shared__ __attribute__((aligned(16))) uint8_t lds[2][(BM + BN) * KB];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;

    // ---- workgroup -> tile: workgroups are dealt round-robin to the 8 XCDs, so give each
    // XCD a contiguous run of tiles (neighbours share X / W panels in that XCD's L2).
    int bid = blockIdx.x;
    const int total = tiles_m * tiles_n;
    if ((total & 7) == 0) bid = (bid & 7) * (total >> 3) + (bid >> 3);
    const int tm = bid % tiles_m, tn = bid / tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;

    const int Kb = K >> 1;                          // packed bytes per row
    const int nk = (Kb + KB - 1) / KB;

    // global load coordinates: thread -> (row, 16-byte chunk)
    const int lrow = tid >> 2, lchunk = tid & 3;
    const uint8_t *xg[LX];
    const uint8_t *wg[LW];
#pragma unroll
    for (int i = 0; i < LX; ++i) {
        int r = m0 + lrow + 64 * i;
        r = r < M ? r : M - 1;
        xg[i] = Xq + (int64_t)r * Kb + lchunk * 16;
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        int r = n0 + lrow + 64 * i;
        r = r < N ? r : N - 1;
        wg[i] = Wq + (int64_t)r * Kb + lchunk * 16;
    }

    uint4 px[LX], pw[LW];
    auto gload = [&](int ks) {
        const int kb = ks * KB;
        const bool ok = kb + lchunk * 16 < Kb;      // K tail (K % 128 == 64): zero codes
#pragma unroll
        for (int i = 0; i < LX; ++i)
            px[i] = ok ? *reinterpret_cast<const uint4 *>(xg[i] + kb) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < LW; ++i)
            pw[i] = ok ? *reinterpret_cast<const uint4 *>(wg[i] + kb) : make_uint4(0, 0, 0, 0);
    };
    auto lstore = [&](int stage) {
        uint8_t *xs_l = lds[stage];
        uint8_t *ws_l = lds[stage] + BM * KB;
#pragma unroll
        for (int i = 0; i < LX; ++i)
            *reinterpret_cast<uint4 *>(xs_l + swz_off(lrow + 64 * i, lchunk)) = px[i];
#pragma unroll
        for (int i = 0; i < LW; ++i)
            *reinterpret_cast<uint4 *>(ws_l + swz_off(lrow + 64 * i, lchunk)) = pw[i];
    };

    v4i acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    const int fr = lane & 15, fg = lane >> 4;       // fragment row / k group of this lane

    gload(0);
    lstore(0);
    __syncthreads();

    for (int ks = 0; ks < nk; ++ks) {
        const int stage = ks & 1;
        if (ks + 1 < nk) gload(ks + 1);

        const uint8_t *xs_l = lds[stage] + (wm * WM) * KB;
        const uint8_t *ws_l = lds[stage] + BM * KB + (wn * WN) * KB;

        v4i xa0[FM], xa1[FM];
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const uint4 p = *reinterpret_cast<const uint4 *>(xs_l + swz_off(j * 16 + fr, fg));
            unpack16(p, xa0[j], xa1[j]);
        }
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const uint4 p = *reinterpret_cast<const uint4 *>(ws_l + swz_off(i * 16 + fr, fg));
            v4i wa0, wa1;
            unpack16(p, wa0, wa1);
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa0, xa0[j], acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa1, xa1[j], acc[i][j], 0, 0, 0);
            }
        }

        if (ks + 1 < nk) lstore(stage ^ 1);
        __syncthreads();
    }

    // ---- epilogue: lane owns token m, output channels n .. n+3 of each MFMA tile ----------
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int m = m0 + wm * WM + j * 16 + fr;
        if (m >= M) continue;
        const float sx = out_i32 ? 0.f : xs[m] * (1.f / 256.f);
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const int n = n0 + wn * WN + i * 16 + fg * 4;
            if (n >= N) continue;
            const v4i a = acc[i][j];
            if (out_i32) {
                int4 o = make_int4(a[0] >> 8, a[1] >> 8, a[2] >> 8, a[3] >> 8);
                *reinterpret_cast<int4 *>(static_cast<int32_t *>(Yv) + (int64_t)m * ldy + n) = o;
            } else {
                const float4 sw = *reinterpret_cast<const float4 *>(ws + n);
                union { __half h[4]; uint2 u; } o;
                o.h[0] = __float2half_rn((float)a[0] * sx * sw.x);
                o.h[1] = __float2half_rn((float)a[1] * sx * sw.y);
                o.h[2] = __float2half_rn((float)a[2] * sx * sw.z);
                o.h[3] = __float2half_rn((float)a[3] * sx * sw.w);
                *reinterpret_cast<uint2 *>(static_cast<__half *>(Yv) + (int64_t)m * ldy + n) = o.u;
            }
        }
    }
}


}  // namespace

hipError_t launch_gemm_prefill(const uint8_t *Xq, const float *xs, const uint8_t *Wq, const float *ws,
                               int64_t M, int64_t N, int64_t K, void *Y, int64_t ldy, int out_i32,
                               hipStream_t st)
{
    // the tile knob selects a tile configuration by number; not set = heuristic
    int variant = 0;
    if (int64_t t; tuned(kTuneGemmTile, t)) variant = (int)t;
    if (K % 256 != 0 || variant == 9) {
        constexpr int BM = 128, BN = 128;
        const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((N + BN - 1) / BN);
        hipLaunchKernelGGL((gemm_w4a4_generic_kernel<BM, BN>), dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, st,
                           Xq, xs, Wq, ws, (int)M, (int)N, (int)K, Y, ldy, out_i32, tiles_m, tiles_n);
        return hipGetLastError();
    }
    const GemmConfig *best = packed_config(packed_shape(M, N, K, compute_units()));
    for (const GemmConfig &c : kPackedConfigs)           // the tile knob
        if (c.id == variant) best = &c;
    switch (best->id) {
        case 14: return launch_tile<128, 128, 2, 2, 2>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st);
        case 15: return launch_tile<256, 128, 4, 2, 1>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st);
        case 20: return launch_tile<128, 128, 2, 2, 1, 2>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st);
        case 17: return launch_tile<128, 64, 4, 2, 2>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st);
        case 18: return launch_tile<192, 128, 2, 4, 1>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st);
        case 19: return launch_tile<64, 128, 2, 4, 2>(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st);
        default: return launch_gemm_w4a4_stream(Xq, xs, Wq, ws, M, N, K, Y, ldy, out_i32, st, best->id / 1000, best->id % 1000);
    }
}

}  // namespace sr
