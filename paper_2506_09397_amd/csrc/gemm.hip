// Projections of the verify step: out[T, N] = X[T, K] * W[N, K]^T over the packed rows of a batch.
//
// Three kernels share the work of bf16 models.  Up to 32 rows (and 4-bit weights up to 64 where K is long) run in gemm_kwave_kernel (both
// operands straight to registers, the k-steps dealt out to the wavefronts); 16-bit weights beyond that in gemm_tile_kernel (both
// operands through LDS); both are described there.  8- and 4-bit weights, batch-invariant models, 65 to 96 rows (three row tiles), and
// the LM head at 97 to 128 rows run in gemm_bf16_kernel, which the following describes.
//
// bf16 path (the one that matters): T is about 100-600 packed rows, so every weight byte is used
// for only T multiply-adds and the kernel is a weight stream bounded by HBM.  It is still a dense
// contraction, so the arithmetic goes through v_mfma_f32_32x32x16_bf16 (the 16x16 shapes run at
// about half its rate on gfx950, which would make them, not HBM, the bound).
//   - Weights sit in HBM in MFMA operand order, k-step-major (see wfrag_offset): a wavefront
//     fetches a 32-row x 16-k tile with one contiguous 1 KiB load straight into registers, no LDS,
//     no transpose, and keeps three pipeline stages of them in flight.
//   - Activations are carried as bf16 PAIRS, x = hi + lo (two planes in operand order, written
//     that way by the producing kernel): a single bf16 rounding of every activation costs more
//     accuracy than the 2e-2 logit tolerance allows at 8B scale, so each weight tile is multiplied
//     with both planes.  All wavefronts of a workgroup need all of them: they go from L2 into a
//     ring of five LDS stage buffers with direct-to-LDS loads, four stages ahead.
//   - A workgroup is 8 wavefronts (two per SIMD), all alike: 2 column groups x 4 k-groups (others for low-bit
//     weights with several blocks of rows and for the LM head; see the shapes below).  A stage is one k-step of 16 per k-group;
//     k-group g works on the g-th of them for the 64 columns (two 32-column
//     tiles) of its column group and all rows of the block (MT 32-row tiles), and the k-groups'
//     sums are exchanged through LDS at the end and added in a fixed order, after which every wavefront stores a
//     share of the outputs.  This shape follows from three
//     per-CU limits that all sit within a factor of two of the HBM time: one wavefront sustains
//     only about 4-5 bytes per clock from L2, so the activation stream (twice the weight bytes per
//     CU) has to be issued by all eight; ds_read_b128 runs at about 64 bytes per clock, so each
//     activation tile read from LDS has to feed four MFMAs; and the MFMAs themselves need two
//     wavefronts per SIMD to hide each other's waits.
//   - Vector-memory loads retire in order under one counter, and the compiler cannot see that the
//     two streams are independent (it drains the counter before any LDS read that might alias a
//     direct-to-LDS load).  Both kinds of loads are therefore issued from inline assembly in a
//     fixed order, and the waits are written by hand from that order.
//   - Weights are read past the caches' replacement order (nt) in all kernels: a step streams gigabytes of them, and loaded as
//     anything else is they push the partial sums and activations, which the next kernel reads, out of Infinity Cache.  Layer
//     times of the 8B shape without and with it, us: 58 rows 146.5-150 -> 140.6-143 (16-bit), 132 -> 128 (8-bit), 86 rows 170-173 -> 168,
//     101 rows 188-190 -> 185; 70B shape, 220 rows 868-873 -> 857-862: the row kernels gain as much as the projections.  8 layers and the head
//     without / with it, us: 8-bit 96 rows 1328 / 1289, 128 1531 / 1491, 256 2521 / 2446, 512 4407 / 4390; 4-bit 96 rows 1260 / 1235,
//     256 2388 / 2379; batch-invariant 16-bit weights, whose row blocks share the narrow shape, 136 rows 2281 / 2279, 192 2401 / 2353,
//     256 2994 / 2946, 512 5611 / 5561 (8-bit 136 rows 2215 / 2163, 4-bit 2099 / 2039): nowhere slower.
//     The ordinary order is kept where two unequal row blocks share the weights and for models that a cache holds (see the launches).
//   - Split-K over blockIdx.y gives every CU work on the narrow projections; partial sums go to a
//     [split, T, N] fp32 buffer that the following row kernel reduces in a fixed order (no float
//     atomics: results are reproducible run to run).
//   - Weights may also be stored in 8 bits (FP8 E4M3, a scale per output row) or 4 bits (FP4 E2M1, a power-of-two
//     scale per row and 32 k): the same tiles at half or a quarter of the bytes, widened to bf16 in registers by
//     the hardware conversions; everything else is unchanged.
//   - The weight tile is the A operand, the activation tile the B operand, so a lane ends up with
//     groups of 4 consecutive output columns of one row: float4 stores, and gate/up pairs for
//     SwiGLU in-lane.
//
// fp32 path: plain FMA kernel, used by fp32 models (correctness configuration).
#include "sled_internal.h"

#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <type_traits>

namespace {

constexpr int PLANES = 2;    // activation planes: hi, lo
constexpr int NW = 2;        // 32-column tiles per wavefront
constexpr int WAVES = 8;     // = k-groups x column groups of a workgroup shape
constexpr int DEPTH = 3;     // weight stages in flight beyond the one in use
constexpr int NBUF = DEPTH + 1;
constexpr int AHEAD = DEPTH + 1;  // activation stages in flight beyond the one being read
constexpr int NXB = AHEAD + 1;    // LDS ring
// Two workgroup shapes (KG k-groups = k-steps of 16 per stage, CG column groups of 64 columns):
//   narrow  KG 4, CG 2: 128 columns, 64 k per stage.  Most workgroups per projection: the shape for one block of
//           33 to 128 rows of 8- and 4-bit weights, for three row tiles of any weights, and for batch-invariant models at any size, where the chip has to be filled by column blocks and K slices alone.
//   wide    KG 2, CG 4: 256 columns, 32 k per stage.  Per MFMA it fetches two thirds of the bytes (half the
//           activations, the same weights): the shape for several row blocks of 8- and 4-bit weights, where the
//           workgroups are many anyway and the L2 -> CU path, not HBM, is what the MFMAs wait for (bf16 weights: the
//           tile kernel below).
//   broad   KG 1, CG 8: 512 columns, 16 k per stage, no sums to exchange at the end.  Per MFMA it fetches half the
//           bytes of the narrow shape; only a matrix with enough columns to fill the chip without K slices can use
//           it (the LM head), and only with four row tiles (a stage's eight activation tiles go one to a wavefront).
constexpr int NARROW_KG = 4, NARROW_CG = 2, WIDE_KG = 2, WIDE_CG = 4, BROAD_KG = 1, BROAD_CG = 8;
constexpr int NARROW_COLS = NARROW_CG * NW * 32;

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float float16_t;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4_t;

// s_waitcnt vmcnt(N) tied to the registers the awaited loads write: the compiler sees the assembly
// loads as complete when issued, so the data dependence has to run through the wait.
template <int N>
__device__ __forceinline__ void wait_loads(u32x4_t& a, u32x4_t& b) {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N) : "memory");
}

// Eight 8-bit weights (FP8 E4M3, the OCP flavour gfx950 converts in hardware) -> a bf16 MFMA operand: one
// instruction per pair, exact (three mantissa bits fit bf16's seven).
__device__ __forceinline__ bf16x8_t cvt_w8(uint32_t lo, uint32_t hi) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_hw;
    const u32x4_t p = {__builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false)),
                       __builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true)),
                       __builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false)),
                       __builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true))};
    return __builtin_bit_cast(bf16x8_t, p);
}

// Eight 4-bit weights (FP4 E2M1, low nibble first) times a power-of-two block scale -> a bf16 MFMA operand; exact
__device__ __forceinline__ bf16x8_t cvt_w4(uint32_t codes, float scale) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_hw;
    const u32x4_t p = {__builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 0)),
                       __builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 1)),
                       __builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 2)),
                       __builtin_bit_cast(uint32_t, (bf16x2_hw)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 3))};
    return __builtin_bit_cast(bf16x8_t, p);
}

// the same for a single register (never pass one register twice to the two-operand form: the second operand would
// be a copy taken while the load is still in flight)
template <int N>
__device__ __forceinline__ void wait_load(u32x4_t& a) {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%1)" : "+v"(a) : "n"(N) : "memory");
}

typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2_t;
// ... and for the two registers of a 4-bit stage (codes and scales)
template <int N>
__device__ __forceinline__ void wait_load4(u32x2_t& a, uint32_t& b) {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N) : "memory");
}

// four consecutive output columns n .. n+3 of row tok: partial sums of K slice `by`, finished values, or SwiGLU of the
// two (gate, up) pairs they hold, written as a bf16 pair in operand order
template <int EPI>
__device__ __forceinline__ void store_cols(const float4_t v, int tok, int n, int by, int T_pad, int N, float* __restrict__ out,
                                           bf16_t* __restrict__ out_act, size_t act_plane, int F_act) {
    if (EPI == SLED_EPI_PARTIAL) {
        *reinterpret_cast<float4_t*>(out + ((size_t)by * T_pad + tok) * N + n) = v;
    } else if (EPI == SLED_EPI_STORE) {
        *reinterpret_cast<float4_t*>(out + (size_t)tok * N + n) = v;
    } else {  // columns are (gate f, up f, gate f+1, up f+1)
        const int f = n >> 1;
        const float a0 = v[0] / (1.f + __expf(-v[0])) * v[1];
        const float a1 = v[2] / (1.f + __expf(-v[2])) * v[3];
        const bf16_t h0 = f32_to_bf16(a0), h1 = f32_to_bf16(a1);
        const bf16_t l0 = f32_to_bf16(a0 - bf16_to_f32(h0)), l1 = f32_to_bf16(a1 - bf16_to_f32(h1));
        const size_t o = frag_offset(tok, f, F_act);
        *reinterpret_cast<uint32_t*>(out_act + o) = (uint32_t)h0 | ((uint32_t)h1 << 16);
        *reinterpret_cast<uint32_t*>(out_act + act_plane + o) = (uint32_t)l0 | ((uint32_t)l1 << 16);
    }
}

// MT: 32-row tiles of activations per block.  WB: bits per weight.  8 (see w8_offset): the wavefront's two column
// tiles come with ONE load per stage, are widened to bf16 in registers, and the accumulators are multiplied by the
// columns' scales on the way out.  4 (see w4_offset): one 8-byte load per stage for the codes and one 2-byte load
// for the two rows' block scales, which the widening instruction applies.
template <int MT, int EPI, int KG, int CG, int WB, bool KEEP>
__global__ __launch_bounds__(64 * WAVES) void gemm_bf16_kernel(const bf16_t* __restrict__ Xp, size_t x_plane,
                                                               const bf16_t* __restrict__ Wp,
                                                               const void* __restrict__ scale_v, int NT, int KS,
                                                               int n_col, int n_split, int n_zb,
                                                               int T, int T_pad, int N, float* __restrict__ out,
                                                               bf16_t* __restrict__ out_act, size_t act_plane,
                                                               int F_act) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int STAGE_TILES = PLANES * MT * KG;  // 1 KiB operand tiles per stage, ordered [plane][row tile][k-step]
    constexpr int MY_TILES = STAGE_TILES / WAVES;  // = MT: tiles of a stage this wavefront fetches
    constexpr bool W8 = WB == 8, W4 = WB == 4;
    static_assert(WB == 16 || W8 || W4, "16-, 8- or 4-bit weights");
    constexpr int NWL = WB == 16 ? NW : 1;         // weight loads per stage
    constexpr int NSL = W4 ? 1 : 0;                // block-scale loads per stage
    constexpr int PER_ITER = MY_TILES + NWL + NSL; // vector-memory instructions a wavefront issues per stage
    const float* scale = static_cast<const float*>(scale_v);
    constexpr unsigned STAGE_BYTES = STAGE_TILES * 1024;
    static_assert(KG * CG == WAVES, "a workgroup is eight wavefronts");
    static_assert(STAGE_TILES % WAVES == 0, "stage does not divide among the wavefronts");
    static_assert(PER_ITER * DEPTH < 64, "too many loads in flight for the counter");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int cg = wv & (CG - 1), kgi = wv / CG;
    // Workgroup -> (column block bx, K slice by, row block bz).  Workgroups go to the eight XCDs round
    // robin by their linear index, and each XCD has its own L2.  The row blocks of one weight tile
    // stream the same weight bytes, so they are given consecutive slots of ONE XCD: they run side by
    // side there and all but the first find the weights in that L2 instead of fetching them from HBM
    // again.  Weight tile t = by * n_col + bx lives on XCD t % 8.
    int bx, by, bz;
    {
        const int w = blockIdx.x, xcd = w & 7, local = w >> 3;
        bz = local % n_zb;
        const int t = (local / n_zb) * 8 + xcd;
        if (t >= n_col * n_split) return;  // the grid is rounded up to whole rounds of eight tiles
        bx = t % n_col;
        by = t / n_col;
    }
    // K slice `by`: K in units of KG * NBUF k-steps (one trip of the stage loop), dealt out as evenly as whole units
    // allow -- the first `urem` slices hold one unit more (the host sees to n_split <= units)
    const int units = KS / (KG * NBUF), ubase = units / n_split, urem = units - ubase * n_split;
    const int ks_begin = (by * ubase + min(by, urem)) * (KG * NBUF);
    const int n_stage = (ubase + (by < urem ? 1 : 0)) * NBUF;  // a positive multiple of NBUF
    const int mt_base = bz * MT;            // first 32-row tile handled by this block

    // ---- activations: this wavefront's tiles of stage 0 and where they land in a stage buffer -----
    const int row_lim = (T + 7) & ~7;
    const bf16_t* xsrc[MY_TILES];
    unsigned xdst[MY_TILES];
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;  // LDS byte address of the ring
#pragma unroll
    for (int j = 0; j < MY_TILES; j++) {
        const int i = j * WAVES + wv;
        const int g = i % KG, pb = i / KG, pl = pb / MT, b = pb - pl * MT;
        // Lanes whose row lies past the last token (rounded up to whole 128-byte lines of 8 rows) re-read
        // the tile's first line instead: the fetch unit merges them into that line's request, so padding
        // rows cost no L2 traffic.  What lands in their LDS bytes only reaches their own output rows.
        // A block may reach past the last row tile (the wide shape always takes four): such a tile re-reads the
        // last one, and its results are not stored.
        const int mt = min(mt_base + b, T_pad / 32 - 1);
        const int row = mt * 32 + (lane & 31);
        const int src_lane = row < row_lim ? lane : (lane & 32) + (lane & 7);
        xsrc[j] = Xp + pl * x_plane + ((size_t)mt * KS + ks_begin + g) * 512 + src_lane * 8;
        xdst[j] = lds_base + i * 1024;
    }
    // one direct-to-LDS load moves a whole operand tile: lane l's 16 bytes land at m0 + 16*l
    auto x_issue_one = [&](int buf, int stage, int j) {
        const bf16_t* src = xsrc[j] + (size_t)stage * (KG * 512);
        const unsigned dst = __builtin_amdgcn_readfirstlane(xdst[j] + (unsigned)buf * STAGE_BYTES);
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst) : "memory");
    };
    auto x_issue = [&](int buf, int stage) {
#pragma unroll
        for (int j = 0; j < MY_TILES; j++) x_issue_one(buf, stage, j);
    };

    // ---- weights: NW tiles per stage, straight into registers ------------------------------------------
    const int nt0 = (bx * CG + cg) * NW;
    const int NTW = WB == 16 ? NT : NT / NW;  // blocks per k-step (an 8- or 4-bit block holds the wavefront's two tiles)
    constexpr int WBLK = W4 ? 256 : 512;      // size of a block and of a lane's share, in 2-byte units
    constexpr int WLANE = W4 ? 4 : 8;
    bool nt_ok[NW];
    const bf16_t* wsrc[NW];
#pragma unroll
    for (int a = 0; a < NW; a++) {
        nt_ok[a] = (nt0 + a) < NT;
        const int blk = WB == 16 ? nt0 + a : nt0 / NW;
        wsrc[a] = Wp + ((size_t)(ks_begin + kgi) * NTW + (nt_ok[a] ? blk : 0)) * WBLK + lane * WLANE;
    }
    // 4-bit weights: the scale bytes of this lane's row in both tiles; those of k-block kb lie kb * NTW * 64 bytes on
    const uint8_t* ssrc = static_cast<const uint8_t*>(scale_v);
    if (W4) ssrc += (size_t)(nt_ok[0] ? nt0 / NW : 0) * 64 + (lane & 31) * 2;
    u32x4_t wreg[NBUF][NWL];
    u32x2_t w4reg[NBUF];
    uint32_t sreg[NBUF];
    auto w_issue_one = [&](int buf, int stage, int a) {  // a: which of the stage's NWL + NSL weight-side loads
        const bf16_t* src = wsrc[a < NWL ? a : 0] + (size_t)stage * KG * NTW * WBLK;
        if (W4) {
            if (a == 0) {
                if constexpr (KEEP)
                    asm volatile("global_load_dwordx2 %0, %1, off" : "=&v"(w4reg[buf]) : "v"(src) : "memory");
                else
                    asm volatile("global_load_dwordx2 %0, %1, off nt" : "=&v"(w4reg[buf]) : "v"(src) : "memory");
            } else
                asm volatile("global_load_ushort %0, %1, off"
                             : "=&v"(sreg[buf])
                             : "v"(ssrc + (size_t)((ks_begin + kgi + stage * KG) >> 1) * NTW * 64)  // a k-block is two k-steps
                             : "memory");
        } else if constexpr (KEEP) {
            asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(wreg[buf][a]) : "v"(src) : "memory");
        } else {
            asm volatile("global_load_dwordx4 %0, %1, off nt" : "=&v"(wreg[buf][a]) : "v"(src) : "memory");
        }
    };
    auto w_issue = [&](int buf, int stage) {
#pragma unroll
        for (int a = 0; a < NWL + NSL; a++) w_issue_one(buf, stage, a);
    };

    float16_t acc[NW][MT];
#pragma unroll
    for (int a = 0; a < NW; a++)
#pragma unroll
        for (int b = 0; b < MT; b++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[a][b][e] = 0.f;

    const bf16_t* xs = reinterpret_cast<const bf16_t*>(smem) + kgi * 512 + lane * 8;
    struct xfrag {
        bf16x8_t hi, lo;
    };
    auto read_x = [&](int xbuf, int b) {
        const bf16_t* xb = xs + (size_t)xbuf * (STAGE_BYTES / 2);
        xfrag f;
        f.hi = *reinterpret_cast<const bf16x8_t*>(xb + (size_t)b * (KG * 512));
        f.lo = *reinterpret_cast<const bf16x8_t*>(xb + (size_t)(MT + b) * (KG * 512));
        return f;
    };
    auto mfma4 = [&](int b, const xfrag& f, const bf16x8_t& w0, const bf16x8_t& w1) {
        acc[0][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0, f.hi, acc[0][b], 0, 0, 0);
        acc[1][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1, f.hi, acc[1][b], 0, 0, 0);
        acc[0][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0, f.lo, acc[0][b], 0, 0, 0);
        acc[1][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1, f.lo, acc[1][b], 0, 0, 0);
    };
    // One stage ("iteration" s): arithmetic of stage s, and the loads of later stages.
    //   - The iteration's PER_ITER loads (activations of stage s+AHEAD, then weights of stage
    //     s+DEPTH, always in that order) leave first, right after the wait.
    //   - LDS reads run one row tile ahead of the MFMAs that use them, and the first row tile of the
    //     next stage is read before the last MFMAs of this one.  `cur` holds row tile 0 of the stage
    //     on entry and row tile 0 of the next stage on exit.
    //   - The barrier before the last row tile says two things: this wavefront's share of stage s+1
    //     has landed (the wait at the top covers it), and its LDS reads of stage s are back, so that
    //     buffer may be refilled.
    // The wait at the top is for the weights of stage s and the activations of stage s+1, both issued
    // DEPTH iterations earlier; AFTER is the number of loads issued since.
    xfrag cur;
    auto stage = [&](auto after_c, int xbuf, auto wbuf_c, bool more, int x_stage, int x_buf, int w_stage) {
        constexpr int AFTER = decltype(after_c)::value, WBUF = decltype(wbuf_c)::value;
        bf16x8_t w0, w1;
        if (W4) {
            wait_load4<AFTER>(w4reg[WBUF], sreg[WBUF]);
            const uint32_t sb = sreg[WBUF];  // E8M0 bytes: 2^(e - 127) is the float with exponent field e
            w0 = cvt_w4(w4reg[WBUF][0], __uint_as_float((sb & 0xffu) << 23));
            w1 = cvt_w4(w4reg[WBUF][1], __uint_as_float((sb >> 8) << 23));
        } else if (W8) {
            wait_load<AFTER>(wreg[WBUF][0]);
            const u32x4_t r = wreg[WBUF][0];
            w0 = cvt_w8(r[0], r[1]);
            w1 = cvt_w8(r[2], r[3]);
        } else {
            wait_loads<AFTER>(wreg[WBUF][0], wreg[WBUF][NWL - 1]);
            w0 = __builtin_bit_cast(bf16x8_t, wreg[WBUF][0]);
            w1 = __builtin_bit_cast(bf16x8_t, wreg[WBUF][NWL - 1]);
        }
        auto issue = [&](int lo, int hi) {  // loads number lo .. hi-1 of this iteration
#pragma unroll
            for (int i = lo; i < hi; i++) {
                if (i < MY_TILES) {
                    if (x_stage >= 0) x_issue_one(x_buf, x_stage, i);
                } else {
                    if (w_stage >= 0) w_issue_one((WBUF + DEPTH) % NBUF, w_stage, i - MY_TILES);
                }
            }
        };
        issue(0, PER_ITER);
#pragma unroll
        for (int b = 0; b + 1 < MT; b++) {
            const xfrag nxt = read_x(xbuf, b + 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma4(b, cur, w0, w1);
            __builtin_amdgcn_sched_barrier(0);
            cur = nxt;
        }
        __builtin_amdgcn_s_waitcnt(7 << 4 | 3 << 14 | 15);  // lgkmcnt(0) only
        __builtin_amdgcn_s_barrier();
        xfrag nxt = cur;
        if (more) nxt = read_x(xbuf == NXB - 1 ? 0 : xbuf + 1, 0);
        __builtin_amdgcn_sched_barrier(0);
        mfma4(MT - 1, cur, w0, w1);
        __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
    };
    using std::integral_constant;

    // prologue: activations of stages 0..DEPTH and weights of stages 0..DEPTH-1, in iteration order
    x_issue(0, 0);
#pragma unroll
    for (int u = 0; u < DEPTH; u++) {
        x_issue(u + 1, u + 1);
        w_issue(u, u);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(DEPTH * PER_ITER) : "memory");  // own tiles of stage 0
    __builtin_amdgcn_s_barrier();                                           // everybody's
    cur = read_x(0, 0);
    int xbuf = 0, fbuf = AHEAD;  // buffer being read; buffer the next activations go to
    int s0 = 0;
    auto advance = [&]() {
        xbuf = xbuf == NXB - 1 ? 0 : xbuf + 1;
        fbuf = fbuf == NXB - 1 ? 0 : fbuf + 1;
    };
    constexpr int STEADY = (DEPTH - 1) * PER_ITER;  // iterations s-DEPTH+1 .. s-1 have issued all their loads
    static_assert(DEPTH == 3 && NBUF == 4, "the trips below are written for three stages in flight");
    for (; s0 + NBUF < n_stage; s0 += NBUF) {
        // buffer fbuf held stage s-1: every reader passed the barrier of the previous iteration
        stage(integral_constant<int, STEADY>{}, xbuf, integral_constant<int, 0>{}, true, s0 + AHEAD, fbuf, s0 + DEPTH);
        advance();
        stage(integral_constant<int, STEADY>{}, xbuf, integral_constant<int, 1>{}, true, s0 + 1 + AHEAD, fbuf, s0 + 1 + DEPTH);
        advance();
        stage(integral_constant<int, STEADY>{}, xbuf, integral_constant<int, 2>{}, true, s0 + 2 + AHEAD, fbuf, s0 + 2 + DEPTH);
        advance();
        stage(integral_constant<int, STEADY>{}, xbuf, integral_constant<int, 3>{}, true, s0 + 3 + AHEAD, fbuf, s0 + 3 + DEPTH);
        advance();
    }
    // last trip: only the weights of the last stage are left to fetch (in its first iteration)
    stage(integral_constant<int, STEADY>{}, xbuf, integral_constant<int, 0>{}, true, -1, 0, s0 + DEPTH);
    advance();
    stage(integral_constant<int, PER_ITER + NWL + NSL>{}, xbuf, integral_constant<int, 1>{}, true, -1, 0, -1);
    advance();
    stage(integral_constant<int, NWL + NSL>{}, xbuf, integral_constant<int, 2>{}, true, -1, 0, -1);
    advance();
    stage(integral_constant<int, 0>{}, xbuf, integral_constant<int, 3>{}, false, -1, 0, -1);
    __syncthreads();  // every stage has been consumed and no load is in flight: the ring is free

    // ---- add the k-groups' sums through LDS ------------------------------------------------------------------------
    // A lane holds, per (column tile a, row tile b), four groups q of four consecutive columns: 4 * MT units
    // u = 4 * b + q per column tile.  The KG wavefronts that share a column group divide the units among themselves
    // in runs (k-group g owns units g * UPW .. (g + 1) * UPW - 1, i.e. whole row tiles when MT is a multiple of KG, so
    // that the stores of one wavefront fill whole 128-byte lines of an output row): each sends the units it does not
    // own to their owners and adds what it receives to its own, always in ascending k-group order.  Afterwards all
    // eight wavefronts hold a disjoint share of the block's outputs and all of them run the epilogue.
    // With two k-groups (the wide shape) k-group 0 owns everything instead and k-group 1 is done after sending: measured
    // 2 % faster there than sharing the epilogue, while with four k-groups four owners beat two (by 2 %) and one (by 20 %).
    constexpr int NOWN = KG == 2 ? 1 : KG;  // owning k-groups (0 .. NOWN-1)
    constexpr int UPW = 4 * MT / NOWN;               // units per owning wavefront and column tile
    auto owner = [](int b2, int q) { return (4 * b2 + q) / UPW; };
    // both column tiles in one pass where the parcels of both fit into the CU's 160 KiB, else one tile per pass
    constexpr int PARCELS_PER_TILE = CG * NOWN * (KG - 1) * UPW;  // KiB
    constexpr int PASSES = PARCELS_PER_TILE * NW <= 160 ? 1 : NW, TILES_PER_PASS = NW / PASSES;
    if (KG > 1) {
        float4_t* red = reinterpret_cast<float4_t*>(smem);
        // parcel (destination k-group, source k-group, unit, column tile within the pass): 64 lanes x 16 bytes
        auto parcel = [&](int dest, int src, int u, int ap) {
            // the destination has no slot of its own; src == dest is never accessed and maps to slot 0 to stay in range
            const int s2 = src < dest ? src : (src > dest ? src - 1 : 0);
            const int slot = ((cg * NOWN + dest) * (KG - 1) + s2) * UPW + (u - dest * UPW);
            return red + ((size_t)(slot * TILES_PER_PASS + ap)) * 64 + lane;
        };
#pragma unroll
        for (int pass = 0; pass < PASSES; pass++) {
#pragma unroll
            for (int ap = 0; ap < TILES_PER_PASS; ap++) {
                const int a = pass * TILES_PER_PASS + ap;
#pragma unroll
                for (int b2 = 0; b2 < MT; b2++)
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        if (owner(b2, q) != kgi)
                            *parcel(owner(b2, q), kgi, 4 * b2 + q, ap) =
                                float4_t{acc[a][b2][4 * q], acc[a][b2][4 * q + 1], acc[a][b2][4 * q + 2], acc[a][b2][4 * q + 3]};
            }
            __syncthreads();
#pragma unroll
            for (int ap = 0; ap < TILES_PER_PASS; ap++) {
                const int a = pass * TILES_PER_PASS + ap;
#pragma unroll
                for (int b2 = 0; b2 < MT; b2++)
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        if (owner(b2, q) == kgi) {
                            const float4_t own = {acc[a][b2][4 * q], acc[a][b2][4 * q + 1], acc[a][b2][4 * q + 2], acc[a][b2][4 * q + 3]};
                            float4_t v = kgi == 0 ? own : *parcel(kgi, 0, 4 * b2 + q, ap);
#pragma unroll
                            for (int src = 1; src < KG; src++) v += kgi == src ? own : *parcel(kgi, src, 4 * b2 + q, ap);
#pragma unroll
                            for (int i = 0; i < 4; i++) acc[a][b2][4 * q + i] = v[i];
                        }
            }
            if (pass + 1 < PASSES) __syncthreads();  // the parcels have been read: the next pass may overwrite them
        }
        if (kgi >= NOWN) return;
    }

    // epilogue: lane holds row (token) mt*32 + lane%32 and, in registers 4q .. 4q+3, the columns
    // nt*32 + 8q + (lane/32)*4 + 0..3; a wavefront stores the units it owns
#pragma unroll
    for (int a = 0; a < NW; a++) {
        if (!nt_ok[a]) continue;
        float4_t sc[4];
        if (W8) {  // 8-bit weights: the columns' scales
#pragma unroll
            for (int q = 0; q < 4; q++) sc[q] = *reinterpret_cast<const float4_t*>(scale + (nt0 + a) * 32 + q * 8 + (lane >> 5) * 4);
        }
#pragma unroll
        for (int b = 0; b < MT; b++) {
            const int tok = (mt_base + b) * 32 + (lane & 31);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                if (owner(b, q) != kgi) continue;
                const int n = (nt0 + a) * 32 + q * 8 + (lane >> 5) * 4;
                float4_t v = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
                if (W8) v *= sc[q];
                if (tok < T) store_cols<EPI>(v, tok, n, by, T_pad, N, out, out_act, act_plane, F_act);  // padding rows are never read
            }
        }
    }
}

// ------------------------------------------------------------------------------------------ tile kernel
// 16-bit weights.  With more than 128 rows the contraction is bound by the matrix pipes, so the workgroup is shaped for them.
// Four wavefronts, ONE per SIMD (512 registers each), own a tile of RT x 32 rows by 256 columns as 2 x 2 quarters; a
// quarter is RT/2 x 4 result tiles.  Both operands go through a ring of LDS stages of one k-step (16 k), filled
// by direct-to-LDS loads that keep as many stages in flight as the 160 KiB hold.  Per stage and wavefront (RT = 6):
// 24 MFMAs (768 clocks of the matrix pipe), 10 ds_read_b128, 5 loads and one barrier, so everything but the MFMAs
// fits into their issue gaps: operands of the next stage are read into a second register set between them.
//   - The k-steps of a slice go to 2 U sums in turn (U k-steps per stage: two sums beyond 128 rows, four in the slim tile),
//     which are added in ascending order at the end: the very sums that the k-groups of the wide and the narrow shape keep, so
//     a sum's rounding grows with a half or a quarter of the slice and a result does not depend on which kernel made it.
//     Two sums are what limits the height: 24 result tiles x 16 registers at RT = 6.  (220 rows x 8192 x 57344 took 387 us with
//     one sum at RT = 8, 408 with two at RT = 4, and 418 in the wide shape; but one sum has about 1.4 times the round-off.)
//   - Against the wide shape above (2 wavefronts per SIMD, weights straight to registers), which ran these cases before,
//     a k-step moves 20 KiB into the CU instead of 24 per 96 MFMAs (RT = 6), reads 40 KiB of LDS instead of 48, and has
//     no sums to exchange at the end; and its height can follow the batch (tile_height).  Gate/up of 372 rows x 4096
//     x 28672: 185 -> 138 us; of 700 rows: 290 -> 270 us = 1.22 PFLOP/s executed (both planes), where a large library
//     product on the same card reaches 1.41.
//   - One block of 33 to 128 rows runs in a slim tile, RT x 32 rows by 128 columns with two k-steps per stage: as many
//     workgroups as the narrow shape above and the same K slices, but no k-group sums to exchange at the end, a cost that a
//     launch of 15 to 60 us feels.  101 rows: gate/up 62.5 -> 61.3, QKV 22.7 -> 20.1 us; 8 layers and the head of the 8B
//     shape 1.54-1.62 -> 1.45-1.55 ms from card to card.  Three row tiles do not run here: they divide into column quarters
//     only, which read 28 KiB of LDS per k-step for 24 MFMAs (four tiles 24 for 32), and whether that is ahead of the narrow
//     shape depends on the card: 8 layers and the head at 84 rows 1.36 against 1.42 ms on one, 1.49 against 1.47 on another,
//     a prompt of 66 tokens 1.28 against 1.32 and 1.39 against 1.35.  (Dealt out as 2 + 1 row tiles it is the narrow shape's
//     time on both.)
// Loads and waits are written by hand as above; all vector-memory operations of the loop are direct-to-LDS loads, so
// no register is ever the target of a load in flight.
constexpr int TILE_WAVES = 4, TILE_CT = 8;
constexpr int SLIM_CT = 4, SLIM_U = 2;
constexpr int tile_stage_kib(int RT, int CT, int U) { return (PLANES * RT + CT) * U; }
// K is dealt out to the slices in units of 8 k-steps; a slice holds at least two units, so never fewer stages than the ring
constexpr int TILE_UNIT = 8, TILE_MIN_STAGES = 16;
static_assert(NARROW_KG * NBUF >= TILE_MIN_STAGES, "sled_launch_gemm has at most K / (16 NARROW_KG NBUF) slices");
// stages in the ring: what LDS holds, an even number, no more k-steps than the shortest slice has
constexpr int tile_ring(int RT, int CT, int U) { return std::min(160 / tile_stage_kib(RT, CT, U) / 2 * 2, TILE_MIN_STAGES / U); }
// a wavefront's sums, in tiles of 16 registers.  Up to eight of them (two row tiles of the slim tile) fit into the 256 registers of a launch bound
// of two wavefronts per SIMD, for which the compiler keeps MFMA results in ordinary registers: they are added up as they are,
// where accumulation registers are read into ordinary ones first.
constexpr int tile_sums(int RT, int CT, int U) { return 2 * U * RT * CT / TILE_WAVES; }

// RT, CT: row and column tiles of the workgroup; U: k-steps per stage; KEEP: weights in the caches' ordinary order
template <int RT, int CT, int U, int EPI, bool KEEP>
__global__ __launch_bounds__(64 * TILE_WAVES, tile_sums(RT, CT, U) <= 8 ? 2 : 1) void gemm_tile_kernel(const bf16_t* __restrict__ Xp, size_t x_plane,
                                                                       const bf16_t* __restrict__ Wp, int NT, int KS, int n_col,
                                                                       int n_split, int n_zb, int T, int T_pad, int N,
                                                                       float* __restrict__ out, bf16_t* __restrict__ out_act,
                                                                       size_t act_plane, int F_act) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int WR = 2, WC = TILE_WAVES / WR;                // wavefronts along rows and columns
    constexpr int HR = RT / WR, HC = CT / WC;                  // row and column tiles of a wavefront's quarter
    constexpr int XT = PLANES * RT * U, ST = XT + CT * U;      // 1 KiB operand tiles per stage: activations [k-step][plane][row tile], then weights [k-step][column tile]
    constexpr int NB = tile_ring(RT, CT, U);                   // stages in the ring = stages in flight
    constexpr int G = 2 * U;                                   // sums: k-step number s of the slice goes to number s % G
    constexpr int XL = XT / TILE_WAVES, WL = CT * U / TILE_WAVES, PER = XL + WL;   // loads per wavefront and stage
    static_assert(RT % WR == 0 && CT % WC == 0 && XT % TILE_WAVES == 0 && CT * U % TILE_WAVES == 0, "tiles do not divide among the wavefronts");
    static_assert(NB % 2 == 0 && TILE_UNIT % (2 * U) == 0 && NB * U <= TILE_MIN_STAGES, "the trips of the stage loop are written for an even ring");
    static_assert((NB - 1) * PER < 64, "too many loads in flight for the counter");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wv / WC, wc = wv % WC;
    // workgroup -> (column block, K slice, row block), as in gemm_bf16_kernel
    int bx, by, bz;
    {
        const int w = blockIdx.x, xcd = w & 7, local = w >> 3;
        bz = local % n_zb;
        const int t = (local / n_zb) * 8 + xcd;
        if (t >= n_col * n_split) return;
        bx = t % n_col;
        by = t / n_col;
    }
    const int units = KS / TILE_UNIT, ubase = units / n_split, urem = units - ubase * n_split;
    const int ks_begin = (by * ubase + min(by, urem)) * TILE_UNIT;
    const int n_stage = (ubase + (by < urem ? 1 : 0)) * (TILE_UNIT / U);   // even, at least the ring's length (the host sees to it)
    const int mt_base = bz * RT, nt_base = bx * CT;

    // ---- sources of this wavefront's loads: a uniform base per tile, advanced stage by stage, and a lane offset
    const int row_lim = (T + 7) & ~7;
    const char* xsrc[XL];
    unsigned xoff[XL];
    const char* wsrc[WL];
#pragma unroll
    for (int j = 0; j < XL; j++) {
        const int i = j * TILE_WAVES + wv, u = i / (PLANES * RT), pl = (i / RT) % PLANES, b = i % RT;
        const int mt = min(mt_base + b, T_pad / 32 - 1);   // a tile past the last one re-reads it; its results are not stored
        // lanes past the last token re-read the tile's first line (see gemm_bf16_kernel)
        const int src_lane = mt * 32 + (lane & 31) < row_lim ? lane : (lane & 32) + (lane & 7);
        xsrc[j] = reinterpret_cast<const char*>(Xp + pl * x_plane + ((size_t)mt * KS + ks_begin + u) * 512);
        xoff[j] = src_lane * 16;
    }
#pragma unroll
    for (int j = 0; j < WL; j++) {
        const int i = j * TILE_WAVES + wv, nt = min(nt_base + i % CT, NT - 1);
        wsrc[j] = reinterpret_cast<const char*>(Wp + ((size_t)(ks_begin + i / CT) * NT + nt) * 512);
    }
    const unsigned woff = lane * 16;
    const size_t wstep = (size_t)NT * (1024 * U);
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem + wv * 1024;
    // load number j of the next stage in order, into ring slot `buf`
    auto issue_one = [&](int buf, int j) {
        const unsigned slot = lds_base + (unsigned)buf * (ST * 1024);
        if (j < XL) {
            const unsigned dst = __builtin_amdgcn_readfirstlane(slot + j * (TILE_WAVES * 1024));
            asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(xoff[j < XL ? j : 0]), "s"(xsrc[j < XL ? j : 0]), "s"(dst) : "memory");
            xsrc[j < XL ? j : 0] += 1024 * U;
        } else {
            const int a = j < XL ? 0 : j - XL;
            const unsigned dst = __builtin_amdgcn_readfirstlane(slot + (XT + a * TILE_WAVES) * 1024);
            if constexpr (KEEP)
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(woff), "s"(wsrc[a]), "s"(dst) : "memory");
            else
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(woff), "s"(wsrc[a]), "s"(dst) : "memory");
            wsrc[a] += wstep;
        }
    };

    // The compiler gives all results of its MFMAs one kind of register, of which there are 256: 16 tiles.  Where there are more, the MFMAs
    // are written here with the first 16 tiles in accumulation registers and the rest in ordinary ones, tied to their places.  The
    // compiler does not know what such an instruction needs: nothing but another MFMA may touch a tile between the zeros below and
    // the wait behind the last stage (compiled code is checked for it).
    constexpr bool MORE_THAN_16 = G * HC * HR > 16;
    constexpr int IN_AGPR = tile_sums(RT, CT, U) <= 8 ? 0 : 16;
    auto in_agpr = [](int g, int a, int b) { return g * HC * HR + a * HR + b < IN_AGPR; };
    float16_t acc[G][HC][HR];

    struct frags {
        bf16x8_t x[U][PLANES][HR], w[U][HC];
    };
    constexpr int RS = PLANES * HR + HC, MS = PLANES * HR * HC;   // LDS reads and MFMAs per k-step ...
    constexpr int NR = RS * U, NM = MS * U;                       // ... and per stage
    const unsigned char* rd = smem + lane * 16;
    auto read_one = [&](frags& f, int buf, int rr) {   // per k-step weights first, then the hi plane, then the lo plane
        const unsigned char* p = rd + (unsigned)buf * (ST * 1024);
        const int u = rr / RS, r = rr - u * RS;
        if (r < HC)
            f.w[u][r < HC ? r : 0] = *reinterpret_cast<const bf16x8_t*>(p + (XT + u * CT + wc * HC + r) * 1024);
        else {
            const int e = r < HC ? 0 : r - HC, pl = e / HR, b = e - pl * HR;
            f.x[u][pl][b] = *reinterpret_cast<const bf16x8_t*>(p + ((u * PLANES + pl) * RT + wr * HR + b) * 1024);
        }
    };
    auto mfma_one = [&](const frags& f, int odd, int ii) {   // per k-step all tiles with the hi plane, then all with the lo plane
        const int u = ii / MS, i = ii - u * MS, pl = i / (HR * HC), e = i - pl * (HR * HC), b = e / HC, a = e - b * HC, g = odd * U + u;
        float16_t& c = acc[g][a][b];
        if (!MORE_THAN_16)
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[u][a], f.x[u][pl][b], c, 0, 0, 0);
        else if (in_agpr(g, a, b))
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(f.w[u][a]), "v"(f.x[u][pl][b]));
        else
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(f.w[u][a]), "v"(f.x[u][pl][b]));
    };
    auto pin_sums = [&]() {
#pragma unroll
        for (int g = 0; g < G; g++)
#pragma unroll
            for (int a = 0; a < HC; a++)
#pragma unroll
                for (int b = 0; b < HR; b++) {
                    if (in_agpr(g, a, b))
                        asm volatile("" : "+a"(acc[g][a][b]));
                    else
                        asm volatile("" : "+v"(acc[g][a][b]));
                }
    };
    // Stage s with its operands in `cur`: the operands of stage s+1 are read into `nxt`, and slot s % NB -- whose last
    // reads, those of stage s, every wavefront has back when it reaches the barrier -- is refilled with stage s+NB.
    // The wait before the barrier is for this wavefront's share of stage s+1; AFTER loads have been issued since.  ODD: s is odd.
    auto stage = [&](auto odd_c, auto after_c, auto load_c, auto more_c, const frags& cur, frags& nxt, int buf, int next_buf) {
        constexpr int ODD = decltype(odd_c)::value, AFTER = decltype(after_c)::value;
        constexpr bool LOAD = decltype(load_c)::value != 0, MORE = decltype(more_c)::value != 0;
        if (MORE) {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(AFTER) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
        constexpr int SPREAD = NM - 6 > NM / 2 ? NM - 6 : NM / 2;
        static_assert(PER <= NM, "one load per slot");
#pragma unroll
        for (int i = 0; i < NM; i++) {
            mfma_one(cur, ODD, i);
            if (LOAD && i < PER) issue_one(buf, i);
#pragma unroll
            for (int q = 0; q < NR; q++)   // the reads are spread over the slots up to the last few
                if (MORE && q * SPREAD / NR == i) read_one(nxt, next_buf, q);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using std::integral_constant;
    typedef integral_constant<int, 1> yes;
    typedef integral_constant<int, 0> no;

#pragma unroll
    for (int s2 = 0; s2 < NB; s2++)
#pragma unroll
        for (int j = 0; j < PER; j++) issue_one(s2, j);
    // zeros while the first loads are under way
#pragma unroll
    for (int g = 0; g < G; g++)
#pragma unroll
        for (int a = 0; a < HC; a++)
#pragma unroll
            for (int b = 0; b < HR; b++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[g][a][b][e] = 0.f;
    pin_sums();
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 1) * PER) : "memory");   // this wavefront's share of stage 0
    __builtin_amdgcn_s_barrier();                                           // everybody's
    asm volatile("" ::: "memory");
    frags f0, f1;
#pragma unroll
    for (int r = 0; r < NR; r++) read_one(f0, 0, r);
    int buf = 0;
    auto next = [&](int b2) { return b2 == NB - 1 ? 0 : b2 + 1; };
    auto trip = [&]() {   // n_stage and NB are even: both stages of a trip have one NB further on
        stage(no{}, integral_constant<int, (NB - 2) * PER>{}, yes{}, yes{}, f0, f1, buf, next(buf));
        buf = next(buf);
        stage(yes{}, integral_constant<int, (NB - 2) * PER>{}, yes{}, yes{}, f1, f0, buf, next(buf));
        buf = next(buf);
    };
    int s = 0;
    if constexpr (NB * U < TILE_MIN_STAGES) {   // there is a trip in every slice: as a do loop it leaves the sums where they are
        do {
            trip();
            s += 2;
        } while (s + NB < n_stage);
    } else {
        for (; s + NB < n_stage; s += 2) trip();
    }
    // the last NB stages fetch nothing: one stage fewer in flight behind the awaited one each time
    auto last = [&](auto self, auto left_c) {   // left: stages still to do
        constexpr int LEFT = decltype(left_c)::value;
        if constexpr (LEFT > 0) {
            constexpr int AFTER = LEFT >= 2 ? (LEFT - 2) * PER : 0;
            if constexpr (LEFT % 2 == 0) stage(no{}, integral_constant<int, AFTER>{}, no{}, yes{}, f0, f1, buf, next(buf));
            else if constexpr (LEFT > 1) stage(yes{}, integral_constant<int, AFTER>{}, no{}, yes{}, f1, f0, buf, next(buf));
            else stage(yes{}, integral_constant<int, 0>{}, no{}, no{}, f1, f0, buf, buf);
            buf = next(buf);
            self(self, integral_constant<int, LEFT - 1>{});
        }
    };
    last(last, integral_constant<int, NB>{});
    if (MORE_THAN_16) {
        asm volatile("s_nop 15\n\ts_nop 7");   // the last MFMA's result (11 wait states for one of eight passes; twice that)
        pin_sums();
    }

    // epilogue: lane holds row (token) mt*32 + lane%32 and, in registers 4q .. 4q+3, the columns nt*32 + 8q + (lane/32)*4 + 0..3
#pragma unroll
    for (int a = 0; a < HC; a++) {
        const int nt = nt_base + wc * HC + a;
        if (nt >= NT) continue;
#pragma unroll
        for (int b = 0; b < HR; b++) {
            const int tok = (mt_base + wr * HR + b) * 32 + (lane & 31);
            if (tok >= T) continue;   // padding rows are never read, or only by their own padding rows
#pragma unroll
            for (int q = 0; q < 4; q++) {
                auto quad = [&](int g) { return float4_t{acc[g][a][b][4 * q], acc[g][a][b][4 * q + 1], acc[g][a][b][4 * q + 2], acc[g][a][b][4 * q + 3]}; };
                float4_t v = quad(0);
#pragma unroll
                for (int g = 1; g < G; g++) v += quad(g);
                store_cols<EPI>(v, tok, nt * 32 + q * 8 + (lane >> 5) * 4, by, T_pad, N, out, out_act, act_plane, F_act);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------ k-wave kernel
// Up to 32 rows: few rows need few MFMAs, so what counts is that the weight stream never pauses and that a launch's fixed part is
// short.  A workgroup of four wavefronts, one per SIMD, owns RT x 32 rows by 128 columns; the k-steps of its slice are dealt
// out to the wavefronts in turn, and each multiplies its k-steps with all columns and all rows.  So no operand is needed by two
// wavefronts: everything goes from memory to registers, SETS k-steps ahead, with no LDS, no barrier and no wait for another
// wavefront in the loop, and the compiler counts the loads by itself.  The price is that the four sums of a result meet in LDS at
// the end (64 KiB per row tile; writing them is what LDS is slowest at, 78 bytes per clock measured, 250 for reading).
//   - Sum g of a result is that of the k-steps g, g + 4, ...; the four are added in ascending order: the sums of the narrow shape and of the
//     slim tile, so a result does not depend on which kernel made it.
//   - At one row, gate/up of 4096 x 28672 takes 37.4 us, 6.3 TB/s, the LM head 6.5 TB/s.  Inside a workgroup of gate/up: 1.4 us until the
//     first loads are out, 29.4 us for the loop, 1.6 us for the sums and SwiGLU; the other 4.8 us are dispatch, the slowest workgroup and the end.
//     Launch times, one row of 16-bit weights, slim tile of one row tile (which this replaced) against this: QKV 11.0 -> 11.2, O 9.6 -> 9.3,
//     gate/up 38.9 -> 37.5, down 21.6 -> 21.1 us; 25 rows of 8-bit weights, narrow shape against this: 10.4 -> 10.0, 8.3 -> 7.5,
//     27.5 -> 26.3, 16.9 -> 15.7; of 4-bit weights: 9.5 -> 8.9, 7.1 -> 6.9, 25.0 -> 21.0, 13.3 -> 13.0.
//   - Four sets of operands in flight saturate the stream; eight delay a short slice's first k-step behind 28 others (QKV 11.2 -> 11.7,
//     O 9.3 -> 10.0 us).  4-bit weights are the exception where a slice is long: the widening of a k-step's weights between the MFMAs
//     of the step before asks for them a step earlier, and there are few bytes to a step (gate/up at 25 rows 22.2 -> 21.0, at 58 rows 34.2 -> 31.1).
//   - More rows: at two row tiles 16- and 8-bit weights are no faster than in the kernels they have (gate/up 47.5 -> 49.0 and 35.8 -> 38.4), 4-bit
//     weights are where the slice is long (35.2 -> 31.1; QKV 14.3 -> 14.0, O 10.2 -> 10.4, down 19.6 -> 19.0 are left alone).
//     Three row tiles lose everywhere (54.4 -> 57.3), four do not fit into the registers.
constexpr int KW_CT = 4, KW_WAVES = 4;
constexpr int KW_MIN_STEPS = 16;     // k-steps of a slice come in multiples of this
// 4-bit slices from here on are long.  Whole steps of models whose gate/up and head have slices of so many k-steps, with eight sets in the slices
// from that length on against none, at 25 rows (four sets instead) and at 58 (the k-group kernel instead): 64 +1.3 and +5.1 %, 112 +1.9 and +4.2, 128 +0.4
// and +1.8, 160 +0.9 and +2.1, 192 +1.7 and +1.1, 256 -1.7 and -4.7, 512 -2.3 and -7.6.
constexpr int KW_DEEP_STEPS = 256;
static_assert(KW_DEEP_STEPS >= 8 * KW_WAVES, "eight sets are filled before the loop");
constexpr int kw_lds(int RT) { return KW_WAVES * KW_CT * RT * 4096; }

// SETS: k-steps whose operands are in registers or on their way; KEEP: weights in the caches' ordinary order
template <int RT, int WB, int SETS, bool KEEP>
__global__ __launch_bounds__(64 * KW_WAVES, 1) void gemm_kwave_kernel(const bf16_t* __restrict__ Xp, size_t x_plane,
                                                                      const unsigned char* __restrict__ Wp, const void* __restrict__ scale_v,
                                                                      int NT, int KS, int n_col, int n_split, int T, int T_pad, int N,
                                                                      float* __restrict__ out, bf16_t* __restrict__ out_act,
                                                                      size_t act_plane, int F_act, int epi) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int TB = 64 * WB;                        // bytes of a 32 x 16 weight tile
    constexpr int WL = WB == 16 ? 4 : 2;               // weight loads per k-step: a tile, or a pair of tiles
    constexpr int WR = WB == 4 ? 2 : 4;                // ... and their registers
    const int tid = threadIdx.x, lane = tid & 63, g = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int by = blockIdx.x / n_col, bx = blockIdx.x - by * n_col;
    const int len = KS / n_split;                      // k-steps of a slice: a multiple of KW_MIN_STEPS (the host sees to it)
    const int ks0 = by * len + g, n = len / KW_WAVES;  // this wavefront's: ks0, ks0 + 4, ...
    const int nt_base = bx * KW_CT;

    const size_t rowb = (size_t)NT * TB;               // bytes of a k-step of the whole matrix
    const char* wsrc = reinterpret_cast<const char*>(Wp) + (size_t)ks0 * rowb;
    const char* ssrc = WB == 4 ? static_cast<const char*>(scale_v) + (size_t)(ks0 >> 1) * (NT / 2) * 64 : nullptr;
    unsigned woff[WL], soff[WL];
#pragma unroll
    for (int i = 0; i < WL; i++) {   // column tiles past the last one re-read it; their results are not stored
        if (WB == 16)
            woff[i] = min(nt_base + i, NT - 1) * 1024 + lane * 16;
        else {
            const int pair = min(nt_base / 2 + i, NT / 2 - 1);
            woff[i] = pair * (2 * TB) + lane * (TB / 32);
            soff[i] = pair * 64 + (lane & 31) * 2;
        }
    }
    const int row_lim = (T + 7) & ~7;
    const char* xsrc[2];
    unsigned xoff[RT];
#pragma unroll
    for (int pl = 0; pl < 2; pl++) xsrc[pl] = reinterpret_cast<const char*>(Xp + pl * x_plane + (size_t)ks0 * 512);
#pragma unroll
    for (int b = 0; b < RT; b++) {
        // lanes past the last token re-read the tile's first line (see gemm_bf16_kernel)
        const int src_lane = b * 32 + (lane & 31) < row_lim ? lane : (lane & 32) + (lane & 7);
        xoff[b] = (unsigned)b * KS * 1024 + src_lane * 16;
    }
    typedef __attribute__((__vector_size__(WR * sizeof(unsigned)))) unsigned wreg_t;
    struct operands {
        bf16x8_t x[2][RT];
        wreg_t w[WL];
        uint32_t sc[WB == 4 ? WL : 1];
    } set[SETS];
    auto load_x = [&](operands& o, int pl, int b, int s) {
        o.x[pl][b] = *reinterpret_cast<const bf16x8_t*>(xsrc[pl] + (size_t)s * (KW_WAVES * 1024) + xoff[b]);
    };
    auto load_w = [&](operands& o, int i, int s) {
        const wreg_t* p = reinterpret_cast<const wreg_t*>(wsrc + (size_t)s * KW_WAVES * rowb + woff[i]);
        if constexpr (KEEP) o.w[i] = *p;
        else o.w[i] = __builtin_nontemporal_load(p);
        if (WB == 4) o.sc[i] = *reinterpret_cast<const uint16_t*>(ssrc + (size_t)s * (KW_WAVES / 2) * (NT / 2) * 64 + soff[i]);
    };

    float16_t acc[KW_CT][RT];
#pragma unroll
    for (int a = 0; a < KW_CT; a++)
#pragma unroll
        for (int b = 0; b < RT; b++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[a][b][e] = 0.f;
    auto widened = [&](const operands& o, int a) {
        const wreg_t& w = o.w[WB == 16 ? a : a / 2];
        if constexpr (WB == 16)
            return __builtin_bit_cast(bf16x8_t, w);
        else if constexpr (WB == 8)
            return a & 1 ? cvt_w8(w[2], w[3]) : cvt_w8(w[0], w[1]);
        else
            return cvt_w4(w[a & 1], __uint_as_float(((o.sc[a / 2] >> (8 * (a & 1))) & 0xffu) << 23));
    };
    // One k-step with the operands in `o`: the loads of the step four further on go into the registers as they fall free, and the
    // next step's weights (in `nx`) are widened between the MFMAs.
    bf16x8_t wb[2][KW_CT];
    auto compute = [&](operands& o, const operands& nx, auto par_c, bool more, bool widen, int s_next) {
        constexpr int PAR = decltype(par_c)::value;
#pragma unroll
        for (int pl = 0; pl < 2; pl++)
#pragma unroll
            for (int b = 0; b < RT; b++) {
                constexpr int GROUPS = 2 * RT, PER = (KW_CT + GROUPS - 1) / GROUPS;
                const int grp = pl * RT + b;
#pragma unroll
                for (int a = 0; a < KW_CT; a++) {
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(WB == 16 ? widened(o, a) : wb[PAR][a], o.x[pl][b], acc[a][b], 0, 0, 0);
                    if (WB != 16 && widen && a < PER && grp * PER + a < KW_CT) {
                        wb[PAR ^ 1][grp * PER + a] = widened(nx, grp * PER + a);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (more) load_x(o, pl, b, s_next);
                if (WB != 16 && more && grp == 0) {
#pragma unroll
                    for (int i = 0; i < WL; i++) load_w(o, i, s_next);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        if (WB == 16 && more) {
#pragma unroll
            for (int i = 0; i < WL; i++) load_w(o, i, s_next);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    using std::integral_constant;
    // four k-steps with the operands in sets BASE .. BASE + 3; those of SETS steps further on are requested if `more`
    auto trip = [&](auto base_c, bool more, int s) {
        constexpr int B0 = decltype(base_c)::value;
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
            compute(set[B0 + j], set[(B0 + j + 1) % SETS], integral_constant<int, 0>{}, more, true, s + j + SETS);
            compute(set[B0 + j + 1], set[(B0 + j + 2) % SETS], integral_constant<int, 1>{}, more, true, s + j + 1 + SETS);
        }
    };
    auto request = [&](auto base_c, int s) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
            operands& o = set[decltype(base_c)::value + j];
#pragma unroll
            for (int i = 0; i < WL; i++) load_w(o, i, s + j);
#pragma unroll
            for (int pl = 0; pl < 2; pl++)
#pragma unroll
                for (int b = 0; b < RT; b++) load_x(o, pl, b, s + j);
        }
    };
    typedef integral_constant<int, 0> low;
    typedef integral_constant<int, SETS - 4> high;
    static_assert(SETS == 4 || SETS == 8, "the trips are written for one or two halves of four sets");
    request(low{}, 0);
    if (SETS == 8) request(high{}, 4);   // n is a multiple of 4 and at least KW_DEEP_STEPS / KW_WAVES here
    if (WB != 16) {
#pragma unroll
        for (int a = 0; a < KW_CT; a++) wb[0][a] = widened(set[0], a);
    }
    int s = 0;
    if constexpr (SETS == 4) {
        for (; s + 4 < n; s += 4) trip(low{}, true, s);
        trip(low{}, false, s);
    } else {
        for (; s + 12 < n; s += 8) {
            trip(low{}, true, s);
            trip(high{}, true, s + 4);
        }
        // 8 or 12 steps are left
        const bool third = s + 8 < n;
        trip(low{}, third, s);
        trip(high{}, false, s);
        if (third) trip(low{}, false, s);
    }

    // The wavefronts' sums meet in LDS: wavefront g adds up column tile g, in ascending order
    float4_t* red = reinterpret_cast<float4_t*>(smem) + lane;
    const int nt = nt_base + g;
    float4_t sc[4];
    if (WB == 8 && nt < NT) {
#pragma unroll
        for (int q = 0; q < 4; q++) sc[q] = *reinterpret_cast<const float4_t*>(static_cast<const float*>(scale_v) + nt * 32 + q * 8 + (lane >> 5) * 4);
    }
#pragma unroll
    for (int a = 0; a < KW_CT; a++)
#pragma unroll
        for (int b = 0; b < RT; b++)
#pragma unroll
            for (int q = 0; q < 4; q++)
                red[(((a * KW_WAVES + g) * RT + b) * 4 + q) * 64] = float4_t{acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
    __syncthreads();
    if (nt >= NT) return;
#pragma unroll
    for (int b = 0; b < RT; b++) {
        const int tok = b * 32 + (lane & 31);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float4_t v = red[((g * KW_WAVES * RT + b) * 4 + q) * 64];
#pragma unroll
            for (int src = 1; src < KW_WAVES; src++) v += red[(((g * KW_WAVES + src) * RT + b) * 4 + q) * 64];
            if (WB == 8) v *= sc[q];
            const int n0 = nt * 32 + q * 8 + (lane >> 5) * 4;
            if (tok >= T) continue;   // padding rows are never read
            if (epi == SLED_EPI_SWIGLU)
                store_cols<SLED_EPI_SWIGLU>(v, tok, n0, by, T_pad, N, out, out_act, act_plane, F_act);
            else   // finished values are slice 0 of one
                store_cols<SLED_EPI_PARTIAL>(v, tok, n0, by, T_pad, N, out, out_act, act_plane, F_act);
        }
    }
}

// ------------------------------------------------------------------------------------------ fp32
// out[t][n] = sum_k X[t][k] W[n][k].  fp32 models are small, so a launch is a chain of memory round trips, not a stream: the
// work is cut fine and the chain kept short.  Workgroup = 16 tokens x 8 columns; the lanes of a wavefront lie along k (256 of it
// per trip, four to a lane), each wavefront has two columns, whose weights go straight to registers, and all share the
// trip's 16 x 256 activations in LDS; the next trip's operands are requested before this one's arithmetic.  At the end the 32
// sums are reduced over the lanes by halving: 32 exchanges, after which every other lane holds one output.
// 20 rows x 256 x 1024 (16 x 64 tiles before, a k at a time from LDS): 87 -> 8 us; x 2048 x 256: 22 -> 4.5 us.
constexpr int F32_T = 16, F32_NC = 2, F32_KC = 256;
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ X, const float* __restrict__ W, int T,
                                                       int N, int K, float* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) float xs[F32_T * F32_KC];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n0 = (blockIdx.x * 4 + wv) * F32_NC, t0 = blockIdx.y * F32_T;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 xr[4], wr[F32_NC];
    auto fetch = [&](int k0) {   // rows of float4: every K of an fp32 model is a multiple of 8
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int t = t0 + i * 4 + wv, k = k0 + lane * 4;
            xr[i] = zero;
            if (t < T && k < K) xr[i] = *reinterpret_cast<const float4*>(X + (size_t)t * K + k);
        }
#pragma unroll
        for (int c = 0; c < F32_NC; c++) {
            const int k = k0 + lane * 4;
            wr[c] = zero;
            if (n0 + c < N && k < K) wr[c] = *reinterpret_cast<const float4*>(W + (size_t)(n0 + c) * K + k);
        }
    };
    float v[F32_NC * F32_T];
#pragma unroll
    for (int i = 0; i < F32_NC * F32_T; i++) v[i] = 0.f;
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += F32_KC) {
        float4 w[F32_NC];
#pragma unroll
        for (int c = 0; c < F32_NC; c++) w[c] = wr[c];
        __syncthreads();   // the last trip's activations have been read
#pragma unroll
        for (int i = 0; i < 4; i++) *reinterpret_cast<float4*>(xs + (i * 4 + wv) * F32_KC + lane * 4) = xr[i];
        __syncthreads();
        if (k0 + F32_KC < K) fetch(k0 + F32_KC);
#pragma unroll
        for (int t = 0; t < F32_T; t++) {
            const float4 x = *reinterpret_cast<const float4*>(xs + t * F32_KC + lane * 4);
#pragma unroll
            for (int c = 0; c < F32_NC; c++) {
                float a = v[c * F32_T + t];
                a = fmaf(x.x, w[c].x, a);
                a = fmaf(x.y, w[c].y, a);
                a = fmaf(x.z, w[c].z, a);
                v[c * F32_T + t] = fmaf(x.w, w[c].w, a);
            }
        }
    }
    static_assert(F32_NC * F32_T == 32, "five halvings leave one value per lane");
#pragma unroll
    for (int s = 0; s < 5; s++) {
        const int off = 32 >> s, half = 16 >> s;
        const bool up = (lane & off) != 0;
#pragma unroll
        for (int i = 0; i < half; i++) {
            float a = v[i], b = v[i + half];
            asm("" : "+v"(a), "+v"(b));   // values, not places: the choice below must not become a dynamic index
            const float send = up ? a : b, keep = up ? b : a;
            v[i] = keep + __shfl_xor(send, off);
        }
    }
    v[0] += __shfl_xor(v[0], 1);
    const int c = lane >> 5, t = t0 + ((lane >> 1) & 15);   // value number lane / 2
    if (!(lane & 1) && n0 + c < N && t < T) out[(size_t)t * N + n0 + c] = v[0];
}

struct gemm_args {
    dim3 grid;
    size_t lds;
    hipStream_t st;
    const bf16_t* X;
    size_t x_plane;
    const bf16_t* W;
    const void* scale;
    int wbits;
    int NT, KS, n_col, n_split, n_zb, T, T_pad, N;
    float* out;
    bf16_t* out_act;
    size_t act_plane;
    int F_act;
};

template <int MT, int EPI, int KG, int CG, int WB, bool KEEP>
int launch_one(const gemm_args& a) {
    // more than 64 KiB of dynamic LDS has to be allowed once per kernel
    static bool allowed = false;
    auto kern = gemm_bf16_kernel<MT, EPI, KG, CG, WB, KEEP>;
    if (!allowed) {
        SLED_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds));
        allowed = true;
    }
    hipLaunchKernelGGL(kern, a.grid, dim3(64 * WAVES), a.lds, a.st, a.X, a.x_plane, a.W, a.scale, a.NT, a.KS, a.n_col,
                       a.n_split, a.n_zb, a.T, a.T_pad, a.N, a.out, a.out_act, a.act_plane, a.F_act);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

template <int RT, int CT, int U, int EPI, bool KEEP>
int launch_tile_one(const gemm_args& a) {
    static bool allowed = false;
    auto kern = gemm_tile_kernel<RT, CT, U, EPI, KEEP>;
    if (!allowed) {
        SLED_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds));
        allowed = true;
    }
    hipLaunchKernelGGL(kern, a.grid, dim3(64 * TILE_WAVES), a.lds, a.st, a.X, a.x_plane, a.W, a.NT, a.KS, a.n_col, a.n_split, a.n_zb,
                       a.T, a.T_pad, a.N, a.out, a.out_act, a.act_plane, a.F_act);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

template <int RT, int WB, int SETS, bool KEEP>
int launch_kwave(int epi, const gemm_args& a) {
    static bool allowed = false;
    auto kern = gemm_kwave_kernel<RT, WB, SETS, KEEP>;
    if (!allowed) {
        SLED_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kw_lds(RT)));
        allowed = true;
    }
    hipLaunchKernelGGL(kern, dim3(a.n_col * a.n_split), dim3(64 * KW_WAVES), kw_lds(RT), a.st, a.X, a.x_plane,
                       reinterpret_cast<const unsigned char*>(a.W), a.scale, a.NT, a.KS, a.n_col, a.n_split, a.T, a.T_pad, a.N, a.out,
                       a.out_act, a.act_plane, a.F_act, epi);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}

template <int RT, int CT = TILE_CT, int U = 1, bool KEEP = false>
int launch_tile(int epi, const gemm_args& a) {
    switch (epi) {
        case SLED_EPI_PARTIAL: return launch_tile_one<RT, CT, U, SLED_EPI_PARTIAL, KEEP>(a);
        case SLED_EPI_SWIGLU: return launch_tile_one<RT, CT, U, SLED_EPI_SWIGLU, KEEP>(a);
        default: return launch_tile_one<RT, CT, U, SLED_EPI_STORE, KEEP>(a);
    }
}

template <int MT, int KG, int CG, int WB, bool KEEP = false>
int launch_epi_wb(int epi, const gemm_args& a) {
    switch (epi) {
        case SLED_EPI_PARTIAL: return launch_one<MT, SLED_EPI_PARTIAL, KG, CG, WB, KEEP>(a);
        case SLED_EPI_SWIGLU: return launch_one<MT, SLED_EPI_SWIGLU, KG, CG, WB, KEEP>(a);
        default: return launch_one<MT, SLED_EPI_STORE, KG, CG, WB, KEEP>(a);
    }
}

template <int MT, int KG, int CG, bool KEEP = false>
int launch_epi(int epi, const gemm_args& a) {
    switch (a.wbits) {
        case 8: return launch_epi_wb<MT, KG, CG, 8, KEEP>(epi, a);
        case 4: return launch_epi_wb<MT, KG, CG, 4, KEEP>(epi, a);
        default: return launch_epi_wb<MT, KG, CG, 16, KEEP>(epi, a);
    }
}

}  // namespace

// Number of K slices for a projection of N columns over K.  More slices mean more workgroups (the
// chip wants at least one per CU) but more partial sums to reduce.  Each slice must hold a multiple
// of 4 stages of 64 k.
static sled_gemm_plan plan_one_block(int N, int K, bool needs_full_k);
static sled_gemm_plan plan_for_rows(sled_gemm_plan base, int N, int K, int T_pad);

sled_gemm_plan sled_gemm_make_plan(const sled_model* m, int N, int K, bool needs_full_k) {
    if (m->s.dtype != SLED_BF16) return sled_gemm_plan{1, 1};
    return plan_one_block(N, K, needs_full_k);
}

static sled_gemm_plan plan_one_block(int N, int K, bool needs_full_k) {
    sled_gemm_plan p{1, 1};
    auto legal = [&](int sp) { return sp >= 1 && (K / 16) % (sp * NARROW_KG * NBUF) == 0; };
    const int n_wg = (N + NARROW_COLS - 1) / NARROW_COLS;
    if (!needs_full_k)
        while (n_wg * p.split < 160 && legal(p.split * 2)) p.split *= 2;
    // a step with several blocks of rows may pick another number of slices, up to twice as many
    p.cap = needs_full_k || p.split == 1 ? p.split : std::min(2 * p.split, K / 16 / (NARROW_KG * NBUF));
    return p;
}

// With more than one block of 128 rows the workgroups of a projection are column blocks x row blocks x K slices, and what
// counts is how many rounds of 256 they make: 288 workgroups take as long as 512.  Fewer K slices also mean fewer
// partial sums to write and to read back.  Estimated time of a launch, in microseconds: rounds x (fixed part +
// stages of 32 k per workgroup x time per stage) + bytes of partial sums written and read / rate.  The slices are those of
// blocks of 128 rows by 256 columns for weights of any width: how many there are is part of how a row's sums are rounded, and
// the tile kernel takes them as they are, whatever its height.
sled_gemm_plan sled_gemm_plan_rows(const sled_model* m, sled_gemm_plan base, int N, int K, int T_pad) {
    if (m->s.dtype != SLED_BF16 || m->batch_invariant) return base;
    return plan_for_rows(base, N, K, T_pad);
}

static sled_gemm_plan plan_for_rows(sled_gemm_plan base, int N, int K, int T_pad) {
    if (base.split <= 1 || T_pad / 32 <= 4) return base;
    constexpr double FIXED_US = 9.0, STAGE_US = 0.8, PARTIAL_BYTES_PER_US = 4.0e6;
    const int n_col = (N / 32 + WIDE_CG * NW - 1) / (WIDE_CG * NW), zb = (T_pad / 32 + 3) / 4;
    const int units = K / 16 / (WIDE_KG * NBUF);   // trips of the stage loop in all of K
    sled_gemm_plan best = base;
    double best_t = -1.0;
    for (int sp = 1; sp <= base.cap && sp <= units; sp++) {
        const int64_t wgs = (int64_t)n_col * zb * sp;
        const int stages = (units + sp - 1) / sp * NBUF;   // of the longest slice
        const double t = (double)((wgs + 255) / 256) * (FIXED_US + stages * STAGE_US) + 2.0 * sp * (double)T_pad * N * 4.0 / PARTIAL_BYTES_PER_US;
        if (best_t < 0 || t < best_t) {
            best_t = t;
            best.split = sp;
        }
    }
    return best;
}

extern "C" int sled_projection_slices(int n_out, int n_in, int T, int* slices /*host out*/, int* max_slices /*host out*/) {
    if (!slices || !max_slices || n_out < 32 || n_in < 16 * NARROW_KG * NBUF || n_out % 32 || n_in % (16 * NARROW_KG * NBUF) || T < 1)
        SLED_FAIL(SLED_EINVAL, "sled_projection_slices: bad argument");
    const sled_gemm_plan base = plan_one_block(n_out, n_in, false);
    *slices = plan_for_rows(base, n_out, n_in, (T + 31) / 32 * 32).split;
    *max_slices = base.cap;
    return SLED_OK;
}

// Row tiles per workgroup of the tile kernel beyond 128 rows, 4 or 6, by the same estimate (without the partial sums, which do not
// depend on it).  Times per k-step on full rounds: 0.35-0.39 us at 4 row tiles (as the wide shape), 0.51-0.54 at 6.  So equal
// rows cost about the same at either height, and what the choice gives is better filled rounds: 372 rows x 4096 x 28672 are 336
// workgroups in two rounds at 4 row tiles (187 us) and 224 in one round at 6 (142 us); 220 x 8192 x 57344 are 448 in two
// rounds at either (415 and 556 us).
static double tile_us(int h, int N, int K, int T_pad, int split, double fixed_us, double step_us) {
    const int n_col = (N / 32 + TILE_CT - 1) / TILE_CT, steps = (K / 16 / TILE_UNIT + split - 1) / split * TILE_UNIT;   // of the longest slice
    const int64_t wgs = (int64_t)n_col * ((T_pad / 32 + h - 1) / h) * split;
    return (double)((wgs + 255) / 256) * (fixed_us + steps * step_us);
}
static int tile_height(int N, int K, int T_pad, int split) {
    constexpr double FIXED_US = 9.0, STEP4_US = 0.40, STEP6_US = 0.59;
    return tile_us(6, N, K, T_pad, split, FIXED_US, STEP6_US) < tile_us(4, N, K, T_pad, split, FIXED_US, STEP4_US) ? 6 : 4;
}

// How long a projection of T rows run by `plan` takes inside a slice of a prompt.  Fitted to the time per layer of slices of 32 to 1024 rows of ten
// models (d_model 1024 to 8192, 16-, 8- and 4-bit weights), which it meets within 8 % nearly everywhere, 12 % at worst.  Up to 128
// rows a launch, the weight stream, and for each further row tile its partial sums and products; beyond, rounds of workgroups as
// above and the partial sums written and read.
double sled_gemm_estimate_us(const sled_model* m, sled_gemm_plan plan, int N, int K, int T) {
    constexpr double LAUNCH_US = 9.0, WEIGHT_BYTES_PER_US = 6.2e6, ROW_TILE_US = 1.75;
    constexpr double FIXED_US = 7.5, STEP4_US = 0.363, STEP6_US = 0.524, STEP_LOWBIT_US = 0.333, PARTIAL_BYTES_PER_US = 4.0e6;
    const int T_pad = (T + 31) / 32 * 32, tiles = T_pad / 32;
    const double weights = (double)N * K;
    if (tiles <= 4)
        return LAUNCH_US + weights * (m->wbits / 8.0 + (m->wbits == 4 ? 1.0 / 32 : 0.0)) / WEIGHT_BYTES_PER_US +
               (tiles - 1) * (ROW_TILE_US + weights * (m->wbits == 16 ? 5.5e-8 : 8.5e-8));
    const int h = m->wbits == 16 ? tile_height(N, K, T_pad, plan.split) : 4;
    const double us = tile_us(h, N, K, T_pad, plan.split, FIXED_US, m->wbits != 16 ? STEP_LOWBIT_US : h == 6 ? STEP6_US : STEP4_US);
    return us + (plan.cap > 1 ? 2.0 * plan.split * (double)T_pad * N * 4.0 / PARTIAL_BYTES_PER_US : 0.0);
}

extern "C" int sled_projection_rows(int n_out, int n_in, int T, int* rows /*host out*/) {
    int slices, cap;
    if (!rows) SLED_FAIL(SLED_EINVAL, "sled_projection_rows: null argument");
    const int rc = sled_projection_slices(n_out, n_in, T, &slices, &cap);
    if (rc != SLED_OK) return rc;
    const int T_pad = (T + 31) / 32 * 32;
    *rows = T_pad <= 128 ? T_pad : 32 * tile_height(n_out, n_in, T_pad, slices);
    return SLED_OK;
}

int sled_launch_gemm(const sled_model* m, const void* X, size_t x_plane, const void* W, const void* scale, int T, int T_pad,
                     int N, int K, int epilogue, sled_gemm_plan plan, float* out_f32, void* out_act, size_t act_plane,
                     int F_act, hipStream_t st) {
    if (m->s.dtype == SLED_BF16) {
        const int NT = N / 32, KS = K / 16;
        if (N % 32 || K % 16 || T_pad % 32 || plan.split < 1 || KS % (NARROW_KG * NBUF) || plan.split > KS / (NARROW_KG * NBUF))   // a slice is never shorter than a trip of the narrow shape and than the tile kernel's ring
            SLED_FAIL(SLED_EINVAL, "gemm: unsupported shape N=%d K=%d T_pad=%d split=%d", N, K, T_pad, plan.split);
        const int mt_total = T_pad / 32;
        // up to 128 rows (4 tiles): k-wave kernel (one tile), slim tile (16-bit weights, two or four tiles) or narrow shape with exactly these tiles; more: the tile kernel at the height that suits
        // (bf16 weights) or blocks of four tiles in the wide shape (8- and 4-bit weights); the last block may reach past the end
        // (a batch-invariant model keeps the narrow shape at every size: the two shapes add the k-steps up in
        // different groupings, so a row's sums would depend on whether its batch has more than 128 rows)
        const bool wide = mt_total > 4 && !m->batch_invariant;
        const int zb = (mt_total + 3) / 4;
        const int MT = wide ? 4 : (mt_total + zb - 1) / zb;
        // one block of four row tiles, no K slices, and column blocks of 512 that fill at least three quarters of the CUs
        const bool broad = !wide && MT == 4 && plan.split == 1 && !m->batch_invariant && (NT + BROAD_CG * NW - 1) / (BROAD_CG * NW) >= 192;
        const int KG = wide ? WIDE_KG : broad ? BROAD_KG : NARROW_KG, CG = wide ? WIDE_CG : broad ? BROAD_CG : NARROW_CG;
        const int RT = wide && m->wbits == 16 ? tile_height(N, K, T_pad, plan.split) : 0;
        gemm_args a;
        a.n_col = (NT + CG * NW - 1) / (CG * NW);
        a.n_split = plan.split;
        a.n_zb = zb;
        a.grid = dim3((a.n_col * a.n_split + 7) / 8 * 8 * a.n_zb, 1, 1);
        // the ring of activation stages; afterwards the same memory holds the parcels the k-groups exchange
        // (every wavefront sends (KG - 1) / KG of its MT * 4 groups of 1 KiB per column tile)
        const size_t parcels = (size_t)WAVES * (KG - 1) * (4 * MT / KG);  // KiB per column tile; both tiles at once if they fit
        a.lds = std::max((size_t)NXB * PLANES * MT * KG * 1024, (parcels * NW <= 160 ? parcels * NW : parcels) * 1024);
        a.st = st;
        a.X = static_cast<const bf16_t*>(X);
        a.x_plane = x_plane;
        a.W = static_cast<const bf16_t*>(W);
        a.wbits = m->wbits;
        a.scale = m->wbits != 16 ? scale : nullptr;
        if (m->wbits != 16 && (!scale || N % 64 || K % 32))
            SLED_FAIL(SLED_EINVAL, "gemm: %d-bit weights need scales, N (%d) a multiple of 64 and K (%d) of 32", m->wbits, N, K);
        a.NT = NT;
        a.KS = KS;
        a.T = T;
        a.T_pad = T_pad;
        a.N = N;
        a.out = out_f32;
        a.out_act = static_cast<bf16_t*>(out_act);
        a.act_plane = act_plane;
        a.F_act = F_act;
        if (RT) {
            a.n_col = (NT + TILE_CT - 1) / TILE_CT;
            a.n_zb = (mt_total + RT - 1) / RT;
            a.grid = dim3((a.n_col * a.n_split + 7) / 8 * 8 * a.n_zb, 1, 1);
            a.lds = (size_t)tile_ring(RT, TILE_CT, 1) * tile_stage_kib(RT, TILE_CT, 1) * 1024;
            if (RT == 6) return launch_tile<6>(epilogue, a);
            // Two row blocks read the same weights, and where the second holds at most half the rows of the first it runs ahead of it: the weights
            // it has passed must still be in a cache then, so they are loaded in the caches' ordinary order (steps of the 8B shape, past the order /
            // in it: 144 rows 7.96 / 7.83 ms, 160 8.18 / 8.03, 192 8.23 / 8.20; with the second block fuller or more of them it is the other way
            // round: 224 rows 8.49 / 8.54, 256 8.57 / 8.68, 384 11.77 / 11.81, 512 15.02 / 15.11).
            return a.n_zb == 2 && mt_total - RT <= RT / 2 ? launch_tile<4, TILE_CT, 1, true>(epilogue, a) : launch_tile<4>(epilogue, a);
        }
        if (wide)
            return m->wbits == 8 ? launch_epi_wb<4, WIDE_KG, WIDE_CG, 8>(epilogue, a) : launch_epi_wb<4, WIDE_KG, WIDE_CG, 4>(epilogue, a);
        const int slice = KS / plan.split;
        if (mt_total <= 4 && (KS % plan.split || slice % KW_MIN_STEPS))   // every plan of one block of rows has equal slices of whole trips
            SLED_FAIL(SLED_EINVAL, "gemm: %d k-steps in %d slices", KS, plan.split);
        auto one_block = [&](auto keep_c) {
            constexpr bool KEEP = decltype(keep_c)::value;
            // up to 32 rows, and 4-bit weights up to 64 in long slices: the k-wave kernel (whose results do not depend on the choice either,
            // so batch-invariant models take it too)
            if (mt_total <= 2) {
                const bool deep = m->wbits == 4 && slice >= KW_DEEP_STEPS;
                a.n_col = (NT + KW_CT - 1) / KW_CT;
                if (mt_total == 1) {
                    switch (m->wbits) {
                        case 8: return launch_kwave<1, 8, 4, KEEP>(epilogue, a);
                        case 4: return deep ? launch_kwave<1, 4, 8, KEEP>(epilogue, a) : launch_kwave<1, 4, 4, KEEP>(epilogue, a);
                        default: return launch_kwave<1, 16, 4, KEEP>(epilogue, a);
                    }
                }
                if (deep) return launch_kwave<2, 4, 8, KEEP>(epilogue, a);
            }
            // one block of 33 or more rows, 16-bit weights: the slim tile kernel (three row tiles: the narrow shape)
            if (!broad && MT != 3 && m->wbits == 16 && !m->batch_invariant) {
                a.n_col = (NT + SLIM_CT - 1) / SLIM_CT;
                a.grid = dim3((a.n_col * a.n_split + 7) / 8 * 8, 1, 1);
                a.lds = (size_t)tile_ring(MT, SLIM_CT, SLIM_U) * tile_stage_kib(MT, SLIM_CT, SLIM_U) * 1024;
                return MT == 2 ? launch_tile<2, SLIM_CT, SLIM_U, KEEP>(epilogue, a) : launch_tile<4, SLIM_CT, SLIM_U, KEEP>(epilogue, a);
            }
            if (broad) return launch_epi<4, BROAD_KG, BROAD_CG>(epilogue, a);   // 98304 columns or more: seldom a model that a cache holds
            switch (MT) {
                case 2: return launch_epi<2, NARROW_KG, NARROW_CG, KEEP>(epilogue, a);
                case 3: return launch_epi<3, NARROW_KG, NARROW_CG, KEEP>(epilogue, a);
                default: return launch_epi<4, NARROW_KG, NARROW_CG, KEEP>(epilogue, a);
            }
        };
        // A model whose matrices Infinity Cache (256 MB) holds beside a step's activations finds them there in the next step, if they are loaded in the
        // caches' ordinary order.  Steps past the order / in it, us, 16-bit weights of 187 MB: one row 170 / 163, 25 195 / 185, 58 227 / 215, 101 275 / 266;
        // of 218 MB 204 / 198, 237 / 226, 277 / 264, 337 / 331; of 248 MB 241 / 250, 280 / 283, 327 / 328, 398 / 403; 4-bit weights of 197 MB with
        // their scales: 25 rows 277 / 260, 58 355 / 341, 101 498 / 485; of 229 MB 327 / 312, 421 / 408, 591 / 592 on one card and even on
        // another; of 261 MB 379 / 382, 487 / 490, 684 / 686.  With more than one block of rows it is even or the other way round (250
        // rows: 218 MB 490 / 494, 229 MB 846 / 861).
        constexpr double KEEP_BYTES = 224e6;
        const double weight_bytes = m->wbits / 8.0 + (m->wbits == 4 ? 1.0 / 32 : 0.0);
        const double matrices = weight_bytes * (m->s.n_layers * ((double)m->n_qkv * m->s.d_model + (double)m->s.d_model * m->s.n_q_heads * m->s.head_dim + 3.0 * m->s.d_ffn * m->s.d_model)
                                                + (double)m->s.vocab * m->s.d_model);
        return mt_total <= 4 && matrices <= KEEP_BYTES ? one_block(std::true_type{}) : one_block(std::false_type{});
    }
    // fp32: no split, plain store (partial buffer with one slice has the same layout)
    dim3 grid((N + 4 * F32_NC - 1) / (4 * F32_NC), (T + F32_T - 1) / F32_T);
    hipLaunchKernelGGL(gemm_f32_kernel, grid, dim3(256), 0, st, static_cast<const float*>(X),
                       static_cast<const float*>(W), T, N, K, out_f32);
    SLED_LAUNCH_CHECK();
    return SLED_OK;
}
