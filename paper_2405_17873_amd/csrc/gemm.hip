// MFMA GEMMs of the quantized-linear hot path for gfx950 (64-wide wavefronts, 32x32 MFMA tiles).
//
//   weight-only : Y = X . dequant(Wq)^T      fp16 / bf16 MFMA (v_mfma_f32_32x32x16_f16 / _bf16), fp32 accumulate
//                 (paper App. C item 2: weight-only layers keep 16-bit floating-point compute; also the layers kept
//                 at 16 bits, Sec. 4.2, whose weights pass unquantised)
//   int8        : ACC = A8 . W8^T            int8 MFMA (v_mfma_i32_32x32x32_i8), int32 accumulate
//                 (paper Sec. 4.3 / App. C item 4: integer GEMM for W8A8; 4-bit codes widened for W4A8)
// and, on the same skeleton, selected by the kernel's MODE: the gated feed-forward projection whose epilogue emits
// value * gelu(gate) as 8-bit codes or fp16, the int8 GEMM on activations that arrive as codes, and the 3x3
// convolution (Sec. 4.1: convolutions are quantised like linears) by addressing the filter taps in the activation loads.
//
// Shared structure
//   * One workgroup = WGM x WGN waves (x KS groups that split k); each wave owns TM x TN MFMA tiles of 32x32.
//   * Both operands go HBM -> LDS directly (buffer loads with the LDS bit: no staging registers) through a
//     pipeline of 2..8 LDS stages with hand-placed vmcnt waits and one barrier per stage; the hand-over to the
//     next stage sits in the middle of a stage, behind the MFMAs of its last two k-steps.
//   * Activations: 128 bytes of K per row per stage, 16-byte pieces XOR-swizzled (on the global side of the
//     copy) so that ds_read_b128 of 32 consecutive rows is conflict free.
//   * Weights stay PACKED in LDS: the kernel layout stores, for every 32-channel x 64-k tile, the 64 lane
//     chunks in lane order, so a tile is copied with one contiguous wave access and a lane later reads its own
//     chunk with one conflict-free ds_read; codes are widened in registers, right before the MFMA.
//   * The MFMA is issued with the weight fragment as the first operand: the 32x32 result then holds, per
//     lane, 4 consecutive output channels of one activation row; the epilogue transposes through LDS and stores
//     16-byte row segments.
//   * k-order inside a stage is permuted identically for both operands (a sum does not care), chosen so
//     that every lane's global and LDS accesses are 16 bytes wide.
//   * Few tiles and a long reduction: several workgroups per tile, partial sums through the caller's workspace,
//     the last-arriving workgroup adds them in a fixed order (no waiting).
//   * Optional residual operand (a skip connection, or the output of the other half of a split concatenated
//     input, Sec. 4.1): a kernel variant (RES) loads it in the accumulator layout and adds it in fp32 before the
//     one rounding; kernels without it contain none of this.
#include <stdio.h>

#include <atomic>
#include <mutex>

#include "gemm_core.h"

namespace mq {

// MODE 0: Y = linear(X).  MODE 1 (int8, two channel tiles per wave): gated feed-forward projection; the wave's first
// channel tile is a value tile, its second the gate tile of the same 32 columns, and the epilogue emits
// value * gelu(gate) as 8-bit codes for the next integer GEMM.  MODE 2 (int8): the activations arrive as codes with
// their parameters; the row sums the epilogue needs are accumulated in the main loop.  MODE 3 / 4: 3x3 convolution
// (16-bit / 8-bit activations).  MODE 5 (int8): the gated projection of MODE 1 without output parameters: it writes
// the fp16 product and one (min, max) pair per workgroup, from which the codes follow in a pass of their own.
// MODE 6 (16-bit activations): the gated projection of the weight-only path with MODE 1's 8-bit output.
template <bool I8, int BITS, int WGM, int WGN, int TM, int TN, int S, int KS, bool BF = false, int MODE = 0,
          bool RES = false>
__global__ __launch_bounds__(WGM* WGN* KS * 64,
                             (TM * TN <= 8 && GemmPlan<I8, BITS, WGM, WGN, TM, TN, S, KS>::LDS_BYTES <= 80 * 1024) ? 2 : 1)
void gemm_kernel(const GemmArgs g) {
    static_assert(!(I8 && BF), "the int8 path writes fp16");
    constexpr bool GEGLU = MODE == 1 || MODE == 5 || MODE == 6, RS_INLINE = MODE == 2 || MODE == 4, CONV = MODE == 3 || MODE == 4;
    constexpr bool RANGE = MODE == 5;    // gated projection that leaves the fp16 product and its range, no codes
    constexpr bool CODES16 = MODE == 6;  // gated projection of the 16-bit-activation path that emits 8-bit codes
    static_assert(MODE == 0 || KS == 1 || (CONV && TM == 1), "in-workgroup k split: plain layers, and convolutions whose waves own one row slab");
    static_assert(!(RES && GEGLU), "the gated projection takes no residual");
    static_assert(!RANGE || (I8 && !BF), "the range output belongs to the int8 gated projection");
    static_assert(!GEGLU || !BF, "the gated projections write fp16 or codes");
    static_assert(!CODES16 || (!I8 && !BF), "MODE 6 is the fp16 weight-only gated projection with 8-bit output");
    static_assert((MODE != 2 && MODE != 4) || I8, "int8 modes");
    static_assert(MODE != 3 || !I8, "MODE 3 is the weight-only convolution");
    static_assert(!GEGLU || TN == 2, "value tile and gate tile per wave");
    using P = GemmPlan<I8, BITS, WGM, WGN, TM, TN, S, KS>;
    constexpr int NW = P::NW, NT = P::NT, BM = P::BM, BN = P::BN, CH = P::CH;
    constexpr int STAGE_BYTES = P::STAGE_BYTES;
    using acc_t = typename std::conditional<I8, int16v, float16v>::type;
    using frag_t = typename std::conditional<I8, int4v, half8>::type;

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int grp = wv / P::NWG, wvg = wv % P::NWG;  // k-split group, wave inside the group
    const int wm = wvg / WGN, wn = wvg % WGN;
    int bm, bn;
    // (the large wave tile has no registers to spare for the split of the reduction over workgroups, and no use
    // for it: its problems have hundreds of tiles)
    constexpr bool CAN_SPLIT = TM * TN <= 4 && TM != 3 && MODE == 0;
    const int splits = CAN_SPLIT ? g.splits : 1;
    uint32_t tile_u = blockIdx.x, sp_u = 0;  // sp: which part of the reduction this workgroup takes
    if (splits > 1) g.fd_splits.divmod(blockIdx.x, tile_u, sp_u);
    const int tile_id = (int)tile_u, sp = (int)sp_u;
    tile_of_block(tile_id, g, bm, bn);
    // n0: first output column of the workgroup (MODE 1: first gated column; it covers BN / 2 of them)
    const int m0 = bm * BM, n0 = GEGLU ? bn * (BN / 2) : bn * BN;
    const int KC = g.K >> 6;
    const int G = (g.N + 31) >> 5;
    const int H = g.N >> 1;  // MODE 1: gated columns
    // local 32-channel group (wave column * TN + channel tile) -> group of weight rows, clamped to an existing one
    auto group_of = [&](int gt) {
        int gi = GEGLU ? ((gt % TN) ? (H >> 5) : 0) + (n0 >> 5) + gt / TN : (n0 >> 5) + gt;
        return gi < G ? gi : G - 1;
    };
    const int l31 = lane & 31, kb = lane >> 5;
    const uint32_t xflip = (I8 && g.w_off) ? 0x80808080u : 0u;
    constexpr int TILE_B = 256 * BITS;
    constexpr int OOB = 0x7FFFF000;  // an offset past the end of any buffer this library accepts

    const int4s ra = make_rsrc(g.a, g.a_bytes);
    const int4s rb = make_rsrc(g.packed, g.packed_bytes);
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;

    // activation loads: lane -> (row, physical slot) of an 8-row group; it fetches the logical piece slot ^ swz(row).
    // Rows past M get an offset past the end of the buffer and therefore read as zero.
    int a_voff[P::DMA_A];
    uint32_t a_lds[P::DMA_A];
    int a_sub[KS == 2 ? P::DMA_A : 1];  // k-split tiles: which of the stage's two k steps the load belongs to
    int a_half[CONV ? P::DMA_A : 1];
    uint32_t a_taps[CONV ? P::DMA_A : 1];
    // convolution: the input pixel that output pixel m is centred on, and which rows and columns of the filter read inside the
    // image there (3 bits each)
    struct Centre {
        int index;
        uint32_t rows, cols;
        __device__ uint32_t taps() const {  // bit r * 3 + s: filter tap (r, s) reads inside the image
            return (rows & 1u ? cols : 0u) | cols << 3 | (rows & 4u ? cols << 6 : 0u);
        }
    };
    auto centre_of = [&](int m) -> Centre {
        uint32_t row, jo, bi, io;
        g.fd_wo.divmod((uint32_t)m, row, jo);
        g.fd_ho.divmod(row, bi, io);
        const int i = (int)io * g.conv_stride, j = (int)jo * g.conv_stride;
        return Centre{((int)bi * g.conv_h + i) * g.conv_w + j, (i > 0 ? 1u : 0u) | 2u | (i + 1 < g.conv_h ? 4u : 0u),
                      (j > 0 ? 1u : 0u) | 2u | (j + 1 < g.conv_w ? 4u : 0u)};
    };
#pragma unroll
    for (int i = 0; i < P::DMA_A; ++i) {
        const int j = i * NW + wv;
        const int sub = j / (BM / 8), row0 = (j % (BM / 8)) * 8;
        const int row = row0 + (lane >> 3);
        const int piece = (lane & 7) ^ swz(row);
        a_voff[i] = m0 + row < g.M ? (int)((long)(m0 + row) * g.a_row_bytes + sub * 128 + piece * 16) : OOB;
        if constexpr (KS == 2) a_sub[i] = __builtin_amdgcn_readfirstlane(sub);
        a_lds[i] = __builtin_amdgcn_readfirstlane((uint32_t)(sub * P::SUB_BYTES + row0 * 128));
        if constexpr (CONV) {
            // row = output pixel; the lane's 16 bytes of a stage lie in one 64-channel chunk (int8: piece / 4 says
            // which of the stage's two), i.e. in one filter tap: per stage it adds that tap's pixel offset, or
            // reads nothing (zero) where the tap falls outside the image
            const bool real = m0 + row < g.M;
            const Centre c = centre_of(real ? m0 + row : g.M - 1);
            a_voff[i] = (int)((long)c.index * g.a_row_bytes) + (I8 ? (piece & 3) : piece) * 16;
            a_half[i] = I8 ? piece >> 2 : 0;
            a_taps[i] = real ? c.taps() : 0u;  // (rows past M read nothing)
        }
    }
    // weight loads: instruction jj of a sub-stage copies piece jj % PCS of weight tile jj / PCS (tile = channel group,
    // chunk)
    constexpr int PCS = P::PIECES;
    constexpr int VALID_LANES = BITS >= 8 ? 64 : 16 * BITS;  // lanes of a 16-byte-per-lane copy that hold tile data
    int b_voff[P::DMA_B];
    uint32_t b_lds[P::DMA_B];
    constexpr bool B_TAIL = I8 || KS == 2;  // a stage may reach past the last 64-k weight tile of the reduction
    int b_chunk[B_TAIL ? P::DMA_B : 1];     // the load's 64-k tile inside its stage
#pragma unroll
    for (int i = 0; i < P::DMA_B; ++i) {
        const int j = i * NW + wv;
        const int sub = j / P::NBI1, jj = j % P::NBI1;
        const int t = jj / PCS, piece = jj % PCS;
        const int gt = t / CH, cc = t % CH;
        const int gi = group_of(gt);
        const bool on = j < P::NBI && lane < VALID_LANES;
        b_voff[i] = on ? (gi * KC + sub * CH + cc) * TILE_B + piece * 1024 + lane * 16 : OOB;
        if constexpr (B_TAIL) b_chunk[i] = sub * CH + cc;
        b_lds[i] = __builtin_amdgcn_readfirstlane(
            j < P::NBI ? (uint32_t)(sub * P::SUB_BYTES + P::A_BYTES + t * P::BSLOT + piece * 1024) : (uint32_t)0xFFFFFFFFu);
    }

    // Weight zero points of the 16-bit-activation path (the int8 path corrects for them in the epilogue): an ordinary
    // load here would be waited for by the compiler with a count that ignores the LDS-writing loads, i.e. until all
    // prologue stages have landed.  So the zero points of the workgroup's channels travel like a stage: one
    // LDS-writing load per 64 channels, issued first (the oldest entry of the counter), into the slot that the int8
    // epilogue uses for its own constants; every lane picks its channel's value up after the first barrier.
    constexpr bool ZP_LDS = !I8 && BITS != 16;
    constexpr int ZP_SLOT = P::CONSTS + 2 * BN * 4;
    if constexpr (ZP_LDS) {
        if (wv < BN / 64) {
            const int ch = wv * 64 + lane;
            int n = group_of(ch >> 5) * 32 + (ch & 31);
            n = n < g.N ? n : g.N - 1;
            const int4s rz = make_rsrc(g.w_zp, (uint32_t)g.N * 4u);
            dma_to_lds_b32(rz, __builtin_amdgcn_readfirstlane(lds_base + ZP_SLOT + wv * 256), n * 4, 0);
        }
    }
    int zc[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) zc[tn] = 0;

    // Without an in-workgroup k split every wave's first k step exists, so its MFMAs take the constant zero as their
    // third operand and the accumulators need no clearing (16 vector instructions per MFMA tile otherwise).
    constexpr bool ZERO_C = KS == 1 && !CONV;  // (the convolution kernels have no registers to spare for the second copy of step 0)
    acc_t acc[TM][TN];
    if constexpr (!ZERO_C) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;
    }

    // Per-channel epilogue inputs of the workgroup's BN channels: thread t fetches those of channel n0 + t now and
    // keeps them in registers; they are combined and parked in LDS after the loop.  These ordinary loads are issued
    // BEFORE the first LDS-writing load, so that they are the oldest entries of the vector-memory counter and the
    // hand-counted waits below see only the stage loads behind them.
    static_assert(BN <= NT, "one thread per channel");
    float c_scale = 0.0f;
    uint32_t c_bias_bits = 0;  // converted where it is used, after the loop: a conversion here would wait for the load
    int c_zp = 0, c_colsum = 0;
    // (the activation parameters are the same for every thread: loaded outside the divergent branch they stay in
    // scalar registers, and nothing waits for them before the epilogue)
    float c_sx = 1.0f;
    int c_zx = 0;
    if constexpr (I8) {
        c_sx = RS_INLINE ? *g.act_scale_p : g.params->scale;
        c_zx = RS_INLINE ? *g.act_zp_p : g.params->zp;
    }
    if (threadIdx.x < BN) {
        int n = group_of((int)threadIdx.x >> 5) * 32 + ((int)threadIdx.x & 31);
        n = n < g.N ? n : g.N - 1;
        c_scale = BITS == 16 ? 1.0f : g.w_scale[n];
        if (g.bias) c_bias_bits = g.bias[n];
        if constexpr (I8) {
            c_zp = g.w_zp[n];
            c_colsum = g.w_colsum[n];
        }
    }
    int rsum[TM];
    // int8 convolution: the row's class of missing taps, first and last filter row in bits 2 and 3, column in bits 0 and 1
    int border[MODE == 4 ? TM : 1];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        int m = m0 + (wm * TM + tm) * 32 + l31;
        m = m < g.M ? m : g.M - 1;
        rsum[tm] = (I8 && !RS_INLINE) ? g.rowsum[m] : 0;
        if constexpr (MODE == 4) {
            const Centre c = centre_of(m);
            border[tm] = (int)((c.rows & 1u ? 0u : 4u) | (c.rows & 4u ? 0u : 8u) | (c.cols & 1u ? 0u : 1u) | (c.cols & 4u ? 0u : 2u));
        }
    }

    // Every wave issues exactly OPS loads per stage (padding loads go to the sink), so that "at most n * OPS loads
    // outstanding" means "all but the n youngest stages have landed" for every wave alike.
    const int KSTEPS = g.k_stages;                // 128-byte k steps
    const int KT_ALL = (KSTEPS + KS - 1) / KS;    // pipeline stages of the whole reduction
    const int kt0 = splits > 1 ? sp * g.kt_q + (sp < g.kt_r ? sp : g.kt_r) : 0;
    const int KT = splits > 1 ? g.kt_q + (sp < g.kt_r ? 1 : 0) : KT_ALL;  // ... of this workgroup
    // The k advance of a stage travels in the load's scalar offset, which the hardware leaves out of its range check
    // (only the lane's own offset is compared with the extent of the buffer).  The last stage may hold a 64-k weight
    // tile or (k-split tiles) a whole k step that does not exist: int8 stages are two weight tiles long and K / 64 may
    // be odd, a k-split stage is two k steps long and their number may be odd.  Loads of such phantom pieces get the
    // out-of-range lane offset, so nothing outside the operands is ever addressed.
    auto issue = [&](int stage, int buf) {
        const int step0 = (kt0 + stage) * KS;  // first k step of the stage
        const int soff_a = __builtin_amdgcn_readfirstlane(step0 * 128);
        const int soff_b = __builtin_amdgcn_readfirstlane(step0 * CH * TILE_B);
        const uint32_t sb = lds_base + buf * STAGE_BYTES;
        const bool tail_a = KS == 2 && step0 + 1 >= KSTEPS;
        const bool tail_b = B_TAIL && (step0 + KS) * CH > KC;
        if constexpr (CONV) {
            // the stage's 64-channel chunks -> (filter tap, chunk inside the tap) -> byte offset from the output pixel
            int tap[KS * CH], delta[KS * CH];
#pragma unroll
            for (int h = 0; h < KS * CH; ++h) {
                const uint32_t ci = (uint32_t)step0 * CH + h;
                const uint32_t t = g.conv_cpt > 1 ? __umulhi(ci, g.conv_cpt_inv) : ci;
                const int cc = (int)(ci - t * g.conv_cpt);
                tap[h] = ci < (uint32_t)KC ? (int)t : 31;  // past the end of K (padding of the last stage): no tap
                // (one scalar: taken apart, its terms meet the lane's offset in vector multiplications, 20 instructions per load)
                delta[h] = __builtin_amdgcn_readfirstlane((((int)t / 3 - 1) * g.conv_w + ((int)t % 3 - 1)) * (int)g.a_row_bytes +
                                                          cc * (I8 ? 64 : 128));
            }
#pragma unroll
            for (int i = 0; i < P::DMA_A; ++i) {
                // (KS == 2: a_sub says whether the load belongs to the stage's second k step)
                const int h0 = KS == 2 ? (a_sub[i] ? CH : 0) : 0;
                const int t0 = h0 ? tap[KS == 2 ? CH : 0] : tap[0], d0 = h0 ? delta[KS == 2 ? CH : 0] : delta[0];
                const int t1 = h0 ? tap[KS * CH - 1] : tap[CH - 1], d1 = h0 ? delta[KS * CH - 1] : delta[CH - 1];
                const int t = CH == 2 && a_half[i] ? t1 : t0, d = CH == 2 && a_half[i] ? d1 : d0;
                const int in = (int)(a_taps[i] << (31 - t)) >> 31;  // all ones where the tap reads inside the image
                const int voff = (in & (a_voff[i] + d)) | (~in & OOB);
                dma_to_lds_b128(ra, __builtin_amdgcn_readfirstlane(sb + a_lds[i]), voff, 0);
            }
        } else if (tail_a) {
            if constexpr (KS == 2) {
#pragma unroll
                for (int i = 0; i < P::DMA_A; ++i)
                    dma_to_lds_b128(ra, __builtin_amdgcn_readfirstlane(sb + a_lds[i]),
                                    step0 + a_sub[i] < KSTEPS ? a_voff[i] : OOB, soff_a);
            }
        } else {
#pragma unroll
            for (int i = 0; i < P::DMA_A; ++i)
                dma_to_lds_b128(ra, __builtin_amdgcn_readfirstlane(sb + a_lds[i]), a_voff[i], soff_a);
        }
        if (tail_b) {
            if constexpr (B_TAIL) {
#pragma unroll
                for (int i = 0; i < P::DMA_B; ++i)
                    dma_to_lds_b128(rb, __builtin_amdgcn_readfirstlane(b_lds[i] == 0xFFFFFFFFu ? lds_base + P::SINK : sb + b_lds[i]),
                                    step0 * CH + b_chunk[i] < KC ? b_voff[i] : OOB, soff_b);
            }
        } else {
#pragma unroll
            for (int i = 0; i < P::DMA_B; ++i)
                dma_to_lds_b128(rb, __builtin_amdgcn_readfirstlane(b_lds[i] == 0xFFFFFFFFu ? lds_base + P::SINK : sb + b_lds[i]),
                                b_voff[i], soff_b);
        }
    };

    // LDS read offsets of this lane: row l31 of the wave's first tile, one register per MFMA step
    const int sw = swz(l31);
    uint32_t rd[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int piece = I8 ? ((s >> 1) * 4 + kb * 2 + (s & 1)) : (kb * 4 + s);
        rd[s] = (uint32_t)(wm * TM * 32 * 128 + l31 * 128 + ((piece ^ sw) << 4));
    }

    long long t0 = 0, t1 = 0, t2 = 0;
    if (g.phase_clk) t0 = clock64();
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < KT) issue(s, s);
    if (g.phase_clk) t1 = clock64();

    // Main loop.  A 32-cycle MFMA leaves room for about five vector ALU instructions on its SIMD (measured: four
    // behind every MFMA cost nothing, eight cost 37 % more time than the MFMAs alone), and a workgroup has one wave
    // per SIMD, so the widening work is spread between the MFMAs and every latency is covered by the wave's own MFMAs:
    //   * the activation fragments of steps 1..3 are requested one or two steps ahead (four register sets);
    //   * the hand-over to the next stage (wait for its loads, barrier, refill of the buffer just read, request of
    //     its first fragments) sits in the MIDDLE of a stage, after the last LDS read of the current stage has
    //     returned and before the MFMAs of steps 2 and 3, which then run while the barrier settles and the first
    //     fragments of the next stage travel.
    WChunk<BITS> wq[TN][CH];
    frag_t xf[4][TM];
    auto request_first = [&](const uint8_t* abuf) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int c = 0; c < CH; ++c)
                read_chunk<BITS>(wq[tn][c], abuf + P::A_BYTES + ((wn * TN + tn) * CH + c) * P::BSLOT, lane);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xf[0][tm] = *(const frag_t*)(abuf + rd[0] + tm * 32 * 128);
    };
    auto widen = [&](frag_t (&wf)[TN], int s) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            if constexpr (I8)
                wf[tn] = widen_step<BITS>(wq[tn][s >> 1], s & 1, xflip);
            else if constexpr (BF && KS == 1)
                wf[tn] = dequant_step_bf16<BITS>(wq[tn][0], s, zc[tn]);
            else
                wf[tn] = dequant_step<BITS>(wq[tn][0], s, zc[tn]);
            if constexpr (BF && KS == 2 && BITS != 16) wf[tn] = half8_to_bf16x8(wf[tn]);  // bf16 bits now
        }
    };
    constexpr int RS_SHARES = WGN == 4 ? 4 : 1;  // waves that share the row sums of the rows they hold
    const int wn_u = __builtin_amdgcn_readfirstlane(wn);
    auto multiply = [&](const frag_t (&wf)[TN], int s, auto fresh_c) {
        constexpr bool FRESH = decltype(fresh_c)::value;  // the accumulators start here: C = 0
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                acc_t c;
                if constexpr (FRESH) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) c[i] = 0;
                } else {
                    c = acc[tm][tn];
                }
                if constexpr (I8)
                    acc[tm][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[tn], xf[s][tm], c, 0, 0, 0);
                else if constexpr (BF)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8, wf[tn]), __builtin_bit_cast(bf16x8, xf[s][tm]), c, 0, 0, 0);
                else
                    acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[tn], xf[s][tm], c, 0, 0, 0);
            }
        // Row sums of the stored activations (bytes a' = code - 128).  Where four waves hold the same rows each takes the
        // fragments of one k-step in four: four dot products per fragment, in every wave, were more vector instructions than the
        // code widening (feed-forward pair 16384 x 640 162 -> 159 us a pass with the share).  Two such waves take all: the turns
        // cut the loop into branches, which costs more than half the sums (1024 x 2560 x 640 at 4 bits, tile 2: 11.35 us with turns,
        // 10.46 without; convolutions of few tiles, tile 4: 2 %; 8-bit tile 1 2 %).
        if constexpr (RS_INLINE) {
            if (RS_SHARES == 1 || s % RS_SHARES == wn_u) {
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    const int4v a = __builtin_bit_cast(int4v, xf[s][tm]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) rsum[tm] = __builtin_amdgcn_sdot4(a[i], 0x01010101, rsum[tm], false);
                }
            }
        }
    };

    // stage 0 must have landed; the younger stages stay in flight
    constexpr int W_FIRST = (S - 1) * P::OPS <= 63 ? (S - 1) * P::OPS : (S > 2 ? (S - 2) * P::OPS : 0);
    if (KT >= S)
        wait_vmcnt<W_FIRST>();
    else
        wait_vmcnt<0>();
    __syncthreads();
    if constexpr (ZP_LDS) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) zc[tn] = *(const int*)(lds + ZP_SLOT + ((wn * TN + tn) * 32 + l31) * 4);
    }
    if constexpr (TM == 1 && TN == 1 && MODE != 0) {
        // One MFMA a step covers neither the LDS round trip of the next step's fragment nor the widening: a stage of the small tile was a chain
        // of four such trips, 600 cycles for 128 of MFMAs.  Its fragments are few, so a wave holds those of two stages: all of the next
        // stage's are requested at the hand-over, the current one's are widened ahead of it and multiplied behind it.  us: convolutions 1 x 20 x 20 x 1280
        // at 4 bits on 16-bit activations 57.4 -> 54.7, on 8-bit ones 45.4 -> 41.8 (8 bits 46.4 -> 43.5), 2 x 32 x 32 x 640 with stride 2 26.9 -> 25.2; on
        // codes 500 x 5120 x 1280 17.2 -> 16.5.  Not plain linears, whose reductions are split further: 0.97 to 1.02, at 8 bits 1.0 to 1.16.
        int buf = 0;
        WChunk<BITS> wq2[2][CH];
        frag_t xf2[2][4];
        auto request = [&](int set, const uint8_t* abuf) {
#pragma unroll
            for (int c = 0; c < CH; ++c) read_chunk<BITS>(wq2[set][c], abuf + P::A_BYTES + (wn * CH + c) * P::BSLOT, lane);
#pragma unroll
            for (int s = 0; s < 4; ++s) xf2[set][s] = *(const frag_t*)(abuf + rd[s]);
        };
        auto stage = [&](int set, int kt) {
            const bool live = KS == 1 || (kt0 + kt) * KS + grp < KSTEPS;
            frag_t wf[4][TN];
#pragma unroll
            for (int c = 0; c < CH; ++c) wq[0][c] = wq2[set][c];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                widen(wf[s], s);
                asm volatile("" : "+v"(wf[s][0]), "+v"(xf2[set][s]));  // here, not behind the requests below
                xf[s][0] = xf2[set][s];
            }
            __builtin_amdgcn_sched_barrier(0);
            const int nb = buf + 1 == S ? 0 : buf + 1;
            if (kt + 1 < KT) {
                // hand-over, as in the loop below
                if (S > 2 && kt + S - 1 < KT)
                    wait_vmcnt<(S > 2 ? (S - 2) * P::OPS : 0)>();
                else
                    wait_vmcnt<0>();
                __syncthreads();
                if (kt + S < KT) issue(kt + S, buf);
                request(set ^ 1, lds + nb * STAGE_BYTES + grp * P::SUB_BYTES);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (ZERO_C && kt == 0)
                multiply(wf[0], 0, std::true_type{});
            else if (live)
                multiply(wf[0], 0, std::false_type{});
            if (live) {
#pragma unroll
                for (int s = 1; s < 4; ++s) multiply(wf[s], s, std::false_type{});
            }
            __builtin_amdgcn_sched_barrier(0);
            buf = nb;
        };
        request(0, lds + grp * P::SUB_BYTES);
        for (int kt = 0; kt < KT; kt += 2) {
            stage(0, kt);
            if (kt + 1 < KT) stage(1, kt + 1);
        }
    } else {
    request_first(lds + grp * P::SUB_BYTES);

    int buf = 0;
    for (int kt = 0; kt < KT; ++kt) {
        const uint8_t* abuf = lds + buf * STAGE_BYTES + grp * P::SUB_BYTES;
        // odd tail of a k-split: the last k step of group 1 does not exist (it still takes part in the barriers)
        const bool live = KS == 1 || (kt0 + kt) * KS + grp < KSTEPS;
        frag_t wf[2][TN];
        // step 0
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xf[1][tm] = *(const frag_t*)(abuf + rd[1] + tm * 32 * 128);
        __builtin_amdgcn_sched_barrier(0);
        widen(wf[0], 0);
        if (ZERO_C && kt == 0)
            multiply(wf[0], 0, std::true_type{});
        else if (live)
            multiply(wf[0], 0, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        // step 1: the last LDS reads of this stage
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xf[2][tm] = *(const frag_t*)(abuf + rd[2] + tm * 32 * 128);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xf[3][tm] = *(const frag_t*)(abuf + rd[3] + tm * 32 * 128);
        __builtin_amdgcn_sched_barrier(0);
        widen(wf[1], 1);
        if (live) multiply(wf[1], 1, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        // the packed weights of this stage are widened completely before their registers are reused
        widen(wf[0], 2);
        widen(wf[1], 3);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)  // materialise them here (the compiler would otherwise sink them past the branch)
            asm volatile("" : "+v"(wf[0][tn]), "+v"(wf[1][tn]));
        __builtin_amdgcn_sched_barrier(0);
        int nb = buf + 1 == S ? 0 : buf + 1;
        if (kt + 1 < KT) {
            // hand-over: stage kt+1 must have landed (the S-2 stages behind it may stay in flight while they exist);
            // the barrier also says that every wave holds its last fragments of stage kt, so its buffer is refilled
            if constexpr (TM == 1 && TN == 1 && KS == 2 && !I8 && !BF) {
                // (The same in a function of its own: the compiler lays this loop out another way.  64 x 64 with two wave groups without a workspace, us:
                // 196 x 4928 x 448 at 8 bits 22.9 -> 21.5, 8 x 3904 x 1176 at 3 bits 19.1 -> 18.3.  Elsewhere written out is the better one:
                // int8 2964 x 1280 x 1280 at 8 bits 12.23, in a function 12.38.)
                auto hand_over = [&](int kt) {
                    if (S > 2 && kt + S - 1 < KT)
                        wait_vmcnt<(S > 2 ? (S - 2) * P::OPS : 0)>();
                    else
                        wait_vmcnt<0>();
                    __syncthreads();
                    if (kt + S < KT) issue(kt + S, buf);
                };
                hand_over(kt);
            } else {
                if (S > 2 && kt + S - 1 < KT)
                    wait_vmcnt<(S > 2 ? (S - 2) * P::OPS : 0)>();
                else
                    wait_vmcnt<0>();
                __syncthreads();
                if (kt + S < KT) issue(kt + S, buf);
            }
            request_first(lds + nb * STAGE_BYTES + grp * P::SUB_BYTES);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (live) {
            multiply(wf[0], 2, std::false_type{});
            multiply(wf[1], 3, std::false_type{});
        }
        __builtin_amdgcn_sched_barrier(0);
        buf = nb;
    }
    }
    __syncthreads();  // every wave is done reading the stages: what follows may overwrite them

    // Row sums in parts: lanes l and l + 32 hold two shares of row l's, the waves that share them and the wave groups one each.
    // They meet in the idle sink of the padding loads.
    constexpr int RS_PARTS = KS * RS_SHARES;
    int* const rs_x = (int*)(lds + P::SINK) + wm * TM * 32 + l31;
    if constexpr (RS_INLINE) {
        static_assert(RS_PARTS == 1 || RS_PARTS * BM * 4 <= P::CONSTS - P::SINK, "shares of the row sums fit the sink");
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            rsum[tm] += __shfl_xor(rsum[tm], 32, 64);
            if (RS_PARTS > 1 && lane < 32 && (RS_SHARES > 1 || wn == 0)) rs_x[(grp * RS_SHARES + (RS_SHARES > 1 ? wn : 0)) * BM + tm * 32] = rsum[tm];
        }
    }

    // Park the per-channel constants in LDS behind the stages: multiplier, additive term and (int8) the two
    // zero-point corrections.
    //   weight-only: y = acc * s_w[n] + bias[n]
    //   int8: stored operands are a' = qx - 128 and b' = qw - w_off; with dx = 128 - z_x, dw = w_off - z_w[n]:
    //         ACC = raw + dw * rowsum_a'[m] + dx * (colsum_b'[n] + K * dw),  colsum_b' = colsum - K * w_off,
    //         y = ACC * (s_x * s_w[n]) + bias[n].  Wrap-around int32 arithmetic is exact because ACC itself fits.
    float* ch_mul = (float*)(lds + P::CONSTS);
    float* ch_add = ch_mul + BN;
    int* ch_dw = (int*)(ch_add + BN);
    int* ch_cn = ch_dw + BN;
    // (int8 convolution: [16][BN], at the end of the idle stages, beyond what the epilogue puts there)
    int* const ch_border = (int*)(lds + S * STAGE_BYTES) - 16 * BN;
    if (threadIdx.x < BN) {
        const int t = threadIdx.x;
        if constexpr (I8) {
            // (nothing derived from the activation parameters is computed before this point: the arithmetic would
            // wait for their load at the top of the kernel, ahead of the first stage's requests)
            asm volatile("" : "+s"(c_zx), "+s"(c_sx));
            const int dx = 128 - c_zx;
            const int dw = g.w_off - c_zp;
            ch_dw[t] = dw;
            const int cn = dx * (c_colsum - g.K * g.w_off + g.K * dw);
            ch_cn[t] = cn;
            if constexpr (MODE == 4) {
                // A filter tap outside the image reads zero bytes, which stand for the code 128, not for the value 0 (code
                // z_x).  cn counts every tap; each class of border pixels takes back dx * sum_c (q_w - z_w) of the
                // taps it does not have: a table of the classes, from which a lane reads its row's constants.  (With the
                // per-tap sums read by the border lanes, the addresses of issue() in vector multiplications and the row sums in
                // every wave, the block 2 x 128 x 128, 320 -> 320 with downsampler at 4 bits took 200 us, now 156.)
                int n = group_of(t >> 5) * 32 + (t & 31);
                n = n < g.N ? n : g.N - 1;
                int tap[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) tap[i] = g.w_tapsum[i * g.N + n];
#pragma unroll
                for (int cls = 0; cls < 16; ++cls) {
                    int missing = 0, taps_missing = 0;
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const int r = i / 3, c = i % 3;
                        if ((r == 0 && (cls & 4)) || (r == 2 && (cls & 8)) || (c == 0 && (cls & 1)) || (c == 2 && (cls & 2))) {
                            missing += tap[i];
                            ++taps_missing;
                        }
                    }
                    ch_border[cls * BN + t] = cn - dx * (missing - taps_missing * (g.conv_cpt * 64) * c_zp);
                }
            }
        }
        // (gated projection: half of the value channels, for two_gelu32)
        const float half_v = GEGLU && !((t >> 5) & 1) ? 0.5f : 1.0f;
        ch_mul[t] = half_v * (c_scale * c_sx);
        asm volatile("" : "+v"(c_bias_bits));  // (keeps the compiler from moving the conversion up to the load)
        ch_add[t] = half_v * (BF ? bf16_bits_to_float((uint16_t)c_bias_bits)
                                 : (float)__builtin_bit_cast(_Float16, (uint16_t)c_bias_bits));
    }

    // k-split: the two groups' partial sums meet through LDS ([register quad][lane], 16 bytes per lane).  With an
    // even number of row slabs per wave each group finishes half of them (it sends the other half across and adds
    // what it receives), so both groups take part in the epilogue; otherwise group 1 sends everything to group 0.
    constexpr bool SPLIT_EPI = KS == 2 && TM % 2 == 0;
    constexpr int TMX = SPLIT_EPI ? TM / 2 : TM;  // slabs one wave sends
    auto owner = [](int tm) { return SPLIT_EPI ? (tm & 1) : 0; };
    if constexpr (KS == 2) {
        using quad_t = typename std::conditional<I8, int4v, float4v>::type;
        constexpr int XW = TMX * TN * 4 * 1024;  // bytes one wave sends
        static_assert(P::NWG * (SPLIT_EPI ? 2 : 1) * XW + (MODE == 4 ? 64 * BN : 0) <= S * STAGE_BYTES, "accumulator exchange must fit the stages");
        auto area = [&](int writer) { return lds + (SPLIT_EPI ? wvg * 2 + writer : wvg) * XW + lane * 16; };
        uint8_t* out = area(grp);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (owner(tm) == grp) continue;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    quad_t v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[tm][tn][4 * q + r];
                    *(quad_t*)(out + (((SPLIT_EPI ? tm >> 1 : tm) * TN + tn) * 4 + q) * 1024) = v;
                }
        }
        __syncthreads();
        const uint8_t* in = area(1 - grp);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (owner(tm) != grp) continue;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const quad_t v = *(const quad_t*)(in + (((SPLIT_EPI ? tm >> 1 : tm) * TN + tn) * 4 + q) * 1024);
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[tm][tn][4 * q + r] += v[r];
                }
        }
        __syncthreads();
    }

    if constexpr (KS == 1) __syncthreads();  // constants visible (the k-split exchange above has its own barriers)
    if constexpr (RS_INLINE && RS_PARTS > 1) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            rsum[tm] = 0;
#pragma unroll
            for (int i = 0; i < RS_PARTS; ++i) rsum[tm] += rs_x[i * BM + tm * 32];
        }
    }

    // Reduction split over workgroups: every workgroup stores its partial sums (register order, one 4-byte value per
    // lane per store: fully coalesced; rows past M skipped), then takes a ticket; the one that draws the last ticket
    // adds the partial sums of all parts, its own included, in part order (so the result does not depend on which
    // workgroup came last) and goes on to the epilogue; the others are done.  Nobody waits for anybody.
    // The partial sums are written and read with device-scope atomic accesses (write-through stores, loads that
    // bypass the L2 of the reader's XCD); every wave waits for its stores to complete, the workgroup meets at a
    // barrier, and one thread draws the ticket with a device-scope acquire-release read-modify-write, which orders
    // the stores of this workgroup before the ticket and the loads of the last workgroup after it.
    unsigned long long* counter = nullptr;
    if (CAN_SPLIT && splits > 1) {
        // (the arguments of the split are read here: the compiler would otherwise request them ahead of the main loop, whose
        // first LDS reads then wait for them, also in calls that do not split: 4 x 1280 x 1280 at 4 bits 7.56 us, 7.39 here)
        auto args = (const __attribute__((address_space(4))) GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        counter = args->counters + tile_id * args->counter_step;
        const unsigned long long split_tag = args->split_tag;
        using elem_t = typename std::conditional<I8, int, float>::type;
        const size_t tile_elems = (size_t)BM * BN;
        elem_t* mine = (elem_t*)(args->partial + ((size_t)tile_id * splits + sp) * tile_elems);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (KS > 1 && owner(tm) != grp) continue;
            if (m0 + (wm * TM + tm) * 32 + l31 >= g.M) continue;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    __hip_atomic_store(mine + (((wvg * TM + tm) * TN + tn) * 16 + i) * 64 + lane, (elem_t)acc[tm][tn][i],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (threadIdx.x == 0) {
            // The tile's arrival counter arrives with unknown contents.  Every part makes sure before it counts that the
            // upper 44 bits hold this launch's tag (a cleared word, then whatever the first exchange found, is replaced;
            // where the second exchange fails another part's has succeeded).  Here the answer travels beside the stores
            // above, which have to be waited for anyway.  (Behind the requests of the first stages the compiler waits for all
            // of those with it: 308 x 2048 x 640 in bf16 19.9 us with the exchange there, 17.2 here.)
            unsigned long long seen = 0;
            if (!__hip_atomic_compare_exchange_strong(counter, &seen, split_tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT) &&
                (seen & ~SPLIT_COUNT) != split_tag)
                __hip_atomic_compare_exchange_strong(counter, &seen, split_tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        }
        wait_vmcnt<0>();  // this wave's stores have completed (reached the level all compute units see)
        __syncthreads();
        uint32_t* ticket = (uint32_t*)(lds + P::SINK);  // the sink of padding loads is idle by now
        if (threadIdx.x == 0)
            *ticket = (uint32_t)__hip_atomic_fetch_add(counter, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) & (uint32_t)SPLIT_COUNT;
        __syncthreads();
        if (*ticket != (uint32_t)(splits - 1)) return;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;
        // (the loads of PU parts are requested together where the registers allow; the additions keep part order)
        constexpr int PU = TM * TN == 1 ? 4 : 1;
        for (int part0 = 0; part0 < splits; part0 += PU) {
            elem_t v[PU][TM][TN][16];
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int part = part0 + u < splits ? part0 + u : splits - 1;
                const elem_t* theirs = (const elem_t*)(args->partial + ((size_t)tile_id * splits + part) * tile_elems);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    if (KS > 1 && owner(tm) != grp) continue;
                    if (m0 + (wm * TM + tm) * 32 + l31 >= g.M) continue;
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                        for (int i = 0; i < 16; ++i)
                            v[u][tm][tn][i] =
                                __hip_atomic_load(theirs + (((wvg * TM + tm) * TN + tn) * 16 + i) * 64 + lane,
                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                if (part0 + u >= splits) break;
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    if (KS > 1 && owner(tm) != grp) continue;
                    if (m0 + (wm * TM + tm) * 32 + l31 >= g.M) continue;
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[tm][tn][i] += v[u][tm][tn][i];
                }
            }
        }
    }
    if (g.phase_clk) t2 = clock64();
    // ---------------------------------------------------------------- epilogue
    // Result element v of a lane is channel 8*(v/4) + 4*kb + v%4 of its 32-channel tile, activation row l31:
    // four consecutive channels of ONE row per lane, so a direct store would scatter 8-byte pieces over 32 rows.
    // Instead every wave transposes through its own slice of the (now idle) LDS stages, in slabs of 32 rows by the
    // wave's TN channel tiles: finished fp16 values are written as 8-byte pieces into a [32 rows][TN*32 channels]
    // image (16-byte chunks XOR-swizzled by row), read back as 16 bytes per lane along rows, and stored with 4*TN
    // lanes covering one contiguous row segment of TN*64 bytes.
    if constexpr (GEGLU) {
        // value * gelu(gate) -> 8-bit codes in the int8 activation layout (a' = code - 128, groups of 8 columns in
        // the order 0,4,1,5,2,6,3,7, columns from H to the row stride zero), optionally the product itself as fp16.
        // A lane holds four consecutive columns of one row; the lane 32 further on holds the other four of the same
        // group of 8, so the two swap their packed words and each keeps one of the group's two output words.
        // Rows are staged through LDS (32 rows x 32 bytes per wave) and leave as 16-byte pieces.
        // (without output parameters the kernel only writes the product and its range: the codes follow in a pass of
        // their own once the range of the whole tensor is known)
        // Vector instructions bound it (the pass of 16384 x 640 -> 2 x 2560 -> 640 with run-time ranges:
        // 178 -> 167 us; waves of two row slabs, three workgroups per compute unit, 10 % slower), so the constants of a
        // register quad are read once for all row slabs and the range is taken from pairs of fp16 values.
        constexpr bool want_codes = (I8 && !RANGE) || CODES16;
        float inv_o = 0.0f, zf_o = 0.0f;
        if constexpr (want_codes) {
            inv_o = __fdiv_rn(1.0f, *g.out_scale_p);
            zf_o = (float)*g.out_zp_p;
        }
        // range of the values as they are stored (fp16), per row slab: a row that does not exist is left out at the end
        uint2v hmn4[TM], hmx4[TM];  // pairs of fp16 values
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            hmn4[tm] = uint2v{0x7C007C00u, 0x7C007C00u};  // infinity
            hmx4[tm] = uint2v{0xFC00FC00u, 0xFC00FC00u};
        }
        constexpr int SLAB = 1024 + 2048;  // codes and fp16 image of 32 rows x 32 columns
        static_assert(P::NWG * TM * SLAB <= S * STAGE_BYTES, "epilogue staging must fit the LDS stages");
        uint8_t* const ep8 = lds + wvg * TM * SLAB;
        uint8_t* const ep16 = ep8 + 1024;
        const int col0 = n0 + wn * 32;  // first gated column of this wave
        const bool real_cols = __builtin_amdgcn_readfirstlane(col0 < H ? 1 : 0);  // (all 32 or none: H is a multiple of 32)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cl_v = (wn * TN) * 32 + 8 * q + 4 * kb, cl_g = cl_v + 32;
            const float4v mul_v = *(const float4v*)(ch_mul + cl_v), add_v = *(const float4v*)(ch_add + cl_v);
            const float4v mul_g = *(const float4v*)(ch_mul + cl_g), add_g = *(const float4v*)(ch_add + cl_g);
            int4v dw_v = {0, 0, 0, 0}, cn_v = dw_v, dw_g = dw_v, cn_g = dw_v;
            if constexpr (I8) {
                dw_v = *(const int4v*)(ch_dw + cl_v), cn_v = *(const int4v*)(ch_cn + cl_v);
                dw_g = *(const int4v*)(ch_dw + cl_g), cn_g = *(const int4v*)(ch_cn + cl_g);
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                uint32_t word = 0;
                float lv[4], tg[4];  // value / 2 and 2 gelu(gate)
                half4 hh;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float lg;
                    if constexpr (I8) {
                        const int av = acc[tm][0][4 * q + r] + __mul24(dw_v[r], rsum[tm]) + cn_v[r];
                        const int ag = acc[tm][1][4 * q + r] + __mul24(dw_g[r], rsum[tm]) + cn_g[r];
                        lv[r] = __fmaf_rn((float)av, mul_v[r], add_v[r]);
                        lg = __fmaf_rn((float)ag, mul_g[r], add_g[r]);
                    } else {
                        lv[r] = __fmaf_rn(acc[tm][0][4 * q + r], mul_v[r], add_v[r]);
                        lg = __fmaf_rn(acc[tm][1][4 * q + r], mul_g[r], add_g[r]);
                    }
                    tg[r] = two_gelu32(lg);
                    if constexpr (!RANGE) {
                        // the fp32 product, rounded once more where it is stored as fp16 (kept apart from that conversion, which
                        // the compiler may otherwise fuse with it: one rounding, and a zero product loses its sign)
                        float h = __fmul_rn(lv[r], tg[r]);
                        asm("" : "+v"(h));
                        if constexpr (want_codes)  // (the conversion saturates to 0..255 and takes NaN to 0)
                            word = __builtin_amdgcn_cvt_pk_u8_f32(__fadd_rn(rintf(__fmul_rn(h, inv_o)), zf_o), r, word);
                        hh[r] = (_Float16)h;
                    }
                }
                if constexpr (RANGE) hh = mul_to_half4(lv, tg);
                if constexpr (RANGE) {
                    const uint2v h2 = __builtin_bit_cast(uint2v, hh);
#pragma unroll
                    for (int p = 0; p < 2; ++p) {  // (written out: the compiler would first canonicalise both operands)
                        asm("v_pk_min_f16 %0, %1, %2" : "=v"(hmn4[tm][p]) : "v"(hmn4[tm][p]), "v"(h2[p]));
                        asm("v_pk_max_f16 %0, %1, %2" : "=v"(hmx4[tm][p]) : "v"(hmx4[tm][p]), "v"(h2[p]));
                    }
                }
                if constexpr (want_codes) {
                    word = real_cols ? word ^ 0x80808080u : 0u;  // code - 128
                    const uint32_t other = (uint32_t)__shfl_xor((int)word, 32, 64);
                    const uint32_t lo = kb ? other : word, hi = kb ? word : other;  // columns 0..3 and 4..7 of the group
                    // v_perm_b32: selector bytes 0..3 pick bytes of the second source, 4..7 of the first
                    const uint32_t out = kb ? __builtin_amdgcn_perm(hi, lo, 0x07030602u) : __builtin_amdgcn_perm(hi, lo, 0x05010400u);
                    *(uint32_t*)(ep8 + tm * SLAB + l31 * 32 + q * 8 + kb * 4) = out;
                }
                // (16-byte chunks XOR-ed with the row bits above those that separate rows inside one turn of the banks)
                if (g.y) *(half4*)(ep16 + tm * SLAB + l31 * 64 + ((q ^ (l31 >> 2)) & 3) * 16 + kb * 8) = hh;
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int mt0 = m0 + (wm * TM + tm) * 32;
            if constexpr (want_codes) {
                const int row = lane >> 1, half = lane & 1;
                const uint4v v = *(const uint4v*)(ep8 + tm * SLAB + row * 32 + half * 16);
                const int m = mt0 + row, col = col0 + half * 16;
                if (m < g.M && col < g.ld8) __builtin_nontemporal_store(v, (uint4v*)(g.a8_out + (long)m * g.ld8 + col));
            }
            if (g.y) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int idx = i * 64 + lane, row = idx >> 2, c = idx & 3;
                    const uint4v v = *(const uint4v*)(ep16 + tm * SLAB + row * 64 + ((c ^ (row >> 2)) & 3) * 16);
                    const int m = mt0 + row, col = col0 + c * 8;
                    if (m < g.M && col < H) __builtin_nontemporal_store(v, (uint4v*)(g.y + (long)m * g.ldy + col));
                }
            }
        }
        if constexpr (RANGE) {  // one pair per workgroup: waves meet through the (idle) sink of the padding loads
            float hmn = INFINITY, hmx = -INFINITY;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool ok = real_cols && m0 + (wm * TM + tm) * 32 + l31 < g.M;
                    hmn = fminf(hmn, ok ? (float)__builtin_bit_cast(half4, hmn4[tm])[r] : INFINITY);
                    hmx = fmaxf(hmx, ok ? (float)__builtin_bit_cast(half4, hmx4[tm])[r] : -INFINITY);
                }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                hmn = fminf(hmn, __shfl_xor(hmn, off, 64));
                hmx = fmaxf(hmx, __shfl_xor(hmx, off, 64));
            }
            float* mm = (float*)(lds + P::SINK);
            if (lane == 0) {
                mm[2 * wv] = hmn;
                mm[2 * wv + 1] = hmx;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                float a = mm[0], b = mm[1];
#pragma unroll
                for (int i = 1; i < NW; ++i) {
                    a = fminf(a, mm[2 * i]);
                    b = fmaxf(b, mm[2 * i + 1]);
                }
                g.mm_out[2 * blockIdx.x] = a;
                g.mm_out[2 * blockIdx.x + 1] = b;
            }
        }
    } else {
    static_assert(TN == 1 || TN == 2 || TN == 4, "channel tiles per wave: 1, 2 or 4");
    constexpr int EP_BYTES = 32 * TN * 64;          // staging bytes of one 32-row slab of a wave
    constexpr int EW = SPLIT_EPI ? NW : P::NWG;     // storing waves
    // Where the idle stages have the room, a wave stages all its slabs at once: the per-channel constants of a
    // register quad are then read from LDS once and serve every slab (a wave that reads them again for each slab
    // spends most of its epilogue waiting for LDS), and one pass of stores follows one pass of conversions.
    constexpr bool ALL_SLABS = KS == 1 && !RES && EW * TM * EP_BYTES + (MODE == 4 ? 64 * BN : 0) <= S * STAGE_BYTES;
    constexpr int WAVE_EP = ALL_SLABS ? TM * EP_BYTES : EP_BYTES;
    static_assert(EW * WAVE_EP + (MODE == 4 ? 64 * BN : 0) <= S * STAGE_BYTES, "epilogue staging must fit the LDS stages");
    uint8_t* ep = lds + (SPLIT_EPI ? wv : wvg) * WAVE_EP;
    const int nw0 = n0 + wn * TN * 32;  // first channel of this wave
    constexpr int CPR = TN * 4;              // 16-byte chunks per staged row
    constexpr int ROWS_PER_PASS = 64 / CPR;  // rows one store instruction covers
    // The chunk index is XOR-ed with the row bits ABOVE those that already separate rows inside one 256-byte
    // turn of the banks (16 / CPR rows): the 8-byte writes of 32 rows then fall on 16 different bank pairs instead
    // of 4 (64-byte rows) or 8 (128-byte rows), and the 16-byte reads of whole rows stay conflict free.
    constexpr int RSH = CPR == 4 ? 2 : (CPR == 8 ? 1 : 0);

    // Residual pieces arrive in the accumulator layout (8 bytes per lane: four channels of the lane's row), all of a
    // 32-row slab at once and, where a wave stores several slabs, one slab ahead of the stores.
    auto load_res = [&](int tm, half4 (&dst)[TN][4]) {
        const int m = m0 + (wm * TM + tm) * 32 + l31;
        long rr = m;
        if constexpr (I8) rr = g.out_map.phys(m);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = nw0 + tn * 32 + 8 * q + 4 * kb;
                half4 z = {0, 0, 0, 0};
                dst[tn][q] = m < g.M && n < g.N ? *(const half4*)(g.res + rr * g.ldr + n) : z;
            }
    };
    auto res_f32 = [&](_Float16 h) -> float {
        if constexpr (BF)
            return __builtin_bit_cast(float, (uint32_t)__builtin_bit_cast(uint16_t, h) << 16);
        else
            return (float)h;
    };
    // RES: a residual operand is present.  A kernel of its own, so that calls without one pay nothing for it.
    constexpr bool has_res = RES;

    // The constants of result quad q of channel tile tn: four consecutive channels.
    struct QuadConst {
        float4v mul, add;
        int4v dw, cn;
    };
    auto quad_const = [&](int tn, int q) {
        const int cl = (wn * TN + tn) * 32 + 8 * q + 4 * kb;  // channel inside the workgroup tile
        QuadConst k;
        k.mul = *(const float4v*)(ch_mul + cl);
        k.add = *(const float4v*)(ch_add + cl);
        if constexpr (I8) {
            k.dw = *(const int4v*)(ch_dw + cl);
            if constexpr (MODE != 4) k.cn = *(const int4v*)(ch_cn + cl);
        }
        return k;
    };
    // int8 path: the exact integer sums of result quad q of tile (tm, tn) with both zero-point corrections.
    auto int_quad = [&](int tm, int tn, int q, const QuadConst& k) {
        int4v a = {0, 0, 0, 0};
        if constexpr (I8) {
            int4v cn = k.cn;
            if constexpr (MODE == 4)  // the constants of the row's class of border pixels
                cn = *(const int4v*)(ch_border + border[tm] * BN + (wn * TN + tn) * 32 + 8 * q + 4 * kb);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                // |dw| <= 255 and |rowsum| <= 128 * K < 2^23: a 24-bit multiply (full rate) is exact
                a[r] = acc[tm][tn][4 * q + r] + __mul24(k.dw[r], rsum[tm]) + cn[r];
        }
        return a;
    };
    // Finishes result quad q of tile (tm, tn) and writes it into the slab image at `slab`.
    auto finish_quad = [&](uint8_t* slab, int tm, int tn, int q, const QuadConst& k, const half4& rq) {
        float4v add = k.add;
        if constexpr (has_res) {  // joins the bias term
#pragma unroll
            for (int r = 0; r < 4; ++r) add[r] += res_f32(rq[r]);
        }
        half4 o;
        if constexpr (I8) {
            const int4v a = int_quad(tm, tn, q, k);
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = (_Float16)((float)a[r] * k.mul[r] + add[r]);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = acc[tm][tn][4 * q + r] * k.mul[r] + add[r];
                if constexpr (BF)
                    o[r] = __builtin_bit_cast(_Float16, float_to_bf16_bits(v));  // bits only
                else
                    o[r] = (_Float16)v;
            }
        }
        const int chunk = tn * 4 + q;
        *(half4*)(slab + l31 * (CPR * 16) + (((chunk ^ (l31 >> RSH)) & (CPR - 1)) << 4) + kb * 8) = o;
    };
    // The integer sums themselves, for the tests that pin them (a pass of its own: the ordinary epilogue carries no
    // trace of it).
    if constexpr (I8) {
        if (g.acc_debug) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                if (KS > 1 && owner(tm) != grp) continue;
                const int m = m0 + (wm * TM + tm) * 32 + l31;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n_real = n0 + (wn * TN + tn) * 32 + 8 * q + 4 * kb;
                        const int4v a = int_quad(tm, tn, q, quad_const(tn, q));
                        if (m < g.M && n_real < g.N) *(int4v*)(g.acc_debug + (long)m * g.N + n_real) = a;
                    }
            }
        }
    }
    // Rows that start inside a 64-byte sector: pieces of two waves meet in it.  A streaming store may leave the XCD's L2 before the other
    // piece has come, and memory then takes the sector twice, in parts.  In the GEMM on codes, whose stages of short reductions leave little
    // time between the stores of one workgroup and the next, such rows are stored the ordinary way (6494 x 448 x 2632 at 4 bits took 20.8 us
    // with row sums in every wave and 28.1 with the faster loop and streaming stores; ordinary stores over streaming ones, 2500 shapes: 0.87 of
    // the time below 512 k, 0.95 from there to 831, 1.01 to 1023, 1.02 beyond; at 8 bits 0.95, 0.98, 1.0).  In the other modes ordinary
    // stores are 0.9 to 0.98 of the time in the mean, but for one call in ten 1.03 to 1.06.
    const bool ragged = MODE == 2 && g.K < 1024 && (((uintptr_t)g.y | (uintptr_t)(uint32_t)g.ldy * 2) & 63) != 0;
    // Reads the slab image back as 16 bytes per lane along rows and stores it: CPR lanes cover one contiguous row
    // segment of TN * 64 bytes.  All reads are requested before the first store (a store that waits for its own read
    // pays the LDS latency every time), and with the identity row map the addresses advance by a constant.
    auto store_slab = [&](const uint8_t* slab, int tm) {
        constexpr int NP = 32 / ROWS_PER_PASS;
        const int r0 = lane / CPR, c = lane % CPR;
        const int m_first = m0 + (wm * TM + tm) * 32 + r0, n = nw0 + c * 8;
        uint4v v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int row = i * ROWS_PER_PASS + r0;
            v[i] = *(const uint4v*)(slab + row * (CPR * 16) + (((c ^ (row >> RSH)) & (CPR - 1)) << 4));
        }
        if (n >= g.N) return;
        // Streaming stores: the output is not read again by this kernel, and a line that is written through as it is
        // produced does not wait in the XCD's L2 for the write-back at the end of the kernel (worth 7 % of the
        // dominant kernel's time).
        bool identity = true;
        if constexpr (I8) identity = g.out_map.rows_per_group <= 0;
        uint16_t* yp = g.y + (long)m_first * g.ldy + n;
        const long step = (long)ROWS_PER_PASS * g.ldy;
        if (identity && ragged) {
            asm volatile("");  // (here and below: or the compiler makes one kind of store of the two)
#pragma unroll
            for (int i = 0; i < NP; ++i)
                if (m_first + i * ROWS_PER_PASS < g.M) *(uint4v*)(yp + i * step) = v[i];
            asm volatile("");
        } else if (identity) {
#pragma unroll
            for (int i = 0; i < NP; ++i)
                if (m_first + i * ROWS_PER_PASS < g.M) __builtin_nontemporal_store(v[i], (uint4v*)(yp + i * step));
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int m = m_first + i * ROWS_PER_PASS;
                if (m < g.M) __builtin_nontemporal_store(v[i], (uint4v*)(g.y + g.out_map.phys(m) * g.ldy + n));
            }
        }
    };
    if constexpr (ALL_SLABS) {
        const half4 none = {0, 0, 0, 0};
        // (the constants of the next quad are requested before the conversions of the current one: the compiler does
        // not move an LDS read above the staging writes by itself)
        QuadConst k = quad_const(0, 0);
#pragma unroll
        for (int i = 0; i < TN * 4; ++i) {
            const QuadConst kn = quad_const((i + 1 < TN * 4 ? i + 1 : i) >> 2, (i + 1 < TN * 4 ? i + 1 : i) & 3);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) finish_quad(ep + tm * EP_BYTES, tm, i >> 2, i & 3, k, none);
            k = kn;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) store_slab(ep + tm * EP_BYTES, tm);
    } else {
        constexpr bool RES_AHEAD = KS == 1 && TM > 1;
        half4 rs[2][TN][4] = {};
        if constexpr (RES_AHEAD && has_res) load_res(0, rs[0]);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (KS > 1 && owner(tm) != grp) continue;  // the finished sums of this slab live in the other group
            if constexpr (has_res) {
                if constexpr (RES_AHEAD) {
                    if (tm + 1 < TM) load_res(tm + 1, rs[(tm + 1) & 1]);
                } else {
                    load_res(tm, rs[tm & 1]);
                }
            }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q) finish_quad(ep, tm, tn, q, quad_const(tn, q), rs[tm & 1][tn][q]);
            __builtin_amdgcn_wave_barrier();
            store_slab(ep, tm);
            __builtin_amdgcn_wave_barrier();
        }
    }
    }
    if (CAN_SPLIT && splits > 1 && threadIdx.x == 0)
        // The word goes back cleared.  (Last: a store ahead of the loads of the partial sums is waited for with them, and
        // takes longer than they do: 1 x 2048 x 1280, 4-bit weights, 8.41 us with it there, 7.75 here.)
        __hip_atomic_store(counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (g.phase_clk && threadIdx.x == 0) {
        long long* o = g.phase_clk + (long)blockIdx.x * 4;
        o[0] = t0;
        o[1] = t1;
        o[2] = t2;
        o[3] = clock64();
    }
}

// ---------------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------------
// Tile table.  index -> workgroup tile (rows x channels), waves, wave tile:
//   0: 128x256, 4 waves (1x4) of 128x64     1: 128x128, 4 waves (2x2) of 64x64     2: 64x64, 4 waves of 32x32
//   3 (unquantised fp16 weights): as 1 and 4: as 2, with a second wave group splitting k inside the workgroup (8 waves)
//   5: 64x128, 4 waves (1x4) of 64x32, two or three LDS stages: the form of tile 1 that puts more workgroups on a
//      compute unit     6 (linear layers, not 8-bit weights under 8-bit activations): 96x256, 4 waves (1x4) of 96x64
//   (int8, plain layers) 7: as 5 with three stages   8, 9: 128x128, 8 waves (2x4) of 64x32, with stages for one or for two
//      workgroups per compute unit
//   10: 96x128, 4 waves (1x4) of 96x32   11 (16-bit activations, plain layers): as 5 with a second wave group splitting k
// A tall wave tile pays: every widened weight fragment then feeds 4 MFMAs (measured: an MFMA hides about five vector
// ALU instructions on its SIMD; what a wave needs beyond that costs time of its own).  256x256 tiles with one wave per
// SIMD and 128x128 tiles with two-wave workgroups were measured slower on every configured shape.
// The number of LDS stages is the largest (<= 4; <= 8 for tile 2, whose problems are latency bound) that lets two
// workgroups share a compute unit and keeps the hand-counted loads within the 6-bit vmcnt.
// 8-bit weights under 8-bit activations, 2 KB per weight tile, leave room for three workgroups of tile 5 and two of tile 10 on a unit (the
// other widths for four and three), with two stages: 1300 tiles of 96x128 (K/V projections of all layers, one prompt) are 512 + 512 + 276.
static int g_force_tile = -1;
static long long* g_phase_clk = nullptr;
static long g_phase_cap = 0;
void set_phase_buffer(long long* p, long workgroups) {
    g_phase_clk = p;
    g_phase_cap = workgroups;
}
void set_force_tile(int t) { g_force_tile = t; }
int forced_tile() { return g_force_tile; }
long long* phase_buffer(long workgroups) { return workgroups <= g_phase_cap ? g_phase_clk : nullptr; }

// ---- reduction split over workgroups ------------------------------------------------------------------------
// Problems with few tiles and a long reduction (K/V projections, a handful of activation rows) are bound by memory
// latency: the only remedy is to have more workgroups request the operands at once.  Their partial sums and one
// arrival counter per tile live in the CALLER's workspace: [counters: tiles x 8 or 128 bytes, rounded up to 256]
// [partial sums: tiles x parts x BM x BN x 4 bytes].  The workspace arrives with unknown contents: a counter word
// counts only under the tag of the launch that reads it (44 bits, another one for every launch; a replayed graph finds
// the zero that the last arrival of the replay before it left), so that no launch of its own has to clear the words
// first.  That launch took 4.5 us beside GEMMs of 10 us.  Whoever owns the workspace owns the hazard, as with any
// workspace: one stream at a time.
static int g_force_splits = 0;  // 0: automatic, 1: never, n > 1: n parts wherever the reduction is long enough
void set_force_splits(int n) { g_force_splits = n < 0 ? 0 : n; }
int forced_splits() { return g_force_splits; }
static int g_force_band = 0;  // 0: automatic, n >= 1: n row blocks per band of the workgroup -> tile map
void set_force_band(int n) { g_force_band = n < 0 ? 0 : n; }
int forced_band() { return g_force_band; }

// Tag of one launch: the upper 44 bits of a Weyl sequence, never zero, so that neither cleared memory nor small numbers
// or 16-bit data left in the workspace look like it.
static unsigned long long next_split_tag() {
    static std::atomic<unsigned long long> count{1};
    const unsigned long long tag = (count.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull) & ~SPLIT_COUNT;
    return tag ? tag : 0xA5A5A5A5A5A00000ull;
}

static constexpr int SPLIT_LINE_WORDS = 16;
static inline size_t split_counter_bytes(long tiles, int step) { return ((size_t)tiles * step * 8 + 255) / 256 * 256; }

// Measured on the SDXL shapes: the large tile wins once it yields two or more workgroups per compute unit; the
// k-split variants only pay where tiles are few and k is long (FF-out at the 640 level, the K/V projections).
static int pick_tile(int M, int N, int K, bool wide_weights = false) {
    if ((g_force_tile >= 0 && g_force_tile <= 4) || g_force_tile == 6) return g_force_tile;
    if (g_force_tile == 5) return 1;  // the half-height form of tile 1: the linear layers' dispatch decides
    const long t0 = (long)((M + 127) / 128) * ((N + 255) / 256);
    // One row block of 65 to 96 rows over very many column tiles (one prompt's 77 text tokens through all K/V
    // projections of the UNet, stacked): the 96x256 tile does three quarters of the large tile's MFMA and widening work
    // on the same weight stream (measured at N = 166400: 13 to 18 % faster with 2- and 4-bit weights, equal at 8).
    if (M > 64 && M <= 96 && t0 >= 256) return 6;
    // (8-bit weights of the int8 path: the large tile leaves LDS for one workgroup per compute unit only, and two
    // co-resident 128x128 workgroups were measured faster on every configured shape)
    if (t0 >= 512 && !wide_weights) return 0;
    const long t1 = (long)((M + 127) / 128) * ((N + 127) / 128);
    if (t1 >= 128) return (t1 < 256 && K >= 2048) ? 3 : 1;
    return K >= 1024 ? 4 : 2;
}

// Tile 1 or its half-height form (tile 5: 64x128, four waves side by side, two or three LDS stages, three to five
// workgroups per compute unit)?  The 128x128 problems of this path have 160 to 640 tiles, one or two workgroups on
// most compute units, and a wave's LDS reads, code widening and MFMAs run one after the other: what is missing is
// other waves on the SIMD to fill the gaps.  Twice the workgroups at half the height fetch every weight tile twice as
// often (weights are the small operand; halving the width instead doubles the activation traffic and was measured
// slower on the 16-bit-activation path).  Measured on operands that are not cached: 8 to 19 % faster on every such
// shape of both paths, except with unquantised 16-bit weights (4 KB per weight tile), which keep tile 1.  Two
// stages instead of three, and eight waves on 64x256, were measured slower.
// The linear layers of the 16-bit-activation path and the convolutions have a third form, 96x128 (tile 10): three MFMAs per
// widened weight fragment instead of two, for fewer workgroups.  A kernel lasts as long as its busiest compute unit, so the form
// is chosen by what that unit multiplies: its number of workgroups times their height (UNITS: compute units).  At equal
// height the taller form is faster, and where the widening costs most also where it takes an eighth more.  Convolutions in us, tile 5 / 10
// (rows of the busiest unit), 16-bit activations, 4-bit weights: 4 x 32 x 32, 1280 -> 1280 (192 / 192) 138 / 129, 3 x 100 x 128, 320 -> 320
// (512 / 480) 93.8 / 86.2, 4 x 64 x 64 x 640 (320 / 384) 126 / 135.
static long busiest(long M, long N, long rows) { return busiest_area(M, N, rows, 128) / 128; }  // rows of the busiest unit, tiles of rows x 128
static bool taller(long M, long N, long num, long den) {  // busiest unit: rows of tile 10 <= num / den of tile 5's
    return den * busiest(M, N, 96) <= num * busiest(M, N, 64);
}

// Linear layers on 16-bit activations (unquantised weights keep tile 1).  Beside each line one pair of times of whole calls in us; all of
// them, and the ratios over thousands of shapes that the lines were drawn by, are in profiles/tile_rules.txt.
template <int BITS>
static int float_tile(int t, const GemmArgs& g, bool bf16) {
    const long M = g.M, N = g.N, K = g.K;
    if (g_force_tile >= 0 && (g_force_tile == 5 || (BITS != 16 && g_force_tile >= 10))) return g_force_tile;
    if (g_force_tile >= 0) return BITS == 16 ? t : t == 1 && bf16 ? 5 : t == 3 ? 11 : t;
    // (one row block of 96 over very many columns keeps tile 6: in fp16 the faster one at 769 to 1024 column tiles, by 10 to 30 %; elsewhere
    // tile 10 would be, by 4 to 17 %, which no rule takes up)
    if (BITS == 16 || t == 6) return t;
    // two such blocks: three quarters of tile 0's rows (154 x 2048 x 166400 at 4 bits: tile 0 141, tile 10 122)
    if (t == 0) return M > 128 && M <= 192 ? 10 : 0;
    const long t2 = ((M + 63) / 64) * ((N + 63) / 64), t5 = ((M + 63) / 64) * ((N + 127) / 128);
    // Where the 64x64 tiles are more than one round of workgroups but those of 64x128 are not, a compute unit would get one wave
    // per SIMD of the latter; with a second wave group on the other half of the reduction (tile 11) it gets two, which short reductions,
    // shorter ones with 8-bit weights, do not repay (1024 x 5120 x 1280: tile 5 31.1, tile 11 25.7; 4096 x 448 x 320 5.8 and 6.1).
    if (t2 > UNITS && t5 <= UNITS) return K >= (BITS == 8 ? 1280 : 640) ? 11 : 5;
    if (t == 1 || t == 3) {
        const bool ragged = g.ldy % 32 != 0;  // (rows that start inside a 64-byte sector, where the pieces of two workgroups meet)
        // bf16, whose widening costs most, takes the taller form at up to an eighth more rows (0.88 to 0.97 of the time there), but short
        // reductions, which the output's stores bound, keep the smaller workgroups if rows are ragged (2877 x 384 x 4728 18.1, 22.1).
        if (bf16) return (K >= 640 || !ragged) && taller(M, N, 9, 8) ? 10 : 5;
        const long r1 = busiest(M, N, 128), r5 = busiest(M, N, 64), r10 = busiest(M, N, 96);
        // fp16 weights beyond 8 MB are streamed once per row block: the full height where neither lower form gives the busiest unit fewer
        // rows (1024 x 3584 x 6352 at 8 bits, tile 1 / 5 / 10: 52.6 / 64.5 / 57.3), but not one workgroup per unit, with nothing beside
        // its reduction (616 x 4992 x 4832 at 3 bits, tile 1 52.0, else 40.7).
        if (N * K * BITS / 8 > (8L << 20) && r1 > 128 && r1 <= r5 && r1 < r10) return 1;
        // one workgroup of tile 10 per unit: two stages of 8-bit weights and nothing beside them (4096 x 2560 x 640: tile 5 20.9, tile 10 22.7)
        const bool one_each = r10 <= 96;
        if (BITS == 8 && one_each) return 5;
        // short reductions, as above (2291 x 384 x 5480 at 2 bits: tile 5 16.6, tile 10 20.9)
        if (K < (ragged && BITS != 8 ? 1280 : 640)) return r10 < r5 && !(ragged && (K < 640 || one_each)) ? 10 : 5;
        // fp16 at an eighth more rows: 0.91 of the time at 8 bits, 0.98 at 3, 1.01 to 1.03 at 2 and 4, which it widens in fewer instructions
        return taller(M, N, BITS == 3 || BITS == 8 ? 9 : 8, 8) ? 10 : 5;
    }
    // Few tiles with 1024 k and more: tile 4 splits its reduction over workgroups from 16 of its stages on (1984 k), tile 2, of twice as
    // many stages, from 1024 k on, where the workspace holds the parts (unsplit its chain is twice as long).  Fewer tiles gain more by it
    // (4 x 1920 x 1280: tile 2 8.0, tile 4 9.8; 32 x 1984 x 2040 9.9 and 8.9; bf16 77 x 1920 x 504 9.2 and 13.2; 4 x 4224 x 3792 20.0 and 21.8).
    const bool few = bf16 ? (K < 1984 && t2 <= (M <= 32 ? 48 : 36)) || (K < 3072 && t2 <= 8) || (K >= 4096 && t2 > 52 && t2 <= 64)
                          : K < 1984 && M <= 32 && t2 <= 24;
    if (t == 4 && few && g.split_ws && g.split_ws_bytes >= split_counter_bytes(t2, 1) + (size_t)(K / 256) * t2 * (64 * 64 * 4)) return 2;
    return t;
}

// The int8 path has more forms of tile 1, by how many workgroups a compute unit gets: with few of them the wait for loads
// counts (more stages, 7, or the eight waves of one 128x128 workgroup over half the L2 -> LDS traffic per operation, 8), with many
// the number of waves.  8-bit weights move twice the bytes, so that the L2 -> LDS path bounds the half height there (96 bytes
// per clock and compute unit at the full MFMA rate, of 55): they have a form of their own for many tiles, 9.  Beside each line one pair of
// times of whole calls with given parameters in us; all of them are in profiles/tile_rules.txt.
template <int BITS>
static int int8_tile(int t, const GemmArgs& g) {
    const long M = g.M, N = g.N, K = g.K;
    if (g_force_tile >= 7) return g_force_tile == 11 ? 5 : BITS != 8 && g_force_tile == 9 ? 8 : g_force_tile;
    const long cols = (N + 127) / 128, t2 = ((M + 63) / 64) * ((N + 63) / 64);
    // Few tiles: the wave groups of tile 4 leave 8-bit weights two stages, tile 2 has four (700 x 5120 x 1280: tile 4 24.6, tile 2 20.2).
    // What tile 4 splits over workgroups stays with it, its parts are fewer (64 x 5120 x 1280 14.3 and 16.0); nearly two rounds of tile 2
    // over a narrow output take tile 7 (2964 x 2560 x 640: tile 2 20.4, tile 7 18.7; wide, 616 x 2560 x 2928, 15.8 and 16.0).
    if (BITS == 8 && t == 4 && g_force_tile < 0) return t2 <= 64 ? (K > 3840 ? 4 : 2) : t2 > 448 && M >= 4 * N ? 7 : 2;
    if (g_force_tile >= 0) return g_force_tile == 5 ? 5 : t == 1 || t == 3 ? (BITS == 8 ? 9 : 1) : t;
    // One or two row blocks of 96 over very many columns (the K/V projections of all layers for one or two prompts of 77 tokens, stacked)
    // stream their weights: several workgroups per compute unit whose loads cover each other's epilogues, at three quarters of the rows
    // (77 x 2048 x 83200 at 8 bits: tile 6 47.6, tile 10 40.0).  2- and 4-bit weights leave room for three workgroups of tile 10 per unit
    // or two of tile 6: just more than three rounds of the one are two of the other (77 x 2048 x 99840 at 4 bits: tile 6 33.4, tile 10 43.3).
    if (BITS != 8 && M > 64 && M <= 96 && cols > 3 * UNITS && cols <= 4 * UNITS) return 6;
    if (((M > 64 && M <= 96) || (M > 128 && M <= 192)) && cols >= 320) return 10;
    if (t != 1 && t != 3) return t;
    const long t1 = ((M + 127) / 128) * cols, t5 = ((M + 63) / 64) * cols;
    // few workgroups of the half height: three stages (2048 x 5120 x 1280 at 4 bits, 320 of them: tile 5 36.9, tile 7 29.9)
    if (t5 <= 384) return 7;
    // one 128x128 workgroup per unit at most, over a reduction that repays its start (3200 x 5120 x 1280 at 8 bits: tile 5 46.8, tile 8 42.1)
    if (t1 <= UNITS && K >= 1536) return 8;
    const long r1 = busiest(M, N, 128), r5 = busiest(M, N, 64), r10 = busiest(M, N, 96);
    const bool big = N * K * BITS / 8 > (8L << 20);
    // 2- and 4-bit weights that do not fit an XCD's L2 by a wide margin are streamed from the last-level cache once per row block, so tall
    // problems keep the full height (1536 x 2560 x 10240: tile 1 49.8, tile 5 50.9); of few row blocks each is better read twice by more
    // workgroups (1024 x 5120 x 5120 41.2 and 37.4), unless the busiest unit gets no fewer rows by it (1024 x 2304 x 7512 26.6 and 28.1).
    if (BITS != 8) return big && (M > 1024 || (t1 <= 2 * UNITS && r1 <= r5)) ? 1 : 5;
    // 8-bit weights: below 640 k the output's stores bound it, and smaller workgroups are the faster ones (8192 x 384 x 6216: tile 5 71.2,
    // tile 9 78.6); many tiles take tile 9 (9000 x 1280 x 1280: tile 5 32.4, tile 9 30.8); in between the form that gives the busiest unit
    // fewest rows (1619 x 2048 x 4504: tile 9 27.6, tile 5 32.8), among them from 2560 k on tile 10 (4096 x 5120 x 1280: tile 9 51.0, tile 10
    // 48.6; 6000 x 5120 x 1280, where it has more rows, 64.8 and 81.9).
    if (K < 640 && !big) return 5;
    if (t1 > 640) {
        // Two workgroups of tile 9 fit a unit: an odd one is alone at the end.  That costs most, and so do the larger stores, where rows start
        // inside a 64-byte sector, whose pieces of two workgroups meet in it (time of tile 9 over tile 5's with 640 to 767 k 1.0 to 1.18, with
        // up to 1400 k 384 rows for 384 1.0 to 1.12, 640 for 576 1.01 to 1.10: 4637 x 1536 x 2456 tile 5 38.5, tile 9 41.2).
        const bool ragged = g.ldy % 32 != 0;
        const long r = ragged ? (r1 + 255) / 256 * 256 : r1;
        return !big && ((ragged && K < 768) || 3 * r >= 4 * r5) ? 5 : 9;
    }
    if (K >= 2560) return r1 < r10 ? 9 : 8 * r10 <= 9 * r5 ? 10 : 5;
    return t1 > UNITS && r1 <= r5 ? 9 : 5;
}

template <bool I8, int BITS, int WGM, int WGN, int TM, int TN, int S, int KS>
constexpr bool stages_fit(int budget) {
    using P = GemmPlan<I8, BITS, WGM, WGN, TM, TN, S, KS>;
    return P::LDS_BYTES <= budget && (S - 2) * P::OPS <= 63;
}

template <bool I8, int BITS, int WGM, int WGN, int TM, int TN, int KS>
constexpr int pick_stages(int budget, int max_stages) {
    if (max_stages >= 8 && stages_fit<I8, BITS, WGM, WGN, TM, TN, 8, KS>(budget)) return 8;
    if (max_stages >= 6 && stages_fit<I8, BITS, WGM, WGN, TM, TN, 6, KS>(budget)) return 6;
    if (max_stages >= 4 && stages_fit<I8, BITS, WGM, WGN, TM, TN, 4, KS>(budget)) return 4;
    if (stages_fit<I8, BITS, WGM, WGN, TM, TN, 3, KS>(budget)) return 3;
    return 2;
}

template <bool I8, int BITS, int WGM, int WGN, int TM, int TN, int KS, int BUDGET, int MAXS, bool BF, int MODE, bool RES>
static int run_gemm_r(GemmArgs& g, int tile_index, hipStream_t st) {
    constexpr int S = pick_stages<I8, BITS, WGM, WGN, TM, TN, KS>(BUDGET, MAXS);
    using P = GemmPlan<I8, BITS, WGM, WGN, TM, TN, S, KS>;
    static_assert(P::LDS_BYTES <= BUDGET && BUDGET <= 160 * 1024, "the plan of the fewest stages exceeds the budget that was asked for");
    g.tiles_m = (g.M + P::BM - 1) / P::BM;
    g.tiles_n = (g.N + P::BN - 1) / P::BN;
    if (MODE == 1 || MODE == 5 || MODE == 6) g.tiles_n = (int)((g.ld8 + P::BN / 2 - 1) / (P::BN / 2));  // gated columns up to the padded row end
    // Split the reduction over workgroups where the tiles alone would leave most compute units idle and the reduction
    // is long: as many parts as fill about two workgroups per compute unit, each at least four pipeline stages long.
    const long tiles = (long)g.tiles_m * g.tiles_n;
    // Height of the bands of the tile walk, measured on operands that are not cached over 1 to 64 row blocks: the
    // int8 path gains 4 to 23 % at 8 to 16 (every shape of the sweep, most at 16384 x 640 x 640 and with 8-bit
    // weights) and loses again from 32 on; unquantised 16-bit weights (the largest weight tiles) gain up to 15 % at
    // 8; quantised weights under 16-bit activations move by -10 (8-bit, 4096 x 2560 x 640) to +2 % at 8, and every
    // weight tile is then fetched once per eight row blocks instead of once per row block.
    set_tile_walk(g, g_force_band > 0 ? g_force_band : (I8 ? 16 : 8));
    const int KT = (g.k_stages + KS - 1) / KS;
    int splits = 1;
    if (g_force_splits > 1) {
        splits = g_force_splits < KT ? g_force_splits : KT;
    } else if (g_force_splits == 0 && tiles <= 64 && KT >= 16 && !(I8 && BITS == 8 && KS == 1 && tiles > 32 && KT < 32)) {
        // (8-bit weights, 77 x 2048 x 320 (10 tiles) 15.5 whole -> 15.2 us split, 640 16.0 -> 15.9, but 1280 (40) 17.3 -> 18.0,
        // 152 x 2048 x 1280 (60) 17.5 -> 19.4, 308 x 2048 x 640 (50) 16.9 -> 18.5; 64 x 3392 x 1280 (20) 17.7 whole, 12.6 split)
        // (measured: handing the sums over costs about as much as eight pipeline stages)
        splits = (int)(512 / tiles);
        if (splits > KT / 4) splits = KT / 4;
        if (splits > 16) splits = 16;
    }
    g.splits = 1;
    if (MODE == 0 && TM * TN <= 4 && TM != 3 && splits > 1) {
        // as many parts as the caller's workspace holds (forced part counts are for tests: they must fit)
        size_t cbytes = split_counter_bytes(tiles, 1);
        const size_t part_bytes = (size_t)tiles * P::BM * P::BN * 4;
        const size_t room = g.split_ws && g.split_ws_bytes > cbytes ? (g.split_ws_bytes - cbytes) / part_bytes : 0;
        if (g_force_splits > 1 && room < (size_t)splits) return MQ_ERR_WORKSPACE_TOO_SMALL;
        if (room < (size_t)splits) splits = (int)room;
        if (splits > 1) {
            g.splits = splits;
            // (a cache line per counter where that takes no part away: every arrival is two atomic accesses, and those to
            // one line wait for each other: 77 x 2048 x 640, 4-bit weights, 8.88 us with shared lines, 8.67 with lines of their own)
            const size_t apart = split_counter_bytes(tiles, SPLIT_LINE_WORDS);
            const bool room_apart = g.split_ws_bytes >= apart + (size_t)splits * part_bytes;
            if (room_apart) cbytes = apart;
            g.counter_step = room_apart ? SPLIT_LINE_WORDS : 1;
            g.counters = (unsigned long long*)g.split_ws;
            g.split_tag = next_split_tag();
            g.partial = (uint32_t*)((uint8_t*)g.split_ws + cbytes);
        }
    }
    g.fd_splits = FastDiv::make((uint32_t)g.splits);
    g.kt_q = KT / g.splits;
    g.kt_r = KT % g.splits;
    g.phase_clk = phase_buffer(tiles * g.splits);
    auto kern = gemm_kernel<I8, BITS, WGM, WGN, TM, TN, S, KS, BF, MODE, RES>;
    // Once per instantiation and device (callers may be on several host threads): allow more than 64 KB of dynamic
    // LDS, name the profiling slot.
    const int slot = prof_gemm_slot(MODE >= 5 ? 3 : (MODE ? 2 + MODE : (I8 ? 1 : (BF ? 2 : 0))), BITS, tile_index);
    static std::mutex prep_mutex;
    static bool prepared[16] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) dev = 0;
    {
        std::lock_guard<std::mutex> lock(prep_mutex);
        if (!prepared[dev]) {
            if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, P::LDS_BYTES) !=
                hipSuccess) {
                set_hip_error((int)hipGetLastError());
                return MQ_ERR_HIP;
            }
            // (the residual variant shares the slot of the plain kernel and leaves the slot's name to it)
            char name[112];
            snprintf(name, sizeof name, "mq::gemm_kernel<%s, %d, %d, %d, %d, %d, %d, %d, %s, %d, false>",
                     I8 ? "true" : "false", BITS, WGM, WGN, TM, TN, S, KS, BF ? "true" : "false", MODE);
            prof_name_slot(slot, name);
            prepared[dev] = true;
        }
    }
    ProfScope prof(st, slot, 2.0 * g.M * g.N * g.K, gemm_alg_bytes(g, I8, BITS, MODE));
    hipLaunchKernelGGL(kern, dim3(g.tiles_m * g.tiles_n * g.splits), dim3(P::NT), P::LDS_BYTES, st, g);
    MQ_HIP_CHECK_LAUNCH();
    return MQ_OK;
}

template <bool I8, int BITS, int WGM, int WGN, int TM, int TN, int KS, int BUDGET, int MAXS, bool BF = false, int MODE = 0>
static int run_gemm(GemmArgs& g, int tile_index, hipStream_t st) {
    if constexpr (MODE != 1 && MODE != 5 && MODE != 6)
        if (g.res) return run_gemm_r<I8, BITS, WGM, WGN, TM, TN, KS, BUDGET, MAXS, BF, MODE, true>(g, tile_index, st);
    return run_gemm_r<I8, BITS, WGM, WGN, TM, TN, KS, BUDGET, MAXS, BF, MODE, false>(g, tile_index, st);
}

template <bool I8, int BITS>
static int dispatch_gemm(GemmArgs& g, hipStream_t st) {
    if (const int form = solo_form(g, I8, BITS, 0); form >= 0) return launch_gemm_solo(g, form, I8, BITS, 0, st);
    // 8-bit weights of the int8 path take 2 KB of LDS per 32x64 tile and unquantised 16-bit weights 4 KB: with the
    // large tile two workgroups per compute unit would not fit, so it runs one per compute unit with a deeper
    // pipeline (and is not chosen automatically)
    constexpr bool WIDE = (I8 && BITS == 8) || BITS == 16;
    int t = pick_tile(g.M, g.N, g.K, WIDE);
    if constexpr (I8) {
        t = int8_tile<BITS>(t, g);
        switch (t) {
            case 7: return run_gemm<I8, BITS, 1, 4, 2, 1, 1, 76 * 1024, 3>(g, 7, st);
            case 8: return run_gemm<I8, BITS, 2, 4, 2, 1, 1, BITS == 8 ? 160 * 1024 : 80 * 1024, 4>(g, 8, st);
            case 9:
                if constexpr (BITS == 8) return run_gemm<I8, BITS, 2, 4, 2, 1, 1, 80 * 1024, 4>(g, 9, st);
        }
    } else {
        t = float_tile<BITS>(t, g, false);
        if constexpr (BITS != 16)
            if (t == 11) return run_gemm<I8, BITS, 1, 4, 2, 1, 2, BITS == 8 ? 160 * 1024 : 80 * 1024, 4>(g, 11, st);
    }
    if constexpr (BITS != 16)
        if (t == 10 || (I8 && BITS == 8 && t == 6)) return run_gemm<I8, BITS, 1, 4, 3, 1, 1, I8 && BITS == 8 ? 60 * 1024 : 53 * 1024, 3>(g, 10, st);
    switch (t) {
        case 0: return run_gemm<I8, BITS, 1, 4, 4, 2, 1, WIDE ? 160 * 1024 : 80 * 1024, 4>(g, 0, st);
        case 1:
            if constexpr (!(I8 && BITS == 8)) return run_gemm<I8, BITS, 2, 2, 2, 2, 1, 80 * 1024, 4>(g, 1, st);
        case 2: return run_gemm<I8, BITS, 2, 2, 1, 1, 1, 80 * 1024, 8>(g, 2, st);
        case 3:
            if constexpr (BITS == 16) return run_gemm<I8, BITS, 2, 2, 2, 2, 2, 160 * 1024, 4>(g, 3, st);
        case 5: return run_gemm<I8, BITS, 1, 4, 2, 1, 1, I8 && BITS != 8 ? 40 * 1024 : 52 * 1024, 3>(g, 5, st);
        case 6:
            if constexpr (!(I8 && BITS == 8)) return run_gemm<I8, BITS, 1, 4, 3, 2, 1, WIDE ? 160 * 1024 : 80 * 1024, 4>(g, 6, st);
        default: return run_gemm<I8, BITS, 2, 2, 1, 1, 2, 80 * 1024, 8>(g, 4, st);
    }
}

// bfloat16 activations: tile 3 and, with unquantised weights, tile 4 fall back to their plain counterparts.  (Tile 4 in place of tile 2 in us:
// 77 x 2048 x 640 9.8 -> 8.7, 77 x 2048 x 1280 15.2 -> 9.7, 308 x 2048 x 640 19 -> 11.2, 616 x 2048 x 1280 14.5 -> 13.1.)
template <int BITS>
static int dispatch_gemm_bf16(GemmArgs& g, hipStream_t st) {
    constexpr bool WIDE = BITS == 16;
    int t = pick_tile(g.M, g.N, g.K, WIDE);
    t = float_tile<BITS>(t == 6 ? 0 : (t == 3 || (BITS == 16 && t == 4) ? t - 2 : t), g, true);
    if constexpr (BITS != 16)
        switch (t) {
            case 4: return run_gemm<false, BITS, 2, 2, 1, 1, 2, 80 * 1024, 8, true>(g, 4, st);
            case 10: return run_gemm<false, BITS, 1, 4, 3, 1, 1, 53 * 1024, 3, true>(g, 10, st);
            case 11: return run_gemm<false, BITS, 1, 4, 2, 1, 2, BITS == 8 ? 160 * 1024 : 80 * 1024, 4, true>(g, 11, st);
        }
    switch (t) {
        case 0: return run_gemm<false, BITS, 1, 4, 4, 2, 1, WIDE ? 160 * 1024 : 80 * 1024, 4, true>(g, 0, st);
        case 1:
            if constexpr (BITS == 16) return run_gemm<false, BITS, 2, 2, 2, 2, 1, 80 * 1024, 4, true>(g, 1, st);
        case 5: return run_gemm<false, BITS, 1, 4, 2, 1, 1, 52 * 1024, 3, true>(g, 5, st);
        default: return run_gemm<false, BITS, 2, 2, 1, 1, 1, 80 * 1024, 8, true>(g, 2, st);
    }
}

int launch_gemm_w_only(const void* x, int M, int K, int ldx, const void* packed, int N, int bits,
                       const float* w_scale, const int32_t* w_zp, const void* bias, void* y, int ldy, int dtype,
                       const void* res, int ldr, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
    GemmArgs g{};
    g.split_ws = split_ws; g.split_ws_bytes = split_ws_bytes;
    g.a = x;
    g.a_row_bytes = (long)ldx * 2;
    g.a_bytes = (uint32_t)(((long)(M - 1) * ldx + K) * 2);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((N + 31) / 32) * (K / 64) * 256 * bits);
    g.M = M; g.N = N; g.K = K;
    g.k_stages = K / 64;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)y; g.ldy = ldy;
    g.res = (const uint16_t*)res; g.ldr = ldr;
    if (dtype == MQ_BF16) {
        switch (bits) {
            case 2: return dispatch_gemm_bf16<2>(g, st);
            case 3: return dispatch_gemm_bf16<3>(g, st);
            case 4: return dispatch_gemm_bf16<4>(g, st);
            case 8: return dispatch_gemm_bf16<8>(g, st);
            case 16: return dispatch_gemm_bf16<16>(g, st);
        }
        return MQ_ERR_UNSUPPORTED_BITS;
    }
    switch (bits) {
        case 2: return dispatch_gemm<false, 2>(g, st);
        case 3: return dispatch_gemm<false, 3>(g, st);
        case 4: return dispatch_gemm<false, 4>(g, st);
        case 8: return dispatch_gemm<false, 8>(g, st);
        case 16: return dispatch_gemm<false, 16>(g, st);
    }
    return MQ_ERR_UNSUPPORTED_BITS;
}

int launch_gemm_a8(const int8_t* a8, const int32_t* rowsum, const ActParams* params, int M, int K,
                   const void* packed, int N, int w_bits, int w_signed, const float* w_scale, const int32_t* w_zp,
                   const int32_t* w_colsum, const void* bias, void* y, int ldy, RowMap out_map, int32_t* acc_debug,
                   const void* res, int ldr, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
    const int Kp = (K + 127) / 128 * 128;
    GemmArgs g{};
    g.split_ws = split_ws; g.split_ws_bytes = split_ws_bytes;
    g.a = a8;
    g.a_row_bytes = Kp;
    g.a_bytes = (uint32_t)((long)M * Kp);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((N + 31) / 32) * (K / 64) * 256 * w_bits);
    g.M = M; g.N = N; g.K = K;
    g.k_stages = Kp / 128;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)y; g.ldy = ldy;
    g.res = (const uint16_t*)res; g.ldr = ldr;
    g.rowsum = rowsum; g.params = params; g.w_colsum = w_colsum;
    g.out_map = out_map; g.acc_debug = acc_debug;
    if (w_bits == 4 || w_bits == 2) {
        g.w_off = 0;
        return w_bits == 4 ? dispatch_gemm<true, 4>(g, st) : dispatch_gemm<true, 2>(g, st);
    }
    if (w_bits == 8) {
        // Unsigned 8-bit codes do not fit a signed MFMA operand: the kernel flips their top bit in registers,
        // which reads them as q - 128 (w_off = 128); signed (symmetric) codes are used as they are.
        g.w_off = w_signed ? 0 : 128;
        return dispatch_gemm<true, 8>(g, st);
    }
    return MQ_ERR_UNSUPPORTED_BITS;
}


// Gated feed-forward projection with 8-bit output (MODE 1).  N = 2H weight rows.
int launch_gemm_a8_geglu(const int8_t* a8, const int32_t* rowsum, const ActParams* params, int M, int K,
                         const void* packed, int H, int w_bits, int w_signed, const float* w_scale, const int32_t* w_zp,
                         const int32_t* w_colsum, const void* bias, const float* out_scale, const int32_t* out_zp,
                         int8_t* a8_out, void* h16, int ldh, float* mm_out, int* mm_pairs, hipStream_t st) {
    const int Kp = (K + 127) / 128 * 128;
    GemmArgs g{};
    g.mm_out = mm_out;
    g.a = a8;
    g.a_row_bytes = Kp;
    g.a_bytes = (uint32_t)((long)M * Kp);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((2 * H + 31) / 32) * (K / 64) * 256 * w_bits);
    g.M = M; g.N = 2 * H; g.K = K;
    g.k_stages = Kp / 128;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)h16; g.ldy = ldh;
    g.rowsum = rowsum; g.params = params; g.w_colsum = w_colsum;
    g.out_scale_p = out_scale; g.out_zp_p = out_zp;
    g.a8_out = a8_out; g.ld8 = (H + 127) / 128 * 128;
    // the large tile (128 gated columns per workgroup) once it yields two workgroups per compute unit
    const bool big = g_force_tile == 0 || (g_force_tile < 0 && (long)((M + 127) / 128) * ((H + 127) / 128) >= 512);
    int rc = MQ_ERR_UNSUPPORTED_BITS;
    if (mm_out) {  // fp16 product and its range, no codes
        if (w_bits == 4) {
            g.w_off = 0;
            if (big) rc = run_gemm<true, 4, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 5>(g, 0, st);
            else rc = run_gemm<true, 4, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 5>(g, 1, st);
        }
        if (w_bits == 2) {
            g.w_off = 0;
            if (big) rc = run_gemm<true, 2, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 5>(g, 0, st);
            else rc = run_gemm<true, 2, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 5>(g, 1, st);
        }
        if (w_bits == 8) {
            g.w_off = w_signed ? 0 : 128;
            if (g_force_tile == 0) rc = run_gemm<true, 8, 1, 4, 4, 2, 1, 160 * 1024, 4, false, 5>(g, 0, st);
            else rc = run_gemm<true, 8, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 5>(g, 1, st);
        }
    } else {
        if (w_bits == 4) {
            g.w_off = 0;
            if (big) rc = run_gemm<true, 4, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 1>(g, 0, st);
            else rc = run_gemm<true, 4, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 1>(g, 1, st);
        }
        if (w_bits == 2) {
            g.w_off = 0;
            if (big) rc = run_gemm<true, 2, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 1>(g, 0, st);
            else rc = run_gemm<true, 2, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 1>(g, 1, st);
        }
        if (w_bits == 8) {
            g.w_off = w_signed ? 0 : 128;
            if (g_force_tile == 0) rc = run_gemm<true, 8, 1, 4, 4, 2, 1, 160 * 1024, 4, false, 1>(g, 0, st);
            else rc = run_gemm<true, 8, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 1>(g, 1, st);
        }
    }
    if (mm_pairs) *mm_pairs = g.tiles_m * g.tiles_n;  // workgroups of the launch: one pair each
    return rc;
}

template <int BITS>
static int dispatch_w_only_geglu(GemmArgs& g, int H, hipStream_t st) {
    const bool big = g_force_tile == 0 || (g_force_tile < 0 && (long)((g.M + 127) / 128) * ((H + 127) / 128) >= 512);
    if (g.a8_out) {  // 8-bit codes out
        if (big) return run_gemm<false, BITS, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 6>(g, 0, st);
        return run_gemm<false, BITS, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 6>(g, 1, st);
    }
    if (big) return run_gemm<false, BITS, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 1>(g, 0, st);
    return run_gemm<false, BITS, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 1>(g, 1, st);
}

// Weight-only gated projection, fp16 out (MODE 1 on the fp16 path).
int launch_gemm_w_only_geglu(const void* x, int M, int K, int ldx, const void* packed, int H, int bits,
                             const float* w_scale, const int32_t* w_zp, const void* bias, void* h16, int ldh,
                             const float* out_scale, const int32_t* out_zp, int8_t* a8_out, hipStream_t st) {
    GemmArgs g{};
    g.out_scale_p = out_scale; g.out_zp_p = out_zp; g.a8_out = a8_out;
    g.a = x;
    g.a_row_bytes = (long)ldx * 2;
    g.a_bytes = (uint32_t)(((long)(M - 1) * ldx + K) * 2);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((2 * H + 31) / 32) * (K / 64) * 256 * bits);
    g.M = M; g.N = 2 * H; g.K = K;
    g.k_stages = K / 64;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)h16; g.ldy = ldh;
    g.ld8 = a8_out ? (H + 127) / 128 * 128 : H;  // without code output the grid covers the H gated columns only
    switch (bits) {
        case 2: return dispatch_w_only_geglu<2>(g, H, st);
        case 3: return dispatch_w_only_geglu<3>(g, H, st);
        case 4: return dispatch_w_only_geglu<4>(g, H, st);
        case 8: return dispatch_w_only_geglu<8>(g, H, st);
    }
    return MQ_ERR_UNSUPPORTED_BITS;
}

// Integer GEMM on activations that arrive as codes in the int8 activation layout (MODE 2).
int launch_gemm_a8_codes(const int8_t* a8, long lda, const float* act_scale, const int32_t* act_zp, int M, int K,
                         const void* packed, int N, int w_bits, int w_signed, const float* w_scale, const int32_t* w_zp,
                         const int32_t* w_colsum, const void* bias, void* y, int ldy, int32_t* acc_debug,
                         const void* res, int ldr, hipStream_t st) {
    const int Kp = (K + 127) / 128 * 128;
    GemmArgs g{};
    g.a = a8;
    g.a_row_bytes = lda;
    g.a_bytes = (uint32_t)((long)(M - 1) * lda + Kp);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((N + 31) / 32) * (K / 64) * 256 * w_bits);
    g.M = M; g.N = N; g.K = K;
    g.k_stages = Kp / 128;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)y; g.ldy = ldy;
    g.res = (const uint16_t*)res; g.ldr = ldr;
    g.w_colsum = w_colsum;
    g.act_scale_p = act_scale; g.act_zp_p = act_zp;
    g.acc_debug = acc_debug;
    g.w_off = w_bits == 8 && !w_signed ? 128 : 0;
    if (const int form = solo_form(g, true, w_bits, 2); form >= 0) return launch_gemm_solo(g, form, true, w_bits, 2, st);
    // no in-workgroup k split here, and not the large tile (no registers to spare for the row sums; the layers this
    // serves, the output linears of feed-forward blocks, are narrow); the half-height tile 5 in place of tile 1
    int t = pick_tile(M, N, K, true);
    t = t == 6 ? 1 : (t >= 3 ? t - 2 : t);
    // Tile 5 (16384 x 2560 x 640 at 4 bits 40 us against 48; 4096 x 5120 x 1280 37.5 against 44.6; at 2 and 4 bits 0 to 30 % faster
    // over 1000 shapes).  8-bit weights move twice the bytes: there tile 1 where two of its workgroups on the busiest compute
    // unit are no more rows than four of the half height (4928 x 5120 x 1280 45.8 us against 58.5; of more rows, 4096 x 5120 x
    // 1280, 44.5 against 42.4), and for many tiles over weights that an XCD's 4 MB L2 does not hold and half the height fetches twice as
    // often (16384 x 5120 x 1280 134 against 145).
    const long t1 = (long)((M + 127) / 128) * ((N + 127) / 128);
    const bool full_height = g_force_tile >= 0 ? g_force_tile != 5
                             : t1 <= 2 * UNITS ? t1 > UNITS && busiest(M, N, 128) <= busiest(M, N, 64)
                                               : t1 > 3 * UNITS && (long)N * K > (4L << 20);
    if (w_bits == 4) {
        if (t <= 1) return run_gemm<true, 4, 1, 4, 2, 1, 1, 40 * 1024, 3, false, 2>(g, 5, st);
        return run_gemm<true, 4, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 2>(g, 2, st);
    }
    if (w_bits == 2) {
        if (t <= 1) return run_gemm<true, 2, 1, 4, 2, 1, 1, 40 * 1024, 3, false, 2>(g, 5, st);
        return run_gemm<true, 2, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 2>(g, 2, st);
    }
    if (w_bits == 8) {
        switch (t) {
            case 0:
            case 1:
                if (!full_height) return run_gemm<true, 8, 1, 4, 2, 1, 1, 52 * 1024, 3, false, 2>(g, 5, st);
                return run_gemm<true, 8, 2, 2, 2, 2, 1, 80 * 1024, 4, false, 2>(g, 1, st);
            default: return run_gemm<true, 8, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 2>(g, 2, st);
        }
    }
    return MQ_ERR_UNSUPPORTED_BITS;
}


// 3x3 convolution, stride 1, zero padding 1, channels-last (MODE 3 weight-only, MODE 4 int8 activations).
static void conv_args(GemmArgs& g, int B, int H, int W, int Cin, int stride, long pix_bytes) {
    g.a_row_bytes = pix_bytes;
    g.a_bytes = (uint32_t)((long)B * H * W * pix_bytes);
    g.conv_stride = stride;
    const int ho = (H - 1) / stride + 1, wo = (W - 1) / stride + 1;
    g.M = B * ho * wo;
    g.K = 9 * Cin;
    g.conv_h = H;
    g.conv_w = W;
    g.fd_ho = FastDiv::make((uint32_t)ho);
    g.fd_wo = FastDiv::make((uint32_t)wo);
    g.conv_cpt = Cin / 64;
    g.conv_cpt_inv = g.conv_cpt > 1 ? (uint32_t)(((1ull << 32) + g.conv_cpt - 1) / g.conv_cpt) : 0u;
}

// Tile of a convolution: no split of the reduction over workgroups (the weight-only entry point has no workspace), and the
// split inside the workgroup (tile 4) only while every workgroup has a compute unit of its own.  A reduction is then 90
// to 270 k steps long and bound by the latency of operands that two wave groups request together (weight-only with twice
// the LDS as stages in flight: 4-bit weights 128 -> 122 us below; the int8 path gains nothing from them).  With a second
// workgroup on the unit the other waves are there already.  Residual blocks, one wave group -> two, us per pass:
//   1 x 20 x 20 x 1280 (140 workgroups): W4A16 142 -> 123, W8A16 145 -> 117, W4A8 122 -> 109, W8A8 115 -> 103
//   1 x 40 x 40, 960 -> 640 (250):       W4A16 93 -> 82, W8A16 94 -> 77, W4A8 90 -> 82, W8A8 83 -> 76
//   1 x 32 x 32, 640 -> 1280 (320):      W4A16 133 -> 141, W8A16 131 -> 134, W4A8 115 -> 121, W8A8 109 -> 117
static int conv_tile(int M, int N, int K, bool wide_weights) {
    const int t = pick_tile(M, N, K, wide_weights);
    if (t == 6 || t == 3) return 1;
    if (t == 4 && g_force_tile < 0 && (long)((M + 63) / 64) * ((N + 63) / 64) > 256) return 2;
    return t;
}

template <int BITS>
static int dispatch_conv_w_only(GemmArgs& g, hipStream_t st) {
    constexpr bool WIDE = BITS == 16;
    if (const int form = solo_form(g, false, BITS, 3); form >= 0) return launch_gemm_solo(g, form, false, BITS, 3, st);
    int t = conv_tile(g.M, g.N, g.K, WIDE);
    // (the large tile only where its 256 channels are filled: the UNet's 320-channel level is better served by 128)
    if (g_force_tile < 0 && t == 0 && g.N < 512) t = 1;
    if (g_force_tile == 10 || (g_force_tile < 0 && t == 1 && taller(g.M, g.N, 9, 8)))
        return run_gemm<false, BITS, 1, 4, 3, 1, 1, 53 * 1024, 3, false, 3>(g, 10, st);
    switch (t) {
        case 0: return run_gemm<false, BITS, 1, 4, 4, 2, 1, 80 * 1024, 4, false, 3>(g, 0, st);
        case 1: return run_gemm<false, BITS, 1, 4, 2, 1, 1, 52 * 1024, 3, false, 3>(g, 5, st);
        case 4: return run_gemm<false, BITS, 2, 2, 1, 1, 2, 160 * 1024, 8, false, 3>(g, 4, st);
        default: return run_gemm<false, BITS, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 3>(g, 2, st);
    }
}

int launch_conv3x3_w_only(const void* x, int B, int H, int W, int Cin, int stride, const void* packed, int N, int bits,
                          const float* w_scale, const int32_t* w_zp, const void* bias, void* y, const void* res,
                          hipStream_t st) {
    GemmArgs g{};
    g.a = x;
    conv_args(g, B, H, W, Cin, stride, (long)Cin * 2);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((N + 31) / 32) * (g.K / 64) * 256 * bits);
    g.N = N;
    g.k_stages = g.K / 64;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)y; g.ldy = N;
    g.res = (const uint16_t*)res; g.ldr = N;
    switch (bits) {
        case 2: return dispatch_conv_w_only<2>(g, st);
        case 3: return dispatch_conv_w_only<3>(g, st);
        case 4: return dispatch_conv_w_only<4>(g, st);
        case 8: return dispatch_conv_w_only<8>(g, st);
    }
    return MQ_ERR_UNSUPPORTED_BITS;
}

int launch_conv3x3_a8(const int8_t* a8, const ActParams* params, int B, int H, int W, int Cin, int stride, const void* packed, int N,
                      int w_bits, int w_signed, const float* w_scale, const int32_t* w_zp, const int32_t* w_colsum,
                      const int32_t* w_tapsum, const void* bias, void* y, int32_t* acc_debug, const void* res,
                      hipStream_t st) {
    GemmArgs g{};
    g.a = a8;
    conv_args(g, B, H, W, Cin, stride, (long)(Cin + 127) / 128 * 128);
    g.packed = (const uint8_t*)packed;
    g.packed_bytes = (uint32_t)((long)((N + 31) / 32) * (g.K / 64) * 256 * w_bits);
    g.N = N;
    g.k_stages = (g.K + 127) / 128;
    g.w_scale = w_scale; g.w_zp = w_zp; g.bias = (const uint16_t*)bias;
    g.y = (uint16_t*)y; g.ldy = N;
    g.res = (const uint16_t*)res; g.ldr = N;
    g.w_colsum = w_colsum; g.w_tapsum = w_tapsum;
    g.act_scale_p = &params->scale; g.act_zp_p = &params->zp;
    g.acc_debug = acc_debug;
    g.w_off = w_bits == 8 && !w_signed ? 128 : 0;
    if (const int form = solo_form(g, true, w_bits, 4); form >= 0) return launch_gemm_solo(g, form, true, w_bits, 4, st);
    // (not the large tile: no registers to spare for the row sums and the tap masks; tile 5 in place of tile 1)
    int t = conv_tile(g.M, N, g.K, true);
    // Or tile 10, see taller(); it has two stages only, so not where a compute unit gets just one workgroup of it (2 x 32 x 32,
    // 1280 -> 1280 at 4 bits 64.2 us with tile 5, 69.9), and 8-bit weights leave room for fewer of them: 4-bit 4 x 32 x 32, 1280 -> 1280
    // 88.6 / 84.2, 3 x 64 x 64 x 640 (an eighth more rows) 65.2 / 63.9, 8-bit 98.4 / 89.1 and 79.0 / 84.6.
    if ((t <= 1 && g_force_tile < 0 && (long)((g.M + 95) / 96) * ((N + 127) / 128) > UNITS &&
         taller(g.M, N, w_bits == 8 ? 1 : 9, w_bits == 8 ? 1 : 8)) || g_force_tile == 10)
        t = 10;
    if (w_bits == 4) {
        if (t == 10) return run_gemm<true, 4, 1, 4, 3, 1, 1, 53 * 1024, 3, false, 4>(g, 10, st);
        if (t <= 1) return run_gemm<true, 4, 1, 4, 2, 1, 1, 40 * 1024, 3, false, 4>(g, 5, st);
        if (t == 4) return run_gemm<true, 4, 2, 2, 1, 1, 2, 80 * 1024, 8, false, 4>(g, 4, st);
        return run_gemm<true, 4, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 4>(g, 2, st);
    }
    if (w_bits == 2) {
        if (t == 10) return run_gemm<true, 2, 1, 4, 3, 1, 1, 53 * 1024, 3, false, 4>(g, 10, st);
        if (t <= 1) return run_gemm<true, 2, 1, 4, 2, 1, 1, 40 * 1024, 3, false, 4>(g, 5, st);
        if (t == 4) return run_gemm<true, 2, 2, 2, 1, 1, 2, 80 * 1024, 8, false, 4>(g, 4, st);
        return run_gemm<true, 2, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 4>(g, 2, st);
    }
    if (w_bits == 8) {
        if (t == 10) return run_gemm<true, 8, 1, 4, 3, 1, 1, 60 * 1024, 3, false, 4>(g, 10, st);
        if (t <= 1) return run_gemm<true, 8, 1, 4, 2, 1, 1, 52 * 1024, 3, false, 4>(g, 5, st);
        if (t == 4) return run_gemm<true, 8, 2, 2, 1, 1, 2, 80 * 1024, 8, false, 4>(g, 4, st);
        return run_gemm<true, 8, 2, 2, 1, 1, 1, 80 * 1024, 8, false, 4>(g, 2, st);
    }
    return MQ_ERR_UNSUPPORTED_BITS;
}

}  // namespace mq
