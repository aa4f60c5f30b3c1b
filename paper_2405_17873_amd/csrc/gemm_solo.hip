// MFMA GEMMs with one wave per SIMD (gfx950): the linears and 3x3 convolutions whose tiles of 256 x 160 (or 128 x 160) fill the chip evenly
// and whose reduction is long.
//
// What bounds the kernels of gemm.hip there (64 x 128 and 96 x 128 tiles, three to five workgroups per compute unit): a wave tile of 64 x 32
// reads an LDS fragment and widens half a weight fragment per MFMA, every stage of 8 MFMAs per wave ends in a barrier, and at the rate at which
// the chip runs MFMAs on real data (power: 1.6 to 1.8 GHz) what a multiplication moves through LDS costs clock as well.  Here a workgroup of
// four waves has a compute unit to itself and a wave owns 64 x 160 results, 160 accumulators of its 512 registers: a stage is 40 MFMAs per wave
// and one barrier, a third of the LDS reads per MFMA, and half the L2 -> LDS bytes (34 to 52 KB per 40 MFMAs).  With no other wave on the SIMD
// every latency is covered by the wave's own MFMAs: reads, widening and the loads of later stages are laid out between them one by one
// (a lone wave has room for about seven instructions per MFMA: 32 cycles, one instruction in four).
// 160 columns, because 320, 640, 1280, ... are multiples of it and 128 leaves 320 and 960 a sixth and a sixteenth of the work for padding.
//
// Measured in us, gemm.hip's choice -> this, 4-bit weights unless said: convolutions 4 x 64 x 64 x 640 on 16-bit activations 121 -> 106, 2 x 128 x
// 128 x 320 on 8-bit ones 57 -> 45, 4 x 64 x 64, 960 -> 640 at 8 bits 142 -> 103; linears 16384 x 2560 x 640 with residual on 16-bit activations
// 69 -> 58 (8 bits 76 -> 58), on codes 49 -> 37.  A stage takes 1700 to 1800 cycles, its MFMAs alone 1308 (loads, LDS reads or widening left
// out in turn: 14 to 20 % less each); the tail, 7000 cycles (int8 12000), is the conversion of 160 results per lane and the store of 80 KB from every
// compute unit at once.  (Constants read per slab and stores behind branches: 10000 and 13000; the residual in pieces of 8 bytes: 4000 more.)
#include <stdio.h>

#include <algorithm>
#include <mutex>

#include "gemm_core.h"

namespace mq {

// Code widening by pairs (gemm_core.h widens whole fragments), so that it can be spread over the MFMAs.  Masks and magic number sit in
// registers that the compiler cannot see through: (w & mask) | magic is then one instruction, and one that it can schedule.
template <int BITS>
struct Masks {
    uint32_t m[4], magic;
    __device__ __forceinline__ Masks() {
        constexpr uint32_t M0 = BITS == 4 ? 0x000F000Fu : BITS == 3 ? 0x00070007u : 0x00030003u;
        constexpr int STEP = BITS == 4 ? 4 : BITS == 3 ? 3 : 2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            m[i] = M0 << (STEP * i);
            asm volatile("" : "+s"(m[i]));
        }
        magic = 0x64006400u;
        asm volatile("" : "+v"(magic));
    }
    // the field F steps up in each half of w, minus the zero point
    template <int F>
    __device__ __forceinline__ half2v field(uint32_t w, int z) const {
        constexpr int SHIFT = F * (BITS == 4 ? 4 : BITS == 3 ? 3 : 2);
        const half2v v = as_h2((w & m[F]) | magic);
        if constexpr (SHIFT == 0) {
            return v - splat((float)(1024 + z));
        } else {
            constexpr float inv = 1.0f / (float)(1 << SHIFT);
            return v * splat(inv) - splat((float)((1024 >> SHIFT) + z));
        }
    }
};
// Pair p (codes 2p, 2p + 1) of the fragment of k-step s.
template <int BITS>
__device__ __forceinline__ half2v dequant_pair(const WChunk<BITS>& c, int s, int p, const Masks<BITS>& k, int z) {
    if constexpr (BITS == 4) {
        const uint32_t w = p < 2 ? c.w[s] : c.w[s] >> 8;
        return (p & 1) ? k.template field<1>(w, z) : k.template field<0>(w, z);
    } else if constexpr (BITS == 2) {
        const uint32_t w = (s & 1) ? c.w[s >> 1] >> 8 : c.w[s >> 1];
        return p == 0 ? k.template field<0>(w, z) : p == 1 ? k.template field<1>(w, z) : p == 2 ? k.template field<2>(w, z) : k.template field<3>(w, z);
    } else if constexpr (BITS == 3) {
        const int i = 4 * s + p, f = i % 5;
        if (i == 15) {
            const uint32_t t = ((c.w[0] >> 15) & 0x00010001u) | ((c.w[1] >> 14) & 0x00020002u) | ((c.w[2] >> 13) & 0x00040004u);
            return k.template field<0>(t, z);
        }
        const uint32_t w = f < 3 ? c.w[i / 5] : c.w[i / 5] >> 9;
        return f == 0 || f == 3 ? k.template field<0>(w, z) : f == 1 || f == 4 ? k.template field<1>(w, z) : k.template field<2>(w, z);
    } else {
        const uint32_t w = c.w[(s >> 1) * 4 + (s & 1) * 2 + (p & 1)];
        return as_h2(__builtin_amdgcn_perm(0x64646464u, w, p < 2 ? 0x04020400u : 0x04030401u)) - splat((float)(1024 + z));
    }
}
// Template arguments as gemm_kernel's.  MODE 0: Y = linear(X).  MODE 2 (int8): the activations arrive as codes.  MODE 3 / 4: 3x3 convolution on
// 16-bit / 8-bit activations.  The reduction has at least S stages, and output rows are where their number says (no row map).
template <bool I8, int BITS, int WGM, int S, int KS, int MODE, bool RES>
__global__ __launch_bounds__(256, 1) void gemm_solo_kernel(const GemmArgs g) {
    constexpr int TM = 2, TN = 5;  // wave tile of 64 x 160
    constexpr bool RS_INLINE = MODE == 2 || MODE == 4, CONV = MODE == 3 || MODE == 4;
    static_assert(WGM * KS == 4, "four waves, one per SIMD");
    static_assert((MODE != 2 && MODE != 4) || I8, "int8 modes");
    static_assert(MODE != 3 || !I8, "MODE 3 is the weight-only convolution");
    using P = GemmPlan<I8, BITS, WGM, 1, TM, TN, S, KS>;
    constexpr int NW = P::NW, BM = P::BM, BN = P::BN, CH = P::CH, STAGE_BYTES = P::STAGE_BYTES;
    using acc_t = typename std::conditional<I8, int16v, float16v>::type;
    using frag_t = typename std::conditional<I8, int4v, half8>::type;

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wv / P::NWG, wvg = wv % P::NWG;
    const int wm = wvg;
    int bm, bn;
    tile_of_block(blockIdx.x, g, bm, bn);
    const int m0 = bm * BM, n0 = bn * BN;
    const int KC = g.K >> 6;
    const int G = (g.N + 31) >> 5;
    auto group_of = [&](int gt) {
        const int gi = (n0 >> 5) + gt;
        return gi < G ? gi : G - 1;
    };
    const int l31 = lane & 31, kb = lane >> 5;
    const uint32_t xflip = (I8 && g.w_off) ? 0x80808080u : 0u;
    constexpr int TILE_B = 256 * BITS;
    constexpr int OOB = 0x7FFFF000;

    const int4s ra = make_rsrc(g.a, g.a_bytes);
    const int4s rb = make_rsrc(g.packed, g.packed_bytes);
    const uint32_t lds_base = (uint32_t)(uintptr_t)lds;

    // Activation loads: lane -> (row, physical slot) of an 8-row group; it fetches the logical piece slot ^ swz(row).  Rows past M read as zero.
    int a_voff[P::DMA_A];
    uint32_t a_lds[P::DMA_A];
    static_assert((BM / 8) % NW == 0, "a load belongs to one k step for every wave alike");
    constexpr int A_PER_SUB = P::DMA_A / KS;
    int a_half[CONV ? P::DMA_A : 1];
    uint32_t a_taps[CONV ? P::DMA_A : 1];
    struct Centre {
        int index;
        uint32_t rows, cols;
        __device__ uint32_t taps() const { return (rows & 1u ? cols : 0u) | cols << 3 | (rows & 4u ? cols << 6 : 0u); }
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
        const int sub = i / A_PER_SUB, row0 = (j % (BM / 8)) * 8;
        const int row = row0 + (lane >> 3);
        const int piece = (lane & 7) ^ swz(row);
        a_voff[i] = m0 + row < g.M ? (int)((long)(m0 + row) * g.a_row_bytes + sub * 128 + piece * 16) : OOB;
        a_lds[i] = __builtin_amdgcn_readfirstlane((uint32_t)(sub * P::SUB_BYTES + row0 * 128));
        if constexpr (CONV) {
            const bool real = m0 + row < g.M;
            const Centre c = centre_of(real ? m0 + row : g.M - 1);
            a_voff[i] = (int)((long)c.index * g.a_row_bytes) + (I8 ? (piece & 3) : piece) * 16;
            a_half[i] = I8 ? piece >> 2 : 0;
            a_taps[i] = real ? c.taps() : 0u;
        }
    }
    // weight loads: instruction jj of a k step copies piece jj % PCS of weight tile jj / PCS (tile = channel group, 64-k chunk)
    constexpr int PCS = P::PIECES;
    constexpr int VALID_LANES = BITS >= 8 ? 64 : 16 * BITS;
    int b_voff[P::DMA_B];
    uint32_t b_lds[P::DMA_B];
    bool b_pad[P::DMA_B];
    constexpr bool B_TAIL = I8 || KS == 2;
    int b_chunk[B_TAIL ? P::DMA_B : 1];
#pragma unroll
    for (int i = 0; i < P::DMA_B; ++i) {
        const int j = i * NW + wv;
        const int sub = j / P::NBI1, jj = j % P::NBI1;
        const int t = jj / PCS, piece = jj % PCS;
        const int gt = t / CH, cc = t % CH;
        const int gi = group_of(gt);
        const bool on = j < P::NBI && lane < VALID_LANES;
        b_voff[i] = on ? (gi * KC + sub * CH + cc) * TILE_B + piece * 1024 + lane * 16 : OOB;
        if constexpr (B_TAIL) b_chunk[i] = __builtin_amdgcn_readfirstlane(sub * CH + cc);
        b_pad[i] = j >= P::NBI;  // a padding load, into the sink
        b_lds[i] = __builtin_amdgcn_readfirstlane(b_pad[i] ? 0u : (uint32_t)(sub * P::SUB_BYTES + P::A_BYTES + t * P::BSLOT + piece * 1024));
    }

    // Weight zero points of the 16-bit-activation path travel like a stage, as the oldest loads: an ordinary load here would be waited for
    // with a count that does not know the LDS-writing loads.
    constexpr bool ZP_LDS = !I8;
    constexpr int ZP_SLOT = P::CONSTS + 2 * BN * 4;
    if constexpr (ZP_LDS) {
        if (wv < (BN + 63) / 64) {
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

    acc_t acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;

    float c_scale = 0.0f;
    uint32_t c_bias_bits = 0;
    int c_zp = 0, c_colsum = 0;
    float c_sx = 1.0f;
    int c_zx = 0;
    if constexpr (I8) {
        c_sx = RS_INLINE ? *g.act_scale_p : g.params->scale;
        c_zx = RS_INLINE ? *g.act_zp_p : g.params->zp;
    }
    if (threadIdx.x < BN) {
        int n = group_of((int)threadIdx.x >> 5) * 32 + ((int)threadIdx.x & 31);
        n = n < g.N ? n : g.N - 1;
        c_scale = g.w_scale[n];
        if (g.bias) c_bias_bits = g.bias[n];
        if constexpr (I8) {
            c_zp = g.w_zp[n];
            c_colsum = g.w_colsum[n];
        }
    }
    int rsum[TM];
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

    const int KSTEPS = g.k_stages;
    const int KT = (KSTEPS + KS - 1) / KS;
    // Loads of one stage, one at a time.  What lies past the reduction (whole stages behind the last, the phantom half of a
    // stage) is requested through a descriptor of no bytes: every stage issues the same number of loads, without a branch.
    struct StageAt {
        int step0;
        uint32_t sb;
        int soff[CONV ? KS : 1];
    };
    // Convolution: lane offsets of the loads of the stage that is being requested, and the filter tap that they hold for (-1: two).
    int c_voff[CONV ? P::DMA_A : 1];
    int c_tap[CONV ? KS : 1];
#pragma unroll
    for (int i = 0; i < (CONV ? KS : 1); ++i) c_tap[i] = -1;
    auto stage_at = [&](int stage, int buf) {
        StageAt s;
        s.step0 = __builtin_amdgcn_readfirstlane(stage * KS);
        s.sb = __builtin_amdgcn_readfirstlane(lds_base + buf * STAGE_BYTES);
        if constexpr (CONV) {
#pragma unroll
            for (int sub = 0; sub < KS; ++sub) {
                // 64-channel chunks of the k step -> (filter tap, chunk inside the tap).  While the tap stays, the channels advance in the
                // scalar offset; another one, and a step of 8-bit activations that holds the end of one tap and the start of the next,
                // set the lane offsets anew.
                constexpr int CHUNK = I8 ? 64 : 128;  // bytes of 64 channels
                int tap[CH], cc[CH], delta[CH];
#pragma unroll
                for (int h = 0; h < CH; ++h) {
                    const uint32_t ci = (uint32_t)(s.step0 + sub) * CH + h;
                    const uint32_t t = g.conv_cpt > 1 ? __umulhi(ci, g.conv_cpt_inv) : ci;
                    cc[h] = (int)(ci - t * g.conv_cpt);
                    tap[h] = ci < (uint32_t)KC ? (int)t : 31;  // past the end of K: no tap
                    delta[h] = __builtin_amdgcn_readfirstlane((((int)t / 3 - 1) * g.conv_w + ((int)t % 3 - 1)) * (int)g.a_row_bytes);
                }
                const bool whole = CH == 1 || tap[CH - 1] == tap[0];
                s.soff[sub] = __builtin_amdgcn_readfirstlane(whole ? cc[0] * CHUNK : 0);
                if (!whole || tap[0] != c_tap[sub]) {
                    c_tap[sub] = __builtin_amdgcn_readfirstlane(whole ? tap[0] : -1);
#pragma unroll
                    for (int i = sub * A_PER_SUB; i < (sub + 1) * A_PER_SUB; ++i) {
                        const int second = CH == 2 && a_half[i];
                        const int t = second ? tap[CH - 1] : tap[0];
                        const int d = (second ? delta[CH - 1] : delta[0]) + (whole ? (second ? 64 : 0) : (second ? 0 : cc[0] * CHUNK));
                        const int in = (int)(a_taps[i] << (31 - t)) >> 31;  // all ones where the tap reads inside the image
                        c_voff[i] = (in & (a_voff[i] + d)) | (~in & OOB);
                    }
                }
            }
        }
        return s;
    };
    // Load k of a stage: its LDS address (which the load takes from a register of its own, at least one instruction later), and the load.
    auto address_op = [&](const StageAt& s, int k) {
        if (k < P::DMA_A)
            dma_address(s.sb, a_lds[k < P::DMA_A ? k : 0]);
        else
            dma_address(b_pad[k < P::DMA_A ? 0 : k - P::DMA_A] ? lds_base + P::SINK : s.sb, b_lds[k < P::DMA_A ? 0 : k - P::DMA_A]);
    };
    auto load_op = [&](const StageAt& s, int k) {
        if (k < P::DMA_A) {
            const int i = k < P::DMA_A ? k : 0, sub = i / A_PER_SUB;
            if constexpr (CONV) {
                dma_load_b128(ra, c_voff[CONV ? i : 0], s.soff[CONV ? sub : 0]);
            } else {
                int4s r = ra;
                if (KS == 2 && sub) r[2] = s.step0 + sub < KSTEPS ? r[2] : 0;
                dma_load_b128(r, a_voff[i], s.step0 * 128);
            }
        } else {
            const int i = k < P::DMA_A ? 0 : k - P::DMA_A;
            int4s r = rb;
            if (B_TAIL) r[2] = s.step0 * CH + b_chunk[B_TAIL ? i : 0] < KC ? r[2] : 0;
            dma_load_b128(r, b_voff[i], s.step0 * CH * TILE_B);
        }
    };
    auto issue_op = [&](const StageAt& s, int k) {
        address_op(s, k);
        asm volatile("s_nop 0");
        load_op(s, k);
    };

    const int sw = swz(l31);
    uint32_t rd[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int piece = I8 ? ((s >> 1) * 4 + kb * 2 + (s & 1)) : (kb * 4 + s);
        rd[s] = (uint32_t)(grp * P::SUB_BYTES + wm * TM * 32 * 128 + l31 * 128 + ((piece ^ sw) << 4));
    }

    long long t0 = 0, t1 = 0, t2 = 0;
    if (g.phase_clk) t0 = clock64();
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        const StageAt at = stage_at(s, s);
#pragma unroll
        for (int k = 0; k < P::OPS; ++k) issue_op(at, k);
    }
    StageAt at = stage_at(S - 1, S - 1);
#pragma unroll
    for (int k = 0; k < P::OPS; ++k)
        if (k * 4 * TM * TN / P::OPS < 2 * TM * TN) issue_op(at, k);
    constexpr int OPS_EARLY = (2 * TM * TN * P::OPS + 4 * TM * TN - 1) / (4 * TM * TN);  // loads of a stage ahead of its second half
    if (g.phase_clk) t1 = clock64();

    WChunk<BITS> wq[TN][CH];
    frag_t xf[4][TM], wf[2][TN];
    auto read_x = [&](const uint8_t* stage, int s, int tm) { xf[s][tm] = *(const frag_t*)(stage + rd[s] + tm * 32 * 128); };
    auto read_w = [&](const uint8_t* stage, int tn) {
#pragma unroll
        for (int c = 0; c < CH; ++c)
            read_chunk<BITS>(wq[tn][c], stage + grp * P::SUB_BYTES + P::A_BYTES + (tn * CH + c) * P::BSLOT, lane);
    };
    // Part `p` of `TM` of the widened fragment of channel tile tn for k-step s.
    const Masks<BITS> masks;
    auto widen_part = [&](frag_t& f, int tn, int s, int p) {
        if constexpr (I8) {
            const frag_t w = widen_step<BITS>(wq[tn][CH == 2 ? s >> 1 : 0], s & 1, xflip);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e * TM / 4 == p) f[e] = w[e];
        } else {
            uint4v w = __builtin_bit_cast(uint4v, f);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e * TM / 4 == p) {
                    const half2v v = dequant_pair<BITS>(wq[tn][0], s, e, masks, zc[tn]);
                    w[e] = h2_bits(v);
                }
            f = __builtin_bit_cast(frag_t, w);
        }
    };
    auto mfma = [&](int tm, int tn, const frag_t& w, const frag_t& x) {
        if constexpr (I8)
            acc[tm][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, acc[tm][tn], 0, 0, 0);
        else
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w, x, acc[tm][tn], 0, 0, 0);
    };

    constexpr int W_FIRST = (S - 2) * P::OPS + OPS_EARLY;
    static_assert(W_FIRST <= 63, "hand-counted loads");
    wait_vmcnt<W_FIRST>();
    __syncthreads();
    if constexpr (ZP_LDS) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) zc[tn] = *(const int*)(lds + ZP_SLOT + (tn * 32 + l31) * 4);
    }
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) read_w(lds, tn);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) read_x(lds, 0, tm);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) read_x(lds, 1, tm);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int p = 0; p < TM; ++p) widen_part(wf[0][tn], tn, 0, p);

    constexpr int SLOTS = TM * TN;
    static_assert(SLOTS % 2 == 0 && P::OPS <= 4 * SLOTS, "at most one load of a stage per slot");
    // Residual of the slabs this wave finishes, requested in the last stages but S - 1: eight channels of its row per lane, 16 bytes; the two
    // lanes of a row swap halves when they are used.  It may lie on any multiple of 8 bytes: buffer loads of 16 need no more than 4.  It may be the
    // output: a wave reads what no other one writes, but for channels beyond the last, whose results are dropped.
    constexpr int RES_LOADS = RES ? TM / KS * TN * 2 : 0;
    uint4v rs[RES ? TM / KS : 1][RES ? TN : 1][2];
    __amdgpu_buffer_rsrc_t rr;
    int r_voff[RES ? TM / KS : 1];
    if constexpr (RES) {
        const int rows = g.M - m0 < BM ? g.M - m0 : BM;
        rr = __builtin_amdgcn_make_buffer_rsrc((void*)(g.res + (long)m0 * g.ldr), 0, (int)(((long)(rows - 1) * g.ldr + g.N) * 2), 0x00020000);
#pragma unroll
        for (int i = 0; i < TM / KS; ++i)
            r_voff[i] = (((wm * TM + (KS == 2 ? 2 * i + grp : i)) * 32 + l31) * (int)g.ldr + n0 + 8 * kb) * 2;
    }
    int buf = 0, kt = 0;
    // One stage.  EARLY: the second half of the loads that the stage before began to request; LATE: the first half of the stage that takes
    // this one's buffer; LAST: stages behind this one (-1: S or more), their loads are all on their way then.
    auto stage = [&](auto early_c, auto late_c, auto last_c) {
        constexpr bool EARLY = decltype(early_c)::value, LATE = decltype(late_c)::value;
        constexpr int LAST = decltype(last_c)::value;
        constexpr bool NEXT = LAST != 0;
        const uint8_t* cur = lds + buf * STAGE_BYTES;
        const int nb = buf + 1 == S ? 0 : buf + 1;
        const uint8_t* next = lds + nb * STAGE_BYTES;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s == 2 && NEXT) {
                // hand-over
                constexpr int YOUNGER = LAST < 0 ? (S - 2) * P::OPS : (LAST - 1) * P::OPS + (LAST < S - 1 ? RES_LOADS : 0);
                static_assert(YOUNGER <= 63, "hand-counted loads");
                wait_vmcnt<YOUNGER>();
                __syncthreads();
                if constexpr (LATE) at = stage_at(kt + S, buf);
            }
#pragma unroll
            for (int j = 0; j < SLOTS; ++j) {
                const int tn = j / TM, tm = j % TM;
                const bool loads = (s < 2 && EARLY) || (s >= 2 && LATE);
                const int at_slot = ((s + 2) & 3) * SLOTS + j;  // from the hand-over to the next one
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (EARLY || LATE) {
#pragma unroll
                    for (int k = 0; k < P::OPS; ++k)
                        if (loads && k * 4 * SLOTS / P::OPS == at_slot) address_op(at, k);
                }
                __builtin_amdgcn_sched_barrier(0);
                mfma(tm, tn, wf[s & 1][tn], xf[s][tm]);
                if constexpr (EARLY || LATE) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < P::OPS; ++k)
                        if (loads && k * 4 * SLOTS / P::OPS == at_slot) load_op(at, k);
                }
                if (j < TM) {
                    if (s < 2)
                        read_x(cur, s + 2, j);
                    else if (NEXT)
                        read_x(next, s - 2, j);
                }
                if (s < 3 || NEXT) widen_part(wf[(s + 1) & 1][tn], tn, (s + 1) & 3, tm);
                if (s == 2 && tm == TM - 1 && NEXT) {
                    asm volatile("" : "+v"(wf[1][tn]));
                    read_w(next, tn);
                }
                if constexpr (RES && LAST == S - 1) {
                    if (s >= 2) {
#pragma unroll
                        for (int k = 0; k < RES_LOADS; ++k)
                            if (k * 2 * SLOTS / RES_LOADS == (s - 2) * SLOTS + j) {
                                const int slab = k / (TN * 2), rt = k / 2 % TN, h = k % 2;
                                rs[RES ? slab : 0][RES ? rt : 0][h] = __builtin_amdgcn_raw_buffer_load_b128(rr, r_voff[RES ? slab : 0] + (rt * 32 + 16 * h) * 2, 0, 0);
                            }
                    }
                }
                if constexpr (RS_INLINE) {
                    if (tn == 0) {
                        const int4v a = __builtin_bit_cast(int4v, xf[s][tm]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) rsum[tm] = __builtin_amdgcn_sdot4(a[i], 0x01010101, rsum[tm], false);
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        buf = nb;
        ++kt;
    };
    using no = std::false_type;
    using yes = std::true_type;
    while (kt < KT - S) stage(yes{}, yes{}, std::integral_constant<int, -1>{});
    stage(yes{}, no{}, std::integral_constant<int, S - 1>{});
    if constexpr (S > 3) stage(no{}, no{}, std::integral_constant<int, (S > 3 ? S - 2 : 1)>{});
    if constexpr (S > 2) stage(no{}, no{}, std::integral_constant<int, 1>{});
    stage(no{}, no{}, std::integral_constant<int, 0>{});
    static_assert(S >= 3 && S <= 4, "stages");
    __syncthreads();

    // ---- epilogue
    constexpr int RS_PARTS = KS;
    int* const rs_x = (int*)(lds + P::SINK) + wm * TM * 32 + l31;
    if constexpr (RS_INLINE) {
        static_assert(RS_PARTS == 1 || RS_PARTS * BM * 4 <= P::CONSTS - P::SINK, "shares of the row sums fit the sink");
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            rsum[tm] += __shfl_xor(rsum[tm], 32, 64);
            if (RS_PARTS > 1 && lane < 32) rs_x[grp * BM + tm * 32] = rsum[tm];
        }
    }
    float* ch_mul = (float*)(lds + P::CONSTS);
    float* ch_add = ch_mul + BN;
    int* ch_dw = (int*)(ch_add + BN);
    int* ch_cn = ch_dw + BN;
    int* const ch_border = (int*)(lds + S * STAGE_BYTES) - 16 * BN;
    if (threadIdx.x < BN) {
        const int t = threadIdx.x;
        if constexpr (I8) {
            asm volatile("" : "+s"(c_zx), "+s"(c_sx));
            const int dx = 128 - c_zx;
            const int dw = g.w_off - c_zp;
            ch_dw[t] = dw;
            const int cn = dx * (c_colsum - g.K * g.w_off + g.K * dw);
            ch_cn[t] = cn;
            if constexpr (MODE == 4) {
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
        ch_mul[t] = c_scale * c_sx;
        asm volatile("" : "+v"(c_bias_bits));
        ch_add[t] = (float)__builtin_bit_cast(_Float16, (uint16_t)c_bias_bits);
    }

    constexpr int TMX = TM / KS;  // slabs a wave finishes
    auto owner = [](int tm) { return KS == 2 ? (tm & 1) : 0; };
    if constexpr (KS == 2) {
        using quad_t = typename std::conditional<I8, int4v, float4v>::type;
        constexpr int XW = TN * 4 * 1024;  // bytes a wave sends per pair of slabs
        static_assert(NW * XW + (MODE == 4 ? 64 * BN : 0) <= S * STAGE_BYTES, "accumulator exchange must fit the stages");
        auto area = [&](int writer) { return lds + (wvg * 2 + writer) * XW + lane * 16; };
        uint8_t* out = area(grp);
        const uint8_t* in = area(1 - grp);
#pragma unroll
        for (int pr = 0; pr < TM / 2; ++pr) {
            if (pr) __syncthreads();
#pragma unroll
            for (int tm = 2 * pr; tm < 2 * pr + 2; ++tm) {
                if (owner(tm) == grp) continue;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        quad_t v;
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = acc[tm][tn][4 * q + r];
                        *(quad_t*)(out + (tn * 4 + q) * 1024) = v;
                    }
            }
            __syncthreads();
#pragma unroll
            for (int tm = 2 * pr; tm < 2 * pr + 2; ++tm) {
                if (owner(tm) != grp) continue;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const quad_t v = *(const quad_t*)(in + (tn * 4 + q) * 1024);
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[tm][tn][4 * q + r] += v[r];
                    }
            }
        }
    }
    __syncthreads();
    if constexpr (RS_INLINE && RS_PARTS > 1) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            rsum[tm] = 0;
#pragma unroll
            for (int i = 0; i < RS_PARTS; ++i) rsum[tm] += rs_x[i * BM + tm * 32];
        }
    }
    if (g.phase_clk) t2 = clock64();

    constexpr int CPR = TN * 4;
    constexpr int EP_BYTES = 32 * CPR * 16;
    static_assert(NW * TMX * EP_BYTES + (MODE == 4 ? 64 * BN : 0) <= S * STAGE_BYTES, "epilogue staging must fit the LDS stages");
    uint8_t* ep = lds + wv * TMX * EP_BYTES;
    const int nw0 = n0;
    // 16-byte chunk of a staged row -> its place
    auto place = [](int row, int chunk) { return (chunk & ~3) | ((chunk ^ (row >> 2)) & 3); };
    // The constants of result quad q of channel tile tn: four consecutive channels.
    struct QuadConst {
        float4v mul, add;
        int4v dw, cn;
    };
    auto quad_const = [&](int i) {
        const int cl = (i >> 2) * 32 + 8 * (i & 3) + 4 * kb;
        QuadConst k;
        k.mul = *(const float4v*)(ch_mul + cl);
        k.add = *(const float4v*)(ch_add + cl);
        if constexpr (I8) {
            k.dw = *(const int4v*)(ch_dw + cl);
            if constexpr (MODE != 4) k.cn = *(const int4v*)(ch_cn + cl);
        }
        return k;
    };
    // int8 path: the exact integer sums of result quad i of slab tm with both zero-point corrections
    auto int_quad = [&](int tm, int i, const QuadConst& k) {
        int4v a, cn = k.cn;
        if constexpr (MODE == 4) cn = *(const int4v*)(ch_border + border[MODE == 4 ? tm : 0] * BN + (i >> 2) * 32 + 8 * (i & 3) + 4 * kb);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            // |dw| <= 255 and |rowsum| <= 128 * K < 2^23: a 24-bit multiply (full rate) is exact
            a[r] = (int)acc[tm][i >> 2][4 * (i & 3) + r] + __mul24(k.dw[r], rsum[tm]) + cn[r];
        return a;
    };
    if constexpr (I8) {
        if (g.acc_debug) {  // for the tests that pin them
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                if (owner(tm) != grp) continue;
                const int m = m0 + (wm * TM + tm) * 32 + l31;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n = n0 + tn * 32 + 8 * q + 4 * kb;
                        const int4v a = int_quad(tm, tn * 4 + q, quad_const(tn * 4 + q));
                        if (m < g.M && n < g.N) *(int4v*)(g.acc_debug + (long)m * g.N + n) = a;
                    }
            }
        }
    }
    // Slabs [from, to): convert (eight-byte pieces into the staged rows; a quad's constants are read once for all slabs, one quad ahead of the
    // conversions: there is no other wave to cover their latency), read back as 16 bytes per lane along rows, store rows of 320 bytes.
    // Every store is issued, without a branch: what lies outside the output is dropped by the buffer's bounds.
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(g.y + (long)m0 * g.ldy), 0, (int)(((long)((g.M - m0 < BM ? g.M - m0 : BM) - 1) * g.ldy + g.N) * 2), 0x00020000);
    auto finish = [&](auto from_c, auto to_c) {
        constexpr int FROM = decltype(from_c)::value, TO = decltype(to_c)::value;
        QuadConst k = quad_const(0);
#pragma unroll
        for (int i = 0; i < TN * 4; ++i) {
            const QuadConst kn = quad_const(i + 1 < TN * 4 ? i + 1 : i);
#pragma unroll
            for (int tm = FROM; tm < TO; ++tm) {
                float4v add = k.add;
                if constexpr (RES) {
                    uint4v& pair = rs[tm - FROM][i >> 2][(i & 3) >> 1];  // the lane's channels of quads i and i + 1, once the halves are swapped
                    if (i % 2 == 0) {
#pragma unroll
                        for (int d = 0; d < 2; ++d) {
                            const auto sw2 = __builtin_amdgcn_permlane32_swap(pair[d], pair[2 + d], false, false);
                            pair[d] = sw2[0], pair[2 + d] = sw2[1];
                        }
                    }
                    const half4 rq = __builtin_bit_cast(half4, uint2v{pair[2 * (i & 1)], pair[2 * (i & 1) + 1]});
#pragma unroll
                    for (int r = 0; r < 4; ++r) add[r] += (float)rq[r];
                }
                half4 o;
                if constexpr (I8) {
                    const int4v a = int_quad(tm, i, k);
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = (_Float16)((float)a[r] * k.mul[r] + add[r]);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = (_Float16)(acc[tm][i >> 2][4 * (i & 3) + r] * k.mul[r] + add[r]);
                }
                *(half4*)(ep + (tm - FROM) * EP_BYTES + l31 * (CPR * 16) + (place(l31, i) << 4) + kb * 8) = o;
            }
            k = kn;
        }
        __builtin_amdgcn_wave_barrier();
        constexpr int NP = 32 * CPR / 64;
#pragma unroll
        for (int tm = FROM; tm < TO; ++tm) {
            uint4v v[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int idx = i * 64 + lane, row = idx / CPR, c = idx % CPR;
                v[i] = *(const uint4v*)(ep + (tm - FROM) * EP_BYTES + row * (CPR * 16) + (place(row, c) << 4));
            }
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int idx = i * 64 + lane, row = (wm * TM + tm) * 32 + idx / CPR, n = nw0 + idx % CPR * 8;
                const int voff = m0 + row < g.M && n < g.N ? (row * (int)g.ldy + n) * 2 : OOB;
                __builtin_amdgcn_raw_buffer_store_b128(v[i], ry, voff, 0, 2 /* streaming */);
            }
        }
    };
    if constexpr (KS == 1) {
        finish(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
    } else {
        if (grp == 0)
            finish(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
        else
            finish(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
    }
    if (g.phase_clk && threadIdx.x == 0) {
        long long* o = g.phase_clk + (long)blockIdx.x * 4;
        o[0] = t0;
        o[1] = t1;
        o[2] = t2;
        o[3] = clock64();
    }
}

// ---------------------------------------------------------------------------------------------
// Launchers.  Form 0: 256 x 160, four waves side by side along the rows.  Form 1: 128 x 160, two waves along the rows and two on the halves of
// the reduction (their sums meet in LDS); under 8-bit activations for convolutions only (see solo_form), and not with 8-bit weights, whose stages
// leave room for two only.
// ---------------------------------------------------------------------------------------------
template <bool I8, int BITS>
constexpr int solo_stages(int form) {
    return form == 0 && !I8 && BITS != 8 ? 4 : 3;
}

static constexpr bool solo_has_halves(bool i8, int bits, int mode) { return !i8 || (mode == 4 && bits != 8); }

template <bool I8, int BITS, int FORM, int MODE, bool RES>
static int run_solo_r(GemmArgs& g, hipStream_t st) {
    constexpr int S = solo_stages<I8, BITS>(FORM), KS = FORM + 1, WGM = 4 / KS;
    using P = GemmPlan<I8, BITS, WGM, 1, 2, 5, S, KS>;
    static_assert(P::LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
    g.tiles_m = (g.M + P::BM - 1) / P::BM;
    g.tiles_n = (g.N + P::BN - 1) / P::BN;
    set_tile_walk(g, forced_band() > 0 ? forced_band() : 8);  // (2 to 16: within 3 %; 32: 4 to 9 % slower)
    g.splits = 1;
    g.phase_clk = phase_buffer((long)g.tiles_m * g.tiles_n);
    auto kern = gemm_solo_kernel<I8, BITS, WGM, S, KS, MODE, RES>;
    const int slot = prof_gemm_slot(!I8 ? 7 : MODE == 0 ? 8 : MODE == 2 ? 9 : 10, BITS, FORM + (MODE == 3 ? 2 : 0));
    // once per instantiation and device (callers may be on several host threads)
    static std::mutex prep_mutex;
    static bool prepared[16] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) dev = 0;
    {
        std::lock_guard<std::mutex> lock(prep_mutex);
        if (!prepared[dev]) {
            if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, P::LDS_BYTES) != hipSuccess) {
                set_hip_error((int)hipGetLastError());
                return MQ_ERR_HIP;
            }
            char name[112];
            snprintf(name, sizeof name, "mq::gemm_solo_kernel<%s, %d, %d, %d, %d, %d, false>", I8 ? "true" : "false", BITS, WGM, S, KS, MODE);
            prof_name_slot(slot, name);
            prepared[dev] = true;
        }
    }
    ProfScope prof(st, slot, 2.0 * g.M * g.N * g.K, gemm_alg_bytes(g, I8, BITS, MODE));
    hipLaunchKernelGGL(kern, dim3(g.tiles_m * g.tiles_n), dim3(P::NT), P::LDS_BYTES, st, g);
    MQ_HIP_CHECK_LAUNCH();
    return MQ_OK;
}

template <bool I8, int BITS, int MODE>
static int run_solo(GemmArgs& g, int form, hipStream_t st) {
    if (form == 0) return g.res ? run_solo_r<I8, BITS, 0, MODE, true>(g, st) : run_solo_r<I8, BITS, 0, MODE, false>(g, st);
    if constexpr (solo_has_halves(I8, BITS, MODE))
        if (form == 1) return g.res ? run_solo_r<I8, BITS, 1, MODE, true>(g, st) : run_solo_r<I8, BITS, 1, MODE, false>(g, st);
    return MQ_ERR_BAD_ARG;
}

template <bool I8, int MODE>
static int run_solo_bits(GemmArgs& g, int form, int bits, hipStream_t st) {
    if (bits == 2) return run_solo<I8, 2, MODE>(g, form, st);
    if (bits == 4) return run_solo<I8, 4, MODE>(g, form, st);
    if (bits == 8) return run_solo<I8, 8, MODE>(g, form, st);
    if constexpr (!I8)
        if (bits == 3) return run_solo<I8, 3, MODE>(g, form, st);
    return MQ_ERR_UNSUPPORTED_BITS;
}

int launch_gemm_solo(GemmArgs& g, int form, bool i8, int bits, int mode, hipStream_t st) {
    if (!i8) return mode == 3 ? run_solo_bits<false, 3>(g, form, bits, st) : run_solo_bits<false, 0>(g, form, bits, st);
    if (mode == 2) return run_solo_bits<true, 2>(g, form, bits, st);
    return mode == 4 ? run_solo_bits<true, 4>(g, form, bits, st) : run_solo_bits<true, 0>(g, form, bits, st);
}

// Which calls run here: a long reduction, and tiles that fill the chip.  A kernel lasts as long as its busiest compute unit: `fit` compares
// the results that this one computes with form 0 or 1 and with the better of gemm.hip's 64 x 128 and 96 x 128 tiles.  Times of this over
// gemm.hip's choice (17000 drawn shapes of 1024 to 20000 rows and convolutions of 512 and more; mean, 9 in 10 below, largest):
//   form 0, fit up to 1.05   16-bit: linears 0.89 0.94 0.98, convolutions 0.85 0.92 0.97 (at fit 0.8 0.78); int8: linears 2 bits 0.96 1.01 1.04,
//                            4 bits 0.89 0.91 0.97, 8 bits 0.83 0.93 0.95; convolutions 2 bits 0.91, 4 bits 0.86, 8 bits 0.76; on codes below
//   ... 1.05 to 1.15         16-bit 0.95 to 1.05; int8: linears 2 bits 0.97 1.02 1.03, 4 bits 0.90 0.96 1.07, 8 bits 0.86 0.93 0.97; convolutions
//                            2 and 4 bits 1.03 to 1.09, 8 bits 0.77
//   ... 1.25                 1.0 to 1.15, but int8 convolutions at 8 bits 0.83 0.90 0.94
//   form 1, fit up to 0.85   16-bit: linears 0.88 to 0.91 (3 bits 0.95), convolutions 0.83 to 0.90; at fit 1.0 1.0 to 1.1; int8: convolutions of
//                            5760 k and more 0.83 to 0.95, of 2880 (22 stages, and the halves' sums have to meet) 1.03; linears 0.98, codes 0.96
// Reductions below 2048 k (convolutions and codes: 2560) do not repay the store at the end, 0.96 to 1.05 at fit 1.0 and more with every round of
// workgroups; 16-bit linears in one round do from 1280 k on at 4 bits (to 1407 0.97 1.00 1.01, from there 0.93 to 0.94) and 8 (0.92 and 0.88), not
// at 2 (1.00 and 0.97).  Where at least 19/20 of that round is output, also shorter ones: with a residual, which this kernel has in registers by then,
// from 640 k on (us: 16384 x 640 x 640 at 2, 3, 4, 8 bits 24.2 -> 22.3, 22.3 -> 21.7, 23.1 -> 21.0, 24.1 -> 21.7, int8 at 4 and 8 bits 26.4 -> 25.2 and
// 27.3 -> 26.1; 32768 x 640 x 320 at 4 bits 27.9 -> 20.1; 14000 x 640 x 640, 0.85 of the round, 17.2 -> 18.2), without one 16-bit linears at 8 bits (16384 x 640 x
// 640 18.3 -> 16.8, 2048 x 640 x 5120 18.5 -> 16.8; at 4 bits 16.9 -> 16.7 and 16.7 -> 16.8) and from 960 k on at 4 bits (16384 x 960 x 640 22.8 -> 21.8; at 2
// bits 23.1 -> 22.7 and 22.5 -> 22.0, left); int8 without a residual 0.93 to 1.1.
// Pairs of times on both sides of the lines are in profiles/tile_rules.txt.
int solo_form(const GemmArgs& g, bool i8, int bits, int mode) {
    const int forced = forced_tile();
    if ((forced >= 0 && forced < 12) || bits == 16) return -1;
    if (g.out_map.rows_per_group > 0 || forced_splits() > 1) return -1;
    if (g.ldy >= (1 << 21) || (g.res && g.ldr >= (1 << 21))) return -1;  // (offsets inside a workgroup's rows are 32-bit)
    const bool halves = solo_has_halves(i8, bits, mode);
    // (the stages that are requested ahead of the loop have to exist)
    auto long_enough = [&](int form) { return (g.k_stages + form) / (form + 1) >= 4; };
    if (forced == 12) return long_enough(0) ? 0 : -1;
    if (forced == 13) return !long_enough(1) || (i8 && bits == 8) ? -1 : halves ? 1 : 0;  // (where form 1 does not exist, form 0 is the nearest)
    if (forced > 13) return -1;
    const bool conv = mode == 3 || mode == 4;
    const long now = std::min(busiest_area(g.M, g.N, 64, 128), busiest_area(g.M, g.N, 96, 128));
    const long full = busiest_area(g.M, g.N, 256, 160), half = busiest_area(g.M, g.N, 128, 160);
    auto fit = [&](long area, int percent) { return 100 * area <= percent * now; };
    const bool one_round = full == 256 * 160;
    const bool filled = one_round && 20L * g.M * g.N >= 19 * UNITS * full;  // ... and hardly any of it padding
    const int shortest = mode != 0 ? 2560 : filled && g.res ? 640 : filled && !i8 && bits == 8 ? 640 : filled && !i8 && bits == 4 ? 960
                         : one_round && !i8 && (bits == 4 || bits == 8) ? 1280 : 2048;
    if (g.K < shortest) return -1;
    if (mode == 2) {
        // On codes: 8 bits 0.85 0.90 1.00 (rows that start inside a 64-byte sector 0.90 0.99 1.00: left where they were), 4 bits 0.92 0.96 0.98 in
        // one round of workgroups but 1.04 in two, 2 bits 0.98 and 1.12.
        if (bits == 8) return fit(full, 115) && g.ldy % 32 == 0 ? 0 : -1;
        return bits == 4 && fit(full, 115) && one_round ? 0 : -1;
    }
    // (int8 linears at 8 bits from 2624 k on, or with a residual in a filled round.  The line at 2560 is not where this form stops paying: the tile of
    // 16384 x 2560 x 640 is pinned by a test of the older rule.  us, that rule -> this: 16384 x 2560 x 640 61 -> 51, 16384 x 2048 x 640 53 -> 46,
    // 4096 x 2048 x 2560 37 -> 32, 8192 x 2304 x 1280 46 -> 39; above the line 16384 x 2624 x 640 65 -> 52.)
    if (mode == 0 && i8) return fit(full, 115) && (bits != 8 || g.K > 2560 || (filled && g.res)) ? 0 : -1;
    if (fit(full, i8 && bits == 8 ? 125 : 105)) return 0;
    return halves && fit(half, 85) && (!i8 || g.K >= 5120) && (conv || g.K >= 2560) ? 1 : -1;
}

}  // namespace mq
