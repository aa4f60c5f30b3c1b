// 8-bit-activation linears that convert their own activations (gfx950): fp16 activations with a run-time range, reductions short enough
// that 64 rows of codes stay in LDS.
//
// One launch in place of two: a workgroup owns 64 rows and a range of 32-channel units; it converts its rows to int8 straight into LDS
// (the same operations as act_quantize_kernel, so the same codes) and multiplies them with every unit of its range.  Nothing of the
// conversion passes through memory.  After the one barrier behind it every wave is on its own: it streams the packed weights of its units
// (one contiguous run of tiles) through a ring of LDS slots that only it uses, multiplies 64 x 32 results at a time and stores them while
// the other waves go on multiplying.
//
// What bounds the two launches at these sizes is their number: conversion 5 to 7 us and GEMM 4.5 to 14, each of it mostly ramp, first loads and
// drain.  What bounds this one is the conversion (about 60 vector instructions for eight values, of 64 rows in every range of channels) and the
// loads ahead of it, so it pays where K is short and the output takes few ranges.  Sixteen waves, 1024 threads: a panel of up to 640 k is one
// round of loads for the conversion (512 threads with two rounds took 1.17 times as long at 16384 x 640 x 640 and 4 bits), and four waves per SIMD cover
// each other's LDS reads, widening and stores.  Whole calls in us, two launches -> this, 4-bit weights, run-time range: 1 x 320 x 320 9.3 -> 7.4, 256 x
// 320 x 320 (8 bits) 10.4 -> 8.4, 4096 x 320 x 320 13 -> 10.4, 16384 x 320 x 320 17.6 -> 13.1, 16384 x 576 x 320 21.6 -> 16.3, 16384 x 640 x 640 24.7 ->
// 19.8.
//
// Compiled with -ffp-contract=off (see act_range.h): fused multiply-adds are written out.
#include <stdio.h>

#include <algorithm>
#include <mutex>

#include "act_range.h"
#include "gemm_core.h"

namespace mq {

struct PanelArgs {
    const _Float16* x;
    long ldx;
    int flat;                // rows follow each other without a gap
    FastDiv K8;
    const float* partials;   // (min, max) pairs of the range pass, where there was one
    int n_partials;
    float* act_scale_out;
    int32_t* act_zp_out;
    int M, N, K;
    const uint8_t* packed;
    const float* w_scale;
    const int32_t* w_zp;
    const int32_t* w_colsum;
    const uint16_t* bias;
    int w_off;
    uint16_t* y;
    long ldy;
    const uint16_t* res;
    long ldr;
    int32_t* acc_debug;
    int units;               // 32-channel units of a workgroup's range
    FastDiv ranges;          // d: ranges of the output's channels
};

static constexpr int PANEL_NT = 1024, PANEL_WAVES = PANEL_NT / 64;
static constexpr int PANEL_MAX_K = 640, PANEL_MAX_UNITS = 20;

// LDS of a workgroup: the panel, 64 rows x 128 bytes per 128 k (pieces swizzled as in the other kernels), per wave D slots of one weight
// tile and a slab of 32 x 32 results on their way out, the constants of the range's channels, the row sums and the waves' extremes.
template <int BITS>
struct PanelPlan {
    static constexpr int D = BITS == 8 ? 2 : 4;
    static constexpr int SLOT = BITS == 8 ? 2048 : 1024;  // (a load writes 16 bytes for every lane, 2-bit tiles have half of them)
    static constexpr int WAVE = D * SLOT + 2048;
    static constexpr size_t bytes(int K, int units) {
        return (size_t)((K + 127) / 128) * 8192 + PANEL_WAVES * WAVE + (size_t)units * 32 * 16 + 64 * 4 + 2 * PANEL_WAVES * 4;
    }
    static_assert(bytes(PANEL_MAX_K, PANEL_MAX_UNITS) <= 160 * 1024, "LDS of a compute unit");
};

// SELF: the tensor is small enough for every workgroup to find its range by itself (one launch in all).
template <int BITS, bool RES, bool SELF>
__global__ __launch_bounds__(PANEL_NT) void gemm_panel_kernel(const PanelArgs g) {
    using P = PanelPlan<BITS>;
    constexpr int D = P::D, NT = PANEL_NT, WAVES = PANEL_WAVES, PCS = BITS == 8 ? 2 : 1, TILE_B = 256 * BITS, OOB = 0x7FFFF000;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l31 = lane & 31, kb = lane >> 5;
    // workgroup -> (64 rows, range of units); the ranges of the same rows run on one XCD
    const int total = gridDim.x, per = total >> 3, bid = blockIdx.x;
    uint32_t rb, range;
    g.ranges.divmod((uint32_t)(bid < per * 8 ? (bid & 7) * per + (bid >> 3) : bid), rb, range);
    const int m0 = (int)rb * 64, KC = g.K >> 6, all_units = (g.N + 31) >> 5;
    const int u0 = (int)range * g.units;
    const int units = all_units - u0 < g.units ? all_units - u0 : g.units;

    const int panel_bytes = (g.K + 127) / 128 * 8192;
    uint8_t* const ring = lds + panel_bytes + wv * P::WAVE;
    uint8_t* const ep = ring + D * P::SLOT;
    float* const ch_mul = (float*)(lds + panel_bytes + WAVES * P::WAVE);
    float* const ch_add = ch_mul + g.units * 32;
    int* const ch_dw = (int*)(ch_add + g.units * 32);
    int* const ch_cn = ch_dw + g.units * 32;
    int* const lsum = ch_cn + g.units * 32;
    float* const smn = (float*)(lsum + 64);

    // this wave's units: a contiguous run, one more for the first waves
    const int share = units / WAVES, more = units % WAVES;
    const int mine = share + (wv < more ? 1 : 0), first = wv * share + (wv < more ? wv : more);
    const int tiles = mine * KC;  // weight tiles of the run, one after the other in memory
    const int4s rw = make_rsrc(g.packed + (long)(u0 + first) * KC * TILE_B, (uint32_t)tiles * TILE_B);
    const uint32_t ring_lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)ring);
    int w_voff[PCS];
#pragma unroll
    for (int i = 0; i < PCS; ++i) w_voff[i] = lane * 16 < TILE_B ? i * 1024 + lane * 16 : OOB;
    // Tile t of the run into its slot.  What lies behind the run is requested through a descriptor of no bytes: every tile is the same number
    // of loads.
    auto issue = [&](int t, int slot) {
        int4s r = rw;
        r[2] = t < tiles ? r[2] : 0;
#pragma unroll
        for (int i = 0; i < PCS; ++i) dma_to_lds_b128(r, ring_lds + (uint32_t)(slot * P::SLOT), (uint32_t)(i * 1024), w_voff[i], t * TILE_B);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) issue(d, d);

    // ---- activations: 64 rows, vectors of eight values
    constexpr int U = 5;  // vectors per thread and round
    const uint32_t K8 = g.K8.d, nvp = 64u * K8;
    half8 v[U];
    uint32_t row[U], piece[U];
    auto request = [&](uint32_t base) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * NT + threadIdx.x;
            g.K8.divmod(i, row[u], piece[u]);
            if (i < nvp && m0 + (int)row[u] < g.M) v[u] = ((const half8*)(g.x + (long)(m0 + (int)row[u]) * g.ldx))[piece[u]];
        }
    };
    request(0);  // on its way while the parameters are derived
    if (threadIdx.x < 64) lsum[threadIdx.x] = 0;
    float mn, mx, s, zf;
    if constexpr (SELF) {
        const RowWalk plain{};
        constexpr int SU = 10;  // (at most two rounds)
        extremes<SU, NT>(g.x, (uint32_t)g.M * K8, g.K8, g.ldx, plain, g.flat, 0, SU * NT, mn, mx);
    } else {
        pair_extremes<NT>(g.partials, g.n_partials, mn, mx);
    }
    group_extremes<NT>(mn, mx, smn, smn + WAVES);
    range_params(mn, mx, s, zf);
    const float inv = 1.0f / s;
    if (bid == 0 && threadIdx.x == 0) {
        if (g.act_scale_out) *g.act_scale_out = s;
        if (g.act_zp_out) *g.act_zp_out = (int)zf;
    }
    for (uint32_t base = 0; base < nvp; base += NT * U) {
        if (base) request(base);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * NT + threadIdx.x;
            if (i < nvp && m0 + (int)row[u] < g.M) {  // (aligned groups of eight lanes agree; rows that do not exist stay unwritten)
                const uint2v w = quantize8(v[u], inv, zf);
                const uint32_t at = (piece[u] >> 4) * 8192 + row[u] * 128 + ((((piece[u] & 15) >> 1) ^ (uint32_t)swz((int)row[u])) << 4) + (piece[u] & 1) * 8;
                *(uint2v*)(lds + at) = w;
                int sum = __builtin_amdgcn_sdot4((int)w[0], 0x01010101, 0, false);
                sum = sum8(__builtin_amdgcn_sdot4((int)w[1], 0x01010101, sum, false));
                if ((lane & 7) == 0) atomicAdd(&lsum[row[u]], sum);
            }
        }
    }
    // constants of the range's channels (gemm_kernel's epilogue explains them)
    const int dx = 128 - (int)zf;
    for (int t = threadIdx.x; t < units * 32; t += NT) {
        int n = u0 * 32 + t;
        n = n < g.N ? n : g.N - 1;
        const int dw = g.w_off - g.w_zp[n];
        ch_dw[t] = dw;
        ch_cn[t] = dx * (g.w_colsum[n] - g.K * g.w_off + g.K * dw);
        ch_mul[t] = g.w_scale[n] * s;
        ch_add[t] = g.bias ? (float)__builtin_bit_cast(_Float16, g.bias[n]) : 0.0f;
    }
    __syncthreads();
    if (mine == 0) {
        wait_vmcnt<0>();
        return;
    }

    // ---- products: one 64 x 32 unit after the other
    const uint32_t xflip = g.w_off ? 0x80808080u : 0u;
    int rsum[2];
#pragma unroll
    for (int tm = 0; tm < 2; ++tm) rsum[tm] = lsum[tm * 32 + l31];
    // Pieces of the two k-steps of an even 64-k tile (two tiles per 128-byte row, two pieces a step); those of an odd one are four pieces on,
    // one bit under the swizzle.  (Four offsets indexed by the tile lie in scratch memory, and every read of that waits for all loads in flight.)
    const int sw = swz(l31);  // (the same for row l31 + 32)
    const uint32_t rd0 = (uint32_t)(l31 * 128 + (((kb * 2) ^ sw) << 4)), rd1 = (uint32_t)(l31 * 128 + (((kb * 2 + 1) ^ sw) << 4));
    auto read_x = [&](int4v (&f)[2], int c, int st) {
        const uint8_t* p = lds + (c >> 1) * 8192 + ((st ? rd1 : rd0) ^ (uint32_t)((c & 1) << 6));
        f[0] = *(const int4v*)p;
        f[1] = *(const int4v*)(p + 32 * 128);
    };
    const __amdgpu_buffer_rsrc_t ry =
        __builtin_amdgcn_make_buffer_rsrc((void*)(g.y + (long)m0 * g.ldy), 0, (int)(((long)((g.M - m0 < 64 ? g.M - m0 : 64) - 1) * g.ldy + g.N) * 2), 0x00020000);
    WChunk<BITS> wq;
    int4v xa[2], xb[2];
    // (a tile has landed when no more than the loads of the D - 1 younger ones are outstanding)
    wait_vmcnt<(D - 1) * PCS>();
    read_chunk<BITS>(wq, ring, lane);
    read_x(xa, 0, 0);
    int t = 0, slot = 0;  // tile, and its slot in the ring
    for (int u = 0; u < mine; ++u) {
        int16v acc[2];
#pragma unroll
        for (int tm = 0; tm < 2; ++tm)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tm][i] = 0;
        for (int c = 0; c < KC; ++c, ++t) {
            int4v w0 = widen_step<BITS>(wq, 0, xflip), w1 = widen_step<BITS>(wq, 1, xflip);
            asm volatile("" : "+v"(w0), "+v"(w1));  // the slot has been read: it may be filled again
            issue(t + D, slot);
            slot = slot + 1 == D ? 0 : slot + 1;
            read_x(xb, c, 1);
            // Tile t + 1 has landed when no more than the D - 1 younger ones are outstanding, and the four stores of the unit before while
            // they are younger than it (every store is issued: what lies outside the output is dropped by the buffer's bounds).
            if (c < D - 1 && u > 0)
                wait_vmcnt<(D - 1) * PCS + 4>();
            else
                wait_vmcnt<(D - 1) * PCS>();
            read_chunk<BITS>(wq, ring + slot * P::SLOT, lane);
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) acc[tm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w0, xa[tm], acc[tm], 0, 0, 0);
            read_x(xa, c + 1 == KC ? 0 : c + 1, 0);
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) acc[tm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w1, xb[tm], acc[tm], 0, 0, 0);
        }
        // epilogue of the unit, a slab of 32 rows at a time
        const int cu = (first + u) * 32, nu = u0 * 32 + cu;  // first channel inside the range, in the output
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const int m = m0 + tm * 32 + l31;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int cl = cu + 8 * q + 4 * kb, n = nu + 8 * q + 4 * kb;
                const float4v mul = *(const float4v*)(ch_mul + cl);
                float4v add = *(const float4v*)(ch_add + cl);
                const int4v dw = *(const int4v*)(ch_dw + cl), cn = *(const int4v*)(ch_cn + cl);
                if constexpr (RES) {
                    half4 rq = {0, 0, 0, 0};
                    if (m < g.M && n < g.N) rq = *(const half4*)(g.res + (long)m * g.ldr + n);
#pragma unroll
                    for (int r = 0; r < 4; ++r) add[r] += (float)rq[r];
                }
                int4v a;
                half4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    a[r] = acc[tm][4 * q + r] + __mul24(dw[r], rsum[tm]) + cn[r];
                    o[r] = (_Float16)__builtin_fmaf((float)a[r], mul[r], add[r]);
                }
                if (g.acc_debug && m < g.M && n < g.N) *(int4v*)(g.acc_debug + (long)m * g.N + n) = a;
                *(half4*)(ep + l31 * 64 + (((q ^ (l31 >> 2)) & 3) << 4) + kb * 8) = o;
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = i * 16 + (lane >> 2), c = lane & 3, n = nu + c * 8;
                const uint4v o = *(const uint4v*)(ep + r * 64 + (((c ^ (r >> 2)) & 3) << 4));
                const int voff = m0 + tm * 32 + r < g.M && n < g.N ? ((tm * 32 + r) * (int)g.ldy + n) * 2 : OOB;
                __builtin_amdgcn_raw_buffer_store_b128(o, ry, voff, 0, 2 /* streaming */);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    wait_vmcnt<0>();  // (the loads of no bytes behind the run)
}

template <int BITS, bool RES, bool SELF>
static int run_panel_s(const PanelArgs& g, int wgs, hipStream_t st) {
    auto kern = gemm_panel_kernel<BITS, RES, SELF>;
    const int slot = prof_gemm_slot(8, BITS, 4 + (SELF ? 1 : 0));
    // once per instantiation and device (callers may be on several host threads)
    static std::mutex prep_mutex;
    static bool prepared[16] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) dev = 0;
    {
        std::lock_guard<std::mutex> lock(prep_mutex);
        if (!prepared[dev]) {
            if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
                set_hip_error((int)hipGetLastError());
                return MQ_ERR_HIP;
            }
            char name[112];
            snprintf(name, sizeof name, "mq::gemm_panel_kernel<%d, false, %s>", BITS, SELF ? "true" : "false");
            prof_name_slot(slot, name);
            prepared[dev] = true;
        }
    }
    ProfScope prof(st, slot, 2.0 * g.M * g.N * g.K, 2.0 * g.M * g.K + (double)g.N * g.K * BITS / 8 + 14.0 * g.N + 2.0 * g.M * g.N);
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(PANEL_NT), PanelPlan<BITS>::bytes(g.K, g.units), st, g);
    MQ_HIP_CHECK_LAUNCH();
    return MQ_OK;
}

template <int BITS>
static int run_panel(const PanelArgs& g, int wgs, bool self, hipStream_t st) {
    if (g.res) return self ? run_panel_s<BITS, true, true>(g, wgs, st) : run_panel_s<BITS, true, false>(g, wgs, st);
    return self ? run_panel_s<BITS, false, true>(g, wgs, st) : run_panel_s<BITS, false, false>(g, wgs, st);
}

// How the output's channels are cut: as many ranges as fill the compute units once, of up to 20 units.
static void panel_split(int M, int N, int* units, int* ranges) {
    const int rows = (M + 63) / 64, all = (N + 31) / 32;
    const int r = std::max(1, (int)(UNITS / rows));
    *units = std::min(PANEL_MAX_UNITS, (all + r - 1) / r);
    *ranges = (all + *units - 1) / *units;
}

// Times of this over the two launches (277 shapes of 1 to 16384 rows, 320 to 1288 channels; mean and largest), by rows, in one round of workgroups:
//   up to 320 k   up to 15 0.83 0.89, up to 511 0.82 0.89, up to 1023 0.87 0.99, beyond 0.80 0.89
//   up to 512 k   up to 15 0.85 0.89, up to 511 0.90 0.97, up to 1023 0.93 1.03, up to 4095 0.89 0.94, up to 8191 0.82 0.91, beyond 0.83 0.90
//   up to 640 k   up to 15 0.84 0.89, up to 511 0.91 1.10, up to 1023 0.94 1.06, up to 4095 0.90 0.94, up to 8191 0.82 0.92, beyond 0.81 0.97
//   in more than one round 1.01 to 1.27
// (pairs in profiles/tile_rules.txt).  The lines beyond 320 k were drawn for a loop that waited for all its loads at every tile and was the slower one
// between 16 and 8191 rows; for this one they are too narrow, and have not been drawn anew.  Calls with given parameters keep their two launches:
// not measured here, and a test pins the tile that each of them runs.
bool panel_takes(int M, int N, int K, long ldy) {
    const int forced = forced_tile();
    if ((forced >= 0 && forced != 14) || forced_splits() > 1 || K < 256 || K > PANEL_MAX_K || ldy >= (1L << 23)) return false;
    if (forced == 14) return true;
    int units, ranges;
    panel_split(M, N, &units, &ranges);
    if ((long)((M + 63) / 64) * ranges > UNITS) return false;
    if (M < 16 || K <= 320) return true;
    return M >= 8192 && N <= 640;
}

int launch_gemm_panel(const void* x, int M, int K, int ldx, const float* partials, int pairs, float* act_scale_out, int32_t* act_zp_out,
                      const void* packed, int N, int w_bits, int w_signed, const float* w_scale, const int32_t* w_zp, const int32_t* w_colsum,
                      const void* bias, void* y, int ldy, int32_t* acc_debug, const void* res, int ldr, hipStream_t st) {
    int units, ranges;
    panel_split(M, N, &units, &ranges);
    PanelArgs g{};
    g.x = (const _Float16*)x; g.ldx = ldx; g.flat = ldx == K; g.K8 = FastDiv::make((uint32_t)K / 8);
    g.partials = partials; g.n_partials = pairs;
    g.act_scale_out = act_scale_out; g.act_zp_out = act_zp_out;
    g.M = M; g.N = N; g.K = K;
    g.packed = (const uint8_t*)packed; g.w_scale = w_scale; g.w_zp = w_zp; g.w_colsum = w_colsum; g.bias = (const uint16_t*)bias;
    g.w_off = w_bits == 8 && !w_signed ? 128 : 0;
    g.y = (uint16_t*)y; g.ldy = ldy; g.res = (const uint16_t*)res; g.ldr = ldr; g.acc_debug = acc_debug;
    g.units = units; g.ranges = FastDiv::make((uint32_t)ranges);
    const int wgs = (M + 63) / 64 * ranges;
    const bool self = pairs == 0;
    if (w_bits == 2) return run_panel<2>(g, wgs, self, st);
    if (w_bits == 4) return run_panel<4>(g, wgs, self, st);
    if (w_bits == 8) return run_panel<8>(g, wgs, self, st);
    return MQ_ERR_UNSUPPORTED_BITS;
}

}  // namespace mq
