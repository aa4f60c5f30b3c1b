// Per-tensor 8-bit activation quantisation (paper Sec. 4.1 "Quantization Scheme": one scale and
// zero point per activation tensor; Sec. 4.3: the FP16->INT8 conversion that precedes the integer GEMM).
//
//   pass 1 (dynamic only; small tensors do without, see act_quantize_kernel): every workgroup reduces the min/max of its rows with wavefront shuffles and
//           writes one partial pair; no atomics, no pre-cleared memory, order independent.
//   pass 2: every workgroup re-reduces the partials (a few KB, L2 resident), derives (scale, zp) with the
//           same fp32 operations as the weight quantiser, then converts its rows:
//               a'[m,k] = clamp(rne(x*inv) + zp, 0, 255) - 128   stored as int8, groups of 8 k in the order
//               0,4,1,5,2,6,3,7, rows padded with zeros to a multiple of 128, and rowsum[m] = sum_k a'[m,k].
//
// Compiled with -ffp-contract=off: each fp32 operation rounds once.
#include "act_range.h"
#include "bos_rows.h"

namespace mq {

static constexpr int kPartialSlots = 512;  // upper bound of pass-1 workgroups
int act_quant_partial_slots() { return kPartialSlots; }

// Both passes are bound by memory latency at the sizes of this path (5 to 80 MB per tensor): what counts is the
// number of bytes requested before the first one arrives.  The tensor is therefore walked as a flat list of 16-byte
// vectors (8 values; vector i is piece i % (K/8) of row i / (K/8)), every lane requests several vectors before it
// touches one, and the grids are sized so that every compute unit holds a few workgroups.
static constexpr int MM_U = 8;  // vectors per lane per round, pass 1
static constexpr int Q_U = 4;   // vectors per lane per round, pass 2 (at most: see the launcher)

// Bound by memory latency up to a few MB and by HBM above.
// (Workgroups of 1024 threads for tensors that need every partial slot left up to half of the slots without work and were
// slower at every size: 8192 x 1280 whole call 21.4 us against 20.4, 16384 x 2560 57.1 against 55.7.)
__global__ __launch_bounds__(256) void act_minmax_kernel(const _Float16* __restrict__ x, uint32_t nv, FastDiv K8,
                                                         long ldx, RowWalk map, int flat, float* __restrict__ partials) {
    constexpr uint32_t STEP = 256 * MM_U;
    float mn, mx;
    extremes<MM_U, 256>(x, nv, K8, ldx, map, flat, blockIdx.x * STEP, gridDim.x * STEP, mn, mx);
    __shared__ float smn[4], smx[4];
    group_extremes<256>(mn, mx, smn, smx);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = mn;
        partials[2 * blockIdx.x + 1] = mx;
    }
}

static constexpr int Q_MAX_ROWS = 128;   // rows per workgroup, pass 2
static constexpr int kQuantGrid = 2048;  // workgroups of a large tensor, pass 2: eight per compute unit
static constexpr long kSmallQuant = 28L * 1000 * 1000;  // values: between 6000 x 4608 and 7000 x 4160 (see the launcher)

// A workgroup converts R whole rows (so that it owns their row sums): R * Kp/8 output vectors, 1024 per round.  Up to a
// few MB it is bound by memory latency, above by HBM as long as a value costs few instructions: one fused multiply-add
// that widens it, one rounding, one addition and one saturating conversion into its byte (the conversion also takes NaN
// to code 0, as the clamp of the formula does), with the division of a vector index by the row length prepared by the
// host.  rowsum == nullptr: the caller's GEMM takes the sums itself, they are left out here.
// BOS: the first `nbos` workgroups compute the BOS rows of a BOS-aware K/V projection instead (they depend on nothing this
// kernel produces; one launch less on a path whose kernels are all bound by launch latency).  They take longest, so they
// come first.
// NT == 1024: a small tensor with a run-time range.  A launch of the range pass costs more than reading such a tensor again, so every
// workgroup finds the range of all of it by itself, with SELF_U vectors per lane on their way at once (see the launcher).
// Whole calls in us, range pass and conversion -> one launch: 1 x 320 -> 64 12.2 -> 8.8, 4 x 1280 -> 1280 12.7 -> 10.7, 64 x 1280 -> 1280 13.5 -> 11.7, 256 x 320 -> 320
// 12.5 -> 10.6, 100 x 1280 -> 1280 13.7 -> 12.8, 128 x 1280 -> 64 13.9 -> 13.1; with four rounds in place of two 250 x 1280 -> 64 14.0 -> 16.0, 154 x 2048 -> 64
// 15.1 -> 17.3, with the BOS rows beside it (four blocks of theirs per workgroup) 77 x 2048 -> 1280 16.7 -> 17.5.
static constexpr int SELF_NT = 1024, SELF_U = 10;
static constexpr uint32_t SELF_VECTORS = 2 * SELF_U * SELF_NT;
static_assert(SELF_VECTORS == ACT_SELF_VECTORS, "sizes that need no pass for the range");
template <bool BOS, int U, int NT = 256>
__global__ __launch_bounds__(NT) void act_quantize_kernel(const _Float16* __restrict__ x, int M, int K, long ldx, int flat, FastDiv K8d,
                                                           RowWalk map, int R, FastDiv Kp8d, const float* __restrict__ partials,
                                                           int n_partials, const float* __restrict__ act_scale,
                                                           const int32_t* __restrict__ act_zp,
                                                           int8_t* __restrict__ a8, int32_t* __restrict__ rowsum,
                                                           ActParams* __restrict__ params,
                                                           float* __restrict__ act_scale_out,
                                                           int32_t* __restrict__ act_zp_out, int nbos, BosWork bw) {
    int blk = (int)blockIdx.x;
    constexpr bool SELF = NT == SELF_NT;
    static_assert(!(BOS && SELF), "the BOS rows take workgroups of 256 threads");
    if constexpr (BOS) {
        __shared__ float part[4][256];
        if (blk < nbos) {  // (whole workgroups: none of them reaches a barrier below)
            bos_block(blk, (int)threadIdx.x, bw, part);
            return;
        }
        blk -= nbos;
    }
    const int lane = threadIdx.x & 63;
    __shared__ float smn[NT / 64], smx[NT / 64];
    __shared__ int lsum[Q_MAX_ROWS];
    const int r0 = blk * R;
    const int Rr = M - r0 < R ? M - r0 : R;
    if (threadIdx.x < Q_MAX_ROWS) lsum[threadIdx.x] = 0;
    const uint32_t K8 = K >> 3;
    const uint32_t Kp = (K + 127) / 128 * 128;  // row stride of the int8 copy; the padding is zero
    const uint32_t Kp8 = Kp8d.d;                // Kp / 8, a multiple of 16: an aligned group of 8 lanes never straddles rows
    const uint32_t nvo = (uint32_t)Rr * Kp8;
    half8 v[U];
    uint32_t lr[U], pp[U];
    auto request = [&](uint32_t base) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * (uint32_t)NT + threadIdx.x;
            Kp8d.divmod(i, lr[u], pp[u]);
            if (i < nvo && pp[u] < K8) v[u] = ((const half8*)(x + map.phys(r0 + lr[u]) * ldx))[pp[u]];
        }
    };
    request(0);  // on its way while the parameters are derived (most workgroups have a single round)
    float s, zf;
    if (SELF || partials) {
        float mn, mx;
        if constexpr (SELF)
            extremes<SELF_U, NT>(x, (uint32_t)M * K8, K8d, ldx, map, flat, 0, SELF_U * NT, mn, mx);
        else
            pair_extremes<NT>(partials, n_partials, mn, mx);
        group_extremes<NT>(mn, mx, smn, smx);
        range_params(mn, mx, s, zf);
    } else {
        s = *act_scale;
        zf = (float)*act_zp;
        __syncthreads();
    }
    const float inv = 1.0f / s;
    if (blk == 0 && threadIdx.x == 0) {
        params->scale = s;
        params->zp = (int)zf;
        if (act_scale_out) *act_scale_out = s;
        if (act_zp_out) *act_zp_out = (int)zf;
    }
    for (uint32_t base = 0; base < nvo; base += (uint32_t)NT * U) {
        if (base) request(base);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * (uint32_t)NT + threadIdx.x;
            const bool valid = i < nvo;
            uint32_t w0 = 0, w1 = 0;
            if (valid && pp[u] < K8) {
                const uint2v w = quantize8(v[u], inv, zf);
                w0 = w[0], w1 = w[1];
            }
            // (streaming store: read next by another kernel, nothing gained by keeping it in this XCD's L2)
            if (valid) {
                const uint2v out = {w0, w1};
                __builtin_nontemporal_store(out, (uint2v*)(a8 + (long)(r0 + lr[u]) * Kp) + pp[u]);
            }
            if (rowsum) {
                int sum = __builtin_amdgcn_sdot4((int)w0, 0x01010101, 0, false);
                sum = sum8(__builtin_amdgcn_sdot4((int)w1, 0x01010101, sum, false));
                if (valid && (lane & 7) == 0) atomicAdd(&lsum[lr[u]], sum);
            }
        }
    }
    if (!rowsum) return;
    __syncthreads();
    if ((int)threadIdx.x < Rr) rowsum[r0 + threadIdx.x] = lsum[threadIdx.x];
}

int launch_act_range(const void* x, int M, int K, int ldx, RowMap in_map, float* partials, int* pairs, hipStream_t st) {
    const uint32_t K8 = (uint32_t)K >> 3;
    const uint32_t nv = (uint32_t)M * K8;  // M * ldx * 2 < 2^31 has been checked: this fits easily
    const long g1 = ((long)nv + 256 * MM_U - 1) / (256 * MM_U);
    const int grid = (int)(g1 > kPartialSlots ? kPartialSlots : g1);
    ProfScope prof(st, PROF_ACT_MINMAX, 0.0, 2.0 * M * K);
    hipLaunchKernelGGL(act_minmax_kernel, dim3(grid), dim3(256), 0, st, (const _Float16*)x, nv, FastDiv::make(K8), (long)ldx,
                       RowWalk::make(in_map), in_map.rows_per_group <= 0 && ldx == K, partials);
    MQ_HIP_CHECK_LAUNCH();
    *pairs = grid;
    return MQ_OK;
}

int launch_act_quant(const void* x, int M, int K, int ldx, RowMap in_map, const float* act_scale,
                     const int32_t* act_zp, int8_t* a8, int32_t* rowsum, ActParams* params, float* partials,
                     float* act_scale_out, int32_t* act_zp_out, const BosWork* bos, hipStream_t st,
                     int given_partials) {
    const uint32_t K8 = (uint32_t)K >> 3;
    const uint32_t nv = (uint32_t)M * K8;
    int grid = 0;  // (min, max) pairs
    const RowWalk walk = RowWalk::make(in_map);
    const bool dynamic = act_scale == nullptr;
    const int flat = in_map.rows_per_group <= 0 && ldx == K;
    const int Kp8 = (K + 127) / 128 * 16;
    if (dynamic && given_partials == 0 && nv <= SELF_VECTORS && !bos) {
        int R = SELF_NT / Kp8;
        R = R < 1 ? 1 : R > Q_MAX_ROWS ? Q_MAX_ROWS : R;
        ProfScope prof(st, PROF_ACT_QUANTIZE, 0.0, 3.0 * M * K + (rowsum ? 4.0 * M : 0.0));
        auto kern = act_quantize_kernel<false, 1, SELF_NT>;
        hipLaunchKernelGGL(kern, dim3((M + R - 1) / R), dim3(SELF_NT), 0, st, (const _Float16*)x, M, K, (long)ldx, flat, FastDiv::make(K8), walk, R,
                           FastDiv::make(Kp8), (const float*)nullptr, 0, act_scale, act_zp, a8, rowsum, params, act_scale_out, act_zp_out, 0,
                           BosWork{});
        MQ_HIP_CHECK_LAUNCH();
        return MQ_OK;
    }
    // given_partials > 0: the producer of x has left that many (min, max) pairs in `partials` already (the gated
    // projection's epilogue does), so the pass over x that would find them is skipped
    if (dynamic && given_partials > 0) {
        grid = given_partials;
    } else if (dynamic) {
        if (const int rc = launch_act_range(x, M, K, ldx, in_map, partials, &grid, st)) return rc;
    }
    // Vectors per lane: as few as keep a row in one round and the grid within eight workgroups per compute unit, so that
    // small tensors have more wavefronts to request them.  Whole calls with 64 output channels in us, four -> two -> one vector:
    //   given parameters 77 x 2048 10.0 -> 9.5 -> 9.3, 256 x 320 7.1 -> 6.5 -> 6.4, 616 x 2048 10.7 -> 10.3 -> 10.1,
    //     4096 x 640 9.5 -> 9.1 -> 8.9, 4096 x 320 8.0 -> 7.6 -> 7.4; 2964 x 1280 (one: 2964 workgroups) 10.5 -> 10.3
    //   run-time range, every workgroup reads the pairs, so one vector only up to a workgroup per compute unit, two up to four:
    //     77 x 2048 13.4 -> 12.4 -> 12.3, 256 x 320 10.3 -> 9.5 -> 9.4, 616 x 2048 14.3 -> 14.0 -> 14.2, 1024 x 640 12.2 -> 11.5 -> 11.6,
    //     4096 x 1280 (two: 1366 workgroups) 17.6 -> 17.6
    // Beyond that grid, rows per workgroup: one round (1024 vectors) while that keeps it within eight workgroups per compute
    // unit.  A larger tensor can take as many rounds per workgroup as bring it there: the parameters are derived (and the pairs read)
    // that many times less often, but the grid may leave compute units idle at its end, the last round lanes, and the rounds
    // of one workgroup do not overlap.  Whole calls in us, one round -> longer:
    //   `full`, a single row is more than half a round and the busiest unit gets hardly more of them:
    //     run-time range 4096 x 5120 41.5 -> 40.4, 5000 x 4608 41.3 -> 39.5; given parameters 3000 x 5120 30.3 -> 29.3,
    //     5000 x 4160 30.3 -> 29.0, 6000 x 4608 33.6 -> 32.3, but 7000 x 4160 34.5 -> 35.1, 6000 x 5120 36.9 -> 38.5;
    //     not full: 2049 x 8192 46.4 -> 47.3 and 38.5 -> 39.9
    //   run-time range, `even`, the grid fills at least 15/16 of its last wave of compute units: 16384 x 1280 31.7 -> 31.4;
    //     not even: 8193 x 2048 (1639 workgroups) 27.2 -> 28.2
    //   thousands of pairs (the gated projection leaves them): 16384 x 2560 126.2 -> 124.1
    //   given parameters otherwise: 16389 x 2560 42.6 -> 45.1, 262144 x 320 79.7 -> 87.2
    int U = Q_U, R = 256 * Q_U / Kp8;
    R = R < 1 ? 1 : R;
    for (int u = 1; u < Q_U && given_partials <= kPartialSlots; u *= 2) {
        const int rows = 256 * u / Kp8;
        if (rows < 1 || (M + rows - 1) / rows > (dynamic ? kQuantGrid / (u == 1 ? 8 : 2) : kQuantGrid)) continue;
        U = u;
        R = rows;
        break;
    }
    if ((M + R - 1) / R > kQuantGrid) {
        int longer = (M + kQuantGrid - 1) / kQuantGrid;
        longer = longer > Q_MAX_ROWS ? Q_MAX_ROWS : longer;
        constexpr int CUS = kQuantGrid / 8;
        const long groups = (M + longer - 1) / longer;
        auto rounds = [&](int rows) {  // ... of the busiest compute unit
            return (((long)M + rows - 1) / rows + CUS - 1) / CUS * (((long)rows * Kp8 + 256 * Q_U - 1) / (256 * Q_U));
        };
        const bool full = R == 1 && rounds(longer) * 10 <= rounds(1) * 11;
        const bool even = groups * 16 >= (groups + CUS - 1) / CUS * CUS * 15;
        if (dynamic ? full || even || given_partials > kPartialSlots : full && (long)M * K <= kSmallQuant) R = longer;
    }
    R = R > Q_MAX_ROWS ? Q_MAX_ROWS : R;
    const int qgrid = (M + R - 1) / R;
    ProfScope prof(st, PROF_ACT_QUANTIZE, 0.0, 3.0 * M * K + (rowsum ? 4.0 * M : 0.0));
    auto kern = bos ? (U == 1 ? act_quantize_kernel<true, 1> : U == 2 ? act_quantize_kernel<true, 2> : act_quantize_kernel<true, 4>)
                    : (U == 1 ? act_quantize_kernel<false, 1> : U == 2 ? act_quantize_kernel<false, 2> : act_quantize_kernel<false, 4>);
    const int nbos = bos ? bos_blocks(*bos) : 0;
    hipLaunchKernelGGL(kern, dim3(nbos + qgrid), dim3(256), 0, st, (const _Float16*)x, M, K, (long)ldx, flat, FastDiv::make(K8),
                       walk, R, FastDiv::make(Kp8), dynamic ? partials : (const float*)nullptr, grid, act_scale, act_zp, a8,
                       rowsum, params, act_scale_out, act_zp_out, nbos, bos ? *bos : BosWork{});
    MQ_HIP_CHECK_LAUNCH();
    return MQ_OK;
}

}  // namespace mq
