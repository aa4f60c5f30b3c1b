// Device-side bodies of the BOS rows of the BOS-aware K/V projection (paper Sec. 3.1): token 0 of every prompt is kept
// out of activation quantisation; its to_k/to_v output is the fp16 linear with the unquantised weights (fp32
// accumulation), or a copy of the vector that was pre-computed offline.  They are functions of a block index so that
// they can run as a kernel of their own or as extra workgroups of the activation-quantise launch.
#pragma once
#include "mq_common.h"

namespace mq {

typedef _Float16 bos_half8 __attribute__((ext_vector_type(8)));

typedef float bos_float4 __attribute__((ext_vector_type(4)));

// 256 threads: one wave per output channel n = 4 * blk + wave.  The wave walks K in rounds of 4 x 64 sixteen-byte
// pieces: it requests the four weight pieces and the matching pieces of BCHUNK prompts' BOS rows before it multiplies
// any, so that one round trip to memory covers 512 k (latency bound: a few MB of weights, a few KB of activations).
// Few prompts: one trip over the weights with four prompts, and more waves at work than 16 channels per workgroup give.
static constexpr int BOS_FEW = 4;
__device__ __forceinline__ void bos_rows_few(int blk, int tid, const BosWork& bw) {
    constexpr int U = 4, BCHUNK = BOS_FEW;
    const int lane = tid & 63;
    const int n = blk * 4 + (tid >> 6);
    if (n >= bw.N) return;
    const int K = bw.K, B = bw.B, T = bw.T, N = bw.N;
    const int K8 = K >> 3;
    const bos_half8* wr = (const bos_half8*)(bw.w_f16 + (size_t)n * K);
    for (int b0 = 0; b0 < B; b0 += BCHUNK) {
        float acc[BCHUNK];
#pragma unroll
        for (int i = 0; i < BCHUNK; ++i) acc[i] = 0.0f;
        for (int p0 = 0; p0 < K8; p0 += 64 * U) {
            bos_half8 wv[U], xv[BCHUNK][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = p0 + u * 64 + lane;
                const int pc = p < K8 ? p : K8 - 1;  // clamped piece: its products are dropped below
                wv[u] = wr[pc];
#pragma unroll
                for (int i = 0; i < BCHUNK; ++i) {
                    const int b = b0 + i < B ? b0 + i : B - 1;
                    xv[i][u] = ((const bos_half8*)(bw.ctx + (size_t)b * T * K))[pc];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (p0 + u * 64 + lane >= K8) continue;
#pragma unroll
                for (int i = 0; i < BCHUNK; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i] += (float)xv[i][u][e] * (float)wv[u][e];
            }
        }
#pragma unroll
        for (int i = 0; i < BCHUNK; ++i) {
            float v = acc[i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane == 0 && b0 + i < B) {
                if (bw.bias) v += (float)bw.bias[n];
                bw.y[(size_t)(b0 + i) * T * N + n] = (_Float16)v;
            }
        }
    }
}

// 256 threads: 16 output channels, 16 prompts at a time, the reduction shared among the four waves (every fourth step of 32 k)
// and their sums added through LDS in wave order.  It is a product of two small matrices, so the matrix unit takes it:
// v_mfma_f32_16x16x32_f16 with the channels as rows (lane l: row or column l % 16, k = 8 (l / 16) + 0..7, which is how both
// operands lie in memory; result: column l % 16, rows 4 (l / 16) + 0..3).  Bound by latency (a few MB of weights, a few KB of
// activations): a wave requests BOS_U steps of both operands before it multiplies one, and all prompts take one trip
// over the weights.  (One wave per channel and a trip for every four prompts, with a wave reduction of every sum: see bos_block.)
static constexpr int BOS_CHANNELS = 16;
static constexpr int BOS_U = 8;
__device__ __forceinline__ void bos_rows_block(int blk, int tid, const BosWork& bw, float (&part)[4][256]) {
    const int lane = tid & 63, wv = tid >> 6, l15 = lane & 15, kb = lane >> 4;
    const int K = bw.K, B = bw.B, T = bw.T, N = bw.N;
    const int n0 = blk * BOS_CHANNELS, steps = K >> 5;
    const int n = n0 + l15 < N ? n0 + l15 : N - 1;  // (channels and prompts that do not exist repeat the last one: not stored)
    const _Float16* wr = bw.w_f16 + (size_t)n * K + kb * 8;
    for (int b0 = 0; b0 < B; b0 += 16) {
        const int b = b0 + l15 < B ? b0 + l15 : B - 1;
        const _Float16* xr = bw.ctx + (size_t)b * T * K + kb * 8;
        bos_float4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int s0 = wv; s0 < steps; s0 += 4 * BOS_U) {
            bos_half8 w[BOS_U], x[BOS_U];
#pragma unroll
            for (int u = 0; u < BOS_U; ++u) {
                const int s = s0 + 4 * u < steps ? s0 + 4 * u : s0;  // (a step past the end: not multiplied)
                w[u] = *(const bos_half8*)(wr + s * 32);
                x[u] = *(const bos_half8*)(xr + s * 32);
            }
#pragma unroll
            for (int u = 0; u < BOS_U; ++u)
                if (s0 + 4 * u < steps) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[u], x[u], acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wv][l15 * 16 + kb * 4 + i] = acc[i];  // [prompt][channel]
        __syncthreads();
        const int ob = b0 + (tid >> 4), on = n0 + (tid & 15);
        float v = part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid];
        if (ob < B && on < N) {
            if (bw.bias) v += (float)bw.bias[on];
            bw.y[(size_t)ob * T * N + on] = (_Float16)v;
        }
        __syncthreads();
    }
}

// 256 threads copy 256 of the B * N pre-computed values.
__device__ __forceinline__ void bos_copy_block(int blk, int tid, const BosWork& bw) {
    const long idx = (long)blk * 256 + tid;
    if (idx >= (long)bw.B * bw.N) return;
    const int b = (int)(idx / bw.N), n = (int)(idx % bw.N);
    bw.y[(size_t)b * bw.T * bw.N + n] = bw.bos_out[n];
}

// One block of the BOS rows, and how many (of 256 threads) there are.  Whole calls at 77 tokens, K = 2048, 8-bit weights, in us,
// few -> matrix unit: 4 prompts 320 channels 18.5 -> 18.9, 1280 channels 19.3 -> 18.9; 8 prompts 21.0 -> 20.3 and 22.3 -> 20.4;
// 16 prompts 26.3 -> 21.3 and 29.5 -> 22.9.
__device__ __forceinline__ void bos_block(int blk, int tid, const BosWork& bw, float (&part)[4][256]) {
    if (bw.bos_out)
        bos_copy_block(blk, tid, bw);
    else if (bw.B <= BOS_FEW)
        bos_rows_few(blk, tid, bw);
    else
        bos_rows_block(blk, tid, bw, part);
}
inline int bos_blocks(const BosWork& bw) {
    if (bw.bos_out) return (int)(((long)bw.B * bw.N + 255) / 256);
    const int channels = bw.B <= BOS_FEW ? 4 : BOS_CHANNELS;
    return (bw.N + channels - 1) / channels;
}

}  // namespace mq
