// Device parts of the activation quantiser that more than one kernel uses: the range of a tensor, its parameters, and the conversion of eight
// values.  Files that include this are compiled with -ffp-contract=off: each fp32 operation rounds once.
#pragma once
#include "mq_common.h"

namespace mq {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

template <typename T, typename Op>
__device__ inline T wave_reduce(T v, Op op) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off, 64));
    return v;
}

// Physical row of logical row r (RowMap::phys with its division prepared by the host).
struct RowWalk {
    FastDiv group;  // d = rows per group; used where `mapped` says so
    int mapped, group_stride, row_offset;
    static RowWalk make(const RowMap& m) {
        return RowWalk{FastDiv::make((uint32_t)(m.rows_per_group > 0 ? m.rows_per_group : 1)), m.rows_per_group > 0,
                       m.group_stride, m.row_offset};
    }
    __device__ inline long phys(uint32_t r) const {
        if (!mapped) return r;
        uint32_t q, rem;
        group.divmod(r, q, rem);
        return (long)q * group_stride + rem + row_offset;
    }
};

// This thread's share of the extremes of the tensor's vectors: U at a time, NT lanes side by side, from `base` on in steps of `step`.
// They are found in pairs of fp16 values (a minimum or maximum of fp16 values is one of them: nothing is lost) and widened
// once at the end; NaN is ignored as by fminf / fmaxf.
template <int U, int NT>
__device__ inline void extremes(const _Float16* __restrict__ x, uint32_t nv, FastDiv K8, long ldx, const RowWalk& map, int flat, uint32_t base,
                                uint32_t step, float& mn, float& mx) {
    half8 mn8, mx8;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        mn8[e] = (_Float16)INFINITY;
        mx8[e] = -(_Float16)INFINITY;
    }
    for (; base < nv; base += step) {
        half8 v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            uint32_t i = base + u * (uint32_t)NT + threadIdx.x;
            i = i < nv ? i : nv - 1;  // a repeated vector does not change a min or a max
            if (flat) {
                v[u] = ((const half8*)x)[i];
            } else {
                uint32_t row, p;
                K8.divmod(i, row, p);
                v[u] = ((const half8*)(x + map.phys(row) * ldx))[p];
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            mn8 = __builtin_elementwise_min(mn8, v[u]);
            mx8 = __builtin_elementwise_max(mx8, v[u]);
        }
    }
    mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        mn = fminf(mn, (float)mn8[e]);
        mx = fmaxf(mx, (float)mx8[e]);
    }
}

// Sum over each aligned group of eight lanes, in every lane of the group (two quad permutes and a mirror of the group:
// register moves inside the vector ALU, no trip through LDS).
__device__ inline int sum8(int v) {
    v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);   // lanes 1 0 3 2
    v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);   // lanes 2 3 0 1
    v += __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);  // lanes 7 6 5 4 3 2 1 0
    return v;
}

// Extremes over a workgroup of NT threads from each thread's own; smn and smx hold NT / 64 values each.  Ends behind a barrier.
template <int NT>
__device__ inline void group_extremes(float& mn, float& mx, float* smn, float* smx) {
    mn = wave_reduce(mn, [](float a, float b) { return fminf(a, b); });
    mx = wave_reduce(mx, [](float a, float b) { return fmaxf(a, b); });
    if ((threadIdx.x & 63) == 0) {
        smn[threadIdx.x >> 6] = mn;
        smx[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        mn = fminf(mn, smn[i]);
        mx = fmaxf(mx, smx[i]);
    }
}

// ... from the (min, max) pairs that a pass over the tensor has left.
template <int NT>
__device__ inline void pair_extremes(const float* __restrict__ partials, int n, float& mn, float& mx) {
    constexpr int PU = 4;  // pairs requested together
    mn = INFINITY, mx = -INFINITY;
    for (int i0 = threadIdx.x; i0 < n; i0 += NT * PU) {
        float2 pr[PU];
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int i = i0 + u * NT;
            pr[u] = ((const float2*)partials)[i < n ? i : n - 1];
        }
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            mn = fminf(mn, pr[u].x);
            mx = fmaxf(mx, pr[u].y);
        }
    }
}

// Scale and zero point (a whole number) of a range: 0 is always in it, a tensor of zeros has scale 1.
__device__ inline void range_params(float mn, float mx, float& s, float& zf) {
    const float lo = fminf(mn, 0.0f), hi = fmaxf(mx, 0.0f);
    s = 1.0f;
    if (hi != lo) {
        const float range = hi - lo;
        s = range / 255.0f;
    }
    const float inv0 = 1.0f / s;
    zf = rintf((-lo) * inv0);
    zf = fminf(fmaxf(zf, 0.0f), 255.0f);
}

// Eight values -> code - 128 as bytes, byte b of word h holding element k8_perm(4 h + b).  A value costs one fused multiply-add that widens it,
// one rounding, one addition and one saturating conversion into its byte (which also takes NaN to code 0, as the clamp of the formula does).
__device__ inline uint2v quantize8(half8 v, float inv, float zf) {
    uint32_t w0 = 0, w1 = 0;
    auto t = [&](int e) { return rintf(__builtin_fmaf((float)v[e], inv, 0.0f)) + zf; };
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        w0 = __builtin_amdgcn_cvt_pk_u8_f32(t(k8_perm(b)), b, w0);
        w1 = __builtin_amdgcn_cvt_pk_u8_f32(t(k8_perm(4 + b)), b, w1);
    }
    return uint2v{w0 ^ 0x80808080u, w1 ^ 0x80808080u};
}

}  // namespace mq
