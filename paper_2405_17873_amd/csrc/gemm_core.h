// What the MFMA GEMM kernels share: operand types, code widening, buffer addressing with LDS-writing loads, the kernel
// arguments, the workgroup -> tile map and the LDS plan of a workgroup.
#pragma once
#include <type_traits>

#include "mq_common.h"

namespace mq {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef int int16v __attribute__((ext_vector_type(16)));
typedef int int4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint3v __attribute__((ext_vector_type(3)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Swizzle of the 16-byte piece index inside a 128-byte LDS row.  Distinct over any 8 consecutive rows and,
// together with the row parity, over any 16 consecutive rows.
__device__ __forceinline__ int swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

__device__ __forceinline__ half2v as_h2(uint32_t u) { return __builtin_bit_cast(half2v, u); }
__device__ __forceinline__ uint32_t h2_bits(half2v h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ half2v splat(float v) {
    half2v r;
    r[0] = (_Float16)v;
    r[1] = (_Float16)v;
    return r;
}

// ---------------------------------------------------------------------------------------------
// Code -> fp16 widening.  0x6400 is 1024.0 in fp16; OR-ing a small integer into its mantissa gives
// 1024 + q (or 1024 + 2^s q for a field that sits s bits up), and one packed add or fma brings it to
// the exact integer q - z.  All intermediate values are integers below 2048, so nothing rounds.
// ---------------------------------------------------------------------------------------------
template <int BITS>
struct WChunk {
    static constexpr int WORDS = BITS == 8 ? 8 : BITS;  // 32-bit words per lane per 64-k tile (16: unquantised)
    uint32_t w[WORDS];
};

// (w & mask) | magic in one instruction.  The compiler emits v_and + v_or here, each with its own 32-bit literal: the
// three-operand form takes no literals on this target, so the mask is handed over in a scalar register and the magic
// number in a vector register (both loop invariant).  It is a third of the widening work of the 2/3/4-bit codes.
__device__ __forceinline__ uint32_t and_or(uint32_t w, uint32_t mask, uint32_t magic) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(mask), "v"(magic));
    return r;
}

template <int SHIFT>
__device__ __forceinline__ half2v field_to_h2(uint32_t w, uint32_t mask, int z) {
    // field value sits at bit SHIFT of each half: magic|field = 1024 + 2^SHIFT q
    const half2v v = as_h2(and_or(w, mask, 0x64006400u));
    if constexpr (SHIFT == 0) {
        return v - splat((float)(1024 + z));
    } else {
        constexpr float inv = 1.0f / (float)(1 << SHIFT);
        return v * splat(inv) - splat((float)((1024 >> SHIFT) + z));
    }
}

// Fragment for MFMA step s (8 consecutive k of this lane's 32): four half2 pairs.
template <int BITS>
__device__ __forceinline__ half8 dequant_step(const WChunk<BITS>& c, int s, int z);

template <>
__device__ __forceinline__ half8 dequant_step<4>(const WChunk<4>& c, int s, int z) {
    uint32_t w = c.w[s];
    half2v p0 = field_to_h2<0>(w, 0x000F000Fu, z);
    half2v p1 = field_to_h2<4>(w, 0x00F000F0u, z);
    w >>= 8;
    half2v p2 = field_to_h2<0>(w, 0x000F000Fu, z);
    half2v p3 = field_to_h2<4>(w, 0x00F000F0u, z);
    return half8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

template <>
__device__ __forceinline__ half8 dequant_step<2>(const WChunk<2>& c, int s, int z) {
    uint32_t w = c.w[s >> 1];
    if (s & 1) w >>= 8;
    half2v p0 = field_to_h2<0>(w, 0x00030003u, z);
    half2v p1 = field_to_h2<2>(w, 0x000C000Cu, z);
    half2v p2 = field_to_h2<4>(w, 0x00300030u, z);
    half2v p3 = field_to_h2<6>(w, 0x00C000C0u, z);
    return half8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

// 3 bit: pair p (0..14) is field p%5 of word p/5; fields 0..2 are read in place, fields 3,4 after >> 9.
template <int F>
__device__ __forceinline__ half2v field3(uint32_t w, int z) {
    if constexpr (F == 0) return field_to_h2<0>(w, 0x00070007u, z);
    if constexpr (F == 1) return field_to_h2<3>(w, 0x00380038u, z);
    if constexpr (F == 2) return field_to_h2<6>(w, 0x01C001C0u, z);
    if constexpr (F == 3) return field_to_h2<0>(w >> 9, 0x00070007u, z);
    return field_to_h2<3>(w >> 9, 0x00380038u, z);
}

template <>
__device__ __forceinline__ half8 dequant_step<3>(const WChunk<3>& c, int s, int z) {
    half2v p0, p1, p2, p3;
    if (s == 0) {
        p0 = field3<0>(c.w[0], z);
        p1 = field3<1>(c.w[0], z);
        p2 = field3<2>(c.w[0], z);
        p3 = field3<3>(c.w[0], z);
    } else if (s == 1) {
        p0 = field3<4>(c.w[0], z);
        p1 = field3<0>(c.w[1], z);
        p2 = field3<1>(c.w[1], z);
        p3 = field3<2>(c.w[1], z);
    } else if (s == 2) {
        p0 = field3<3>(c.w[1], z);
        p1 = field3<4>(c.w[1], z);
        p2 = field3<0>(c.w[2], z);
        p3 = field3<1>(c.w[2], z);
    } else {
        p0 = field3<2>(c.w[2], z);
        p1 = field3<3>(c.w[2], z);
        p2 = field3<4>(c.w[2], z);
        const uint32_t t = ((c.w[0] >> 15) & 0x00010001u) | ((c.w[1] >> 14) & 0x00020002u) |
                           ((c.w[2] >> 13) & 0x00040004u);
        p3 = field_to_h2<0>(t, 0x00070007u, z);
    }
    return half8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

// 8 bit: step s uses the two words of group (s & 1) in piece (s >> 1): bytes c0,c4,c1,c5 | c2,c6,c3,c7.
template <>
__device__ __forceinline__ half8 dequant_step<8>(const WChunk<8>& c, int s, int z) {
    const uint32_t wa = c.w[(s >> 1) * 4 + (s & 1) * 2], wb = c.w[(s >> 1) * 4 + (s & 1) * 2 + 1];
    const half2v zz = splat((float)(1024 + z));
    // v_perm_b32: selector bytes 0..3 pick bytes of the second source, 4..7 of the first
    half2v p0 = as_h2(__builtin_amdgcn_perm(0x64646464u, wa, 0x04020400u)) - zz;  // c0,c1
    half2v p1 = as_h2(__builtin_amdgcn_perm(0x64646464u, wb, 0x04020400u)) - zz;  // c2,c3
    half2v p2 = as_h2(__builtin_amdgcn_perm(0x64646464u, wa, 0x04030401u)) - zz;  // c4,c5
    half2v p3 = as_h2(__builtin_amdgcn_perm(0x64646464u, wb, 0x04030401u)) - zz;  // c6,c7
    return half8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

// 16 bit: the weights are unquantised fp16 (or bf16) values, piece s is the operand of step s as it stands.
template <>
__device__ __forceinline__ half8 dequant_step<16>(const WChunk<16>& c, int s, int) {
    const uint4v v = {c.w[4 * s], c.w[4 * s + 1], c.w[4 * s + 2], c.w[4 * s + 3]};
    return __builtin_bit_cast(half8, v);
}

// bfloat16 variant: the widened weights are small integers (|q - z| <= 255), exact in fp16, in fp32 and in bf16 alike.
// Where two wave groups share a reduction: the fp16 fragment is converted pair by pair, two fp16 -> fp32 conversions and one byte permute that
// keeps the upper halves (which for these values is the exact bf16), five instructions a pair in all.
__device__ __forceinline__ half8 half8_to_bf16x8(half8 h) {  // (bf16 bits)
    uint4v o;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t f0 = __float_as_uint((float)h[2 * p]), f1 = __float_as_uint((float)h[2 * p + 1]);
        o[p] = __builtin_amdgcn_perm(f1, f0, 0x07060302u);
    }
    return __builtin_bit_cast(half8, o);
}
// Elsewhere the pair with the magic number in it, 1024 + 2^SHIFT q, becomes q - z in fp32 by one mixed-precision multiply-add a half: four
// instructions a pair.  us, five -> four: 16384 x 640 x 640 20.8 -> 19.3 (2 bits), 21.2 -> 20.7 (4 bits), 4096 x 5120 x 1280 63.7 -> 60.7 (3 bits), 4096 x
// 2560 x 640 25.1 -> 25.3; two wave groups, one wave per SIMD each: 535 x 3904 x 2520 (3 bits) 25.6 -> 26.5.
template <int SHIFT>
__device__ __forceinline__ uint32_t magic_to_bf16x2(uint32_t v, int z) {
    const float c = -(float)((1024 >> SHIFT) + z);
    float inv = 1.0f / (float)(1 << SHIFT);
    asm("" : "+s"(inv));  // (a multiplication by a visible 1 would become a conversion and an addition)
    const half2v h = as_h2(v);
    const float f0 = __builtin_fmaf((float)h[0], inv, c), f1 = __builtin_fmaf((float)h[1], inv, c);
    return __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
}
template <int SHIFT>
__device__ __forceinline__ uint32_t field_to_bf16x2(uint32_t w, uint32_t mask, int z) {
    uint32_t magic = 0x64006400u;
    asm("" : "+s"(mask));  // (as and_or, but left to the compiler to schedule)
    asm("" : "+v"(magic));
    return magic_to_bf16x2<SHIFT>((w & mask) | magic, z);
}
template <int BITS>
__device__ __forceinline__ half8 dequant_step_bf16(const WChunk<BITS>& c, int s, int z) {  // (bf16 bits)
    uint4v o;
    if constexpr (BITS == 4) {
        const uint32_t w = c.w[s], v = w >> 8;
        o = uint4v{field_to_bf16x2<0>(w, 0x000F000Fu, z), field_to_bf16x2<4>(w, 0x00F000F0u, z), field_to_bf16x2<0>(v, 0x000F000Fu, z),
                   field_to_bf16x2<4>(v, 0x00F000F0u, z)};
    } else if constexpr (BITS == 2) {
        const uint32_t w = (s & 1) ? c.w[s >> 1] >> 8 : c.w[s >> 1];
        o = uint4v{field_to_bf16x2<0>(w, 0x00030003u, z), field_to_bf16x2<2>(w, 0x000C000Cu, z), field_to_bf16x2<4>(w, 0x00300030u, z),
                   field_to_bf16x2<6>(w, 0x00C000C0u, z)};
    } else if constexpr (BITS == 3) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {  // as dequant_step<3>: pair 4 s + p is field % 5 of word / 5, the last one scattered
            const int i = 4 * s + p, f = i % 5;
            if (i == 15) {
                const uint32_t t = ((c.w[0] >> 15) & 0x00010001u) | ((c.w[1] >> 14) & 0x00020002u) | ((c.w[2] >> 13) & 0x00040004u);
                o[p] = field_to_bf16x2<0>(t, 0x00070007u, z);
            } else {
                const uint32_t w = f < 3 ? c.w[i / 5] : c.w[i / 5] >> 9;
                o[p] = f == 0 || f == 3 ? field_to_bf16x2<0>(w, 0x00070007u, z) : f == 1 || f == 4 ? field_to_bf16x2<3>(w, 0x00380038u, z)
                                                                                                   : field_to_bf16x2<6>(w, 0x01C001C0u, z);
            }
        }
    } else if constexpr (BITS == 8) {
        const uint32_t wa = c.w[(s >> 1) * 4 + (s & 1) * 2], wb = c.w[(s >> 1) * 4 + (s & 1) * 2 + 1];
        o = uint4v{magic_to_bf16x2<0>(__builtin_amdgcn_perm(0x64646464u, wa, 0x04020400u), z), magic_to_bf16x2<0>(__builtin_amdgcn_perm(0x64646464u, wb, 0x04020400u), z),
                   magic_to_bf16x2<0>(__builtin_amdgcn_perm(0x64646464u, wa, 0x04030401u), z), magic_to_bf16x2<0>(__builtin_amdgcn_perm(0x64646464u, wb, 0x04030401u), z)};
    } else {
        return dequant_step<BITS>(c, s, z);  // unquantised
    }
    return __builtin_bit_cast(half8, o);
}

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// ---------------------------------------------------------------------------------------------
// Buffer addressing.  Both operands are read through buffer resources: a lane's offset is a 32-bit
// register computed once, the k advance is a scalar offset, and anything past the end of the buffer reads
// as zero instead of faulting (rows beyond M, the k padding of the int8 activation copy).
// ---------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Raw buffer resource (stride 0): base address, byte extent, gfx9-family format word.
typedef int int4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int4s make_rsrc(const void* p, uint32_t bytes) {
    const uint64_t a = (uint64_t)(uintptr_t)p;
    int4s r;
    r[0] = (int)(uint32_t)a;
    r[1] = (int)(uint32_t)((a >> 32) & 0xFFFFu);
    r[2] = (int)bytes;
    r[3] = 0x00020000;
    // the descriptor is wave-uniform: keep it in scalar registers
    r[0] = __builtin_amdgcn_readfirstlane(r[0]);
    r[1] = __builtin_amdgcn_readfirstlane(r[1]);
    r[2] = __builtin_amdgcn_readfirstlane(r[2]);
    return r;
}

// 16 bytes per lane from the buffer straight into LDS: lane L of the wave writes lds_wave_base + 16 * L; a lane
// whose offset lies past the end of the buffer writes zeros.  Issued as inline assembly on purpose: the compiler
// would otherwise order every later LDS read behind ALL pending loads of this kind (it cannot tell the stage being
// filled from the stage being read), which serialises the pipeline.  The waits are placed by hand (vmcnt below).
__device__ __forceinline__ void dma_to_lds_b128(int4s rsrc, uint32_t lds_wave_base, int voff, int soff) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %2, %3 offen lds"
        :
        : "s"(lds_wave_base), "v"(voff), "s"(rsrc), "s"(soff)
        : "memory");  // m0 is a reserved register: the compiler rewrites it before each of its own uses
}

// The same with the LDS address as a sum of two scalars, and in two halves: between the address and the load has to lie one other instruction.
__device__ __forceinline__ void dma_address(uint32_t lds_stage, uint32_t lds_offset) {
    asm volatile("s_add_u32 m0, %0, %1" : : "s"(lds_stage), "s"(lds_offset) : "memory", "scc");
}
__device__ __forceinline__ void dma_load_b128(int4s rsrc, int voff, int soff) {
    asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" : : "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ void dma_to_lds_b128(int4s rsrc, uint32_t lds_stage, uint32_t lds_offset, int voff, int soff) {
    dma_address(lds_stage, lds_offset);
    asm volatile("s_nop 0");
    dma_load_b128(rsrc, voff, soff);
}

// The same for 4 bytes per lane (256 contiguous bytes per wave).
__device__ __forceinline__ void dma_to_lds_b32(int4s rsrc, uint32_t lds_wave_base, int voff, int soff) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dword %1, %2, %3 offen lds"
        :
        : "s"(lds_wave_base), "v"(voff), "s"(rsrc), "s"(soff)
        : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A lane's chunk of one 64-k weight tile, read from the tile's LDS copy (lane order, so consecutive lanes read
// consecutive addresses).
template <int BITS>
__device__ __forceinline__ void read_chunk(WChunk<BITS>& c, const uint8_t* tile, int lane) {
    if constexpr (BITS == 4) {
        const uint4v v = *(const uint4v*)(tile + lane * 16);
        c.w[0] = v[0]; c.w[1] = v[1]; c.w[2] = v[2]; c.w[3] = v[3];
    } else if constexpr (BITS == 2) {
        const uint2v v = *(const uint2v*)(tile + lane * 8);
        c.w[0] = v[0]; c.w[1] = v[1];
    } else if constexpr (BITS == 3) {
        const uint32_t* p = (const uint32_t*)(tile + lane * 12);
        c.w[0] = p[0]; c.w[1] = p[1]; c.w[2] = p[2];
    } else if constexpr (BITS == 16) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint4v v = *(const uint4v*)(tile + s * 1024 + lane * 16);
            c.w[4 * s] = v[0]; c.w[4 * s + 1] = v[1]; c.w[4 * s + 2] = v[2]; c.w[4 * s + 3] = v[3];
        }
    } else {
        const uint4v v0 = *(const uint4v*)(tile + lane * 16);
        const uint4v v1 = *(const uint4v*)(tile + 1024 + lane * 16);
        c.w[0] = v0[0]; c.w[1] = v0[1]; c.w[2] = v0[2]; c.w[3] = v0[3];
        c.w[4] = v1[0]; c.w[5] = v1[1]; c.w[6] = v1[2]; c.w[7] = v1[3];
    }
}

// xflip = 0x80808080 turns unsigned 8-bit codes q into the signed bytes q - 128 (0 for signed codes).
template <int WBITS>
__device__ __forceinline__ int4v widen_step(const WChunk<WBITS>& c, int s /*0..1 inside the 64-k tile*/,
                                            uint32_t xflip) {
    if constexpr (WBITS == 8) {
        return int4v{(int)(c.w[4 * s] ^ xflip), (int)(c.w[4 * s + 1] ^ xflip), (int)(c.w[4 * s + 2] ^ xflip),
                     (int)(c.w[4 * s + 3] ^ xflip)};
    } else if constexpr (WBITS == 2) {
        // Word s holds codes 16s..16s+15, pair (c[2p], c[2p+1]) in bits [2p, 2p+2) and [16+2p, 16+2p+2):
        // (w >> 2t) & 0x03030303 = bytes c[2t], c[2t+8], c[2t+1], c[2t+9].  The activations of a group of 8 sit in
        // the order 0,4,1,5,2,6,3,7: two byte permutes per pair of extracts put the codes in that order.
        const uint32_t w = c.w[s];
        const uint32_t e0 = w & 0x03030303u, e1 = (w >> 2) & 0x03030303u, e2 = (w >> 4) & 0x03030303u,
                       e3 = (w >> 6) & 0x03030303u;
        // v_perm_b32: selector bytes 0..3 pick bytes of the second source, 4..7 of the first
        return int4v{(int)__builtin_amdgcn_perm(e2, e0, 0x06020400u),   // c0,c4,c1,c5
                     (int)__builtin_amdgcn_perm(e3, e1, 0x06020400u),   // c2,c6,c3,c7
                     (int)__builtin_amdgcn_perm(e2, e0, 0x07030501u),   // c8,c12,c9,c13
                     (int)__builtin_amdgcn_perm(e3, e1, 0x07030501u)};  // c10,c14,c11,c15
    } else {
        const uint32_t w0 = c.w[2 * s], w1 = c.w[2 * s + 1];
        return int4v{(int)(w0 & 0x0F0F0F0Fu), (int)((w0 >> 4) & 0x0F0F0F0Fu), (int)(w1 & 0x0F0F0F0Fu),
                     (int)((w1 >> 4) & 0x0F0F0F0Fu)};
    }
}

// ---------------------------------------------------------------------------------------------
// GELU of the gated feed-forward epilogue: gelu(g) = 0.5 g (1 + erf(g / sqrt 2)), single fp32 operations without
// contraction, library call or division, with erf(x) = 1 - exp(-x P(x)) on [0, 4.3] (x is held at 4.3 beyond), P a
// degree-6 polynomial fitted to -ln(erfc(x)) / x (error of the fit below 2e-7), and the exponential by the hardware's
// 2^t instruction (1 ulp, i.e. 1.2e-7 of a value that is at most 1; the rounding of its argument, at most 30 in
// magnitude, matters only where exp(-t) is below 1e-8): |error of erf| < 3e-7.  A range reduction with a degree-6
// polynomial in its place costs twelve more instructions per element: the gated feed-forward pair runs 2 to 3 %
// slower with it.
// ---------------------------------------------------------------------------------------------
// Returns 2 gelu(g) = g (1 + erf): the factor 1/2 rides in the value's constants (exact, a multiplication less).
__device__ __forceinline__ float two_gelu32(float g) {
    const float x = fminf(__fmul_rn(fabsf(g), 0.70710678f), 4.3f);
    float p = -5.95750535e-05f;
    p = __fmaf_rn(p, x, 0.000253331062f);
    p = __fmaf_rn(p, x, 0.00176583871f);
    p = __fmaf_rn(p, x, -0.0206223261f);
    p = __fmaf_rn(p, x, 0.103378408f);
    p = __fmaf_rn(p, x, 0.636503041f);
    p = __fmaf_rn(p, x, 1.12838686f);
    const float e = __builtin_amdgcn_exp2f(__fmul_rn(__fmul_rn(p, x), -1.44269504f));  // v_exp_f32: 2^t, 1 ulp
    const float erf_g = copysignf(__fsub_rn(1.0f, e), g);
    return __fmul_rn(g, __fadd_rn(1.0f, erf_g));
}

// Four products a[r] * b[r] rounded once, to fp16, one instruction each: the mixed-precision multiply-add writes one half of
// its destination (the compiler, where the results are used as a vector, multiplies in fp32 and packs in instructions of their
// own).  A zero product is stored as +0.  For the run-time-range form, whose product is needed in fp16 only; the forms with given
// output parameters have the fp32 product in hand and convert that.
__device__ __forceinline__ half4 mul_to_half4(const float (&a)[4], const float (&b)[4]) {
    uint2v o;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(o[0]) : "v"(a[0]), "v"(b[0]));
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(o[1]) : "v"(a[2]), "v"(b[2]));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(o[0]) : "v"(a[1]), "v"(b[1]));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(o[1]) : "v"(a[3]), "v"(b[3]));
    return __builtin_bit_cast(half4, o);
}

// ---------------------------------------------------------------------------------------------
// The GEMM kernel.  I8 == false: weight-only, fp16 activations straight from X, 64 k per stage.
//                   I8 == true : int8 activation copy (row stride Kp = K rounded up to 128, padding zero),
//                                128 k per stage = two 64-k weight tiles.
// A stage of the activation operand is BM rows x 128 bytes.  It is brought in by buffer loads that write LDS
// directly (each lane 16 bytes, a wave instruction fills 8 rows), XOR-swizzled on the global side so that the
// later ds_read_b128 of 32 consecutive rows is conflict free.  S LDS stages rotate; the loads of the next S-1 stages
// are in flight while a stage is multiplied.
// ---------------------------------------------------------------------------------------------
// Low bits of a split reduction's counter word, the arrivals of one tile; the launch's tag lies above them.  A part is at
// least one pipeline stage of 64 or more k, and (N + 31) * K < 2^31 with N >= 8 is checked: fewer than 2^20 parts.
static constexpr unsigned long long SPLIT_COUNT = 0xFFFFFull;

struct GemmArgs {
    const void* a;        // X fp16 [M, lda] or int8 copy [M, Kp]
    long a_row_bytes;     // byte stride between rows of a
    uint32_t a_bytes;     // valid extent of a in bytes
    const uint8_t* packed;
    uint32_t packed_bytes;
    int M, N, K;          // K: true reduction length
    int k_stages;         // number of 128-byte stages
    const float* w_scale;
    const int32_t* w_zp;
    const uint16_t* bias;  // fp16 or bf16 bits
    uint16_t* y;
    long ldy;
    int tiles_m, tiles_n;
    int band_rows;        // row blocks per band of the workgroup -> tile map (>= 1)
    FastDiv fd_band_tiles, fd_band_rows, fd_last_rows;  // divisors of that map: tiles per band, rows of a band, of the last
    FastDiv fd_splits;
    int kt_q, kt_r;       // pipeline stages per part of a split reduction: kt_q, and one more for the first kt_r parts
    // int8 only
    const int32_t* rowsum;
    const ActParams* params;
    const int32_t* w_colsum;
    int w_off;
    long long* phase_clk;  // optional: 4 shader-clock samples per workgroup (start, loop, epilogue, end)
    RowMap out_map;
    int32_t* acc_debug;
    // split of the reduction over `splits` workgroups per tile (1 = none): partial accumulators in `partial`
    // ([tile][split][BM * BN] 4-byte values, register order), one arrival counter per tile (counts under the launch's tag)
    int splits;
    uint32_t* partial;
    unsigned long long* counters;
    unsigned long long split_tag;
    int counter_step;  // words between the counters of two tiles
    // (host side only) the caller's workspace that partial sums and counters are carved from; may be null
    void* split_ws;
    size_t split_ws_bytes;
    // MODE 1 (gated feed-forward projection, 8-bit output): N = 2H weight rows; codes of the gated product go to
    // a8_out (row stride ld8 bytes, the int8 activation layout), optionally the product itself as fp16 to y
    const float* out_scale_p;
    const int32_t* out_zp_p;
    int8_t* a8_out;
    // optional (int8 gated projection): one (min, max) pair per workgroup over the fp16 gated products it wrote
    float* mm_out;
    long ld8;
    // MODE 2 (activations arrive as int8 codes): their parameters; row sums are taken inside the main loop
    const float* act_scale_p;
    const int32_t* act_zp_p;
    // MODE 3 / 4 (3x3 convolution, stride 1, zero padding 1, channels-last): a is the [B*H*W, Cin] activation tensor
    // (a_row_bytes per pixel), K = 9 * Cin, row m is output pixel m; the k order is (filter row, filter column, c)
    int conv_h, conv_w;      // input image
    int conv_stride;         // 1 or 2: output pixel (i, j) is centred on input pixel (stride * i, stride * j)
    int conv_cpt;            // 64-channel chunks per filter tap (Cin / 64)
    uint32_t conv_cpt_inv;   // ceil(2^32 / conv_cpt) for conv_cpt > 1
    FastDiv fd_ho, fd_wo;    // output image ho x wo: (H - 1) / stride + 1, likewise W; M = B * ho * wo
    const int32_t* w_tapsum; // MODE 4: [9][N] sums of the weight codes per filter tap
    // optional residual [M, ldr] (16-bit, the dtype of y; rows as the rows of y): added in fp32 before the rounding
    const uint16_t* res;
    long ldr;
};

// Workgroup id -> tile.  Consecutive workgroup ids land on different XCDs (8 of them, each with its own L2),
// so the ids an XCD receives are mapped onto a contiguous run of tiles.  The run walks the tile grid in bands of
// `band_rows` row blocks, inside a band column by column: the workgroups an XCD runs at the same time then cover
// band_rows row blocks times a few column blocks, the band's activation rows stay in that L2 while the band walks
// along N, and every weight tile is fetched once per band instead of once per row block.
__device__ __forceinline__ void tile_of_block(int bid, const GemmArgs& g, int& bm, int& bn) {
    const int total = g.tiles_m * g.tiles_n;
    const int per = total >> 3;  // tiles of the leftover (total % 8) keep their own index
    const uint32_t t = (uint32_t)(bid < (per << 3) ? (bid & 7) * per + (bid >> 3) : bid);
    uint32_t band, r, col, row;
    g.fd_band_tiles.divmod(t, band, r);
    const int first = (int)band * g.band_rows;
    if (g.tiles_m - first < g.band_rows)  // (the last band may be lower)
        g.fd_last_rows.divmod(r, col, row);
    else
        g.fd_band_rows.divmod(r, col, row);
    bn = (int)col;
    bm = first + (int)row;
}

// LDS plan of one workgroup: S stages, each KS sub-stages of [activation tile BM x 128 B][weight tiles]; a 1 KB sink
// for padding loads; the per-channel epilogue constants.  The accumulator exchange (KS == 2) and the epilogue staging
// reuse the stages.
//
// KS == 2 splits the reduction inside the workgroup: a second group of WGM x WGN waves works on the same output
// tile and takes every other 128-byte k step.  It is for problems with few tiles: a compute unit then still has two
// waves per SIMD to alternate between while fragments travel from LDS, without any extra global traffic; the two
// accumulator sets meet once, through LDS, before the epilogue.
template <bool I8, int BITS, int WGM, int WGN, int TM, int TN, int S, int KS>
struct GemmPlan {
    static constexpr int NWG = WGM * WGN;                     // waves of one group
    static constexpr int NW = NWG * KS, NT = NW * 64;
    static constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32;
    static constexpr int CH = I8 ? 2 : 1;                     // 64-k weight tiles per 128-byte k step
    static constexpr int A_BYTES = BM * 128;
    static constexpr int BSLOT = BITS == 16 ? 4096 : BITS == 8 ? 2048 : 1024;  // LDS slot of one weight tile
    static constexpr int PIECES = BITS == 16 ? 4 : BITS == 8 ? 2 : 1;           // 1 KB wave loads per weight tile
    static constexpr int NBT = (BN / 32) * CH;                // weight tiles per sub-stage
    static constexpr int B_BYTES = NBT * BSLOT;
    static constexpr int SUB_BYTES = A_BYTES + B_BYTES;
    static constexpr int STAGE_BYTES = KS * SUB_BYTES;
    static constexpr int NAI = KS * (BM / 8);                 // LDS-writing loads per stage, activations
    static constexpr int DMA_A = NAI / NW;                    // ... per wave
    static constexpr int NBI1 = NBT * PIECES;                 // LDS-writing loads per sub-stage, weights
    static constexpr int NBI = KS * NBI1;
    static constexpr int DMA_B = (NBI + NW - 1) / NW;         // per wave (padded with loads into the sink)
    static constexpr int OPS = DMA_A + DMA_B;                 // vector-memory operations per wave per stage
    static constexpr int SINK = S * STAGE_BYTES;
    static constexpr int CONSTS = SINK + (TM == 3 && TN == 1 ? 1536 : 1024);  // (the shares of 96 row sums, see rs_x)
    static constexpr int LDS_BYTES = CONSTS + BN * 16;
    static_assert(NAI % NW == 0, "tile rows must split over the waves");
};

// ---- host side ------------------------------------------------------------------------------------------------
// Number of compute units, and what the busiest of them computes of an M x N output with tiles of rows x cols and a unit per tile: a kernel
// lasts as long as that one.
static constexpr long UNITS = 256;
inline long busiest_area(long M, long N, long rows, long cols) {
    return rows * cols * (((M + rows - 1) / rows * ((N + cols - 1) / cols) + UNITS - 1) / UNITS);
}

// The workgroup -> tile map of a grid of tiles_m x tiles_n (see tile_of_block).
inline void set_tile_walk(GemmArgs& g, int band_rows) {
    g.band_rows = band_rows < g.tiles_m ? band_rows : g.tiles_m;
    if (g.band_rows < 1) g.band_rows = 1;
    g.fd_band_tiles = FastDiv::make((uint32_t)(g.band_rows * g.tiles_n));
    g.fd_band_rows = FastDiv::make((uint32_t)g.band_rows);
    g.fd_last_rows = FastDiv::make((uint32_t)(g.tiles_m % g.band_rows ? g.tiles_m % g.band_rows : g.band_rows));
}

// Algorithmic bytes of one launch (a convolution reads each input pixel once, not nine times: the whole input tensor).
inline double gemm_alg_bytes(const GemmArgs& g, bool i8, int bits, int mode) {
    const double abytes = mode == 3 || mode == 4 ? (double)g.a_bytes : (i8 ? 1.0 * g.M * g.K + (mode == 0 ? 4.0 * g.M : 0.0) : 2.0 * g.M * g.K);
    const double ybytes = mode == 1 || mode == 6 ? 1.0 * g.M * g.ld8 + (g.y ? 1.0 * g.M * g.N : 0.0) : (mode == 5 ? 1.0 * g.M * g.N : 2.0 * g.M * g.N);
    return abytes + (double)g.N * g.K * bits / 8 + (i8 ? 14.0 : 10.0) * g.N + ybytes;
}

// Test and measurement hooks (mq_tune_*, mq_prof_phase_buffer), kept in gemm.hip.
int forced_band();      // 0: automatic
long long* phase_buffer(long workgroups);  // where the shader clocks of that many workgroups go, or null

// One wave per SIMD (gemm_solo.hip): the form that runs a call (-1: none of them), and the launch.  mode as for gemm_kernel: 0, 2, 3 or 4.
int solo_form(const GemmArgs& g, bool i8, int bits, int mode);
int launch_gemm_solo(GemmArgs& g, int form, bool i8, int bits, int mode, hipStream_t st);

}  // namespace mq
