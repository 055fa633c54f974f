// Device helpers shared by the gfx950 kernels of libprox: wave64 reductions
// and scans, matrix-core and dot-product wrappers and 16-bit float
// conversions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.hpp"

namespace prox {

constexpr int kWave = 64;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// 16-bit float conversions (exact widening, round-to-nearest-even narrowing)
// ---------------------------------------------------------------------------

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ float f16_bits_to_float(uint32_t h) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

template <int DT>
__device__ __forceinline__ float lo_to_float(uint32_t w) {
    if constexpr (DT == kBF16) return bf16_lo(w);
    else return f16_bits_to_float(w & 0xFFFFu);
}
template <int DT>
__device__ __forceinline__ float hi_to_float(uint32_t w) {
    if constexpr (DT == kBF16) return bf16_hi(w);
    else return f16_bits_to_float(w >> 16);
}
template <int DT>
__device__ __forceinline__ float half_to_float(uint16_t h) {
    return lo_to_float<DT>((uint32_t)h);
}

// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t float_to_bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
// fp32 -> fp16 bits; the hardware conversion rounds to nearest even.
__device__ __forceinline__ uint16_t float_to_f16_rne(float v) {
    return __builtin_bit_cast(uint16_t, (_Float16)v);
}
template <int DT>
__device__ __forceinline__ uint16_t float_to_half(float v) {
    if constexpr (DT == kBF16) return float_to_bf16_rne(v);
    else return float_to_f16_rne(v);
}

// Two-term dot product with fp32 accumulation: a.lo*b.lo + a.hi*b.hi + c.
template <int DT>
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a),
                                               __builtin_bit_cast(bf16x2, b), c, false);
    else
        return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b),
                                      c, false);
}

// INT4 dequant by exponent OR: a nibble n under the bits of M (128.0 in bf16,
// 1024.0 in fp16) is exactly the 16-bit value M + n, so a code q stored as
// n = q + 8 reads back as q after subtracting offset = M + 8 once per sum.
template <int DT>
struct Int4Magic;
template <>
struct Int4Magic<kBF16> {
    static constexpr uint32_t pair = 0x43004300u;   // (128.0, 128.0)
    static constexpr uint32_t one = 0x3F803F80u;    // (1.0, 1.0)
    static constexpr float offset = 136.0f;
};
template <>
struct Int4Magic<kF16> {
    static constexpr uint32_t pair = 0x64006400u;   // (1024.0, 1024.0)
    static constexpr uint32_t one = 0x3C003C00u;
    static constexpr float offset = 1032.0f;
};

// Codes of 8 columns of four kept rows (4 bytes a row: column 2k in the low nibble
// of byte k) as B operands of four-row MFMAs, in the dtype of x, so that x enters
// the product as it is, at any exponent.  A nibble n = q + 8 under an exponent is
// exact: fp16 64 + n (n at bits 4..7, where the high one already is), bf16 16 + n
// (the top four of its seven mantissa bits, both nibbles move).  The bias comes off
// with the sum of x.  (Under fp16's 1024.0 the low nibble needs no move, nor under
// bf16's 128.0, but fp32 sums then round at 1032 or 136 times that sum.)
// bf16: the bytes of two rows and two columns go side by side, so that one shift
// and one v_and_or serve four codes, and a second v_perm puts the exponent's byte
// next to each: 36 instructions for the quad (40 with halves shifted one by one;
// fp16 takes 32).
template <int DT>
struct Int4Quad {
    static constexpr float bias = DT == kBF16 ? 16.0f + 8.0f : 64.0f + 8.0f;
    static constexpr bool kB = DT == kBF16;
    uint32_t mask_lo = kB ? 0x41414141u : 0x000F000Fu;   // bf16: the exponent's byte
    uint32_t mask = kB ? 0x78787878u : 0x00F000F0u;
    uint32_t M = kB ? 0x80808080u : 0x54005400u;
    // Constants the compiler cannot see through, so that (p & mask) | M is one
    // v_and_or_b32 rather than two instructions with literals.  (Not as inline
    // asm: the compiler must see what an MFMA next to it reads and overwrites.)
    __device__ __forceinline__ Int4Quad() {
        if constexpr (kB) asm("" : "+v"(mask_lo), "+s"(mask), "+v"(M));
        else asm("" : "+s"(mask_lo), "+s"(mask), "+v"(M));
    }
    // Columns 4h .. 4h + 3 (h = 0, 1).
    __device__ __forceinline__ void columns(const uint32_t (&w)[4], int h, uint2 (&op)[4]) const {
        if constexpr (kB) {
            const uint32_t sel = 0x05010400u + (uint32_t)h * 0x02020202u;
            const uint32_t p01 = __builtin_amdgcn_perm(w[1], w[0], sel);
            const uint32_t p23 = __builtin_amdgcn_perm(w[3], w[2], sel);
            const uint32_t l01 = ((p01 << 3) & mask) | M, l23 = ((p23 << 3) & mask) | M;
            const uint32_t h01 = ((p01 >> 1) & mask) | M, h23 = ((p23 >> 1) & mask) | M;
            auto half = [&](uint32_t v, uint32_t s) { return __builtin_amdgcn_perm(v, mask_lo, s); };
            op[0] = make_uint2(half(l01, 0x00050004u), half(l23, 0x00050004u));
            op[1] = make_uint2(half(h01, 0x00050004u), half(h23, 0x00050004u));
            op[2] = make_uint2(half(l01, 0x00070006u), half(l23, 0x00070006u));
            op[3] = make_uint2(half(h01, 0x00070006u), half(h23, 0x00070006u));
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t sel = (uint32_t)(2 * h + k) | ((uint32_t)(2 * h + k + 4) << 16);
                const uint32_t p01 = __builtin_amdgcn_perm(w[1], w[0], sel);
                const uint32_t p23 = __builtin_amdgcn_perm(w[3], w[2], sel);
                op[2 * k] = make_uint2(((p01 & mask_lo) << 4) | M, ((p23 & mask_lo) << 4) | M);
                op[2 * k + 1] = make_uint2((p01 & mask) | M, (p23 & mask) | M);
            }
        }
    }
};

// (v & mask) | bits as one v_and_or_b32 (the compiler otherwise emits two VOP2
// instructions with literals).
__device__ __forceinline__ uint32_t and_or(uint32_t v, uint32_t mask, uint32_t bits) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(mask), "v"(bits));
    return r;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

typedef short v4s __attribute__((ext_vector_type(4)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// D += A B on the matrix cores, 16 x 16 x 16 with fp32 accumulation.  Lane l
// holds A[l % 16][4 (l / 16) + e] and B[4 (l / 16) + e][l % 16] for e = 0..3
// (four 16-bit values in a uint2) and gets D[4 (l / 16) + e][l % 16].
template <int DT>
__device__ __forceinline__ v4f mfma16(uint2 a, uint2 b, v4f c) {
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, a),
                                                         __builtin_bit_cast(v4s, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(v4h, a),
                                                     __builtin_bit_cast(v4h, b), c, 0, 0, 0);
}

// The same for 16 blocks of 4 x 4 x 4: block l / 4, A[l % 4][e] and B[e][l % 4],
// D[e][l % 4].
template <int DT>
__device__ __forceinline__ v4f mfma4(uint2 a, uint2 b, v4f c) {
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(v4s, a),
                                                      __builtin_bit_cast(v4s, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(v4h, a),
                                                  __builtin_bit_cast(v4h, b), c, 0, 0, 0);
}

// 16- and 8-byte streaming loads (non-temporal hint: weights are read once
// per call).
__device__ __forceinline__ uint4 load_stream16(const void *p) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 load_stream8(const void *p) {
    const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p));
    return make_uint2(v.x, v.y);
}

// Bounds-checked loads from [p, p + bytes): past the end they return 0, at no
// instruction's cost.  off: per lane, in bytes.  The whole offset is the per-lane
// one (the compiler moves up to 4095 of it into the instruction): these two are
// what the range check covers, while the scalar offset is left out of it by the
// intrinsics' description and stays 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ uint32_t buffer_load32(__amdgpu_buffer_rsrc_t rs, int off) {
    return __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
}
__device__ __forceinline__ uint32_t buffer_load16(__amdgpu_buffer_rsrc_t rs, int off) {
    return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
}
__device__ __forceinline__ uint2 buffer_load64(__amdgpu_buffer_rsrc_t rs, int off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
    return make_uint2(v[0], v[1]);
}
__device__ __forceinline__ uint4 buffer_load128(__amdgpu_buffer_rsrc_t rs, int off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

// Gate activation of the gated FFN: SiLU (act 0) or GELU z * Phi(z) (act 1),
// with Phi(z) = erfc(-z / sqrt 2) / 2 (no cancellation in the negative tail).
__device__ __forceinline__ float gate_act(float z, int act) {
    return act == 0 ? silu(z) : 0.5f * z * erfcf(-z * 0.70710678118654752f);
}

// ---------------------------------------------------------------------------
// Wave64 collectives
// ---------------------------------------------------------------------------

// Orders a wave's LDS writes before its later LDS reads by other lanes (the LDS
// serves a wave's instructions in order; this holds the compiler to it).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Cross-lane moves on the VALU (no LDS round trip): DPP within 16-lane rows,
// and the gfx950 row / half swaps.  swap16(v) is v + lane^16's v, swap32(v)
// is v + lane^32's v; both lanes of a pair get the same bits.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
constexpr int kDppXor1 = 0xB1;     // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;     // quad_perm [2,3,0,1]
constexpr int kDppRor4 = 0x124;    // row_ror:4
constexpr int kDppRor8 = 0x128;    // row_ror:8 (lane ^ 8 within a row)
__device__ __forceinline__ float add_swap16(float v) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_swap32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the wave in a fixed order, returned in every lane (lane 0's value).
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_move<kDppXor1>(v);
    v += dpp_move<kDppXor2>(v);    // quads uniform
    v += dpp_move<kDppRor4>(v);
    v += dpp_move<kDppRor8>(v);    // rows summed
    v = add_swap16(v);
    v = add_swap32(v);
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// Number of set bits of `mask` in lanes below this one.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Inclusive prefix sum over the wave (every lane active).  Shifts of 1, 2, 4
// and 8 inside each 16-lane row (lanes shifted in from outside the row read
// 0), then each row adds the totals of the rows below it.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
              r2 = __builtin_amdgcn_readlane(v, 47);
    const int row = lane_id() >> 4;
    return v + (row >= 1 ? r0 : 0) + (row >= 2 ? r1 : 0) + (row >= 3 ? r2 : 0);
}

// Sum over each quad of lanes (lanes 4j .. 4j+3), in every lane of the quad.
__device__ __forceinline__ uint32_t quad_sum_u32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppXor1, 0xF, 0xF, false);
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kDppXor2, 0xF, 0xF, false);
}

}  // namespace prox
