// In-register dequantisation of packed codes to 16-bit MFMA operands (Sec. 3.1 "standard unpacking",
// grouped affine form s * (q - z)).
//
// A thread always holds one "unit": 32 consecutive codes of one weight row = BITS 32-bit words, all in one
// quantisation group (group sizes are multiples of 32).  dequant8<BITS,BF16>(w, part, c) returns codes
// [8*part, 8*part+8) of the unit, in k order, as eight 16-bit floats, each rounded once from the exact product.
//
// fp16: a code is dropped into the mantissa of the constant 1024.0 (bits 0x6400), giving 1024 + c * 2^p exactly
// for a code sitting at bit p of a 16-bit lane; one packed fma with (2^-p, -(1024 * 2^-p + z)) yields the exact
// small integer c - z, and one packed multiply applies the scale.  bf16: there is no packed bf16 arithmetic.  The
// same fp16 values 1024 + c * 2^p (fp32 holds their products with a scale exactly: 11 bits each) go through one
// mixed-precision fma per code, (1024 + c * 2^p) * (s * 2^-p) - (1024 * 2^-p + z) * s = s (c - z) exactly, and are packed
// with the hardware bf16 conversion: 2.0 to 3.0 instructions per code where extracting and converting every code by
// itself took 2.5 to 3.4.  8-bit codes keep that form: v_cvt_f32_ubyte takes any byte of a word, and the mixed-precision
// form was 1 to 7 % slower where the pass has little else to do (17 tokens, 13824 -> 5120, no adapter: 36.6 against 34.1 us).
#pragma once
#include "common.hpp"

namespace qlora {

template <int BITS, bool BF16>
struct DequantConst;

template <int BITS>
struct DequantConst<BITS, false> {
    half2_t s2;        // (s, s)
    half2_t off[2];    // additive constants per code-pair pattern
    __device__ __forceinline__ void set(float s, float z)
    {
        s2 = half2_t{(half_t)s, (half_t)s};
        if constexpr (BITS == 4) {
            off[0] = half2_t{(half_t)(-(1024.f + z)), (half_t)(-(64.f + z))};
        } else if constexpr (BITS == 2) {
            off[0] = half2_t{(half_t)(-(1024.f + z)), (half_t)(-(256.f + z))};
            off[1] = half2_t{(half_t)(-(64.f + z)), (half_t)(-(16.f + z))};
        } else if constexpr (BITS == 3) {
            off[0] = half2_t{(half_t)(-(1024.f + z)), (half_t)(-(128.f + z))};
        } else {
            off[0] = half2_t{(half_t)(-(1024.f + z)), (half_t)(-(1024.f + z))};
        }
    }
};

template <int BITS>
struct DequantConst<BITS, true> {
    // codes sit at bit p = STEP i of a 16-bit lane, i < NP
    static constexpr int NP = BITS == 2 ? 4 : (BITS == 8 ? 1 : 2), STEP = BITS;
    float mul[NP], off[NP];     // s * 2^-p and -(1024 * 2^-p + z) * s (8-bit codes: s and -z * s)
    __device__ __forceinline__ void set(float sc, float z)
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float inv = 1.f / (float)(1 << (STEP * i));
            mul[i] = sc * inv;
            off[i] = BITS == 8 ? -z * sc : -(1024.f * inv + z) * sc;
        }
    }
};

// (byte b of x) -> [b, 0x64, b, 0x64]: the byte in the low byte of both 16-bit lanes, the exponent byte of 1024.0
// above it, picked from the first source of the byte permute (selector 5 = its byte 1).  Masking the unwanted code
// bits away (with the 0x64 bytes kept by the mask) leaves the two fp16 values 1024 + c * 2^p.
__device__ __forceinline__ uint32_t spread_byte(uint32_t x, int b)
{
    return __builtin_amdgcn_perm(0x64006400u, x, 0x05000500u | ((uint32_t)b << 16) | (uint32_t)b);
}

// (x & mask) | magic in one instruction: the mask from a scalar register, the magic from a vector register (as literals
// the two constants would take two instructions; small-token backward pass, fp16, 16 tokens, gate and up: INT2 23.9 -> 22.7 us,
// INT4 30.8 -> 30.2)
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t magic)
{
    uint32_t d;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(d) : "v"(x), "s"(mask), "v"(magic));
    return d;
}

__device__ __forceinline__ uint32_t h2_bits(half2_t v) { return __builtin_bit_cast(uint32_t, v); }

// SCALE false: the exact integers q - z are returned and the caller applies the group's scale to its sums
template <bool SCALE = true>
__device__ __forceinline__ uint32_t fp16_pair(uint32_t bits, half2_t mul, half2_t off, half2_t s2)
{
    const half2_t h = __builtin_bit_cast(half2_t, bits);
    if constexpr (SCALE) return h2_bits((h * mul + off) * s2);
    else return h2_bits(h * mul + off);
}

// 32-bit window of the unit starting at bit `bit` (compile-time after unrolling).
template <int BITS>
__device__ __forceinline__ uint32_t window(const uint32_t (&w)[BITS], int bit)
{
    const int wi = bit >> 5, sh = bit & 31;
    if (sh == 0) return w[wi];
    const uint32_t hi = wi + 1 < BITS ? w[wi + 1] : 0u;
    return __builtin_amdgcn_alignbit(hi, w[wi], (uint32_t)sh);
}

template <int BITS, bool BF16, bool SCALE = true>     // SCALE false: c was set with scale 1, the result is q - z
__device__ __forceinline__ u16x8_t dequant8(const uint32_t (&w)[BITS], int part, const DequantConst<BITS, BF16> &c)
{
    u32x4_t out;
    if constexpr (!BF16) {
        constexpr uint32_t MAGIC = 0x64006400u;   // (1024.0h, 1024.0h)
        if constexpr (BITS == 4) {
            const uint32_t x = w[part];
            const half2_t mul = {(half_t)1.f, (half_t)0.0625f};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[i] = fp16_pair<SCALE>(spread_byte(x, i) & (0x00F0000Fu | MAGIC), mul, c.off[0], c.s2);
        } else if constexpr (BITS == 2) {
            const uint32_t x = w[part >> 1];
            const half2_t mul0 = {(half_t)1.f, (half_t)0.25f}, mul1 = {(half_t)0.0625f, (half_t)0.015625f};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t p = spread_byte(x, 2 * (part & 1) + i);
                out[2 * i] = fp16_pair<SCALE>(p & (0x000C0003u | MAGIC), mul0, c.off[0], c.s2);
                out[2 * i + 1] = fp16_pair<SCALE>(p & (0x00C00030u | MAGIC), mul1, c.off[1], c.s2);
            }
        } else if constexpr (BITS == 8) {
            const half2_t one = {(half_t)1.f, (half_t)1.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t x = w[2 * part + (i >> 1)];
                const uint32_t sel = (i & 1) ? 0x05030502u : 0x05010500u;   // [b0,0x64,b1,0x64] or [b2,0x64,b3,0x64]
                out[i] = fp16_pair<SCALE>(__builtin_amdgcn_perm(MAGIC, x, sel), one, c.off[0], c.s2);
            }
        } else {   // BITS == 3: eight codes = 24 bits starting at bit 24*part
            const uint32_t x = window<BITS>(w, 24 * part);
            const half2_t mul = {(half_t)1.f, (half_t)0.125f};
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[i] = fp16_pair<SCALE>(spread_byte(x >> (6 * i), 0) & (0x00380007u | MAGIC), mul, c.off[0], c.s2);
        }
    } else {
        typedef float float2_t __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        constexpr uint32_t MAGIC = 0x64006400u;
        // two neighbouring codes as (1024 + c * 2^p, 1024 + c' * 2^p'), p and p' given by their index into c.mul
        auto pair = [&](uint32_t bits, int p0, int p1) {
            const half2_t h = __builtin_bit_cast(half2_t, bits);
            const float2_t f = {__builtin_fmaf((float)h[0], c.mul[p0], c.off[p0]),
                                __builtin_fmaf((float)h[1], c.mul[p1], c.off[p1])};
            return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
        };
        if constexpr (BITS == 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) out[i] = pair(spread_byte(w[part], i) & (0x00F0000Fu | MAGIC), 0, 1);
        } else if constexpr (BITS == 2) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t p = spread_byte(w[part >> 1], 2 * (part & 1) + i);
                out[2 * i] = pair(p & (0x000C0003u | MAGIC), 0, 1);
                out[2 * i + 1] = pair(p & (0x00C00030u | MAGIC), 2, 3);
            }
        } else if constexpr (BITS == 8) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t b = w[2 * part + (i >> 1)] >> (16 * (i & 1));
                const float2_t f = {__builtin_fmaf((float)(b & 0xffu), c.mul[0], c.off[0]),
                                    __builtin_fmaf((float)((b >> 8) & 0xffu), c.mul[0], c.off[0])};
                out[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
            }
        } else {
            const uint32_t x = window<BITS>(w, 24 * part);
#pragma unroll
            for (int i = 0; i < 4; ++i) out[i] = pair(spread_byte(x >> (6 * i), 0) & (0x00380007u | MAGIC), 0, 1);
        }
    }
    return __builtin_bit_cast(u16x8_t, out);
}

}  // namespace qlora
