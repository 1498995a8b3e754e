// Device-side decoders of the packed chunk formats: one octet (8 codes of one plane of a
// layout block) -> 8 BF16 values in one 16-byte word.  Shared by every kernel that reads
// packed chunks; the values are the ones a load writes into the cache:
// bf16_rne(fma(code, scale, zero)) for the integer formats, exact for FP8 and GSE-8.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace ha_rag {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u32x4 ld16(const uint8_t *p)
{
    return *reinterpret_cast<const u32x4 *>(p);
}

template <bool NT>
__device__ __forceinline__ void st16(uint8_t *p, u32x4 v)
{
    if (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(p));
    else *reinterpret_cast<u32x4 *>(p) = v;
}

__device__ __forceinline__ float h2f(uint32_t h16)
{
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h16);
}

// two fp32 -> one dword of two BF16 (round to nearest even), a in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ float byte_f(uint32_t w, int k)
{
    return (float)((w >> (8 * k)) & 0xFFu);  // one byte-to-float conversion each
}

// 8 int4 codes (one dword) of one plane -> 8 BF16 (16 bytes)
__device__ __forceinline__ u32x4 dequant_octet4(uint32_t c, uint32_t m)
{
    const float s = h2f(m & 0xFFFFu), z = h2f(m >> 16);
    const uint32_t ev = c & 0x0F0F0F0Fu;         // codes 0,2,4,6 one per byte
    const uint32_t od = (c >> 4) & 0x0F0F0F0Fu;  // codes 1,3,5,7
    u32x4 r;
    r.x = pack_bf16(__builtin_fmaf(byte_f(ev, 0), s, z), __builtin_fmaf(byte_f(od, 0), s, z));
    r.y = pack_bf16(__builtin_fmaf(byte_f(ev, 1), s, z), __builtin_fmaf(byte_f(od, 1), s, z));
    r.z = pack_bf16(__builtin_fmaf(byte_f(ev, 2), s, z), __builtin_fmaf(byte_f(od, 2), s, z));
    r.w = pack_bf16(__builtin_fmaf(byte_f(ev, 3), s, z), __builtin_fmaf(byte_f(od, 3), s, z));
    return r;
}

// 8 int8 codes (two dwords) of one plane -> 8 BF16
__device__ __forceinline__ u32x4 dequant_octet8(uint32_t c0, uint32_t c1, uint32_t m)
{
    const float s = h2f(m & 0xFFFFu), z = h2f(m >> 16);
    u32x4 r;
    r.x = pack_bf16(__builtin_fmaf(byte_f(c0, 0), s, z), __builtin_fmaf(byte_f(c0, 1), s, z));
    r.y = pack_bf16(__builtin_fmaf(byte_f(c0, 2), s, z), __builtin_fmaf(byte_f(c0, 3), s, z));
    r.z = pack_bf16(__builtin_fmaf(byte_f(c1, 0), s, z), __builtin_fmaf(byte_f(c1, 1), s, z));
    r.w = pack_bf16(__builtin_fmaf(byte_f(c1, 2), s, z), __builtin_fmaf(byte_f(c1, 3), s, z));
    return r;
}

// 8 FP8 codes (two dwords) of one plane -> 8 BF16: one conversion per two codes.  Every FP8 value is a BF16 value, so
// with scale 1 nothing is rounded.  (By way of binary32 and a byte permute of the upper halves, two instructions: 16 requests x
// 5,120 tokens, two layers, 12 query tokens 105.7 -> 103.0 us, 30 (512- and 300-token documents) 135.2 -> 132.2, one query token
// of 32 requests 128.5 -> 127.2.)
template <bool E5M2>
__device__ __forceinline__ u32x4 decode_octet_fp8(uint32_t c0, uint32_t c1)
{
    auto two = [](uint32_t c, auto high) -> uint32_t {
        bf16x2 v;
        if (E5M2) v = __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(c, 1.0f, decltype(high)::value);
        else v = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c, 1.0f, decltype(high)::value);
        return __builtin_bit_cast(uint32_t, v);
    };
    u32x4 r;
    r.x = two(c0, std::false_type{});
    r.y = two(c0, std::true_type{});
    r.z = two(c1, std::false_type{});
    r.w = two(c1, std::true_type{});
    return r;
}

// GSE-8: value = +-field * 2^n with n = min(base + 3 index, top), where base = e_lo + 2 - 2 and top = e_hi - 2 are the
// tile's exponent bounds already lowered by the 2 fraction places of the field; exact in BF16.  With
// least = min(base, top) that is field * 2^least, one of eight BF16 words per tile, with min(3 index, top - least)
// added to its exponent.  The eight words are kept as a table of low and one of high bytes, from which one byte permute
// takes the bytes of four codes; the exponents are raised two codes at a time in 16-bit halves.  Byte permutes and
// packed 16-bit operations take a SIMD 4.2 clocks as conversions, bit-field extracts, minima and ldexp do, but those
// served one code each: 27 clocks per code and lane then, 16 now.  Attention of 32 requests over ten documents of 512
// tokens, us per layer: 105 -> 82 at one query token, 136 -> 108 at 12, 167 -> 138 at 24, 227 -> 188 at 64; a load of
// ten such documents, bound by memory, 168.4 -> 167.0.
struct Gse8Tab {
    uint32_t lo0, lo1, hi0, hi1;  // low / high bytes of field * 2^least, fields 0..3 and 4..7
    uint32_t lim;                 // (top - least) << 7, in both halves
};

// range: the first dword of the block that follows the tile's payload
__device__ __forceinline__ Gse8Tab gse8_tab(uint32_t range)
{
    const int base = (int)(int8_t)(range & 0xFFu), top = (int)(int8_t)((range >> 8) & 0xFFu) - 2;
    const int least = base < top ? base : top;
    // three significant bits: the upper halves of the binary32 numbers are the BF16 values.  (The format's
    // e_lo is at least -126, so subnormal ones can only be there where least = top: nothing is added to their exponents.)
    uint32_t w[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) w[f] = __builtin_bit_cast(uint32_t, __builtin_ldexpf((float)f, least));
    Gse8Tab t;
    uint32_t by2[4];  // fields 2 i and 2 i + 1: low bytes, then high bytes
#pragma unroll
    for (int i = 0; i < 4; ++i) by2[i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x07030602u);
    t.lo0 = __builtin_amdgcn_perm(by2[1], by2[0], 0x05040100u);
    t.hi0 = __builtin_amdgcn_perm(by2[1], by2[0], 0x07060302u);
    t.lo1 = __builtin_amdgcn_perm(by2[3], by2[2], 0x05040100u);
    t.hi1 = __builtin_amdgcn_perm(by2[3], by2[2], 0x07060302u);
    t.lim = (uint32_t)(top - least) * (128u * 0x00010001u);
    return t;
}

// four codes (one dword) -> two dwords of two BF16
__device__ __forceinline__ void decode_quad_gse8(uint32_t c, const Gse8Tab &t, uint32_t &r01, uint32_t &r23)
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const uint32_t field = c & 0x07070707u;
    const uint32_t lo = __builtin_amdgcn_perm(t.lo1, t.lo0, field);
    const uint32_t hi = __builtin_amdgcn_perm(t.hi1, t.hi0, field) | (c & 0x80808080u);
    // a zero field is zero whatever its index
    const uint32_t k = c & __builtin_amdgcn_perm(0xFFFFFFFFu, 0xFFFFFF00u, field) & 0x78787878u;
    auto pair = [&](uint32_t spread, uint32_t bytes) {
        const u16x2 k8 = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(0u, k, spread));  // 8 * index
        const u16x2 up = __builtin_elementwise_min((u16x2)(k8 * u16x2{48, 48}), __builtin_bit_cast(u16x2, t.lim));
        return __builtin_amdgcn_perm(hi, lo, bytes) + __builtin_bit_cast(uint32_t, up);  // no half overflows
    };
    r01 = pair(0x0C010C00u, 0x05010400u);
    r23 = pair(0x0C030C02u, 0x07030602u);
}

// 8 codes (two dwords) of one plane -> 8 BF16
__device__ __forceinline__ u32x4 decode_octet_gse8(uint32_t c0, uint32_t c1, const Gse8Tab &t)
{
    uint32_t r0, r1, r2, r3;
    decode_quad_gse8(c0, t, r0, r1);
    decode_quad_gse8(c1, t, r2, r3);
    return u32x4{r0, r1, r2, r3};
}

}  // namespace ha_rag
