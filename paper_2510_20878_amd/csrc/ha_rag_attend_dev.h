// Device-side pieces shared by the attention kernels over packed chunks: the per-format block
// geometry, the decoders that give the BF16 values a load would write, and small helpers.
#pragma once
#include "ha_rag_kernels.h"
#include "ha_rag_decode.h"
#include <cstring>

namespace ha_rag {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <uint32_t PREC>
struct Fmt {
    static constexpr uint32_t kWords = PREC == kInt4 ? 1u : PREC == kP16 ? 4u : 2u;  // 16-byte words per lane and block
    static constexpr uint32_t kPayload = 1024u * kWords;
    static constexpr bool kMeta = PREC == kInt4 || PREC == kInt8;
};

// Integer codes -> binary32 of fma(code, scale, zero), the very values of dequant_octet4 / 8.  Two
// codes lie in the halves of a dword: read as binary16 such a half is the subnormal code * 2^-24,
// which the mixed fma takes as it is next to scale * 2^24 (exact) and the binary16 zero: the product
// is code * scale, the sum is rounded once.  No conversion per code.
template <int HALF>
__device__ __forceinline__ float code_fma(uint32_t codes, float scale24, uint32_t meta)
{
    float r;
    if (HALF == 0) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(codes), "v"(scale24), "v"(meta));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(codes), "v"(scale24), "v"(meta));
    return r;
}

__device__ __forceinline__ float scale24(uint32_t meta) { return h2f(meta & 0xFFFFu) * 16777216.0f; }

// 8 int4 codes (one dword) / 8 int8 codes (two) of one octet -> 8 binary32
__device__ __forceinline__ void octet4_f32(uint32_t c, uint32_t m, float (&f)[8])
{
    const float s = scale24(m);
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // codes k and k + 4
        const uint32_t h = (c >> (4 * k)) & 0x000F000Fu;
        f[k] = code_fma<0>(h, s, m);
        f[k + 4] = code_fma<1>(h, s, m);
    }
}

__device__ __forceinline__ void octet8_f32(uint32_t c0, uint32_t c1, uint32_t m, float (&f)[8])
{
    const float s = scale24(m);
    const uint32_t h[4] = {__builtin_amdgcn_perm(0u, c0, 0x0C010C00u), __builtin_amdgcn_perm(0u, c0, 0x0C030C02u),
                           __builtin_amdgcn_perm(0u, c1, 0x0C010C00u), __builtin_amdgcn_perm(0u, c1, 0x0C030C02u)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[2 * k] = code_fma<0>(h[k], s, m);
        f[2 * k + 1] = code_fma<1>(h[k], s, m);
    }
}

__device__ __forceinline__ u32x4 pack_octet(const float (&f)[8])
{
    return u32x4{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7])};
}

// the raw codes of one octet (x: int4; x, y: 8-bit formats; all four: 16-bit) -> 8 BF16
template <uint32_t PREC>
__device__ __forceinline__ u32x4 decode_octet(u32x4 raw, uint32_t meta, const Gse8Tab &tab)
{
    if (PREC == kInt4 || PREC == kInt8) {
        float f[8];
        if (PREC == kInt4) octet4_f32(raw.x, meta, f);
        else octet8_f32(raw.x, raw.y, meta, f);
        return pack_octet(f);
    }
    if (PREC == kE4M3) return decode_octet_fp8<false>(raw.x, raw.y);
    if (PREC == kE5M2) return decode_octet_fp8<true>(raw.x, raw.y);
    if (PREC == kGSE8) return decode_octet_gse8(raw.x, raw.y, tab);
    return raw;
}

// Two octets of the same dims and two tokens a, b -> t[p] = {value p of a, value p of b}: the integer
// formats are rounded straight into these pairs, the others' words or codes are regrouped.
template <uint32_t PREC>
__device__ __forceinline__ void decode_octets_by_token(u32x4 ra, u32x4 rb, uint32_t ma, uint32_t mb, const Gse8Tab &tab,
                                                       uint32_t (&t)[8])
{
    if (PREC == kInt4 || PREC == kInt8) {
        float a[8], b[8];
        if (PREC == kInt4) {
            octet4_f32(ra.x, ma, a);
            octet4_f32(rb.x, mb, b);
        } else {
            octet8_f32(ra.x, ra.y, ma, a);
            octet8_f32(rb.x, rb.y, mb, b);
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) t[p] = pack_bf16(a[p], b[p]);
    } else if (PREC == kP16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            t[2 * q] = __builtin_amdgcn_perm(rb[q], ra[q], 0x05040100u);
            t[2 * q + 1] = __builtin_amdgcn_perm(rb[q], ra[q], 0x07060302u);
        }
    } else {  // the codes are regrouped: half as many bytes
        const uint32_t a[2] = {ra.x, ra.y}, b[2] = {rb.x, rb.y};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4 raw = {__builtin_amdgcn_perm(b[h], a[h], 0x05010400u), __builtin_amdgcn_perm(b[h], a[h], 0x07030602u), 0u, 0u};
            const u32x4 v = decode_octet<PREC>(raw, 0u, tab);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[4 * h + q] = v[q];
        }
    }
}

// plane j of the words a lane loaded from a payload block
template <uint32_t PREC>
__device__ __forceinline__ u32x4 plane_raw(const u32x4 *w, int j)
{
    u32x4 r = {0u, 0u, 0u, 0u};
    if (PREC == kInt4) r.x = w[0][j];
    else if (PREC == kP16) r = w[j];
    else {
        r.x = w[j >> 1][(j & 1) * 2];
        r.y = w[j >> 1][(j & 1) * 2 + 1];
    }
    return r;
}

// The first instruction that reads an MFMA result has to come a fixed number of cycles after
// the MFMA (11 for the 8-pass 16x16x32).  The compiler inserts that wait where both are in one
// basic block; with a branch between them it was found to leave the wait out, and the reader
// then sees what the registers held before.  Called right after a chain whose result is first
// read behind a branch: nothing is scheduled across it, and it idles for 12 cycles.
__device__ __forceinline__ void mfma_result_wait()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7\n\ts_nop 3");
    __builtin_amdgcn_sched_barrier(0);
}

// how far a score may exceed a row's running maximum before that maximum is brought up to
// date, in units of log2: weights stay below 2^8
constexpr float kLazyMaxSlack = 8.0f;
// and how far above the largest score the reference is then put: the two together are what the
// scores may still grow by before it has to be moved again, which is a hundred-odd instructions for
// the wave.  With 0, one pair of blocks in eight moved it (every row of a wave has a say, and every
// document brings keys of another spread); the weights are relative to it, so nothing is lost.
constexpr float kLazyMaxLift = 8.0f;

// Adds two BF16 weights (one dword) to `sum`.  The output is normalised by the sum of the very
// weights that multiplied V, so that what rounding does to a weight does not also scale the result
// (a row with one dominant key gets that key's value exactly); the log-sum-exp keeps the
// unrounded sum.  One instruction per two weights.  Relative error of the output against 64 bits,
// without and with it, over ten documents of 512 tokens (two 16-bit, three int8, five int4): one request at
// one query token 0.62e-3 and 0.21e-3, 32 requests 1.1e-3 and 0.67e-3, at 64 query tokens 1.2e-3 and 0.80e-3.
// It costs k6_attend_shared 1 to 2 % where the decode is long (32 requests over GSE-8, 24 query tokens: 164 ->
// 166 us, with the decode as it was then).
__device__ __forceinline__ float add_weights(uint32_t pair, float sum)
{
    const uint32_t ones = 0x3F803F80u;
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, ones), sum, false);
}

__device__ __forceinline__ float neg_inf() { return -__builtin_huge_valf(); }

// orders the LDS accesses of one wave: what its lanes wrote before is visible to all its
// lanes after.  The hardware executes the LDS instructions of a wave in issue order, so
// nothing has to be waited for; the fences keep the compiler from moving accesses across
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the launch-wide scalars a workgroup needs, read from the argument buffer once
struct AttendHdr {
    uint32_t n_kv_heads, n_q_heads, layer;
    float scale_log2;
};

// keeps a value in a scalar register from here on: everything pinned at the top of the kernel
// is fetched from the argument buffer by loads issued together, not one by one where the
// values are first used
__device__ __forceinline__ void pin(uint32_t &v) { asm volatile("" : "+s"(v)); }
__device__ __forceinline__ void pin(float &v) { asm volatile("" : "+s"(v)); }
template <class T>
__device__ __forceinline__ void pin(T *&v)
{
    uint64_t a = reinterpret_cast<uint64_t>(v);
    asm volatile("" : "+s"(a));
    v = reinterpret_cast<T *>(a);
}

// Everything the attention kernels read or write outside LDS lies in global memory; saying so lets the
// loads run as global instructions (scalar base, 32-bit lane offset), which do not count
// against the LDS counter the way loads through generic pointers do.
typedef const uint8_t __attribute__((address_space(1))) *gbytes;
typedef float __attribute__((address_space(1))) *gfloats;

__device__ __forceinline__ u32x4 ldg16(gbytes p)
{
    return *(const u32x4 __attribute__((address_space(1))) *)p;
}

// the same, past the last-level cache if ONCE
template <bool ONCE>
__device__ __forceinline__ u32x4 ldg16_of(gbytes p)
{
    if (ONCE) return __builtin_nontemporal_load((const u32x4 __attribute__((address_space(1))) *)p);
    return ldg16(p);
}

// max of a value over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (one per lane group), in every
// lane.  The row swaps exchange registers between lane rows without a trip through LDS: after
// swapping the odd rows of one copy with the even rows of another, the two copies hold the
// value of rows r and r ^ 1 side by side; the same with halves of 32 lanes.
__device__ __forceinline__ float max_over_lane_groups(float x)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const unsigned xi = __builtin_bit_cast(unsigned, x);
    const u2 r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    const unsigned r0 = r.x, r1 = r.y;  // copied out first: a bit cast of a vector element reads element 0
    const float y = __builtin_fmaxf(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1));
    const unsigned yi = __builtin_bit_cast(unsigned, y);
    const u2 t = __builtin_amdgcn_permlane32_swap(yi, yi, false, false);
    const unsigned t0 = t.x, t1 = t.y;
    return __builtin_fmaxf(__builtin_bit_cast(float, t0), __builtin_bit_cast(float, t1));
}

// the sum over the same four lanes, in every lane, the same way
__device__ __forceinline__ float sum_over_lane_groups(float x)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const unsigned xi = __builtin_bit_cast(unsigned, x);
    const u2 r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    const unsigned r0 = r.x, r1 = r.y;
    const unsigned yi = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1));
    const u2 t = __builtin_amdgcn_permlane32_swap(yi, yi, false, false);
    const unsigned t0 = t.x, t1 = t.y;
    return __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1);
}

// Launches a kernel of one argument from where the argument lies.  (The launch syntax passes it by value
// first: another copy of up to 36 KiB.)  What it reports is the thread's last error, fetched, as the other launchers
// do: left there, it would be taken for the next call's.
template <class P>
inline hipError_t launch_args(void (*kernel)(const P), dim3 grid, dim3 block, uint32_t lds_bytes, hipStream_t stream, P &p)
{
    void *args[] = {&p};
    (void)hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, args, lds_bytes, stream);
    return hipGetLastError();
}

// launch(p), or launch of a copy of p in the structure of few where that holds what p does (see K6ParamsOf).
template <class F>
inline hipError_t launch_few_or_all(K6Params &p, F launch)
{
    if (p.doc_end > K6ParamsFew::kMaxDocs) return launch(p);  // doc_end lies behind the runs (check_k6_args)
    K6ParamsFew f;
    f.n_kv_heads = p.n_kv_heads;
    f.n_q_heads = p.n_q_heads;
    f.layer = p.layer;
    f.n_runs = p.n_runs;
    f.mtw = p.mtw;
    f.scale_log2 = p.scale_log2;
    f.doc_first = p.doc_first;
    f.doc_end = p.doc_end;
    f.past = p.past;
    f.heads_first = p.heads_first;
    std::memcpy(f.doc, p.doc, p.doc_end * sizeof(K6Doc));
    return launch(f);
}

}  // namespace ha_rag
