// gfx950 kernels for attention over packed chunks when a request has more query rows than one
// wave can keep (more than two 16-row tiles: the question's prefill of Sec. 2.1, tens of query
// tokens times the query heads of a KV head), and for requests of two tiles next to such.
//
//  k6_attend_shared<W>   one workgroup of W waves (2 or 4) per (run of blocks across a request's
//      documents in list order, KV head, group of 2 W query tiles).  Every wave owns two query
//      tiles for the whole run: their queries, reference maxima, sums and output rows stay in its
//      registers.  The layout blocks are taken W at a time: half the waves decode the keys and
//      half the values of the round, two blocks each (W = 2: one wave each), to BF16 (the values a load would write)
//      and leave them in LDS in the form the MFMAs take their operands in; after one barrier
//      every wave scores all W blocks against its own tiles, two blocks (a pair) at a time.  A
//      block is therefore fetched and decoded once per 32 W query rows.  The rounds alternate
//      between two sets of LDS buffers, so one barrier per round is enough: a wave that writes
//      round r + 1 has passed barrier r, which every wave reaches only after it has read all of
//      round r - 1.
//  k6_attend_roles    the same with waves of two kinds: four or eight that score (two tiles each, so 128
//      or 256 query rows) and four that decode the next round of eight blocks meanwhile.  Described at
//      the kernel.
// Which of them a call takes, and in runs of what length, follows from what each is expected to cost (kForms in
// ha_rag_attend.hip).
//
// Block geometry as for k6_attend_partial: lane (c = lane / 16, n = lane % 16) of the wave that
// reads a block holds, in plane j, token 4 j + c, dims 8 n .. 8 n + 7.
//   V: that is what the product P V takes from a lane, so the decoding wave stores its eight
//      operand words lane by lane, those of a pair's first and second block side by side (16
//      bytes per lane and operand), and every wave reads them back lane by lane: one 16x16x32
//      MFMA then contracts over the 32 tokens of the pair.
//   K: the score MFMA wants, per lane, 8 dims of the token of its column; the decoding wave
//      stores octet o of token t at 16-byte slot (o ^ t) of row t (256 bytes a row), which
//      both its own stores and the readers' loads reach without bank conflicts.
// A pair's buffer is 16 KiB: K of its first block, K of its second block, V of both (the layout of
// k6_attend_roles differs in the rows of K: kRoleKeyRow).
#include "ha_rag_attend_dev.h"
#include <atomic>
#include <type_traits>

namespace ha_rag {

namespace {

constexpr uint32_t kSharedBlockLds = 8192;  // LDS per block: K operands 4 KiB, V operands 4 KiB (laid out per pair)


struct SharedState {  // a wave's two query tiles
    bf16x8 qb[2][4];
    float m_run[2], l_run[2];
    float r_run[2];  // the sum of the weights as they multiply V (add_weights); l_run: before rounding
    f32x4 O[2][8];
};

struct SharedSide {  // the keys or the values of one document's (layer, head) tile (uniform values)
    gbytes tile, meta;
    uint32_t meta_blk, gsh;
    Gse8Tab tab;  // GSE-8
};

struct SharedLane {
    uint32_t lane, c_, n_;  // MFMA coordinates: lane group, lane column
    uint32_t k_rd;          // where the lane reads its K operand 0 inside a block's buffer; operand y: ^ 16 y
    uint32_t k_wr;          // where it writes the keys of its plane 0; plane j: (^ 64 j) + 1024 j
};

// a fresh copy of a lane constant: what is derived from it is computed where it is used and
// does not occupy registers across the whole loop
__device__ __forceinline__ uint32_t fresh(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// the eight weights of a pair
__device__ __forceinline__ float add_weights8(const bf16x8 &w, float sum)
{
    const u32x4 pk = __builtin_bit_cast(u32x4, w);
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = add_weights(pk[i], sum);
    return sum;
}

// Two blocks (a pair) against the wave's two tiles, in three steps: S^T = K Q^T of both blocks
// (shared_qk_pair), the running softmax (shared_softmax_pair), O += P V (shared_pv_pair).
//
// The product P V contracts over tokens, 16 per block; the 16x16x32 MFMA contracts over 32, so
// the two blocks of a pair share one: contraction index 8 c_ + i is token 4 i + c_ of the pair's
// first block for i < 4 and token 4 (i - 4) + c_ of its second block for i >= 4.  For the lane
// that is the weights of the first block next to those of the second (P8) and, per dim, the
// values of the first block next to those of the second, which is how the decoding waves lay
// the pair's V operands out (16 bytes per lane and operand: first block, second block).  Half
// the MFMAs of the 16x16x16 form, which is no faster per instruction.

// S[e][mt][jj] = q k (unscaled) of token 4 jj + c_ of block e of the pair and query row n_ of tile mt
__device__ __forceinline__ void shared_qk_pair(const uint8_t *pair, const SharedLane &ln, const SharedState &st,
                                               f32x4 (&S)[2][2])
{
    const uint32_t k_rd = fresh(ln.k_rd);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        bf16x8 ka[4];
#pragma unroll
        for (uint32_t y = 0; y < 4; ++y)
            ka[y] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(pair + e * 4096u + (k_rd ^ (16u * y))));
        // both tiles side by side, so that their MFMA chains overlap
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) S[e][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                S[e][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[y], st.qb[mt][y], S[e][mt], 0, 0, 0);
    }
}

// From the scores of the pair that starts at block b to the weights P8 (the A operands of P V).
// `end` = the first token that does not count: the document's end, or the end of the run's last
// block; only a pair that reaches beyond it is masked.  The caller sees to it that S is not read
// too early after its MFMAs (mfma_result_wait).
__device__ __forceinline__ void shared_softmax_pair(f32x4 (&S)[2][2], uint32_t b, uint32_t end, float scale_log2,
                                                    const SharedLane &ln, SharedState &st, bf16x8 (&P8)[2])
{
    if (b * 16u + 32u > end) {  // a ragged last block, or a last block without a partner
        const uint32_t tok = b * 16u + (fresh(ln.lane) >> 4);  // computed only here
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    if (tok + 16u * e + 4u * jj >= end) S[e][mt][jj] = neg_inf();
    }
    float mx[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const float a = __builtin_fmaxf(__builtin_fmaxf(S[0][mt][0], S[0][mt][1]), __builtin_fmaxf(S[0][mt][2], S[0][mt][3]));
        const float bb = __builtin_fmaxf(__builtin_fmaxf(S[1][mt][0], S[1][mt][1]), __builtin_fmaxf(S[1][mt][2], S[1][mt][3]));
        mx[mt] = __builtin_fmaxf(a, bb) * scale_log2;
    }
    // The running maximum of a row is only a reference point for the exponentials, so it need
    // not be the true maximum: it is brought up to date (a reduction over the lane groups and a
    // rescaling of what is accumulated) only when some lane meets a score more than
    // kLazyMaxSlack above it, which bounds every weight by 2^kLazyMaxSlack.  After the first
    // blocks that almost never happens, and a pair costs one comparison instead of the reduction.
    if (__any(mx[0] > st.m_run[0] + kLazyMaxSlack || mx[1] > st.m_run[1] + kLazyMaxSlack)) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const float m_new = __builtin_fmaxf(st.m_run[mt], max_over_lane_groups(mx[mt]) + kLazyMaxLift);
            const float alpha = __builtin_amdgcn_exp2f(st.m_run[mt] - m_new);  // 0 at the first block, 1 if nothing moved
            st.l_run[mt] *= alpha;
            st.r_run[mt] *= alpha;
            st.m_run[mt] = m_new;
            const uint32_t c_ = fresh(ln.lane) >> 4;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const float ar = __shfl(alpha, (int)(4u * c_ + jj));  // factor of output row 4 c_ + jj
#pragma unroll
                for (int pp = 0; pp < 8; ++pp) st.O[mt][pp][jj] *= ar;
            }
        }
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        float pr[2][4];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                pr[e][jj] = __builtin_amdgcn_exp2f(__builtin_fmaf(S[e][mt][jj], scale_log2, -st.m_run[mt]));
        st.l_run[mt] += ((pr[0][0] + pr[0][1]) + (pr[0][2] + pr[0][3])) + ((pr[1][0] + pr[1][1]) + (pr[1][2] + pr[1][3]));
        const u32x4 pk = {pack_bf16(pr[0][0], pr[0][1]), pack_bf16(pr[0][2], pr[0][3]),
                          pack_bf16(pr[1][0], pr[1][1]), pack_bf16(pr[1][2], pr[1][3])};
        P8[mt] = __builtin_bit_cast(bf16x8, pk);
        st.r_run[mt] = add_weights8(P8[mt], st.r_run[mt]);
    }
}

// O += P V of a pair; `vsrc` = its V operands
__device__ __forceinline__ void shared_pv_pair(const uint8_t *vsrc, const SharedLane &ln, SharedState &st,
                                               const bf16x8 (&P8)[2])
{
    const uint32_t v_rd = fresh(ln.lane) * 16u;
    u32x4 vq[8];
#pragma unroll
    for (int pp = 0; pp < 8; ++pp) vq[pp] = *reinterpret_cast<const u32x4 *>(vsrc + pp * 1024u + v_rd);
#pragma unroll
    for (int pp = 0; pp < 8; ++pp) {
        const bf16x8 v = __builtin_bit_cast(bf16x8, vq[pp]);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
            st.O[mt][pp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P8[mt], v, st.O[mt][pp], 0, 0, 0);
    }
}

// The rounds of one document for a wave that decodes one side (IS_K: the keys) of format P:
// decoder number r of its side takes blocks 2 r and 2 r + 1 of every round of W blocks.
template <uint32_t P, bool IS_K, int W>
__device__ __forceinline__ void shared_rounds(const SharedSide &sd, uint32_t T, uint32_t b0, uint32_t b1,
                                              float scale_log2, uint32_t r, bool active, const SharedLane &ln,
                                              uint8_t (*lds)[W][kSharedBlockLds], uint32_t &set, SharedState &st)
{
    typedef Fmt<P> F;
    const uint32_t lane = ln.lane, c_ = ln.c_;
    u32x4 w[2][F::kWords], m[2];
    m[0] = m[1] = u32x4{0u, 0u, 0u, 0u};
    // the block is clamped to the range's last one instead of skipping the loads: no branch
    // around them, so nothing waits for them before they are needed
    auto fetch = [&](int e, uint32_t b) {
        b = b < b1 ? b : b1 - 1u;
#pragma unroll
        for (uint32_t a = 0; a < F::kWords; ++a)
            w[e][a] = ldg16(sd.tile + ((uint64_t)b * F::kPayload + a * 1024u + lane * 16u));
        if (F::kMeta) m[e] = ldg16(sd.meta + ((uint64_t)b * sd.meta_blk + ((lane * 8u) >> sd.gsh) * 16u));
    };
    fetch(0, b0 + 2u * r);
    fetch(1, b0 + 2u * r + 1u);
    for (uint32_t rb = b0; rb < b1; rb += W) {  // a round: blocks rb .. rb + W - 1
        // ---- this wave's two blocks of the round: decode into the round's buffers
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t blk = rb + 2u * r + e;
            uint8_t *pair = lds[set][2u * r];  // this decoder's pair of the round: K 4 KiB + 4 KiB, then V 8 KiB
            if (blk >= b1) {
                // no such block.  If its partner exists, the pair's MFMAs still take this half of
                // the V operands, with weight zero: it must hold numbers (what the keys' half
                // holds does not matter, its scores are replaced)
                if (!IS_K && e == 1 && blk - 1u < b1) {
#pragma unroll
                    for (int pp = 0; pp < 8; ++pp)
                        *reinterpret_cast<u32x2 *>(pair + 8192u + pp * 1024u + fresh(lane) * 16u + 8u) = u32x2{0u, 0u};
                }
                continue;
            }
            uint8_t *dst = pair + e * 4096u;
            u32x4 o[4];  // o[j] = token 4 j + c_, dims 8 n_ .. 8 n_ + 7 as BF16
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = decode_octet<P>(plane_raw<P>(w[e], j), m[e][j], sd.tab);
            if (IS_K) {
                // token t = 4 j + c_, octet n_: slot (n_ ^ t) of row t
                const uint32_t k_wr = fresh(ln.k_wr);
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j)
                    *reinterpret_cast<u32x4 *>(dst + ((k_wr ^ (64u * j)) + 1024u * j)) = o[j];
            } else {
                if (blk * 16u + 16u > T) {  // rows past the document's end
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j)
                        if (blk * 16u + 4u * j + c_ >= T) o[j] = u32x4{0u, 0u, 0u, 0u};
                }
                // operand pp of P V: value pp of the octet of each of the lane's four tokens; the
                // pair's second block fills the second half of the lane's 16 bytes
                uint8_t *vdst = pair + 8192u + fresh(lane) * 16u + e * 8u;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    u32x2 lo, hi;
                    lo.x = __builtin_amdgcn_perm(o[1][q], o[0][q], 0x05040100u);
                    lo.y = __builtin_amdgcn_perm(o[3][q], o[2][q], 0x05040100u);
                    hi.x = __builtin_amdgcn_perm(o[1][q], o[0][q], 0x07060302u);
                    hi.y = __builtin_amdgcn_perm(o[3][q], o[2][q], 0x07060302u);
                    *reinterpret_cast<u32x2 *>(vdst + (2 * q) * 1024u) = lo;
                    *reinterpret_cast<u32x2 *>(vdst + (2 * q + 1) * 1024u) = hi;
                }
            }
        }
        __syncthreads();
        // the wave's blocks of the next round: in flight while this round is scored.  Issued
        // after the barrier, which waits for every memory access of the wave still under way
        fetch(0, rb + W + 2u * r);
        fetch(1, rb + W + 2u * r + 1u);

        // ---- every wave: its two tiles against the round's blocks, two blocks at a time.  The
        // loop over the pairs is kept a loop: unrolled, the pairs' operand loads and temporaries
        // overlap and the registers do not reach (the 16-bit instances then spill into the path
        // of the prefetch, whose wait a reload shares).
        if (active) {
            const uint32_t nb = b1 - rb < (uint32_t)W ? b1 - rb : (uint32_t)W;
            const uint32_t end = b1 * 16u < T ? b1 * 16u : T;  // the first token that does not count
            const uint8_t *base = lds[set][0];
#pragma unroll 1
            for (uint32_t pr = 0; 2u * pr < nb; ++pr) {
                {
                    const uint8_t *pair = base + pr * (2u * kSharedBlockLds);
                    f32x4 S[2][2];
                    bf16x8 P8[2];
                    shared_qk_pair(pair, ln, st, S);
                    mfma_result_wait();
                    shared_softmax_pair(S, rb + 2u * pr, end, scale_log2, ln, st, P8);
                    shared_pv_pair(pair + 8192u, ln, st, P8);
                }
            }
        }
        set ^= 1u;
    }
    // what follows the document's last P V MFMAs (moves of the output rows between registers, the
    // records) lies behind branches
    mfma_result_wait();
}

template <bool IS_K, int W>
__device__ __forceinline__ void shared_rounds_any(uint32_t prec, const SharedSide &sd, uint32_t T, uint32_t b0,
                                                  uint32_t b1, float scale_log2, uint32_t r, bool active,
                                                  const SharedLane &ln, uint8_t (*lds)[W][kSharedBlockLds],
                                                  uint32_t &set, SharedState &st)
{
    switch (prec) {
    case kP16: shared_rounds<kP16, IS_K, W>(sd, T, b0, b1, scale_log2, r, active, ln, lds, set, st); break;
    case kInt8: shared_rounds<kInt8, IS_K, W>(sd, T, b0, b1, scale_log2, r, active, ln, lds, set, st); break;
    case kInt4: shared_rounds<kInt4, IS_K, W>(sd, T, b0, b1, scale_log2, r, active, ln, lds, set, st); break;
    case kE4M3: shared_rounds<kE4M3, IS_K, W>(sd, T, b0, b1, scale_log2, r, active, ln, lds, set, st); break;
    case kE5M2: shared_rounds<kE5M2, IS_K, W>(sd, T, b0, b1, scale_log2, r, active, ln, lds, set, st); break;
    default: shared_rounds<kGSE8, IS_K, W>(sd, T, b0, b1, scale_log2, r, active, ln, lds, set, st); break;
    }
}

__device__ __forceinline__ SharedSide shared_side(const uint8_t *first, uint32_t prec, uint32_t gsh, uint32_t h,
                                                  uint32_t nblk)
{
    SharedSide sd;
    const bool has_meta = prec == kInt4 || prec == kInt8;
    const uint32_t pay = prec == kInt4 ? 1024u : prec == kP16 ? 4096u : 2048u;
    sd.gsh = gsh;
    sd.meta_blk = has_meta ? 8192u >> gsh : 0u;
    // `first` points at the layer's tile of head 0; the heads' tile records follow one another
    sd.tile = (gbytes)first + (uint64_t)h * ((uint64_t)nblk * (pay + sd.meta_blk) + (prec == kGSE8 ? 16u : 0u));
    sd.meta = sd.tile + (uint64_t)nblk * pay;
    sd.tab = Gse8Tab{};
    if (prec == kGSE8)  // the tile's exponent range follows its payload
        sd.tab = gse8_tab(*(const uint32_t __attribute__((address_space(1))) *)(sd.tile + (uint64_t)nblk * 2048u));
    return sd;
}


// ---- the same with waves of two kinds -----------------------------------------------------------

// Orders LDS accesses of the whole workgroup across a barrier, and only those: global loads under
// way stay under way (__syncthreads() would wait for them).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr uint32_t kRoleDecoders = 4;                      // waves of a workgroup besides the scoring ones
constexpr uint32_t kRoleBlocks = 8;                       // layout blocks per round
// LDS of a pair of blocks: the keys of each block as 16 rows of 256 bytes, 16 bytes apart so that
// the lanes of a column reach different banks with constant offsets (an exclusive-or of row and
// octet does the same, but costs an instruction per access), then the values of both.
constexpr uint32_t kRoleKeyRow = 272, kRoleKeys = 16 * kRoleKeyRow, kRolePair = 2 * kRoleKeys + 8192;
constexpr uint32_t kRoleSet = kRoleBlocks / 2 * kRolePair;  // 66 KiB; two sets

struct RoleLane {
    uint32_t lane, c_, n_;  // MFMA coordinates: lane group, lane column
    uint32_t key;           // a scorer: where its K operands start in a block; a decoder: where plane 0 goes
};

// One block of one side: decode what the lane has fetched and leave it in the pair's buffer
// (`pair`, e = 0 / 1: first / second block of the pair).
template <uint32_t P, bool IS_K>
__device__ __forceinline__ void role_decode(const u32x4 *w, const u32x4 &m, const SharedSide &sd, uint32_t blk, uint32_t T,
                                            uint8_t *pair, int e, const RoleLane &ln)
{
    if (IS_K) {
        uint8_t *dst = pair + e * kRoleKeys + ln.key;  // token 4 j + c_, octet n_
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            *reinterpret_cast<u32x4 *>(dst + j * (4u * kRoleKeyRow)) =
                decode_octet<P>(plane_raw<P>(w, j), m[j], sd.tab);
        return;
    }
    // Operand pp of P V: value pp of the octet of each of the lane's four tokens; the pair's
    // second block fills the second half of the lane's 16 bytes.
    uint32_t t01[8], t23[8];  // value pp of tokens 4 * 0 + c_ and 4 * 1 + c_, of 4 * 2 + c_ and 4 * 3 + c_
    decode_octets_by_token<P>(plane_raw<P>(w, 0), plane_raw<P>(w, 1), m[0], m[1], sd.tab, t01);
    decode_octets_by_token<P>(plane_raw<P>(w, 2), plane_raw<P>(w, 3), m[2], m[3], sd.tab, t23);
    if (blk * 16u + 16u > T) {  // rows past the document's end
        uint32_t keep[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) keep[j] = blk * 16u + 4u * j + ln.c_ < T ? 0xFFFFu : 0u;
#pragma unroll
        for (int pp = 0; pp < 8; ++pp) {
            t01[pp] &= keep[0] | (keep[1] << 16);
            t23[pp] &= keep[2] | (keep[3] << 16);
        }
    }
    uint8_t *vdst = pair + 2u * kRoleKeys + ln.lane * 16u + e * 8u;
#pragma unroll
    for (int pp = 0; pp < 8; ++pp) *reinterpret_cast<u32x2 *>(vdst + pp * 1024u) = u32x2{t01[pp], t23[pp]};
}

// The rounds of one document for decoder r (0, 1) of one side: blocks 4 r .. 4 r + 3 of every
// round.  A block's words of the next round are requested as soon as this round's are decoded and
// stay under way across the barrier.
template <uint32_t P, bool IS_K>
__device__ __forceinline__ void role_decode_rounds(const SharedSide &sd, uint32_t T, uint32_t b0, uint32_t b1, uint32_t r,
                                                   const RoleLane &ln, uint8_t *lds, uint32_t &set)
{
    typedef Fmt<P> F;
    u32x4 w[4][F::kWords], m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) m[i] = u32x4{0u, 0u, 0u, 0u};
    // Issued whether or not the block exists (a block past the end is replaced by the last one), in
    // the order the blocks are decoded in, here and in the loop: only then does a wait for one
    // block leave the others' loads under way.
    auto fetch = [&](int i, uint32_t b) {
        b = b < b1 ? b : b1 - 1u;
#pragma unroll
        for (uint32_t a = 0; a < F::kWords; ++a)
            w[i][a] = ldg16(sd.tile + ((uint64_t)b * F::kPayload + a * 1024u + ln.lane * 16u));
        if (F::kMeta) m[i] = ldg16(sd.meta + ((uint64_t)b * sd.meta_blk + ((ln.lane * 8u) >> sd.gsh) * 16u));
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) fetch(i, b0 + 4u * r + i);
    uint32_t rb = b0;
    for (; rb + kRoleBlocks <= b1; rb += kRoleBlocks) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t blk = rb + 4u * r + i;
            role_decode<P, IS_K>(w[i], m[i], sd, blk, T, lds + set * kRoleSet + (2u * r + i / 2) * kRolePair, i & 1, ln);
            fetch(i, blk + kRoleBlocks);
        }
        lds_barrier();
        set ^= 1u;
    }
    if (rb >= b1) return;
    // The document's (or run's) last round, if it is not a whole one.  A block that does not exist is left
    // out: the keys' scores are replaced whatever the buffer holds, and only if its partner exists the
    // values, which the MFMAs then take with weight zero, have to be zeros.  Decoding absent blocks as well cost
    // lists of short documents more than the eight-wave kernel took that decoded in turn (30 documents of 16
    // tokens in the paper's formats, 64 query tokens, 16 requests: 72.6 us per layer, 66.7 then, 49.8 now);
    // leaving them out by a branch in the loop above cost whole rounds 1 %.
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t blk = rb + 4u * r + i;
        uint8_t *pair = lds + set * kRoleSet + (2u * r + i / 2) * kRolePair;
        if (blk < b1) role_decode<P, IS_K>(w[i], m[i], sd, blk, T, pair, i & 1, ln);
        else if (!IS_K && (i & 1) && blk - 1u < b1) {
#pragma unroll
            for (int pp = 0; pp < 8; ++pp)
                *reinterpret_cast<u32x2 *>(pair + 2u * kRoleKeys + pp * 1024u + ln.lane * 16u + 8u) = u32x2{0u, 0u};
        }
    }
    lds_barrier();
    set ^= 1u;
}

template <bool IS_K>
__device__ __forceinline__ void role_decode_any(uint32_t prec, const SharedSide &sd, uint32_t T, uint32_t b0, uint32_t b1,
                                                uint32_t r, const RoleLane &ln, uint8_t *lds, uint32_t &set)
{
    switch (prec) {
    case kP16: role_decode_rounds<kP16, IS_K>(sd, T, b0, b1, r, ln, lds, set); break;
    case kInt8: role_decode_rounds<kInt8, IS_K>(sd, T, b0, b1, r, ln, lds, set); break;
    case kInt4: role_decode_rounds<kInt4, IS_K>(sd, T, b0, b1, r, ln, lds, set); break;
    case kE4M3: role_decode_rounds<kE4M3, IS_K>(sd, T, b0, b1, r, ln, lds, set); break;
    case kE5M2: role_decode_rounds<kE5M2, IS_K>(sd, T, b0, b1, r, ln, lds, set); break;
    default: role_decode_rounds<kGSE8, IS_K>(sd, T, b0, b1, r, ln, lds, set); break;
    }
}

// The wave's queries as the B operand of S^T = K Q^T: lane (c_, n_) holds, for MFMA y, dims
// 32 c_ + 8 y .. + 7 of query row n_ of the tile (zero rows beyond M); nothing accumulated yet.
__device__ __forceinline__ void shared_load_queries(const K6Run &c, const AttendHdr &hdr, uint32_t h, uint32_t tile0,
                                                    uint32_t M, uint32_t c_, uint32_t n_, SharedState &st)
{
    const uint32_t G = hdr.n_q_heads / hdr.n_kv_heads;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const uint32_t row = (tile0 + mt) * 16u + n_;
        u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int y = 0; y < 4; ++y) st.qb[mt][y] = __builtin_bit_cast(bf16x8, z);
        if (row < M) {
            const uint32_t qt = row / G, gq = row - qt * G;
            gbytes qp = (gbytes)c.q + ((uint64_t)(qt * hdr.n_q_heads + h * G + gq) * 128u + 32u * c_) * 2u;
#pragma unroll
            for (int y = 0; y < 4; ++y) st.qb[mt][y] = __builtin_bit_cast(bf16x8, ldg16(qp + 16 * y));
        }
        st.m_run[mt] = neg_inf();
        st.l_run[mt] = st.r_run[mt] = 0.0f;
#pragma unroll
        for (int pp = 0; pp < 8; ++pp) st.O[mt][pp] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// The wave's results, straight from its registers: lane (c_, n_) holds rows 4 c_ + jj, dims
// 8 n_ + pp of each tile.
__device__ __forceinline__ void shared_write_results(const K6Run &c, const AttendHdr &hdr, uint32_t h, uint32_t tile0,
                                                     uint32_t M, uint32_t c_, uint32_t n_, SharedState &st)
{
    const uint32_t G = hdr.n_q_heads / hdr.n_kv_heads, n_mt = (M + 15u) >> 4;
    uint32_t final = c.final;
    pin(final);
    const float *lse_ptr = c.lse;
    pin(lse_ptr);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const uint32_t tile = tile0 + mt;
        if (tile >= n_mt) continue;
        const float l_tot = sum_over_lane_groups(st.l_run[mt]), r_tot = sum_over_lane_groups(st.r_run[mt]);
        if (final) {
            // The run is everything the request attends to: what the merge would do with its one
            // record is done here.  l_tot of row n_ is in every lane of column n_; the rows this
            // lane holds are 4 c_ + jj.
            gfloats out = (gfloats)c.part;
#pragma unroll
            for (uint32_t jj = 0; jj < 4; ++jj) {
                const uint32_t row = 4u * c_ + jj, mrow = tile * 16u + row;
                const float r_row = __shfl(r_tot, (int)row);
                if (mrow >= M) continue;
                const uint32_t qt = mrow / G, gq = mrow - qt * G;
                f32x4 __attribute__((address_space(1))) *dst = (f32x4 __attribute__((address_space(1))) *)(
                    out + ((uint64_t)qt * hdr.n_q_heads + h * G + gq) * 128u + 8u * n_);
                f32x4 w0, w1;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    w0[e] = r_row > 0.0f ? st.O[mt][e][jj] / r_row : 0.0f;
                    w1[e] = r_row > 0.0f ? st.O[mt][4 + e][jj] / r_row : 0.0f;
                }
                dst[0] = w0;
                dst[1] = w1;
            }
            const uint32_t mrow = tile * 16u + n_;
            if (c_ == 0 && lse_ptr && mrow < M) {
                const uint32_t qt = mrow / G, gq = mrow - qt * G;
                ((gfloats)lse_ptr)[(uint64_t)qt * hdr.n_q_heads + h * G + gq] =
                    l_tot > 0.0f ? (st.m_run[mt] + __builtin_log2f(l_tot)) * 0.69314718055994531f : neg_inf();
            }
            continue;
        }
        gfloats rec = (gfloats)c.part + ((uint64_t)h * n_mt + tile) * kAttendRecFloats;
#pragma unroll
        for (uint32_t jj = 0; jj < 4; ++jj) {
            const uint32_t row = 4u * c_ + jj;
            const float fit = __shfl(r_tot > 0.0f ? l_tot / r_tot : 0.0f, (int)row);  // the merge divides by l
            if (tile * 16u + row >= M) continue;  // no query in this row: the merge never reads it
            f32x4 __attribute__((address_space(1))) *dst =
                (f32x4 __attribute__((address_space(1))) *)(rec + row * 128u + 8u * n_);
            dst[0] = f32x4{st.O[mt][0][jj], st.O[mt][1][jj], st.O[mt][2][jj], st.O[mt][3][jj]} * fit;
            dst[1] = f32x4{st.O[mt][4][jj], st.O[mt][5][jj], st.O[mt][6][jj], st.O[mt][7][jj]} * fit;
        }
        if (c_ == 0) {
            rec[2048 + n_] = st.m_run[mt];
            rec[2048 + 16 + n_] = l_tot;
        }
    }
}

// How large the sum of a lane's eight weights of a pair and tile may get before the row's reference
// maximum is brought up to date: no weight exceeds 2^kLazyMaxSlack.
constexpr float kRoleMaxSum = 256.0f;
// The reference of a row that has none yet: the lowest number there is, which a row's first pair moves
// (its weights overflow) unless its scores lie there themselves, and then their weights are right as they
// are.  Finite: a masked score (-inf) minus it is still -inf.
constexpr float kRoleNoRef = -__FLT_MAX__;
constexpr int kRoleEarlyV = 6;  // V operands read before the softmax; the last two would not fit the registers

// The weights of one tile and pair relative to the row's reference, and their sum in this lane.
__device__ __forceinline__ float role_weights(const f32x4 &s0, const f32x4 &s1, float scale_log2, float ref, bf16x8 &P8)
{
    float pr[8];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        pr[jj] = __builtin_amdgcn_exp2f(__builtin_fmaf(s0[jj], scale_log2, -ref));
        pr[4 + jj] = __builtin_amdgcn_exp2f(__builtin_fmaf(s1[jj], scale_log2, -ref));
    }
    const u32x4 pk = {pack_bf16(pr[0], pr[1]), pack_bf16(pr[2], pr[3]), pack_bf16(pr[4], pr[5]), pack_bf16(pr[6], pr[7])};
    P8 = __builtin_bit_cast(bf16x8, pk);
    return ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
}

// What the rounds before this one came to, for a scorer with registers to spare (S = 4).  A round's rows are scaled by
// what rounding did to that round's weights (their sum before over their sum after) when they are added here, so that a
// long run is about as exact as runs of one round each, whose records the merge adds up the same way.  Error against 64 bits
// of 8 requests x 4 x 512 tokens at 12 query tokens: runs of 8 blocks 0.44e-3, of 32 with one factor a run 0.76e-3, with one a
// round 0.48e-3.  Over the 28 of 70 calls (1 to 32 requests, 3 to 402 query tokens) that S = 4 took over, 0.94 times the error
// they had, 0.55 to 1.12.
struct RoleTotal {
    f32x4 O[2][8];
    float l_run[2];
};

// Adds a round to the total; the next one's first products overwrite st.O.  The factors come first, while the round's
// last MFMAs run.  (Sums below the smallest normal number have no reciprocal; their rows' factor is 1.)
__device__ __forceinline__ void role_add_round(const RoleLane &ln, SharedState &st, RoleTotal &tot)
{
    const uint32_t c_ = fresh(ln.lane) >> 4;
    float f[2][4];  // of output rows 4 c_ + jj
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const float l = sum_over_lane_groups(st.l_run[mt]), r = sum_over_lane_groups(st.r_run[mt]);
        const float fit = r >= __FLT_MIN__ * 4.0f ? l * __builtin_amdgcn_rcpf(r) : 1.0f;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) f[mt][jj] = __shfl(fit, (int)(4u * c_ + jj));
        tot.l_run[mt] += st.l_run[mt];
        st.l_run[mt] = st.r_run[mt] = 0.0f;
    }
    mfma_result_wait();
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int pp = 0; pp < 8; ++pp)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) tot.O[mt][pp][jj] = __builtin_fmaf(st.O[mt][pp][jj], f[mt][jj], tot.O[mt][pp][jj]);
}

// A round of a scorer: its two tiles against `nb` blocks, two (a pair) at a time.  The LDS reads are
// issued ahead of what hides them: the keys of a pair's first block before the P V MFMAs of the
// pair before, those of the second before the first's MFMAs, the values before the softmax.
// The reference maximum is looked at after the fact: weights are formed with the reference there
// is, and only if their sum says that one of them may be too large (or there is no reference yet)
// the row maxima are taken, what is accumulated is rescaled and the weights are formed again.
// That saves the maxima of every pair, a fifth of the softmax's instructions.
template <bool TOTAL>
__device__ __forceinline__ void role_score_round(const uint8_t *base, uint32_t rb, uint32_t nb, uint32_t end,
                                                 float scale_log2, const RoleLane &ln, SharedState &st, RoleTotal &tot)
{
    u32x4 ka0[4], ka1[4];
    const uint8_t *key = base + ln.key;
#pragma unroll
    for (uint32_t y = 0; y < 4; ++y) ka0[y] = *reinterpret_cast<const u32x4 *>(key + 16u * y);
#pragma unroll 1
    for (uint32_t pr = 0; 2u * pr < nb; ++pr) {
        f32x4 S[2][2];
        bf16x8 P8[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) S[e][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        key = base + pr * kRolePair + fresh(ln.key);
#pragma unroll
        for (uint32_t y = 0; y < 4; ++y) ka1[y] = *reinterpret_cast<const u32x4 *>(key + kRoleKeys + 16u * y);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                S[0][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka0[y]), st.qb[mt][y], S[0][mt], 0, 0, 0);
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
                S[1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka1[y]), st.qb[mt][y], S[1][mt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        u32x4 vq[8];
        const uint8_t *val = base + pr * kRolePair + 2u * kRoleKeys + fresh(ln.lane) * 16u;
#pragma unroll
        for (int pp = 0; pp < kRoleEarlyV; ++pp) vq[pp] = *reinterpret_cast<const u32x4 *>(val + pp * 1024u);
        mfma_result_wait();
        const uint32_t b = rb + 2u * pr;
        if (b * 16u + 32u > end) {  // a ragged last block, or a last block without a partner
            const uint32_t tok = b * 16u + (fresh(ln.lane) >> 4);
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
                        if (tok + 16u * e + 4u * jj >= end) S[e][mt][jj] = neg_inf();
        }
        float sum[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            sum[mt] = role_weights(S[0][mt], S[1][mt], scale_log2, st.m_run[mt], P8[mt]);
            __builtin_amdgcn_sched_barrier(0);  // one tile after the other: registers are short
        }
        if (__builtin_amdgcn_ballot_w64(sum[0] > kRoleMaxSum || sum[1] > kRoleMaxSum) != 0ull) {
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                const float a = __builtin_fmaxf(__builtin_fmaxf(S[0][mt][0], S[0][mt][1]), __builtin_fmaxf(S[0][mt][2], S[0][mt][3]));
                const float bb = __builtin_fmaxf(__builtin_fmaxf(S[1][mt][0], S[1][mt][1]), __builtin_fmaxf(S[1][mt][2], S[1][mt][3]));
                const float m_new = __builtin_fmaxf(st.m_run[mt], max_over_lane_groups(__builtin_fmaxf(a, bb) * scale_log2) + kLazyMaxLift);
                const float alpha = __builtin_amdgcn_exp2f(st.m_run[mt] - m_new);  // 0 where there was no reference, 1 if nothing moved
                st.l_run[mt] *= alpha;
                st.r_run[mt] *= alpha;
                if (TOTAL) tot.l_run[mt] *= alpha;
                st.m_run[mt] = m_new;
                const uint32_t c_ = fresh(ln.lane) >> 4;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const float ar = __shfl(alpha, (int)(4u * c_ + jj));  // factor of output row 4 c_ + jj
#pragma unroll
                    for (int pp = 0; pp < 8; ++pp) {
                        st.O[mt][pp][jj] *= ar;
                        if (TOTAL) tot.O[mt][pp][jj] *= ar;
                    }
                }
                sum[mt] = role_weights(S[0][mt], S[1][mt], scale_log2, m_new, P8[mt]);
            }
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            st.l_run[mt] += sum[mt];
            st.r_run[mt] = add_weights8(P8[mt], st.r_run[mt]);
        }
        __builtin_amdgcn_sched_barrier(0);
        val = base + pr * kRolePair + 2u * kRoleKeys + fresh(ln.lane) * 16u;
#pragma unroll
        for (int pp = kRoleEarlyV; pp < 8; ++pp) vq[pp] = *reinterpret_cast<const u32x4 *>(val + pp * 1024u);
        key = base + (2u * pr + 2u < nb ? pr + 1u : pr) * kRolePair + fresh(ln.key);
#pragma unroll
        for (uint32_t y = 0; y < 4; ++y) ka0[y] = *reinterpret_cast<const u32x4 *>(key + 16u * y);
        __builtin_amdgcn_sched_barrier(0);
        if (TOTAL && pr == 0u) {
#pragma unroll
            for (int pp = 0; pp < 8; ++pp) {
                const bf16x8 v = __builtin_bit_cast(bf16x8, vq[pp]);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    st.O[mt][pp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P8[mt], v, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int pp = 0; pp < 8; ++pp) {
                const bf16x8 v = __builtin_bit_cast(bf16x8, vq[pp]);
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
                    st.O[mt][pp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(P8[mt], v, st.O[mt][pp], 0, 0, 0);
            }
        }
    }
    if (TOTAL) role_add_round(ln, st, tot);
}

}  // namespace

// W = 2 or 4 waves, half of them decoding keys and half values; two waves per SIMD keep 256 registers
// each (two tiles of output, their queries, the raw words of two blocks).
// Bound: instructions.  Of 4,080 clocks a round (W = 2, 16 query tokens, 32 requests x 5,120 tokens) a wave decodes 1,290 and
// scores 1,970, waits 210 for its loads and 320 at the barrier; another wave on its SIMD does the same.  (16-bit documents:
// 2,480 of 6,300 wait for loads.)
// W = 4 is for calls of five to eight tiles whose requests leave k6_attend_roles<4> with a third of its compute units idle or
// a round nearly empty; two of its workgroups share a compute unit.  us a layer, k6_attend_roles<4> / this: 25 requests of 11 x
// 1,024 tokens at 21 query tokens 254 / 213, 12 of 11 x 129 at 13 38.7 / 33.1; 27 of 2 x 256 at 18 23.0 / 26.1.
template <int W, class P>
__global__ void __launch_bounds__(64 * W, 2) k6_attend_shared(const P p)
{
    // two sets of W block buffers
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_bytes[];
    uint8_t (*lds)[W][kSharedBlockLds] = reinterpret_cast<uint8_t (*)[W][kSharedBlockLds]>(lds_bytes);
    K6Run c = p.run[blockIdx.y];
    AttendHdr hdr = {p.n_kv_heads, p.n_q_heads, p.layer, p.scale_log2};
    pin(c.k);
    pin(c.v);
    pin(c.q);
    pin(c.part);
    pin(c.n_tokens);
    pin(c.info);
    pin(c.n_q);
    pin(hdr.n_kv_heads);
    pin(hdr.n_q_heads);
    pin(hdr.scale_log2);
    uint32_t run = c.n_docs, more = c.more;  // the run's documents: this one, then descriptors more, more + 1, ..
    uint32_t first_block = c.first_block, end_block = c.end_block;  // where the run starts in its first and ends in its last
    pin(run);
    pin(more);
    pin(first_block);
    pin(end_block);
    const uint32_t H = hdr.n_kv_heads, G = hdr.n_q_heads / H, M = c.n_q * G;
    const uint32_t n_mt = (M + 15u) >> 4;
    const uint32_t n_mtg = (n_mt + 2u * W - 1u) / (2u * W);
    const uint32_t u = blockIdx.x;
    if (u >= H * n_mtg) return;  // the grid is as wide as the widest run
    const uint32_t mtg = u % n_mtg, h = u / n_mtg;

    SharedLane ln;
    ln.lane = threadIdx.x & 63u;
    ln.c_ = ln.lane >> 4;
    ln.n_ = ln.lane & 15u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t tile0 = (mtg * W + wave) * 2u;  // this wave's tiles: tile0, tile0 + 1
    const bool active = tile0 < n_mt;              // a wave without a tile still decodes
    const bool is_k = wave < (uint32_t)W / 2u;
    const uint32_t r = is_k ? wave : wave - (uint32_t)W / 2u;
    // where this lane reads its K operands: the token of MFMA row n_ is 4 (n_ % 4) + n_ / 4, so
    // that score register jj of lane group c_ belongs to token 4 jj + c_, the token whose values
    // the lane group's plane jj holds
    {
        const uint32_t tau = 4u * (ln.n_ & 3u) + (ln.n_ >> 2);
        ln.k_rd = tau * 256u + (((4u * ln.c_) ^ tau) & 15u) * 16u;  // octet 4 c_ + y of token tau: slot (4 c_ ^ tau) ^ y
        ln.k_wr = ln.c_ * 256u + ((ln.n_ ^ ln.c_) & 15u) * 16u;     // n_ ^ (4 j + c_) = (n_ ^ c_) ^ 4 j
    }

    SharedState st;
    shared_load_queries(c, hdr, h, tile0, M, ln.c_, ln.n_, st);

    uint32_t set = 0;
    for (uint32_t d = 0; d < run; ++d) {
        // ---- the document: descriptor d of the run (its first is already here)
        const uint8_t *dk = c.k, *dv = c.v;
        uint32_t T = c.n_tokens, dinfo = c.info;
        if (d) {
            const K6Doc &cd = p.doc[more + d - 1u];
            dk = cd.k;
            dv = cd.v;
            T = cd.n_tokens;
            dinfo = cd.info;
        }
        const uint32_t nblk = (T + 15u) >> 4;
        const uint32_t b0 = d ? 0u : first_block;
        const uint32_t b1 = d + 1u == run ? end_block : nblk;
        if (b0 >= b1) continue;  // cannot happen with a checked launch
        if (is_k) {
            const uint32_t prec = dinfo & 0xFu;
            const SharedSide sd = shared_side(dk, prec, (dinfo >> 4) & 0xFu, h, nblk);
            shared_rounds_any<true, W>(prec, sd, T, b0, b1, hdr.scale_log2, r, active, ln, lds, set, st);
        } else {
            const uint32_t prec = (dinfo >> 8) & 0xFu;
            const SharedSide sd = shared_side(dv, prec, (dinfo >> 12) & 0xFu, h, nblk);
            shared_rounds_any<false, W>(prec, sd, T, b0, b1, hdr.scale_log2, r, active, ln, lds, set, st);
        }
    }

    // ---- the wave's results, straight from its registers: lane (c_, n_) holds rows
    // 4 c_ + jj, dims 8 n_ + pp of each tile
    if (!active) return;
    shared_write_results(c, hdr, h, tile0, M, ln.c_, ln.n_, st);
}

// S = 4 or 8 waves score, two query tiles each (up to 128 or 256 query rows a workgroup), four decode: two the
// keys and two the values of a round of eight blocks, for the round after the one that is being
// scored.  One barrier per round, for LDS only.  With S = 8 three waves per SIMD (168 registers): two scorers,
// whose registers hold no raw words, and a decoder that fills their gaps.  With S = 4 one scorer and one decoder per
// SIMD: a round takes 2.2 us instead of 3.1 to 4.3, so that a call with compute units to spare, or with no more than
// eight tiles a request, is done sooner.  Without the rounds' factors (role_add_round, a tenth of the time) a scorer takes
// 3,600 clocks a round and a decoder 3,800 to 4,000; eight decoders, loads two rounds ahead and 32x32x16 MFMAs over two
// pairs at a time all measured the same or worse.
// S = 4 against what took these calls before, us a layer: one request of 8 x 512 tokens, 64 query tokens (S = 8): 25.8 -> 22.0;
// two of 4 x 512: 25.5 -> 21.7; one of 8 x 1,024, 16 query tokens (k6_attend_shared): 26.3 -> 21.2; 32 requests x 5,120 tokens,
// 32 query tokens (k6_attend_shared<4>): 146 -> 142.
//
// S = 8 is bound by the SIMDs' instruction slots and the clock.  32 requests x 5,120 tokens x 64 query tokens
// x 32 heads (172 GFLOP a layer, one workgroup per CU, one run per request): 215-227 us with eight waves
// that decoded and scored in turn, 182-192 now = 907-944 TFLOP/s, against 1,390 of a large matrix
// product.  Of 383,000 clocks the matrix cores work 164,000 and vector instructions take about
// 160,000, which overlap with them only in part (two waves of 16 MFMAs and 64 fused multiply-adds
// each take 355 ns where the MFMAs alone take 273); under this load the card runs at 2.07 GHz.  What gave how
// much: the split into two kinds of waves 10 %; operands read ahead of what hides them 2 %; the maxima
// after the fact, keys without address arithmetic, codes without conversions and values rounded
// straight into operands 4 %; the reference lifted above the maximum 3 %; loads issued in the order they are
// decoded in (before, the compiler waited for all of them at the top of the loop) 2 %.
// The tile groups of a head read the same blocks.  Numbered one after the other they are dealt to the eight XCDs, each
// of which fetches the blocks into an L2 of its own, and the last group of a head, which has fewer tiles, falls on the same XCDs
// each time.  With the heads first (heads_first) the groups of a head meet in one L2 if there are eight heads, and the
// shorter groups are spread.  us for two layers, without / with, 8 KV heads: two requests of 16 x 1,024 tokens in 16 bits, 256 query
// tokens, 64 query heads 550 / 516; eight of 10 x 512 and 200 at 90 to 256 486 / 454; three of 16 documents of up to 1,024 at 96 to
// 201 418 / 404; eight of 4 x 512 at 100 147 / 142.  By KV heads, calls of requests of one kind in runs of 96 blocks and more, mean
// (least to most) of the ratio: 2 1.00 (0.98-1.02), 3 0.96 (0.94-0.99), 4 0.98 (0.96-1.01), 5 0.97 (0.94-1.01), 6 0.99 (0.96-1.01),
// 7 0.98 (0.93-1.01), 8 0.95 (0.91-0.99), 10 0.97 (0.95-0.99), 12 0.98 (0.94-1.00), 16 0.96 (0.91-0.99).  Calls of shorter runs only may
// lose by it, whose groups all wait for the same lines at their start: 16 to 40 blocks a run 0.92 to 1.11.  Next to longer runs
// shorter ones gain too, so it is the call's longest run that decides: four requests of 1,790 tokens at 100 and 30 of 2 x 512 at 200
// 367 / 341 (366 with the long ones alone ordered so); 170 random calls of long and short runs 0.98 (0.85-1.05; above 1.02 with two
// and four heads only).
// Scoring with 32x32x16
// MFMAs took 6 % fewer clocks at a clock 5 % lower, 186.5 -> 189.5 us, as at a power limit.
template <int S, class P>
__global__ void __launch_bounds__(64 * (S + kRoleDecoders), (S + kRoleDecoders) / 4) k6_attend_roles(const P p)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_bytes[];
    K6Run c = p.run[blockIdx.y];
    AttendHdr hdr = {p.n_kv_heads, p.n_q_heads, p.layer, p.scale_log2};
    pin(c.k);
    pin(c.v);
    pin(c.q);
    pin(c.part);
    pin(c.n_tokens);
    pin(c.info);
    pin(c.n_q);
    pin(hdr.n_kv_heads);
    pin(hdr.n_q_heads);
    pin(hdr.scale_log2);
    uint32_t run = c.n_docs, more = c.more;  // the run's documents: this one, then descriptors more, more + 1, ..
    uint32_t first_block = c.first_block, end_block = c.end_block;
    pin(run);
    pin(more);
    pin(first_block);
    pin(end_block);
    const uint32_t H = hdr.n_kv_heads, G = hdr.n_q_heads / H, M = c.n_q * G;
    const uint32_t n_mt = (M + 15u) >> 4;
    const uint32_t n_mtg = (n_mt + 2u * (uint32_t)S - 1u) / (2u * (uint32_t)S);
    const uint32_t u = blockIdx.x;
    if (u >= H * n_mtg) return;  // the grid is as wide as the widest run
    const bool heads_first = S == 8 && p.heads_first;
    const uint32_t h = heads_first ? u % H : u / n_mtg, mtg = heads_first ? u / H : u % n_mtg;

    RoleLane ln;
    ln.lane = threadIdx.x & 63u;
    ln.c_ = ln.lane >> 4;
    ln.n_ = ln.lane & 15u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t set = 0;

    if (wave >= (uint32_t)S) {
        ln.key = ln.c_ * kRoleKeyRow + ln.n_ * 16u;
        const uint32_t dec = wave - (uint32_t)S;
        const bool is_k = dec < kRoleDecoders / 2u;
        const uint32_t r = dec & 1u;
        for (uint32_t d = 0; d < run; ++d) {
            const uint8_t *dp = is_k ? c.k : c.v;
            uint32_t T = c.n_tokens, info = is_k ? c.info : c.info >> 8;
            if (d) {
                const K6Doc &cd = p.doc[more + d - 1u];
                dp = is_k ? cd.k : cd.v;
                T = cd.n_tokens;
                info = is_k ? cd.info : cd.info >> 8;
            }
            const uint32_t nblk = (T + 15u) >> 4;
            const uint32_t b0 = d ? 0u : first_block;
            const uint32_t b1 = d + 1u == run ? end_block : nblk;
            if (b0 >= b1) continue;  // cannot happen with a checked launch
            const uint32_t prec = info & 0xFu;
            const SharedSide sd = shared_side(dp, prec, (info >> 4) & 0xFu, h, nblk);
            if (is_k) role_decode_any<true>(prec, sd, T, b0, b1, r, ln, lds_bytes, set);
            else role_decode_any<false>(prec, sd, T, b0, b1, r, ln, lds_bytes, set);
        }
        return;
    }

    const uint32_t tile0 = (mtg * (uint32_t)S + wave) * 2u;  // this wave's tiles: tile0, tile0 + 1
    const bool active = tile0 < n_mt;
    // the token of MFMA row n_ is 4 (n_ % 4) + n_ / 4, so that score register jj of lane group c_
    // belongs to token 4 jj + c_, the token whose values the lane group's plane jj holds
    ln.key = (4u * (ln.n_ & 3u) + (ln.n_ >> 2)) * kRoleKeyRow + ln.c_ * 64u;
    SharedState st;
    shared_load_queries(c, hdr, h, tile0, M, ln.lane >> 4, ln.lane & 15u, st);
    st.m_run[0] = st.m_run[1] = kRoleNoRef;
    RoleTotal tot = {};
    for (uint32_t d = 0; d < run; ++d) {
        const uint32_t T = d ? p.doc[more + d - 1u].n_tokens : c.n_tokens;
        const uint32_t nblk = (T + 15u) >> 4;
        const uint32_t b0 = d ? 0u : first_block;
        const uint32_t b1 = d + 1u == run ? end_block : nblk;
        if (b0 >= b1) continue;
        const uint32_t end = b1 * 16u < T ? b1 * 16u : T;  // the first token that does not count
        for (uint32_t rb = b0; rb < b1; rb += kRoleBlocks) {
            lds_barrier();
            if (active) {
                const uint32_t nb = b1 - rb < kRoleBlocks ? b1 - rb : kRoleBlocks;
                role_score_round<S == 4>(lds_bytes + set * kRoleSet, rb, nb, end, hdr.scale_log2, ln, st, tot);
            }
            set ^= 1u;
        }
        mfma_result_wait();
    }
    if (!active) return;
    if (S == 4) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            st.l_run[mt] = st.r_run[mt] = tot.l_run[mt];  // rounding is accounted for
#pragma unroll
            for (int pp = 0; pp < 8; ++pp) st.O[mt][pp] = tot.O[mt][pp];
        }
    }
    const uint32_t lane_ = fresh(ln.lane);
    shared_write_results(c, hdr, h, tile0, M, lane_ >> 4, lane_ & 15u, st);
}

// k6_attend_roles takes 132 KiB of LDS per workgroup; more than 64 KiB has to be asked for
// once per device.  Called when a context is created on the device (not from inside a launch
// that a caller may be capturing into a graph) and, as a fallback, before the first such launch.
hipError_t prepare_k6_shared()
{
    static std::atomic<uint64_t> asked{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (asked.load(std::memory_order_acquire) >> dev & 1u) return hipSuccess;
    for (const void *k : {reinterpret_cast<const void *>(k6_attend_roles<4, K6Params>), reinterpret_cast<const void *>(k6_attend_roles<8, K6Params>),
                          reinterpret_cast<const void *>(k6_attend_roles<4, K6ParamsFew>), reinterpret_cast<const void *>(k6_attend_roles<8, K6ParamsFew>)}) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(2u * kRoleSet));
        if (e != hipSuccess) return e;
    }
    asked.fetch_or(1ull << dev, std::memory_order_release);
    return hipSuccess;
}

hipError_t launch_k6_shared(K6Params &p, SharedForm form, hipStream_t stream, bool check_only)
{
    if (p.n_runs == 0) return hipSuccess;
    if (form > SharedForm::kRoles8) return hipErrorInvalidValue;
    const uint32_t waves = scoring_waves(form);
    uint32_t max_mt = 1;
    bool narrow = true;
    hipError_t e = check_k6_args(p, &max_mt, &narrow);
    if (e != hipSuccess) return e;
    const uint64_t width = (uint64_t)p.n_kv_heads * ((max_mt + 2u * waves - 1u) / (2u * waves));
    if (width > 0x7FFFFFFFull) return hipErrorInvalidValue;
    p.mtw = 2;
    if (check_only) return hipSuccess;
    dim3 grid((uint32_t)width, p.n_runs);
    if (form == SharedForm::kRoles4 || form == SharedForm::kRoles8) {
        e = prepare_k6_shared();  // done at ha_rag_create; a no-op from then on
        if (e != hipSuccess) return e;
    }
    return launch_few_or_all(p, [&](auto &q) {
        typedef std::remove_reference_t<decltype(q)> P;
        const dim3 roles(64u * (waves + kRoleDecoders));
        switch (form) {
        case SharedForm::kShared2: return launch_args(k6_attend_shared<2, P>, grid, dim3(128), 2u * 2u * kSharedBlockLds, stream, q);
        case SharedForm::kShared4: return launch_args(k6_attend_shared<4, P>, grid, dim3(256), 2u * 4u * kSharedBlockLds, stream, q);
        case SharedForm::kRoles4: return launch_args(k6_attend_roles<4, P>, grid, roles, 2u * kRoleSet, stream, q);
        default: return launch_args(k6_attend_roles<8, P>, grid, roles, 2u * kRoleSet, stream, q);
        }
    });
}

}  // namespace ha_rag
