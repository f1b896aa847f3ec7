// K side of decode attention as device functions: Rule 1 level per K column, and the streaming q.K~ pass
// over one tile of tokens.
// "Quantization of K-Cache": from q and K_colmax estimate the magnitude of the 128 addends of one logit,
// align them to the coarsest one (Rule 1), read each column of K at the bit width its addend needs.
#pragma once
#include <type_traits>

#include "akv_common.h"

namespace akv {

// q as binary32 in LDS, for the kernels that read it there (rows of neighbouring heads four banks apart)
template <int G, bool USED> struct KSharedQ {};
template <int G> struct KSharedQ<G, true> { alignas(16) float q[G][kD + 4]; };
// LDS of the K side of one (sequence, KV head).  In groups of eight k_tile multiplies on the matrix cores, which take q from LDS.
template <int G>
struct KShared : KSharedQ<G, G == 8> {
    static constexpr bool kNew = false;
    static constexpr int kHeads = G;
    static constexpr bool kMatrix = G == 8;
    int emax[2][G];                     // largest addend exponent per query head, of the columns of wave 0 / wave 1
    uint64_t need_mid[2], need_lo[2];   // bit d%64 of word d/64: column d is read at level >= 1 / = 2
    uint16_t kread[kD];                 // fused append: the new token's K row as it is read at the column levels
};
// ... of a kernel that appends a token itself
template <int G>
struct KSharedNew : KShared<G>, KSharedQ<G, true> {
    static_assert(G < 8, "one q");
    static constexpr bool kNew = true;
    float knew[kD];                     // the new token's K row as it will be read at the column levels
    float new_logit[G];                 // q . knew, accumulated in channel order
};

// Rule 1 for the 128 columns of (b, h), in two steps so that a caller can put other loads in flight between the
// issue of the loads here and their first use.  Both are called by every thread of a workgroup of at least 128
// threads (the second contains barriers); afterwards ks holds the level masks.
// k_new_bits: fp16 bits of channel tid of a token that is being appended in the same kernel, else -1: K_colmax then counts that token, and
// its row, read at the column levels, is left in ks.kread for k_tile (ks a KSharedNew: with q as fp32 in ks.knew and ks.q for new_token_logit()).
template <int G>
struct KLevelsIn {
    uint32_t cm;         // K_colmax of channel tid as stored
    uint32_t qbits[G];   // fp16 bits of q[g][tid]
};

template <int G>
__device__ __forceinline__ void k_levels_load(const DecodeArgs& a, int b, int h, KLevelsIn<G>& in)
{
    const int tid = threadIdx.x;
    const size_t bh = size_t(b) * a.s.Hkv + h;
    in.cm = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) in.qbits[g] = 0;
    if (tid < kD) {
        in.cm = a.colmax[bh * kD + tid];
#pragma unroll
        for (int g = 0; g < G; ++g) in.qbits[g] = a.q[(size_t(b) * a.s.Hq + size_t(h) * G + g) * kD + tid];
    }
}

// Returns the K_colmax of channel tid (tid < 128) that the levels used.
// stat_len: tokens of the sequence the levels apply to (for the counters of akv_stats; used with export_levels).
template <int G, typename KS>
__device__ __forceinline__ uint32_t k_levels_finish(const DecodeArgs& a, int b, int h, KS& ks, bool export_levels,
                                                    int k_new_bits, const KLevelsIn<G>& in, int stat_len)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t bh = size_t(b) * a.s.Hkv + h;
    float P[G];
    uint32_t colmax_used = 0;
    if (tid < kD) {   // waves 0 and 1 (wave-uniform): channel tid
        uint32_t cm = in.cm;
        if (k_new_bits >= 0) cm = max(cm, uint32_t(k_new_bits) & 0x7FFFu);
        colmax_used = cm;
        cm = cm < 0x0400u ? 0x0400u : cm;               // below the smallest normal: its places are 2^-14's
        const float cmf = half_bits_to_float(cm);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float qf = half_bits_to_float(in.qbits[g]);
            if constexpr (KS::kNew || KS::kMatrix) ks.q[g][tid] = qf;
            P[g] = qf * cmf;                             // exact: 11-bit x 11-bit significands
            // the maximum over the wave's 64 columns in the vector ALU (LDS atomics of 64 lanes on one address take a
            // cycle per lane of the LDS unit that all workgroups of the compute unit share)
            const int em = wave_max_int(P[g] != 0.0f ? float_exp_field(P[g]) : -1);
            if (lane == 0) ks.emax[wave][g] = em;
        }
    }
    __syncthreads();
    if (tid < kD) {
        int lv = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (P[g] != 0.0f) {
                const int emax = max(ks.emax[0][g], ks.emax[1][g]);
                const int l = level_for_mantissa_bits(10 + a.guard_bits - (emax - float_exp_field(P[g])));
                lv = l > lv ? l : lv;
            }
        }
        if (a.force_level >= 0) lv = a.force_level;
        const uint64_t b1 = __ballot(lv >= 1), b2 = __ballot(lv >= 2);
        if (lane == 0) {
            ks.need_mid[wave] = b1;
            ks.need_lo[wave] = b2;
        }
        if (a.dbg.lvlK && export_levels) a.dbg.lvlK[bh * kD + tid] = (uint8_t)lv;
        if (a.stats && export_levels && lane == 0) {   // 64 columns of this wave: how many at each level, times the tokens
            const unsigned long long n2 = __builtin_popcountll(b2), n1 = __builtin_popcountll(b1) - n2, n = (unsigned long long)stat_len;
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->k_elems[0]), (64ull - n1 - n2) * n);
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->k_elems[1]), n1 * n);
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->k_elems[2]), n2 * n);
        }
        if (k_new_bits >= 0) {
            const uint32_t kb = read_at(uint32_t(k_new_bits), lv);
            if constexpr (KS::kNew) ks.knew[tid] = half_bits_to_float(kb);
            else ks.kread[tid] = (uint16_t)kb;
        }
    }
    __syncthreads();
    return colmax_used;
}

// Fused append: the logit of the token that is being appended, from ks.knew, with the same arithmetic as a
// tile lane (fp32, channels ascending).  One thread per query head of the group.
template <int G>
__device__ __forceinline__ float new_token_logit(const KSharedNew<G>& ks, int g)
{
    float acc = 0.0f;
    for (int d0 = 0; d0 < kD; d0 += 16) {   // operands fetched 16 at a time, the additions stay in channel order
        float qv[16], kv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            qv[i] = ks.q[g][d0 + i];
            kv[i] = ks.knew[d0 + i];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) acc = fmaf(qv[i], kv[i], acc);
    }
    return acc;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{   // readfirstlane returns a signed int: widen through uint32_t
    const uint32_t lo32 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi32 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (uint64_t(hi32) << 32) | uint64_t(lo32);
}

// One wave, one unit of 64*TPL tokens of (b, h): lane -> tokens TPL*lane .. TPL*lane+TPL-1 of the unit; the logit of a
// token is accumulated in fp32 over channels in ascending order inside its lane (no reduction).  TPL = 4: a unit is a
// 256-token block, the form that streams best (2-KB and 1-KB runs).  TPL = 2: half a block, in the head kernel, for calls with so few blocks
// that the time is one wave's walk through its unit: twice the waves, half as many dependent groups each (the call below: 24.8 -> 22.3 us).
// Channels are processed U = 32 / TPL at a time, 4 KB per group in either form.  For TPL = 4 the wave fetches per group the 2-KB run of K_hi (8 columns x 256 B,
// contiguous in the channel-major block) with two 16-B loads per lane, and the 1-KB runs of K_mid / K_lo with one
// 16-B load per lane each, lane -> (column lane/8, 16 bytes): a column whose level does not ask for a plane is
// left out by sending its 8 lanes out of range (nothing is fetched, zeros come back).  Four vector-memory
// instructions per group instead of one per column and plane: the address unit of a CU takes about as long
// for a 2-byte-per-lane load as for a 16-byte one, and the count of such instructions, not their bytes, bounded
// this pass.  The loaded registers are in "memory order"; the nibbles become low bytes there (one lane holds 32 tokens of
// one column: 4 words of each nibble plane, the fill a constant per lane), then HI and low bytes are written to a 4-KB
// wave-private LDS area and read back in "token order" (lane -> its 4 tokens of every column: two words per column, the
// reads of the whole group issued before the first is used).  q comes through scalar loads as fp16 pairs and goes into the
// multiply-adds as it is.  No branch in a group: a branch per column on its level had made every LDS read wait for the one
// before (13.9 us for one wave's block).  Measured against that form: B 1, 32 heads, 1024 tokens 29.1 -> 24.8 us a call;
// groups of eight heads 172 -> 106 registers; calls bound by memory 1-2 % faster.
// Logits go to a.logits and are left in acc; the maximum over the unit's valid tokens is returned for every query head of the
// group (same value in all lanes).
constexpr int kKStage = 4096;     // bytes of LDS staging per wave

// Byte offset (inside a block's HI plane) of the 16-byte piece this lane fetches of the first half of a group that starts at
// column 0; the second half lies kHiHalf<TPL> further, column d0 starts at d0 * 256.  A piece whose tokens all lie at or
// past len is out of range: nothing of it is fetched (8193 tokens: 3 % of the bytes).
template <int TPL>
__device__ __forceinline__ uint32_t k_hi_lane_offset(int unit, int len)
{
    const uint32_t lane = threadIdx.x & 63, sub = uint32_t(unit) % (4 / TPL), t = (lane % (4 * TPL)) * 16;
    return unit * (64 * TPL) + int(t) < len ? (lane / (4 * TPL)) * kTB + sub * (64 * TPL) + t : kSkip;
}
template <int TPL> constexpr uint32_t kHiHalf = (16 / TPL) * kTB;

// HI bytes of the first three groups of a unit, issued before the levels are known (they are always read):
// pre[] is handed to k_tile (use_pre = true) for the same unit.
template <bool NT = true, int TPL = 4>
__device__ __forceinline__ void k_tile_pre(const DecodeArgs& a, int b, int h, int unit, int len, u32x4_t (&pre)[6])
{
    const size_t bh = size_t(b) * a.s.Hkv + h;
    const __amdgpu_buffer_rsrc_t rh = make_rsrc(a.k_hi + (bh * a.s.Ncap + size_t(unit / (4 / TPL)) * kTB) * kD, uint32_t(kTB) * kD);
    const uint32_t off = k_hi_lane_offset<TPL>(unit, len);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const uint32_t at = off + i * kHiHalf<TPL>;   // past the end of the buffer (nothing is fetched) if off is kSkip
        pre[i] = NT ? buf_load_b128_nt(rh, at) : buf_load_b128(rh, at);
    }
}

// NT: the block's bytes are read with the non-temporal hint (they are read once per step); a caller that is about to
// store into the block's lines (fused append) reads that one block without it, so that the lines stay in L2.
// lds_lg: where a kernel keeps the logits of its (sequence, KV head) in LDS (query head g at lds_lg + g * lds_stride
// floats, token t at index t), or NULL: they go to a.logits.  With LDS logits a.logits is written as well only if it
// is the caller's export buffer (a.dbg.logits).
// hq0: first of the G consecutive query heads whose logits are computed.
// NEW: token at_new of the unit is being appended; its values come from ks.kread and not from the planes (whose bytes may be stored meanwhile).
template <int G, bool NT = true, int TPL = 4, bool NEW = false, typename KS>
__device__ __forceinline__ void k_tile(const DecodeArgs& a, int b, int h, size_t hq0, int unit, int len, const KS& ks,
                                       float (&tile_max)[G], const u32x4_t (&pre)[6], bool use_pre,
                                       float (&acc)[G][TPL], uint8_t* stage, float* lds_lg = nullptr, int lds_stride = 0, int at_new = 0)
{
    static_assert(TPL == 4 || TPL == 2, "");
    constexpr int U = 32 / TPL;       // columns per group
    constexpr int kUnit = 64 * TPL;   // tokens of the unit
    constexpr int kAux = NT ? kAuxNt : 0;
    const int lane = threadIdx.x & 63;
    const int Hkv = a.s.Hkv, Ncap = a.s.Ncap;
    const size_t bh = size_t(b) * Hkv + h;
    unit = __builtin_amdgcn_readfirstlane(unit);   // wave-uniform by contract: scalar addressing
    const int blk = unit / (4 / TPL), sub = unit % (4 / TPL);

#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < TPL; ++i) acc[g][i] = 0.0f;

    // the level masks live in scalar registers for the whole loop
    const uint64_t nm0 = uniform64(ks.need_mid[0]), nm1 = uniform64(ks.need_mid[1]);
    const uint64_t nl0 = uniform64(ks.need_lo[0]), nl1 = uniform64(ks.need_lo[1]);
    // bits of the U columns starting at d0 (d0 % U == 0, so a group never straddles the two words)
    auto bits_at = [&](uint64_t w0, uint64_t w1, int d0) -> uint32_t {
        return d0 < kD ? (uint32_t)((d0 < 64 ? w0 : w1) >> (d0 & 63)) & (uint32_t)((1ull << U) - 1) : 0u;
    };
    const uint8_t* hi_blk = a.k_hi + (bh * Ncap + size_t(blk) * kTB) * kD;
    const uint8_t* mid_blk = a.k_mid + (bh * Ncap + size_t(blk) * kTB) * (kD / 2);
    const uint8_t* lo_blk = a.k_lo + (bh * Ncap + size_t(blk) * kTB) * (kD / 2);
    // q of the group as fp16 pairs: uniform addresses in constant memory space, scalar loads
    const uint32_t __attribute__((address_space(4)))* qw[G];
#pragma unroll
    for (int g = 0; g < G; ++g) qw[g] = (const uint32_t __attribute__((address_space(4)))*)(uintptr_t)(a.q + (hq0 + g) * kD);
    const uint32_t voff = uint32_t(lane) * 16;
    // Groups of eight heads: the multiply-adds on the matrix cores, a column at a time.  One 4x4x1 product is sixteen blocks of four
    // lanes: its rows are four query heads, its columns the four lanes' tokens, and a lane receives its own token's sums for the four
    // heads -- one binary32 multiply-add per element and column, in channel order, the same bits as the vector ALU's.  235 vector
    // instructions a group of columns for four heads become 83 and 32 products of half a multiply-add's time.  Us a call, 64/8 heads:
    // B 4 16384 tokens 79.9 -> 75.8, B 8 8192 78.6 -> 74.7, B 3 13000 64.1 -> 62.3, B 1 8192 42.3 -> 41.8.  Groups of four are bound by
    // memory: -2 to +2 %, left on the vector ALU.
    constexpr bool MX = KS::kMatrix;
    static_assert(!MX || G % 4 == 0, "four heads per product");
    constexpr int S = MX ? G / 4 : 1;
    f32x4_t dx[MX ? TPL : 1][S];
#pragma unroll
    for (int i = 0; i < (MX ? TPL : 1); ++i)
#pragma unroll
        for (int s = 0; s < S; ++s) dx[i][s] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t hoff = k_hi_lane_offset<TPL>(unit, len);
    const uint32_t col = uint32_t(lane) / (2 * TPL);   // the column of the group this lane fetches nibbles of (32 tokens of it)
    const bool nib_in = unit * kUnit + int(uint32_t(lane) % (2 * TPL)) * 32 < len;   // some of the lane's 32 tokens are inside the sequence
    const uint32_t noff = col * (kTB / 2) + uint32_t(sub) * (kUnit / 2) + (uint32_t(lane) % (2 * TPL)) * 16;

    struct Group {
        u32x4_t h0, h1;   // 16 HI bytes of a column of the first / second half of the group
        u32x4_t m, l;     // 16 MID / LO bytes of column col
    };
    // groups past the last column are issued through descriptors of size zero: nothing is fetched
    auto issue_hi = [&](Group& gr, int d0) {
        const __amdgpu_buffer_rsrc_t rh = make_rsrc(hi_blk, d0 < kD ? uint32_t(kTB) * kD : 0u);
        gr.h0 = __builtin_amdgcn_raw_buffer_load_b128(rh, hoff, d0 * kTB, kAux);
        gr.h1 = __builtin_amdgcn_raw_buffer_load_b128(rh, hoff + kHiHalf<TPL>, d0 * kTB, kAux);
    };
    auto issue_nib = [&](Group& gr, int d0) {
        const uint32_t bm = bits_at(nm0, nm1, d0), bl = bits_at(nl0, nl1, d0);
        const uint32_t size = d0 < kD ? uint32_t(kTB) * (kD / 2) : 0u;
        const __amdgpu_buffer_rsrc_t rm = make_rsrc(mid_blk, size), rl = make_rsrc(lo_blk, size);
        const uint32_t base = noff + uint32_t(d0 < kD ? d0 : 0) * (kTB / 2);
        gr.m = __builtin_amdgcn_raw_buffer_load_b128(rm, nib_in && ((bm >> col) & 1u) ? base : kSkip, 0, kAux);
        gr.l = __builtin_amdgcn_raw_buffer_load_b128(rl, nib_in && ((bl >> col) & 1u) ? base : kSkip, 0, kAux);
    };
    auto issue = [&](Group& gr, int d0) {
        issue_hi(gr, d0);
        issue_nib(gr, d0);
    };
    auto compute = [&](const Group& gr, int d0) {
        // the low bytes of the lane's 32 tokens of column col, from their nibbles (planes that were not read came back
        // as zeros) and the column's fill, in token order
        const uint32_t bm = bits_at(nm0, nm1, d0) >> col, bl = bits_at(nl0, nl1, d0) >> col;
        const uint32_t fill = (bl & 1u) ? 0u : ((bm & 1u) ? 0x08080808u : 0x80808080u);
        const uint32_t mw[4] = {gr.m.x, gr.m.y, gr.m.z, gr.m.w}, lw[4] = {gr.l.x, gr.l.y, gr.l.z, gr.l.w};
        uint32_t low[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t ev = bit_select(0xF0F0F0F0u, mw[i] << 4, lw[i]) | fill;   // tokens 0, 2, 4, 6 of eight
            const uint32_t od = bit_select(0xF0F0F0F0u, mw[i], lw[i] >> 4) | fill;   // tokens 1, 3, 5, 7
            low[2 * i] = __builtin_amdgcn_perm(od, ev, 0x05010400u);
            low[2 * i + 1] = __builtin_amdgcn_perm(od, ev, 0x07030602u);
        }
        // memory order -> token order through the wave's LDS area (LDS serves a wave's accesses in order)
        __builtin_amdgcn_wave_barrier();
        *reinterpret_cast<u32x4_t*>(stage + voff) = gr.h0;
        *reinterpret_cast<u32x4_t*>(stage + 1024 + voff) = gr.h1;
        *reinterpret_cast<u32x4_t*>(stage + 2048 + 2 * voff) = u32x4_t{low[0], low[1], low[2], low[3]};
        *reinterpret_cast<u32x4_t*>(stage + 2048 + 2 * voff + 16) = u32x4_t{low[4], low[5], low[6], low[7]};
        if (NEW && lane < U) {   // behind the stores above: LDS serves a wave's accesses in order
            const uint32_t kb = ks.kread[d0 + lane];
            stage[lane * kUnit + at_new] = (uint8_t)(kb >> 8);
            stage[2048 + lane * kUnit + at_new] = (uint8_t)kb;
        }
        __builtin_amdgcn_wave_barrier();
        typedef std::conditional_t<TPL == 4, uint32_t, uint16_t> word_t;   // TPL bytes
        uint32_t hh[U], ll[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            hh[u] = *reinterpret_cast<const word_t*>(stage + u * kUnit + lane * TPL);
            ll[u] = *reinterpret_cast<const word_t*>(stage + 2048 + u * kUnit + lane * TPL);
        }
        f32x4_t qx[S][U / 4];   // q of head lane % 4 (+ 4 s), the group's columns
        if constexpr (MX)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int v = 0; v < U / 4; ++v) qx[s][v] = *reinterpret_cast<const f32x4_t*>(&ks.q[4 * s + (lane & 3)][d0 + 4 * v]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float k[TPL];
            const uint32_t p0 = __builtin_amdgcn_perm(hh[u], ll[u], 0x05010400u);   // tokens (0,1)
            k[0] = lo_half(p0);
            k[1] = hi_half(p0);
            if constexpr (TPL == 4) {
                const uint32_t p1 = __builtin_amdgcn_perm(hh[u], ll[u], 0x07030602u);   // tokens (2,3)
                k[2] = lo_half(p1);
                k[3] = hi_half(p1);
            }
            if constexpr (MX) {
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int i = 0; i < TPL; ++i) dx[i][s] = __builtin_amdgcn_mfma_f32_4x4x1f32(qx[s][u / 4][u % 4], k[i], dx[i][s], 0, 0, 0);
                continue;
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const uint32_t qp = qw[g][(d0 + u) >> 1];
                const float qd = (u & 1) ? hi_half(qp) : lo_half(qp);
                // q*k is exact in fp32, so the fused form rounds exactly like multiply-then-add
#pragma unroll
                for (int i = 0; i < TPL; ++i) acc[g][i] = fmaf(qd, k[i], acc[g][i]);
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    // three groups rotate by name: all three are issued before the first is consumed, and a group is issued again
    // as soon as it has been consumed (8 to 12 KB in flight per wave)
    Group A, B, C;
    if (use_pre) {   // uniform: the HI bytes of the first three groups are already in flight (k_tile_pre)
        A.h0 = pre[0];
        A.h1 = pre[1];
        B.h0 = pre[2];
        B.h1 = pre[3];
        C.h0 = pre[4];
        C.h1 = pre[5];
        issue_nib(A, 0);
        issue_nib(B, U);
        issue_nib(C, 2 * U);
    } else {
        issue(A, 0);
        issue(B, U);
        issue(C, 2 * U);
    }
#pragma unroll 1
    for (int d0 = 0; d0 < kD; d0 += 3 * U) {
        compute(A, d0);
        issue(A, d0 + 3 * U);
        if (d0 + U < kD) compute(B, d0 + U);   // kD is not a multiple of 3 * U: the last round is partial
        issue(B, d0 + 4 * U);
        if (d0 + 2 * U < kD) compute(C, d0 + 2 * U);
        issue(C, d0 + 5 * U);
    }

    if constexpr (MX)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < TPL; ++i) acc[g][i] = dx[i][g / 4][g % 4];

    // ---- logits out, tile maxima -----------------------------------------------------------------
    // Written for other workgroups they go with the non-temporal hint, which is also how the V kernel of a group of four or eight reads
    // them: B 8, 32/8, 32768 tokens (34 MB) 169.5 -> 161.5 us a call, B 4, 32/8, up to 131072 246 -> 241; of one or two heads where there
    // are many (a.lg_nt; 17 MB, B 16, 32 heads, 8193 with append 283.5 -> 274; 8 MB equal; 4 MB, which the caches hold until they are
    // read again: B 4, 32 heads, 8192 84.2 -> 85.1).  Groups of four and eight always: few logits lose up to 1.2 % (plain stores and
    // loads / the hint: B 1, 32/8, 1024 25.17/25.35, 8192 33.7/34.0, 32768 (4 MB) 49.8/50.4; B 1, 64/8, 16384 (4 MB) 45.7/45.9; from
    // 6 MB on the hint is ahead: B 3, 64/8, 8192 51.1/50.9, B 4, 32/8, 32768 110.9/108.4), but choosing by the size costs all calls as
    // much (stores by size 0.2 to 0.7 % more, loads too 0.5 to 3 %).  The head kernel reads its own soon after: without.
    const bool lg_nt = !KS::kNew && (KS::kHeads >= 4 || a.lg_nt);
    const int t0 = unit * kUnit + lane * TPL;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const size_t hq = hq0 + g;
        const __amdgpu_buffer_rsrc_t rs_lg = make_rsrc(a.logits + hq * Ncap, uint32_t(Ncap) * 4u);
        typedef std::conditional_t<TPL == 4, u32x4_t, u32x2_t> vec_t;
        vec_t w;
#pragma unroll
        for (int i = 0; i < TPL; ++i) w[i] = float_bits(acc[g][i]);
        if (lds_lg) *reinterpret_cast<vec_t*>(lds_lg + g * lds_stride + t0) = w;
        if (!lds_lg || a.dbg.logits) {
            auto store = [&](auto aux) {
                if constexpr (TPL == 4) __builtin_amdgcn_raw_buffer_store_b128(w, rs_lg, uint32_t(t0) * 4u, 0, aux());
                else __builtin_amdgcn_raw_buffer_store_b64(w, rs_lg, uint32_t(t0) * 4u, 0, aux());
            };
            if (lg_nt) store(std::integral_constant<int, kAuxNt>());   // uniform
            else store(std::integral_constant<int, 0>());
        }
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < TPL; ++i)
            if (t0 + i < len) m = fmaxf(m, acc[g][i]);
        tile_max[g] = wave_max(m);
    }
}

}  // namespace akv
