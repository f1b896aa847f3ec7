// V side of decode attention as device functions: Rule 2 per element, fetch per token row, softmax
// weights, O = S V~.
// "Quantization of V-Cache": with O_est known, every addend s_t * v_td is aligned to the precision of the
// result (Rule 2); the bit width of the addend is the bit width V is read at.
#pragma once
#include "akv_common.h"

namespace akv {

// Byte-parallel form of Rule 2 for one token row.  With w_d = guard - 5 - Ehat_d and s = Ahat_t the
// mantissa bits element (t,d) needs are m = ev' + w_d + s (ev' = max(exponent field, 1)); the row is read
// at level >= 1 iff some m >= 3 and at level 2 iff some m >= 7.  Per byte: S = ev + B_d + (s + 64) with
// B_d = clamp(w_d + 61, 4, 132) reaches 128 exactly when ev + w_d + s reaches 3, and 132 exactly when it
// reaches 7: bit 7 of S and bit 7 of S - 4 are the two answers (no carry and no borrow: 4 <= S <= 227).
// The clamps only cut cases that are decided for every ev in 0..31 and s in -64..0.  ev' differs from ev
// only for ev = 0, which adds the row-independent test 1 + max_d w_d + s >= 3 (resp. 7).
__device__ __forceinline__ uint32_t clamp_byte(int v) { return (uint32_t)(v < 4 ? 4 : (v > 132 ? 132 : v)); }

// Per-lane constants of Rule 2 for the lane's 128 / LPR channels (LPR lanes per row: lane -> channel slice lane % LPR)
template <int LPR = 8>
struct VRule {
    static constexpr int kWords = 32 / LPR;
    uint32_t B[kWords];
    int ehat[4 * kWords];   // only read by the variant that exports per-element needs
    int wmax;       // max over all 128 channels of w_d
    int force;      // -1, or the level every row is read at (then B = 4: no byte ever reaches bit 7)
};

// The constants in LDS: thread d < 128 of the workgroup (two waves) lays down those of its channel, v_rule_load takes them up behind a
// barrier (a lane working out its 16 or 32 channels by itself took 600 or 1500 cycles of every workgroup)
struct VRuleShared {
    alignas(16) uint8_t B[kD];
    int wmax[2];    // of channels 0..63, 64..127
    int ehat[kD];
};
__device__ __forceinline__ void v_rule_store(VRuleShared& sh, int d, int ehat, int guard_bits)
{
    const int w = guard_bits - 5 - ehat;
    sh.B[d] = (uint8_t)clamp_byte(w + 61);
    sh.ehat[d] = ehat;
    sh.wmax[d >> 6] = wave_max_int(w);
}
template <int LPR>
__device__ __forceinline__ void v_rule_load(const VRuleShared& sh, int force_level, VRule<LPR>& vr)
{
    const int cl = threadIdx.x % LPR;
#pragma unroll
    for (int i = 0; i < vr.kWords; i += 4) {
        const u32x4_t w = *reinterpret_cast<const u32x4_t*>(&sh.B[(cl * vr.kWords + i) * 4]);
#pragma unroll
        for (int k = 0; k < 4; ++k) vr.B[i + k] = force_level >= 0 ? 0x04040404u : w[k];
    }
#pragma unroll
    for (int i = 0; i < 4 * vr.kWords; ++i) vr.ehat[i] = sh.ehat[cl * vr.kWords * 4 + i];   // dead but in the variant that exports
    vr.wmax = max(sh.wmax[0], sh.wmax[1]);
    vr.force = force_level;
}

// OR over the 8 (4) lanes of a row, result in all of them: two exchanges inside the quads, and one with the mirrored lane of
// the 8-lane half row.
template <int LPR = 8>
__device__ __forceinline__ uint32_t or_over_row(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);    // quad_perm [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);    // quad_perm [2,3,0,1]
    if (LPR == 8) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);   // row_half_mirror
    return v;
}

// the row-independent tests 1 + max_d w_d + Ahat >= 3 and >= 7 (or the forced level) as bounds of Ahat + 64 in every byte
template <int LPR>
__device__ __forceinline__ uint32_t v_bound_word(const VRule<LPR>& vr, int need, int level)
{
    const int at = vr.force >= 0 ? (vr.force >= level ? 0 : 127) : min(max(need + 63 - vr.wmax, 0), 127);
    return (uint32_t)__builtin_amdgcn_readfirstlane(at * 0x01010101);
}
// levels >= 1 / = 2 needed by some element of the row, from the lane's words of HI bytes (result in all LPR lanes of the row);
// ss: Ahat + 64 in every byte
template <int LPR>
__device__ __forceinline__ void v_row_needs(const uint32_t (&hw)[32 / LPR], const VRule<LPR>& vr, uint32_t ss, uint32_t row1, uint32_t row2,
                                            bool& need1, bool& need2)
{
    uint32_t any1 = 0, any2 = 0;
#pragma unroll
    for (int i = 0; i < 32 / LPR; ++i) {
        const uint32_t evp = (hw[i] >> 2) & 0x1F1F1F1Fu;
        const uint32_t S = evp + vr.B[i] + ss;
        any1 |= S;
        any2 |= S - 0x04040404u;
    }
    // bit 7 of a byte: level >= 1 needed; bit 6: level 2 needed (which implies the former)
    const uint32_t flags = or_over_row<LPR>((any1 & 0x80808080u) | ((any2 >> 1) & 0x40404040u));
    need1 = flags != 0 || ss >= row1;
    need2 = (flags & 0x40404040u) != 0 || ss >= row2;   // ss: the same byte four times
}

// HI bytes of the first NPRE batches of a wave, issued early by a caller that has idle time before the V side can
// start (they depend on nothing but the row range).  Rows at or past len are not fetched.
template <int KG, int NPRE, bool NT = false>
__device__ __forceinline__ void v_prefetch_hi(const DecodeArgs& a, int b, int h, int t_first, int batch_stride, int len,
                                              u32x4_t (&hi)[NPRE][KG])
{
    const int lane = threadIdx.x & 63;
    const size_t bh = size_t(b) * a.s.Hkv + h;
    const __amdgpu_buffer_rsrc_t rs_hi = make_rsrc(a.v_hi + bh * a.s.Ncap * kD, uint32_t(len) * kD);
    const uint32_t voff = uint32_t(t_first) * kD + uint32_t(lane >> 3) * kD + uint32_t(lane & 7) * 16;
#pragma unroll
    for (int n = 0; n < NPRE; ++n)
#pragma unroll
        for (int gr = 0; gr < KG; ++gr) hi[n][gr] = NT ? buf_load_b128_nt(rs_hi, voff + uint32_t(n * batch_stride + gr * 8) * kD) : buf_load_b128(rs_hi, voff + uint32_t(n * batch_stride + gr * 8) * kD);
}

// DEBUG: what a lane has counted for akv_stats (rows at each level; elements in all and those that need levels 1 and 2), added
// once per wave
__device__ __forceinline__ void v_add_stats(const DecodeArgs& a, const unsigned (&rows)[3], const unsigned (&need)[3])
{
    unsigned v6[6] = {rows[0], rows[1], rows[2], need[0] - need[1] - need[2], need[1], need[2]};
#pragma unroll
    for (int i = 0; i < 6; ++i)
        for (int o = 1; o < 64; o <<= 1) v6[i] += __shfl_xor(v6[i], o);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->v_row_elems[i]), (unsigned long long)v6[i] * kD);
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->v_need_elems[i]), (unsigned long long)v6[3 + i]);
        }
    }
}
// DEBUG: the exports of one lane for its W words of HI bytes of row t of (b, h): the level applied, the level each element needs
template <int W>
__device__ __forceinline__ void v_export(const DecodeArgs& a, size_t bh, int t, int cl, int applied, int ahat, const uint32_t (&hw)[W],
                                         const int (&ehat)[4 * W], unsigned (&st_rows)[3], unsigned (&st_need)[3])
{
    if (a.dbg.appliedV && cl == 0) a.dbg.appliedV[bh * a.s.Ncap + t] = (uint8_t)applied;
    if (cl == 0) {
        st_rows[0] += applied == 0;
        st_rows[1] += applied == 1;
        st_rows[2] += applied == 2;
    }
    if (!a.dbg.needV && !a.stats) return;
    uint32_t nv[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
        nv[i] = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int ev = (int)((hw[i] >> (8 * k + 2)) & 31u);
            ev = ev < 1 ? 1 : ev;
            int need = level_for_mantissa_bits(10 + a.guard_bits - (ehat[i * 4 + k] - (ahat + ev - 15)));
            if (a.force_level >= 0) need = a.force_level;
            nv[i] |= (uint32_t)need << (8 * k);
            st_need[1] += need == 1;
            st_need[2] += need == 2;
        }
    }
    st_need[0] += 4 * W;
    if (a.dbg.needV)
#pragma unroll
        for (int i = 0; i < W; i += 4)
            *reinterpret_cast<uint4*>(a.dbg.needV + (bh * a.s.Ncap + t) * kD + (cl * W + i) * 4) = make_uint4(nv[i], nv[i + 1], nv[i + 2], nv[i + 3]);
}

// One wave walks token rows of (b, h) in batches of 8*KG rows (KG groups of 8 rows; lane -> row lane/8 of the
// group and the 16-channel slice lane%8): batch i covers rows t_first + i*batch_stride .. + 8*KG - 1,
// i < nbatches.  Three stages per batch, software-pipelined over DL + 1 named buffers:
//   L  issue the HI loads and the logit load (lane j < 8*KG*G holds the logit of row j / G of the batch for query
//      head j % G: one load for all heads; single heads: one load for four batches);
//   D  softmax weight and score exponent once per (row, head), in that lane, handed to the 8 lanes of the row by lane
//      permutes;
//      Rule 2 on the HI bytes; MID / LO loads of the rows that need them (the others are issued out of
//      range: nothing is fetched);
//   F  assemble the fp16 values, multiply-adds.
// Round i runs D(i+1), L(i+DL), F(i): every load has at least a whole round of arithmetic to arrive; a kernel
// with few waves per SIMD raises DL to keep enough bytes in flight.
// The descriptors end at row len, so rows at or past len read as zero without any per-lane test; their weight
// is forced to zero.  acc accumulates sum_t p_t * v~_td per lane (to be reduced over the 8 row lanes, then
// over waves, by the caller); z accumulates sum_t p_t per lane (to be summed over all 64 lanes).
// NPRE > 0: pre holds the HI bytes of batches 0 .. NPRE-1 (v_prefetch_hi) if pre_ok.
// lds_lg / lds_stride: the logits in LDS (query head g at lds_lg + g * lds_stride, token t at index t), or NULL: a.logits.
// Mlane: the global max of query head lane % G.  ready(): called when the first loads are on their way; vr is read after it.
// NT: the HI bytes are read with the non-temporal hint (measured: it pays in the token-split V kernel, where the logits
// and the chunk partials of other workgroups share the caches, and costs in the head-per-workgroup kernel); the MID
// and LO bytes always are (it pays in both).
template <int G, int KG, bool DEBUG, int NPRE, int DL, bool NT, typename READY>
__device__ __forceinline__ void v_rows(const DecodeArgs& a, int b, int h, int t_first, int batch_stride, int nbatches,
                                       int len, const VRule<>& vr, float Mlane, float (&acc)[G][16],
                                       float (&z)[G], const u32x4_t (&pre)[NPRE > 0 ? NPRE : 1][KG], bool pre_ok,
                                       const float* lds_lg, int lds_stride, READY ready)
{
    constexpr int RB = 8 * KG;
    // wave-uniform by contract: scalar registers, scalar loop control
    nbatches = __builtin_amdgcn_readfirstlane(nbatches);
    t_first = __builtin_amdgcn_readfirstlane(t_first);
    if (nbatches <= 0) {
        ready();
        return;
    }
    const int lane = threadIdx.x & 63;
    const int r = lane >> 3, cl = lane & 7;
    // lane j < RB * G computes the score of row j / G of the batch for query head j % G: every (row, head) pair once
    static_assert(RB * G <= 64 && (G == 1 || G == 2 || G == 4), "one lane per (row of the batch, query head)");
    const int jrow = lane / G, jg = lane % G;
    const bool jlane = lane < RB * G;
    const int Hkv = a.s.Hkv, Hq = a.s.Hq, Ncap = a.s.Ncap;
    const size_t bh = size_t(b) * Hkv + h;

    // the logits of the G query heads of the group lie Ncap floats apart: one descriptor over all of them
    const __amdgpu_buffer_rsrc_t rs_lg = make_rsrc(a.logits + (size_t(b) * Hq + size_t(h) * G) * Ncap, uint32_t(G) * uint32_t(Ncap) * 4u);
    const __amdgpu_buffer_rsrc_t rs_hi = make_rsrc(a.v_hi + bh * Ncap * kD, uint32_t(len) * kD);
    const __amdgpu_buffer_rsrc_t rs_mid = make_rsrc(a.v_mid + bh * Ncap * (kD / 2), uint32_t(len) * (kD / 2));
    const __amdgpu_buffer_rsrc_t rs_lo = make_rsrc(a.v_lo + bh * Ncap * (kD / 2), uint32_t(len) * (kD / 2));
    uint32_t row1 = 0, row2 = 0;
    const uint32_t voff_hi = uint32_t(r) * kD + uint32_t(cl) * 16;
    const uint32_t voff_nib = uint32_t(r) * (kD / 2) + uint32_t(cl) * 8;
    const uint32_t voff_lg = (uint32_t(jg) * uint32_t(Ncap) + uint32_t(jrow)) * 4u;
    int src[KG];                                   // byte address of the first score lane of row gr*8 + r, for the lane permutes
#pragma unroll
    for (int gr = 0; gr < KG; ++gr) src[gr] = (gr * 8 + r) * G * 4;
    float zl = 0.0f;                               // sum of this lane's weights (rows j / G of the batches, head j % G)
    unsigned st_rows[3] = {0u, 0u, 0u}, st_need[3] = {0u, 0u, 0u};   // DEBUG: this lane's counts for akv_stats

    struct Batch {
        u32x4_t hi[KG];
        float lg;
        u32x2_t mid[KG], lo[KG];
        float p[KG][G];
        uint32_t fill[KG];
    };
    auto row0 = [&](int bt) { return t_first + bt * batch_stride; };
    // a batch past the wave's last one is issued out of range: nothing is fetched
    auto Lhi = [&](Batch& X, int bt) {
        const uint32_t base = bt < nbatches ? uint32_t(row0(bt)) * kD : kSkip;
#pragma unroll
        for (int gr = 0; gr < KG; ++gr) X.hi[gr] = NT ? buf_load_b128_nt(rs_hi, voff_hi + base + gr * 8 * kD) : buf_load_b128(rs_hi, voff_hi + base + gr * 8 * kD);
    };
    auto Llg = [&](Batch& X, int bt) {   // one load for all heads; rows at or past len and idle lanes ask out of range
        const bool on = bt < nbatches && jlane && row0(bt) + jrow < len;
        if (lds_lg) X.lg = on ? lds_lg[jg * lds_stride + row0(bt) + jrow] : 0.0f;   // uniform branch: the kernel keeps its logits in LDS
        else X.lg = bits_float(buf_load_b32(rs_lg, on ? voff_lg + uint32_t(row0(bt)) * 4u : kSkip));
    };
    // Single heads in a ring of four (SB): the scores of the four batches of a round of the ring are computed together, one row
    // per lane (lane / 16 = batch, lane % 16 = row), a quarter of the score instructions and of the logit loads: B 1, 32 heads,
    // 1024 tokens 22.7 -> 22.1 us a call, B 8 4096 71.9 -> 70.2, B 16 step of 8193 285.3 -> 282.
    constexpr bool SB = G == 1 && KG == 2 && DL == 3;
    float lg_n = 0.0f, sb_p = 0.0f;                // logits of the block to come; weights of the present one
    uint32_t sb_ss = 0;
    auto sb_load = [&](int b0) {                   // logits of batches b0 .. b0 + 3
        const int bt = b0 + (lane >> 4), t = row0(bt) + (lane & 15);
        const bool on = bt < nbatches && t < len;
        if (lds_lg) lg_n = on ? lds_lg[t] : 0.0f;
        else lg_n = bits_float(buf_load_b32(rs_lg, on ? uint32_t(t) * 4u : kSkip));
    };
    auto sb_scores = [&](int b0) {
        const int bt = b0 + (lane >> 4);
        const float x = score_x(lg_n, Mlane, a.c);
        sb_p = bt < nbatches && row0(bt) + (lane & 15) < len ? __builtin_amdgcn_exp2f(x) : 0.0f;
        zl += sb_p;
        const int ahat = score_a(x);
        sb_ss = __builtin_amdgcn_perm(0u, uint32_t(ahat + 64), 0x00000000u);
    };
    // k: the batch's place in its round of the ring (used with SB)
    auto D = [&](Batch& X, int bt, int k) {
        uint32_t offm[KG], offl[KG];
#pragma unroll
        for (int gr = 0; gr < KG; ++gr) offm[gr] = offl[gr] = kSkip;
        if (bt < nbatches) {   // uniform; arithmetic only -- the loads below are issued in any case
            const int t0 = row0(bt);
            const int nvalid = min(len - t0, RB);       // rows of the batch inside the sequence (may be <= 0)
            float pj;
            uint32_t ssw;
            if constexpr (SB) {
                pj = sb_p;
                ssw = sb_ss;
            } else {
                const float x = score_x(X.lg, Mlane, a.c);
                int ahat = score_a(x);                  // then the maximum over the G heads of the row (adjacent lanes)
                pj = jlane && jrow < nvalid ? __builtin_amdgcn_exp2f(x) : 0.0f;
                zl += pj;
                if (G >= 2) ahat = max(ahat, __builtin_amdgcn_update_dpp(ahat, ahat, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
                if (G >= 4) ahat = max(ahat, __builtin_amdgcn_update_dpp(ahat, ahat, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
                ssw = __builtin_amdgcn_perm(0u, uint32_t(ahat + 64), 0x00000000u);   // (Ahat + 64) in every byte
            }
            const int sk = SB ? 64 * k : 0;   // the batch's sixteen score lanes
#pragma unroll
            for (int gr = 0; gr < KG; ++gr) {
                const uint32_t ss = (uint32_t)__builtin_amdgcn_ds_bpermute(src[gr] + sk, (int)ssw);
#pragma unroll
                for (int g = 0; g < G; ++g) X.p[gr][g] = bits_float((uint32_t)__builtin_amdgcn_ds_bpermute(src[gr] + sk + 4 * g, (int)float_bits(pj)));
                const uint32_t hw[4] = {X.hi[gr].x, X.hi[gr].y, X.hi[gr].z, X.hi[gr].w};
                bool need1, need2;
                v_row_needs<8>(hw, vr, ss, row1, row2, need1, need2);
                const uint32_t off = voff_nib + uint32_t(t0) * (kD / 2) + gr * 8 * (kD / 2);
                offm[gr] = need1 ? off : kSkip;
                offl[gr] = need2 ? off : kSkip;
                X.fill[gr] = need2 ? 0u : (need1 ? 0x08080808u : 0x80808080u);

                if (DEBUG) {
                    const int t = t0 + gr * 8 + r;
                    if (t < len) v_export<4>(a, bh, t, cl, need2 ? 2 : (need1 ? 1 : 0), int(ss & 0xFFu) - 64, hw, vr.ehat, st_rows, st_need);
                }
            }
        }
#pragma unroll
        for (int gr = 0; gr < KG; ++gr) {
            X.mid[gr] = buf_load_b64_nt(rs_mid, offm[gr]);
            X.lo[gr] = buf_load_b64_nt(rs_lo, offl[gr]);
        }
    };
    auto F = [&](const Batch& X, int bt) {
        if (bt >= nbatches) return;
#pragma unroll
        for (int gr = 0; gr < KG; ++gr) {
            uint32_t pa[4], pb[4];
            assemble8_fill(X.hi[gr].x, X.hi[gr].y, X.mid[gr].x, X.lo[gr].x, X.fill[gr], pa);   // channels 0..7 of the slice
            assemble8_fill(X.hi[gr].z, X.hi[gr].w, X.mid[gr].y, X.lo[gr].y, X.fill[gr], pb);   // channels 8..15
            const float v[16] = {lo_half(pa[0]), lo_half(pa[1]), hi_half(pa[0]), hi_half(pa[1]),
                                 lo_half(pa[2]), lo_half(pa[3]), hi_half(pa[2]), hi_half(pa[3]),
                                 lo_half(pb[0]), lo_half(pb[1]), hi_half(pb[0]), hi_half(pb[1]),
                                 lo_half(pb[2]), lo_half(pb[3]), hi_half(pb[2]), hi_half(pb[3])};
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[g][i] = fmaf(X.p[gr][g], v[i], acc[g][i]);
        }
    };

    // R = DL + 1 named buffers: round i runs D(i + 1), L(i + DL), F(i); the buffer L fills is the one F emptied in
    // the round before.  The loop is unrolled R times so that every buffer index is a constant.  Loads come back in
    // the order they were issued, so the wait of F(i) for its MID / LO bytes (asked for by D(i), one round earlier) is
    // also a wait for every load issued before them: D issues ahead of L in a round, so that this never includes the HI
    // bytes L asked for in that round.
    constexpr int R = DL + 1;
    static_assert(DL >= 2 && NPRE <= DL, "the HI loads run at least two batches ahead");
    Batch ring[R];
#pragma unroll
    for (int k = 0; k < DL; ++k) {
        if (k < NPRE) {
#pragma unroll
            for (int gr = 0; gr < KG; ++gr) ring[k].hi[gr] = pre[k < NPRE ? k : 0][gr];
            if (!pre_ok) Lhi(ring[k], k);
        } else {
            Lhi(ring[k], k);
        }
        if (!SB) Llg(ring[k], k);
    }
    if (SB) sb_load(0);
    ready();
    row1 = v_bound_word(vr, 3, 1);
    row2 = v_bound_word(vr, 7, 2);
    if (SB) sb_scores(0);
    D(ring[0], 0, 0);
#pragma unroll 1
    for (int i = 0; i < nbatches; i += R) {   // rounds past the last batch issue nothing and compute nothing
#pragma unroll
        for (int k = 0; k < R; ++k) {
            if (SB && k == 0) sb_load(i + R);
            if (SB && k == R - 1) sb_scores(i + R);
            D(ring[(k + 1) % R], i + k + 1, (k + 1) % R);
            Lhi(ring[(k + DL) % R], i + k + DL);
            if (!SB) Llg(ring[(k + DL) % R], i + k + DL);
            F(ring[k], i + k);
        }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) z[g] += jg == g ? zl : 0.0f;
    if (DEBUG && a.stats) v_add_stats(a, st_rows, st_need);
}

// Sum acc over the 8 row lanes of a wave (lanes with the same lane % 8) and z over all lanes: afterwards a lane holds the wave's totals of
// channels 16 (lane % 8) + row_lane_column(lane), + 1 in sum and every lane the wave's z
template <int G>
__device__ __forceinline__ void v_reduce_rows(const float (&acc)[G][16], float (&z)[G], float (&sum)[G][2])
{
#pragma unroll
    for (int g = 0; g < G; ++g) {
        z[g] = wave_sum<1>(z[g]);
        sum_row_lanes(acc[g], sum[g]);
    }
}

// ---- Groups of four and eight query heads (the token-split V kernel): the rows of all waves of a workgroup are shared.
// Every wave fetches, tests and assembles its own rows, once, and leaves them in LDS with their weights; after a barrier the
// sum over the rows of the round, for all query heads at once, is a matrix product on the matrix cores:
// D[m][line] += sum_rows W[m][row] * V[row][line], wave w taking lines 32 w .. 32 w + 31.
constexpr int kSRows = 16;        // rows of a wave's batch: lane -> row lane / 4, 32-channel slice lane % 4
// LDS: the rows of a round, each as sixteen 16-byte words (word 4 k + c: channels 32 c + 8 k .. + 7), and the weights of these
// rows, line g the high part and line G + g the low part of query head g's weight (two fp16 numbers whose sum carries 22
// bits).  The matrix instruction wants four consecutive rows of one value per lane: the transposing LDS read turns them on the
// way out, so that a lane lays a row down with 16-byte stores.  The words of a row are permuted by its number
// (v_word_turn), so that neither side has bank conflicts.  Two buffers alternate by round.
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
struct VShare {
    static constexpr int kRows = kVWaves * kSRows;   // rows of a round
    alignas(16) u32x4_t vr[2][kRows][16];
    alignas(16) uint16_t pt[2][16][kRows + 8];
};
// a store takes rows 2 i, 2 i + 1 (four lanes each) at a time, a transposing read rows 4 i .. 4 i + 3 (two words each)
__device__ __forceinline__ int v_word_turn(int row) { return ((row & 1) << 2) | (row & 2); }
// the channel of value `line` (0..127) of a row as it lies in VShare::vr: assemble8_fill leaves channels (0,2), (1,3), (4,6),
// (5,7) of eight in its four words
__device__ __forceinline__ int line_channel(int line)
{
    const int word = line >> 3, pos = line & 7;
    return 32 * (word & 3) + 8 * (word >> 2) + ((pos >> 1) & 1) + 4 * (pos >> 2) + 2 * (pos & 1);
}
constexpr float kVWeightScale = 16384.0f;   // weights are at most 1: scaled by 2^14 their fp16 parts reach down to 2^-38
// workgroup barrier that waits for this wave's LDS traffic only: the loads from memory that are in flight stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Batch i of this wave covers rows t_first + i * kVWaves * kSRows .. + 15; all waves of the workgroup call with the same nbatches.
// Stages L, D, A + matrix product as in v_rows.  Four lanes per row: they are also the lanes that compute the row's scores
// (lane -> query heads lane % 4, + 4), so that nothing is exchanged but the maximum over a quad, and a MID or LO row takes one
// 16-byte load per lane: five vector-memory instructions a batch instead of seven, a quarter of the vector instructions less.
// Measured against eight lanes per row, scores handed over by lane permutes, batches of 8 rows for groups of eight (us a call, the
// non-temporal hint on the logits on both sides): B 8, 32/8, 32768 tokens, few MID and LO rows, 160.6 -> 161.3, with many 190 -> 181; B 4, 32/8,
// up to 131072 246 -> 236; B 16, 32/8, 5000 80.7 -> 75.9; B 3, 64/8, up to 13000, with the matrix products of its K tile, 67.8 -> 64.2.
// What bounds it now is the loads: without assembly, LDS and matrix products (timing only) the call takes as long, without Rule 2's test
// and its MID / LO bytes 8 us less, without the logits 10 us less.  The two halves of a lane's 32 HI bytes share a line, so the HI loads
// keep the line in the caches (temporal: 175 -> 168, at an earlier state).
// acc: the wave's two 16x16 result tiles (four words each: rows 4 * (lane / 16) .. + 3 of W, line 16 * (2 w + tile) + lane % 16),
// scaled by kVWeightScale.  Ml[s]: the global max of query head lane % 4 + 4 s.  ready(): as in v_rows.  z[s]: this lane's sum of the weights of head lane % 4 + 4 s.
template <int G, bool DEBUG, int DL, typename READY>
__device__ __forceinline__ void v_rows_shared(const DecodeArgs& a, int b, int h, int t_first, int nbatches, int len, const VRule<4>& vr,
                                              const float (&Ml)[G / 4], float (&acc)[8], float (&z)[G / 4], VShare& sh, READY ready)
{
    static_assert(G == 4 || G == 8, "high and low parts of all heads are the 16 rows of W");
    static_assert(kVWaves * 32 == kD, "four waves share the 128 lines");
    constexpr int S = G / 4, kStride = VShare::kRows;
    nbatches = __builtin_amdgcn_readfirstlane(nbatches);
    t_first = __builtin_amdgcn_readfirstlane(t_first);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane >> 2, c = lane & 3;
    const int Hq = a.s.Hq, Ncap = a.s.Ncap;
    const size_t bh = size_t(b) * a.s.Hkv + h;
    // the logits of the G query heads of the group lie Ncap floats apart: one descriptor over all of them
    const __amdgpu_buffer_rsrc_t rs_lg = make_rsrc(a.logits + (size_t(b) * Hq + size_t(h) * G) * Ncap, uint32_t(G) * uint32_t(Ncap) * 4u);
    // ... and the rows end at len: rows at or past it read as zeros, their weight is forced to zero
    const __amdgpu_buffer_rsrc_t rs_hi = make_rsrc(a.v_hi + bh * Ncap * kD, uint32_t(len) * kD);
    const __amdgpu_buffer_rsrc_t rs_mid = make_rsrc(a.v_mid + bh * Ncap * (kD / 2), uint32_t(len) * (kD / 2));
    const __amdgpu_buffer_rsrc_t rs_lo = make_rsrc(a.v_lo + bh * Ncap * (kD / 2), uint32_t(len) * (kD / 2));
    uint32_t row1 = 0, row2 = 0;
    const uint32_t voff_hi = uint32_t(r) * kD + uint32_t(c) * 32, voff_nib = uint32_t(r) * (kD / 2) + uint32_t(c) * 16;
    const uint32_t voff_lg = (uint32_t(c) * uint32_t(Ncap) + uint32_t(r)) * 4u;
    unsigned st_rows[3] = {0u, 0u, 0u}, st_need[3] = {0u, 0u, 0u};   // DEBUG: this lane's counts for akv_stats

    struct Batch {
        u32x4_t hi[2], mid, lo;
        float lg[S], p[S];
        uint32_t fill;
    };
    auto row0 = [&](int bt) { return t_first + bt * kStride; };
    // a batch past the wave's last one is issued out of range: nothing is fetched
    auto L = [&](Batch& X, int bt) {
        const uint32_t base = bt < nbatches ? uint32_t(row0(bt)) * kD : kSkip;
#pragma unroll
        for (int i = 0; i < 2; ++i) X.hi[i] = buf_load_b128(rs_hi, voff_hi + base + 16 * i);
        const bool on = bt < nbatches && row0(bt) + r < len;
#pragma unroll
        for (int s = 0; s < S; ++s) X.lg[s] = bits_float(buf_load_b32_nt(rs_lg, on ? voff_lg + (uint32_t(row0(bt)) + uint32_t(4 * s) * uint32_t(Ncap)) * 4u : kSkip));
    };
    auto D = [&](Batch& X, int bt) {
        uint32_t offm = kSkip, offl = kSkip;
        if (bt < nbatches) {   // uniform; arithmetic only -- the loads below are issued in any case
            const int t = row0(bt) + r;
            int ahat = kAMin;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float x = score_x(X.lg[s], Ml[s], a.c);
                ahat = max(ahat, score_a(x));
                X.p[s] = t < len ? __builtin_amdgcn_exp2f(x) : 0.0f;
                z[s] += X.p[s];
            }
            ahat = max(ahat, __builtin_amdgcn_update_dpp(ahat, ahat, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
            ahat = max(ahat, __builtin_amdgcn_update_dpp(ahat, ahat, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
            const uint32_t ss = __builtin_amdgcn_perm(0u, uint32_t(ahat + 64), 0x00000000u);     // (Ahat + 64) in every byte
            const uint32_t hw[8] = {X.hi[0].x, X.hi[0].y, X.hi[0].z, X.hi[0].w, X.hi[1].x, X.hi[1].y, X.hi[1].z, X.hi[1].w};
            bool need1, need2;
            v_row_needs<4>(hw, vr, ss, row1, row2, need1, need2);
            const uint32_t off = voff_nib + uint32_t(row0(bt)) * (kD / 2);
            offm = need1 ? off : kSkip;
            offl = need2 ? off : kSkip;
            X.fill = need2 ? 0u : (need1 ? 0x08080808u : 0x80808080u);
            if (DEBUG && t < len) v_export<8>(a, bh, t, c, need2 ? 2 : (need1 ? 1 : 0), ahat, hw, vr.ehat, st_rows, st_need);
        }
        X.mid = buf_load_b128_nt(rs_mid, offm);
        X.lo = buf_load_b128_nt(rs_lo, offl);
    };
    const int turn = v_word_turn(r);
    auto A = [&](const Batch& X, int bt) {
        const int buf = bt & 1;
        u32x4_t* row = sh.vr[buf][wave * kSRows + r];
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // channels 8 k .. 8 k + 7 of the slice
            uint32_t w[4];
            assemble8_fill(X.hi[k >> 1][2 * (k & 1)], X.hi[k >> 1][2 * (k & 1) + 1], X.mid[k], X.lo[k], X.fill, w);
            row[(4 * k + c) ^ turn] = u32x4_t{w[0], w[1], w[2], w[3]};
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float ws = X.p[s] * kVWeightScale;
            const _Float16 whi = (_Float16)ws;
            const _Float16 wlo = (_Float16)(ws - (float)whi);
            sh.pt[buf][c + 4 * s][wave * kSRows + r] = __builtin_bit_cast(uint16_t, whi);
            sh.pt[buf][G + c + 4 * s][wave * kSRows + r] = __builtin_bit_cast(uint16_t, wlo);
        }
    };
    f32x4_t d0 = {0.0f, 0.0f, 0.0f, 0.0f}, d1 = {0.0f, 0.0f, 0.0f, 0.0f};   // the wave's two result tiles
    auto F = [&](int bt) {
        const int buf = bt & 1;
        const int n = lane & 15, kq = lane >> 4;
#pragma unroll
        for (int kb = 0; kb < VShare::kRows / 32; ++kb) {   // 32 rows: a lane's k are rows 8 kq .. 8 kq + 7
            const half8_t w8 = *reinterpret_cast<const half8_t*>(&sh.pt[buf][n][kb * 32 + 8 * kq]);
            short4_t v[2][2];   // [tile][rows 0..3, 4..7 of the lane's eight]
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 2; ++e) {   // lane n of sixteen reads four values of row n / 4 and receives value n of all four rows
                    const int row = kb * 32 + 8 * kq + 4 * e + (n >> 2), word = 4 * wave + 2 * t + ((n >> 1) & 1);
                    typedef __attribute__((address_space(3))) short4_t* lds_ptr;
                    v[t][e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(reinterpret_cast<short4_t*>(&sh.vr[buf][row][word ^ v_word_turn(row)]) + (n & 1)));
                }
            d0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w8, __builtin_bit_cast(half8_t, __builtin_shufflevector(v[0][0], v[0][1], 0, 1, 2, 3, 4, 5, 6, 7)), d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w8, __builtin_bit_cast(half8_t, __builtin_shufflevector(v[1][0], v[1][1], 0, 1, 2, 3, 4, 5, 6, 7)), d1, 0, 0, 0);
        }
    };
    constexpr int R = DL + 1;   // rounds and buffers as in v_rows
    Batch ring[R];
#pragma unroll
    for (int k = 0; k < DL; ++k) L(ring[k], k);
    if constexpr (2 * G < 16) {   // the rows of W no head uses stay zero in both buffers (ordered before the first read by the first barrier)
        constexpr int kRows = VShare::kRows;
        for (int idx = threadIdx.x; idx < 2 * (16 - 2 * G) * kRows; idx += 64 * kVWaves) {
            const int bf = idx / ((16 - 2 * G) * kRows), rest = idx % ((16 - 2 * G) * kRows);
            sh.pt[bf][2 * G + rest / kRows][rest % kRows] = 0;
        }
    }
    ready();
    row1 = v_bound_word(vr, 3, 1);
    row2 = v_bound_word(vr, 7, 2);
    D(ring[0], 0);
#pragma unroll 1
    for (int i = 0; i < nbatches; i += R) {   // rounds past the last batch issue nothing and compute nothing
#pragma unroll
        for (int k = 0; k < R; ++k) {
            D(ring[(k + 1) % R], i + k + 1);
            L(ring[(k + DL) % R], i + k + DL);
            if (i + k < nbatches) {   // the same for every wave of the workgroup
                A(ring[k], i + k);
                lds_barrier();
                F(i + k);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[i] = d0[i];
        acc[4 + i] = d1[i];
    }
    if (DEBUG && a.stats) v_add_stats(a, st_rows, st_need);
}

// write out[b][h*G + g][:] = o / zsum for channel d (or zero for an empty sequence)
__device__ __forceinline__ void store_out(const DecodeArgs& a, size_t hq, int d, float res)
{
    if (a.out_dtype == 0) reinterpret_cast<float*>(a.out)[hq * kD + d] = res;
    else reinterpret_cast<_Float16*>(a.out)[hq * kD + d] = (_Float16)res;
}

}  // namespace akv
