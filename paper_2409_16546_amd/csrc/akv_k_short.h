// K side of short calls: Rule 1 and the q.K~ pass by waves that each take a small unit of tokens and ask for nothing from their
// neighbours.  For calls whose units are too few to fill the device, where the time is one wave's walk and not its bytes.
#pragma once
#include "akv_common.h"
#include "akv_k_tile.h"

namespace akv {

// q of the group as binary32 (rows of neighbouring heads four banks apart).  Every wave writes all of it and reads only what it has
// written itself, so no barrier is needed: the words of other waves are the same.
template <int G> struct KShortQ { alignas(16) float q[G][kD + 4]; };

// What a lane asks for at the start: K_colmax and q of channels 2 lane, 2 lane + 1 (fp16 pairs).
template <int G> struct KPairIn { uint32_t cm, knew, q[G]; };
template <int G>
__device__ __forceinline__ void k_pairs_load(const DecodeArgs& a, int b, int h, KPairIn<G>& in)
{
    const int lane = threadIdx.x & 63;
    in.cm = reinterpret_cast<const uint32_t*>(a.colmax + (size_t(b) * a.s.Hkv + h) * kD)[lane];
    in.knew = a.k_new ? reinterpret_cast<const uint32_t*>(a.k_new + (size_t(b) * a.s.Hkv + h) * kD)[lane] : 0u;   // uniform; fused append
#pragma unroll
    for (int g = 0; g < G; ++g) in.q[g] = reinterpret_cast<const uint32_t*>(a.q + (size_t(b) * a.s.Hq + size_t(h) * G + g) * kD)[lane];
}

// Columns read at level >= 1 / = 2: bit l of word e is channel 2 l + e
struct KPairLevels { uint64_t mid[2], lo[2]; };

// Rule 1 by one wave for all 128 channels: no LDS between the loads and the masks, no barrier.  The largest magnitude of a head's
// products has the largest exponent; a product that is not a number counts as larger than all, as its exponent field says.  The level of a
// channel is that of the head whose addend lies closest to its head's coarsest one.
// q goes to ks.q for the multiply-adds of the same wave.  stat_len, export_levels: as in k_levels_finish (one wave of the pair).
template <int G>
__device__ __forceinline__ KPairLevels k_pair_levels(const DecodeArgs& a, int b, int h, KShortQ<G>& ks, const KPairIn<G>& in, bool export_levels, int stat_len)
{   // in.cm with the appended token's magnitudes already in it
    typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63;
    const uint32_t cm = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, in.cm), u16x2_t{0x0400, 0x0400}));
    const float c0 = lo_half(cm), c1 = hi_half(cm);
    int m0[G], m1[G], mx[G];   // bits of the products' magnitudes
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float q0 = lo_half(in.q[g]), q1 = hi_half(in.q[g]);
        *reinterpret_cast<float2*>(&ks.q[g][2 * lane]) = make_float2(q0, q1);
        m0[g] = int(float_bits(q0 * c0) & 0x7FFFFFFFu);
        m1[g] = int(float_bits(q1 * c1) & 0x7FFFFFFFu);
        mx[g] = max(m0[g], m1[g]);
    }
    wave_max_ints(mx);
    int gap0 = -1000, gap1 = -1000;   // largest (exponent of the addend - that of the head's coarsest)
#pragma unroll
    for (int g = 0; g < G; ++g) {
        int em = mx[g] >> 23;
        em = em == 0 ? 1000 : em;       // a head whose products are all zero asks for nothing
        gap0 = max(gap0, (m0[g] >> 23) - em);   // a zero product lies 89 and more below any other
        gap1 = max(gap1, (m1[g] >> 23) - em);
    }
    int lv0 = level_for_mantissa_bits(10 + a.guard_bits + gap0), lv1 = level_for_mantissa_bits(10 + a.guard_bits + gap1);
    if (a.force_level >= 0) lv0 = lv1 = a.force_level;
    KPairLevels lv;
    lv.mid[0] = __ballot(lv0 >= 1);
    lv.mid[1] = __ballot(lv1 >= 1);
    lv.lo[0] = __ballot(lv0 >= 2);
    lv.lo[1] = __ballot(lv1 >= 2);
    if (export_levels && (a.dbg.lvlK || a.stats)) {
        if (a.dbg.lvlK) {
            uint8_t* to = a.dbg.lvlK + (size_t(b) * a.s.Hkv + h) * kD + 2 * lane;
            to[0] = uint8_t(lv0);
            to[1] = uint8_t(lv1);
        }
        if (a.stats && lane == 0) {
            const unsigned long long n2 = __builtin_popcountll(lv.lo[0]) + __builtin_popcountll(lv.lo[1]);
            const unsigned long long n1 = __builtin_popcountll(lv.mid[0]) + __builtin_popcountll(lv.mid[1]) - n2, n = (unsigned long long)stat_len;
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->k_elems[0]), (128ull - n1 - n2) * n);
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->k_elems[1]), n1 * n);
            atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats->k_elems[2]), n2 * n);
        }
    }
    return lv;
}

// fused append: the new token's K row (pairs: channels 2 lane, 2 lane + 1) as it is read at the column levels, channel 32 i + lane % 32 in word i
__device__ __forceinline__ void k_pair_read(uint32_t pairs, const KPairLevels& lv, uint32_t (&knew)[4])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = 32 * i + lane % 32;
        const uint64_t mid = (c & 1) ? lv.mid[1] : lv.mid[0], lo = (c & 1) ? lv.lo[1] : lv.lo[0];
        const uint32_t w = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (c / 2), (int)pairs);
        knew[i] = read_at((c & 1) ? w >> 16 : w & 0xFFFFu, int((mid >> (c / 2)) & 1u) + int((lo >> (c / 2)) & 1u));
    }
}

// maximum over the 64 lanes for every one of G values: afterwards lane l holds that of value l / (64 / G)
template <int G>
__device__ __forceinline__ float wave_max_each(const float (&v)[G])
{
    float a[G];
#pragma unroll
    for (int g = 0; g < G; ++g) a[g] = v[g];
    auto pairs = [](float x, float y, bool wide) {
        if (wide) {
            const auto s = __builtin_amdgcn_permlane32_swap(float_bits(x), float_bits(y), false, false);
            return fmaxf(bits_float(s[0]), bits_float(s[1]));
        }
        const auto s = __builtin_amdgcn_permlane16_swap(float_bits(x), float_bits(y), false, false);
        return fmaxf(bits_float(s[0]), bits_float(s[1]));
    };
    constexpr int G32 = G > 1 ? G / 2 : 1, G16 = G32 > 1 ? G32 / 2 : 1;
#pragma unroll
    for (int i = 0; i < G32; ++i) a[i] = pairs(a[i], G > 1 ? a[i + G32] : a[i], true);
#pragma unroll
    for (int i = 0; i < G16; ++i) a[i] = pairs(a[i], G32 > 1 ? a[i + G16] : a[i], false);
    auto dpp = [](float x, auto ctrl) { return bits_float((uint32_t)__builtin_amdgcn_update_dpp((int)float_bits(x), (int)float_bits(x), ctrl(), 0xF, 0xF, false)); };
    using std::integral_constant;
#pragma unroll
    for (int i = 0; i < G16; ++i) a[i] = fmaxf(a[i], dpp(a[i], integral_constant<int, 0x128>()));   // row_ror:8
    if (G16 == 2) a[0] = (threadIdx.x & 8) ? a[G16 - 1] : a[0];                                      // eight values: eight lanes each
    a[0] = fmaxf(a[0], dpp(a[0], integral_constant<int, 0x141>()));                                  // row_half_mirror
    a[0] = fmaxf(a[0], dpp(a[0], integral_constant<int, 0x4E>()));                                   // quad_perm [2,3,0,1]
    return fmaxf(a[0], dpp(a[0], integral_constant<int, 0xB1>()));                                   // quad_perm [1,0,3,2]
}

// One wave, one unit of 64 tokens of (b, h), a token per lane.  Channels go 32 at a time, 4 KB of LDS per group as in k_tile, but a lane's
// pieces are the same 32 tokens of one column in all three planes (32 + 16 + 16 bytes), so that it puts the fp16 values together in front
// of the turn: one LDS read per column and nothing but a conversion behind it.  All HI bytes are asked for at the start, in front of
// the levels, all MID and LO bytes as soon as these are known: one round trip to memory each.
// What bounds a short call is the number of instructions of one wave: a wave that has a SIMD to itself takes 4.5 to 5.5 cycles for each,
// whatever its loads.  So a unit is as small as lanes allow.  Against half a block per wave by k_tile, and two waves
// per block in groups of eight, us a call: 8 pairs of four heads 1024 tokens 25.0 -> 20.5, 8192 36.0 -> 28.7; of eight heads 8192 41.8 -> 33.2;
// 32 single heads 4096 28.4 -> 28.8
constexpr int kSUnit = 64, kSCols = 32, kSGroups = kD / kSCols, kSPerBlk = kTB / kSUnit;
struct KShortHi { u32x4_t w[kSGroups][2]; };
__device__ __forceinline__ void k_short_hi(const DecodeArgs& a, int b, int h, int unit, int len, KShortHi& hi)
{
    const uint32_t lane = threadIdx.x & 63, col = lane >> 1, t = (lane & 1) * 32;
    const size_t blk = (size_t(b) * a.s.Hkv + h) * (a.s.Ncap / kTB) + unit / kSPerBlk;
    const __amdgpu_buffer_rsrc_t rh = make_rsrc(a.k_hi + blk * kTB * kD, uint32_t(kTB) * kD);
    // pieces whose tokens all lie at or past len are asked for out of range: nothing is fetched
    const uint32_t off = unit * kSUnit + int(t) < len ? col * kTB + uint32_t(unit % kSPerBlk) * kSUnit + t : kSkip;
#pragma unroll
    for (int i = 0; i < kSGroups; ++i) {
        hi.w[i][0] = buf_load_b128(rh, off + i * kSCols * kTB);
        hi.w[i][1] = buf_load_b128(rh, off + i * kSCols * kTB + 16);
    }
}

// the token of a lane, and the place of a token in an LDS row (assemble8_fill's order; the exchange is its own inverse)
__device__ __forceinline__ int k_short_token(int lane) { return (lane & ~3) | ((lane & 1) << 1) | ((lane >> 1) & 1); }

// acc[g]: the logit of token unit * 64 + k_short_token(lane) for query head g, by the same multiply-adds in the same order as in k_tile
// at_new: the token of the unit that is being appended, or -1; its values come from knew, channel 32 i + lane % 32 in word i, and not from the planes.
template <int G>
__device__ __forceinline__ void k_short_tile(const DecodeArgs& a, int b, int h, int unit, int len, const KPairLevels& lv, const KShortHi& hi,
                                             const KShortQ<G>& ks, uint8_t* stage, float (&acc)[G], int at_new, const uint32_t (&knew)[kSGroups])
{
    constexpr bool MX = G % 4 == 0;       // groups of four and eight: matrix products of depth one, as in k_tile
    constexpr int S = MX ? G / 4 : 1;
    const int lane = threadIdx.x & 63;
    const uint32_t col = uint32_t(lane) >> 1, t = (lane & 1) * 32;
    const size_t blk = (size_t(b) * a.s.Hkv + h) * (a.s.Ncap / kTB) + unit / kSPerBlk;
    const __amdgpu_buffer_rsrc_t rm = make_rsrc(a.k_mid + blk * kTB * (kD / 2), uint32_t(kTB) * (kD / 2));
    const __amdgpu_buffer_rsrc_t rl = make_rsrc(a.k_lo + blk * kTB * (kD / 2), uint32_t(kTB) * (kD / 2));
    const uint32_t noff = unit * kSUnit + int(t) < len ? (col * kTB + uint32_t(unit % kSPerBlk) * kSUnit + t) / 2 : kSkip;
    // the lane's column of group i is channel 32 i + col: bit 16 i + col / 2 of the word of its parity
    const uint64_t mid_l = ((col & 1) ? lv.mid[1] : lv.mid[0]) >> (col / 2), lo_l = ((col & 1) ? lv.lo[1] : lv.lo[0]) >> (col / 2);
    u32x4_t m[kSGroups], l[kSGroups];
#pragma unroll
    for (int i = 0; i < kSGroups; ++i) {
        m[i] = buf_load_b128(rm, (mid_l >> (i * kSCols / 2)) & 1u ? noff + i * kSCols * (kTB / 2) : kSkip);
        l[i] = buf_load_b128(rl, (lo_l >> (i * kSCols / 2)) & 1u ? noff + i * kSCols * (kTB / 2) : kSkip);
    }
    f32x4_t dx[S];
#pragma unroll
    for (int s = 0; s < S; ++s) dx[s] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = 0.0f;
    // LDS: column c of the group is a row of 64 halves in pieces of eight tokens (16 bytes); the pieces of a row are permuted by its
    // number, so that the lanes of a store meet on few banks.  Inside a piece tokens lie as 0 2 1 3 4 6 5 7 (assemble8_fill).  The transposing
    // read hands a lane the values of four columns at its own place: lane n of sixteen reads four values of row n / 4 and receives value n of all
    // four rows.
    constexpr uint32_t kRow = kSUnit * 2;
    const uint32_t n = lane & 15, piece = 2 * (lane >> 4) + ((n & 3) >> 1);
    uint32_t rd[2], wr[4];   // rd: of rows 8 v .. 8 v + 3 and of the next four
#pragma unroll
    for (int e = 0; e < 2; ++e) rd[e] = (4 * e + (n >> 2)) * kRow + ((piece ^ (4 * e + (n >> 2))) << 4) + 8 * (n & 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) wr[k] = col * kRow + (((t / 8 + k) ^ (col & 7)) << 4);
#pragma unroll
    for (int i = 0; i < kSGroups; ++i) {
        const bool need1 = (mid_l >> (i * kSCols / 2)) & 1u, need2 = (lo_l >> (i * kSCols / 2)) & 1u;
        const uint32_t fill = need2 ? 0u : (need1 ? 0x08080808u : 0x80808080u);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 4; ++k) {   // eight tokens
            uint32_t w[4];
            assemble8_fill(hi.w[i][k >> 1][2 * (k & 1)], hi.w[i][k >> 1][2 * (k & 1) + 1], m[i][k], l[i][k], fill, w);
            *reinterpret_cast<u32x4_t*>(stage + wr[k]) = u32x4_t{w[0], w[1], w[2], w[3]};
        }
        if (at_new >= 0 && lane < kSCols) {   // behind the stores above: LDS serves a wave's accesses in order
            const uint32_t c = uint32_t(lane), place = k_short_token(at_new);
            *reinterpret_cast<uint16_t*>(stage + c * kRow + (((place >> 3) ^ (c & 7)) << 4) + 2 * (place & 7)) = (uint16_t)knew[i];
        }
        __builtin_amdgcn_wave_barrier();
        short4_t x[kSCols / 4];   // of four columns each
#pragma unroll
        for (int v = 0; v < kSCols / 4; ++v) {
            typedef __attribute__((address_space(3))) short4_t* lds_ptr;
            x[v] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)reinterpret_cast<short4_t*>(stage + rd[v & 1] + (v >> 1) * 8 * kRow));
        }
#pragma unroll
        for (int v = 0; v < kSCols / 4; ++v) {
            f32x4_t qx[MX ? S : G];   // four columns of head lane % 4 (+ 4 s), or of every head
#pragma unroll
            for (int s = 0; s < (MX ? S : G); ++s) qx[s] = *reinterpret_cast<const f32x4_t*>(&ks.q[MX ? 4 * s + (lane & 3) : s][i * kSCols + 4 * v]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float k = half_bits_to_float((uint16_t)x[v][u]);
                if constexpr (MX) {
#pragma unroll
                    for (int s = 0; s < S; ++s) dx[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(qx[s][u], k, dx[s], 0, 0, 0);
                } else {
#pragma unroll
                    for (int g = 0; g < G; ++g) acc[g] = fmaf(qx[g][u], k, acc[g]);
                }
            }
        }
        // The sums are wanted here: left to itself the compiler puts the multiply-adds of all groups behind the last one and holds their operands
        // until then (one head 180 registers instead of 104, two heads 282 instead of 112, one workgroup per compute unit).  us a call: 32 pairs
        // of two heads 8192 tokens 42.3 -> 36.2, ragged 34.9 -> 29.0, 160 pairs 2048 48.2 -> 40.6, 640 pairs 512 55.9 -> 48.7; 128 single
        // heads 2048 30.5 -> 29.8, 320 pairs 1024 37.0 -> 35.9
        if constexpr (!MX)
#pragma unroll
            for (int g = 0; g < G; ++g) asm volatile("" : "+v"(acc[g]));
    }
    __builtin_amdgcn_wave_barrier();
    if constexpr (MX)
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = dx[g / 4][g % 4];
}

}  // namespace akv
