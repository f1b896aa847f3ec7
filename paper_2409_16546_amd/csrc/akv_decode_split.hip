// Decode attention, token-split path: the tokens of every (sequence, KV head) are spread over many
// workgroups (long contexts, few heads).  Three kernels:
//   K kernel          Rule 1 levels + q.K~, a 256-token block per wave, or a quarter of one in calls of few blocks (akv_k_short.h);
//   selection kernel  one workgroup per (sequence, query head): max, approximate top-k, O_est and the result exponents;
//   V kernel          Rule 2 + S.V~ over chunks of tokens; the workgroup that finishes last combines the chunks.
// Sections "Quantization of K-Cache", "Quantization of V-Cache", "Runtime of AlignedKV".
#include <type_traits>
#include "akv_common.h"
#include "akv_k_short.h"
#include "akv_k_tile.h"
#include "akv_mid_step.h"
#include "akv_v_rows.h"

namespace akv {

// Fused append: one token per sequence.  Its K row is in no plane yet when the tiles run: they take its values from k_new.  The workgroup of the
// K kernel that walks its block stores its V row, which the kernels behind read; its K bytes and K_colmax, which they do not, are stored by that
// workgroup as well or by the selection kernel (a.k_late).  The V kernel moves the length.
__device__ __forceinline__ void count_flags(const DecodeArgs& a, const SeqLen& sl, int h, int at)
{
    if (at || h || threadIdx.x) return;
    if (sl.stored + (sl.appended ? 1 : 0) > a.max_len) atomicAdd(&a.flags[AKV_FLAG_MAXLEN], 1);
    if (a.k_new && !sl.appended) atomicAdd(&a.flags[AKV_FLAG_OVERFLOW], 1);   // a full sequence keeps its tokens
}
struct NewToken {
    int k_bits = -1;                  // of one channel
    uint32_t old_m = 0, old_l = 0;    // the nibble bytes the new token shares with its neighbour
    __device__ __forceinline__ void load(const DecodeArgs& a, const SeqLen& sl, size_t bh, int d, bool stores)
    {
        if (!sl.appended || d < 0 || d >= kD) return;
        k_bits = a.k_new[bh * kD + d];
        if (stores && (sl.stored & 1)) {   // an even place opens its nibble byte
            const size_t nib = k_nibble_index(bh, a.s.Ncap, sl.stored, d);
            old_m = a.k_mid[nib];
            old_l = a.k_lo[nib];
        }
    }
    __device__ __forceinline__ uint32_t store_k(const DecodeArgs& a, const SeqLen& sl, size_t bh, int d, bool nt) const
    {
        return store_token_k(const_cast<uint8_t*>(a.k_hi), const_cast<uint8_t*>(a.k_mid), const_cast<uint8_t*>(a.k_lo), bh, a.s.Ncap, sl.stored, d,
                             uint32_t(k_bits), old_m, old_l, nt);
    }
};
__device__ __forceinline__ void store_new_v(const DecodeArgs& a, const SeqLen& sl, size_t bh, int d)
{
    store_token_v(const_cast<uint8_t*>(a.v_hi), const_cast<uint8_t*>(a.v_mid), const_cast<uint8_t*>(a.v_lo), bh, a.s.Ncap, sl.stored, d, a.v_new + bh * kD);
}

// K kernel: workgroup = kKWaves waves of one (sequence, KV head).  A wave walks one 256-token block (k_tile) and leaves its logits and the
// block's maxima in the workspace.
template <int G>
__global__ __launch_bounds__(64 * kKWaves) void split_k_kernel(DecodeArgs a)
{
    __shared__ __align__(16) uint8_t kstage[kKWaves][kKStage];
    __shared__ KShared<G> ks;

    const int h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63;
    const int Hq = a.s.Hq, Ncap = a.s.Ncap;
    const SeqLen sl(a, b);
    const int len = sl.len;
    const int wave_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int blk = blockIdx.x * kKWaves + wave_u;
    if (blockIdx.x * kKWaves * kTB >= len) return;   // whole workgroup beyond the sequence (uniform)

    const size_t bh = size_t(b) * a.s.Hkv + h;
    count_flags(a, sl, h, blockIdx.x);
    KLevelsIn<G> in;
    k_levels_load<G>(a, b, h, in);
    const int d = threadIdx.x;
    NewToken nt;
    const bool owner = sl.owner(kTB * kKWaves, blockIdx.x);
    nt.load(a, sl, bh, d, owner && !a.k_late);
    const uint32_t colmax_used = k_levels_finish<G>(a, b, h, ks, blockIdx.x == 0, nt.k_bits, in, len);
    if (blk * kTB < len) {                    // else this wave's block is beyond the sequence
        float tm[G];
        const u32x4_t zero4 = {0u, 0u, 0u, 0u};
        const u32x4_t none[6] = {zero4, zero4, zero4, zero4, zero4, zero4};
        float lg[G][4];
        const size_t hq0 = size_t(b) * Hq + size_t(h) * G;
        if (sl.attend_new() && blk == sl.stored / kTB) k_tile<G, true, 4, true>(a, b, h, hq0, blk, len, ks, tm, none, false, lg, &kstage[wave_u][0], nullptr, 0, sl.stored % kTB);
        else k_tile<G>(a, b, h, hq0, blk, len, ks, tm, none, false, lg, &kstage[wave_u][0]);
        if (lane == 0)
#pragma unroll
            for (int g = 0; g < G; ++g) a.tilemax[(hq0 + g) * (Ncap / kMinUnit) + blk] = tm[g];
    }
    if (owner && d < kD) {
        if (!a.k_late) {
            nt.store_k(a, sl, bh, d, false);
            const_cast<uint16_t*>(a.colmax)[bh * kD + d] = (uint16_t)colmax_used;
        }
        store_new_v(a, sl, bh, d);
    }
}

// The same for calls with few blocks (akv_k_short.h): the four waves of a workgroup take a quarter of its block each, find the levels
// by themselves and have all their HI bytes in flight meanwhile.
template <int G>
__global__ __launch_bounds__(64 * kKWaves) void split_k_short_kernel(DecodeArgs a)
{
    static_assert(kKWaves * kSUnit == kTB, "a block per workgroup");
    __shared__ __align__(16) uint8_t kstage[kKWaves][kKStage];
    __shared__ KShortQ<G> ks;
    __shared__ float best_s[kKWaves][G];

    const int h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63;
    const int Hq = a.s.Hq, Ncap = a.s.Ncap;
    KPairIn<G> in;
    k_pairs_load<G>(a, b, h, in);
    const SeqLen sl(a, b);
    const int len = sl.len;
    const int wave_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const unsigned turned = blockIdx.x + unsigned(b * a.s.Hkv + h) * unsigned(a.kturn);
    const int at = int(turned < gridDim.x ? turned : turned - gridDim.x);   // the block of this workgroup
    const int unit = at * kKWaves + wave_u;
    if (at * kTB >= len) return;   // whole workgroup beyond the sequence (uniform)
    KShortHi hi;
    k_short_hi(a, b, h, unit, len, hi);
    const size_t bh = size_t(b) * a.s.Hkv + h;
    count_flags(a, sl, h, at);
    const bool owner = sl.owner(kTB, at);
    NewToken nt;
    nt.load(a, sl, bh, threadIdx.x, owner);
    if (sl.appended) in.cm = max_halves(in.cm, in.knew & 0x7FFF7FFFu);
    const KPairLevels lv = k_pair_levels<G>(a, b, h, ks, in, unit == 0, len);
    const size_t hq0 = size_t(b) * Hq + size_t(h) * G;
    float best = -INFINITY;   // of head lane / (64 / G)
    if (unit * kSUnit < len) {                    // else this wave's unit is beyond the sequence
        float lg[G], m[G];
        uint32_t knew[kSGroups] = {};
        const int at_new = sl.attend_new() && unit == sl.stored / kSUnit ? sl.stored % kSUnit : -1;   // uniform
        if (at_new >= 0) k_pair_read(in.knew, lv, knew);
        k_short_tile<G>(a, b, h, unit, len, lv, hi, ks, &kstage[wave_u][0], lg, at_new, knew);
        const int t = unit * kSUnit + k_short_token(lane);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            a.logits[(hq0 + g) * Ncap + t] = lg[g];
            m[g] = t < len ? lg[g] : -INFINITY;
        }
        best = wave_max_each<G>(m);
    }
    if (lane % (64 / G) == 0) best_s[wave_u][lane / (64 / G)] = best;
    __syncthreads();
    if (threadIdx.x < G) {
        float m = best_s[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kKWaves; ++w) m = fmaxf(m, best_s[w][threadIdx.x]);
        a.tilemax[(hq0 + threadIdx.x) * (Ncap / kMinUnit) + at] = m;
    }
    if (owner) {   // a.k_late is for calls of many blocks
        if (threadIdx.x < kD) {
            nt.store_k(a, sl, bh, threadIdx.x, false);
            store_new_v(a, sl, bh, threadIdx.x);
        }
        if (threadIdx.x < 64) reinterpret_cast<uint32_t*>(const_cast<uint16_t*>(a.colmax + bh * kD))[lane] = in.cm;
    }
}

// Mid step: one workgroup per (sequence, query head) does all of it -- the global max logit, the approximate top-k, O_est
// and the result exponents of its head.  Each wave finds M by itself and takes a contiguous range of the blocks, in token order:
//   pass 1  the histogram of its tokens' score exponents (LDS);
//   cut     from the totals, and from the waves in front of it how many selected tokens precede its range;
//   pass 2  ballots place the selected tokens.
// Up to kKeep blocks per wave it reads all of them at the start, beside the maxima, and keeps their logits in registers.  Of longer sequences
// it reads only the K blocks that can hold a selected token: every block maximum the K kernel left behind is itself a token, and so is the
// largest of those that fall on one lane (block i on lane i % 64); the bucket Jb in which the running count of the lanes' maxima reaches k'
// is an upper bound of the cut bucket, and a block whose best token lies beyond Jb holds nothing that counts (the floor bucket needs no
// count: it is what is left of the range).  Pass 2 fetches the blocks up to the cut again (from L2) only where a wave had more than kKeep, or
// the cut is the floor bucket; a block whose best token is in the cut bucket itself is then passed over once enough tokens of it have been seen.
// Bound by its chain of dependent steps, not by bytes: a wave takes 4.5 to 5.5 cycles an instruction, 25 to 30 where a scalar one needs the
// result of a vector one, and two or three round trips to memory of some 900 cycles; so a head has a workgroup of its own, and its
// loops run over blocks that are there only.
// Measured against a histogram of the block maxima by LDS atomics, two barriers more, and code for every slot whether it held a block or
// not: B 1, 32/8, 1024 tokens 18.4 -> 16.9 us a call, 4096 22.3 -> 21.0, 8192 27.0 -> 24.8, B 3, 64/8, 13000 57.0 -> 55.6; longer ones equal.
// kKeep: four blocks of a wave leave 54 registers, four workgroups of 512 threads to a compute unit; eight took 86 and two workgroups, and calls
// of many heads paid for it (eight / four, us a call: 4096 heads 256 tokens 70.9/63.3, 2048 214.5/205.3, 2048 heads 1024 72.3/68.2, 1024 heads
// 512 51.2/50.3; fewer heads and long sequences equal).
// NT: 512 threads, or 1024 where every head can have a compute unit to itself and has more than 16 blocks (512 / 1024: B 1, 32/8, 1024 tokens
// 16.9/17.6, 4096 21.0/21.0, 32768 47.1/45.9, B 3, 64/8, 13000 57.4/55.6; with 512 heads of 16 blocks 57.7/61.1).
// LATE: a.k_late (a variant of its own: other calls run nothing of it)
template <int NT, bool LATE>
__global__ __launch_bounds__(NT, LATE && NT == 512 ? 8 : 1) void split_select_kernel(DecodeArgs a)
{
    constexpr int kWaves = NT / 64, kKeep = 4;   // kKeep: blocks of a wave in flight
    __shared__ MidShared ms;
    __shared__ int hist_s[kWaves][64 + 64];      // per wave: buckets 0..63, and a place per lane for tokens that need no count

    const int hq_i = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Hq = a.s.Hq, Hkv = a.s.Hkv, Ncap = a.s.Ncap;
    const SeqLen sl(a, b);
    const int len = sl.len;
    if (tid == 0) a.tilemax[(size_t(b) * Hq + hq_i) * (Ncap / kMinUnit) + Ncap / kTB] = bits_float((uint32_t)len);   // for the V kernel, which moves lens
    if (len <= 0) return;   // uniform: an empty sequence has no selection (the V kernel writes its zeros)
    const int G = Hq / Hkv;
    const size_t hq = size_t(b) * Hq + hq_i, bh = size_t(b) * Hkv + hq_i / G;
    // fused append, a.k_late: the workgroups of a group's heads store an equal share of the new token's channels each, by waves 2 and 3, which have
    // nothing to do while O_est is added up
    static_assert(NT >= 2 * kD, "");
    const int d_new = tid - kD;
    const bool stores = LATE && sl.appended && d_new >= 0 && d_new < kD && d_new * G / kD == hq_i % G;
    NewToken nt;
    uint32_t colmax = 0;
    if (stores) {
        nt.load(a, sl, bh, d_new, true);
        colmax = a.colmax[bh * kD + d_new];
    }
    const int nblk = (len + kTB - 1) / kTB;
    const int kk = a.topk < len ? a.topk : len;
    const int b0 = int((long long)nblk * wave / kWaves), b1 = int((long long)nblk * (wave + 1) / kWaves);   // the wave's blocks
    const bool all = nblk <= kKeep * kWaves;   // every wave reads all of its blocks, and keeps them
    const __amdgpu_buffer_rsrc_t rs_tm = make_rsrc(a.tilemax + hq * (Ncap / kMinUnit), uint32_t(Ncap / kTB) * 4u);
    const __amdgpu_buffer_rsrc_t rs_lg = make_rsrc(a.logits + hq * Ncap, uint32_t(Ncap) * 4u);
    int nb = 0, blk[kKeep];   // the blocks at hand (uniform) and their logits (lane -> four consecutive tokens)
    u32x4_t w[kKeep];
    auto ask = [&](int u, int block) {
        blk[u] = block;
        w[u] = buf_load_b128(rs_lg, uint32_t(block) * (kTB * 4u) + uint32_t(lane) * 16u);
    };

    // ---- the global max logit (exact, order-free)
    float m = -INFINITY;   // of the blocks of this lane
    for (int i0 = 0; i0 < nblk; i0 += 4 * 64) {
        float t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = bits_float(buf_load_b32(rs_tm, uint32_t(i0 + 64 * i + lane) * 4u));
        if (all) {   // nothing to decide first: the logits are on their way beside the maxima (one turn: nblk <= 64)
            nb = b1 - b0;
#pragma unroll
            for (int u = 0; u < kKeep; ++u)
                if (u < nb) ask(u, b0 + u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) m = fmaxf(m, i0 + 64 * i + lane < nblk ? t[i] : -INFINITY);
    }
    hist_s[wave][lane] = 0;   // read and written by this wave alone up to the cut
    const float M = wave_max(m);
    // score and score exponent of the tokens of block blk[u] (score_x, score_a); -1000 past the sequence
    auto score4 = [&](int u, float (&x)[4], int (&e)[4]) {
        const float lv[4] = {bits_float(w[u].x), bits_float(w[u].y), bits_float(w[u].z), bits_float(w[u].w)};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = score_x(lv[i], M, a.c);
            e[i] = floor_int(fmaxf(x[i], (float)kAMin));   // the maximum passes over a score that is not a number
        }
        if ((blk[u] + 1) * kTB > len)   // uniform
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = blk[u] * kTB + lane * 4 + i < len ? e[i] : -1000;
    };
    // buckets before `top` are counted by LDS atomics, bucket `top` in the lanes (n_top), later ones not at all: atomics of a whole wave on one
    // address take a cycle per lane, and where scores are flat nearly all tokens of a long sequence are in the cut bucket (B 1, 32/8, 131072
    // tokens of equal scores: every bucket by atomics 217 us a call, so 125)
    int n_top = 0;
    auto count = [&](int top) {
#pragma unroll
        for (int u = 0; u < kKeep; ++u) {
            if (u >= nb) break;   // uniform
            float x[4];
            int e[4];
            score4(u, x, e);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                atomicAdd(&hist_s[wave][e[i] > -top ? -e[i] : 64 + lane], 1);
                n_top += e[i] == -top;
                if (a.dbg.a && e[i] >= kAMin) a.dbg.a[hq * Ncap + blk[u] * kTB + lane * 4 + i] = (int8_t)e[i];
            }
        }
    };
    // bucket of the best token of block c0 + lane (1000 past the range)
    auto best_of = [&](int c0) {
        const float best = bits_float(buf_load_b32(rs_tm, uint32_t(c0 + lane) * 4u));
        return c0 + lane < b1 ? -score_a(score_x(best, M, a.c)) : 1000;
    };
    // takes up to kKeep blocks off the mask
    auto take = [&](int c0, uint64_t& mask) {
        nb = min((int)__builtin_popcountll(mask), kKeep);
#pragma unroll
        for (int u = 0; u < kKeep; ++u) {
            if (u >= nb) break;   // uniform
            ask(u, c0 + __builtin_ctzll(mask));
            mask &= mask - 1;
        }
    };
    // ---- pass 1
    bool kept = all;
    if (all) {
        count(64);
    } else {
        // the bound of the cut: the smallest bucket that k' lanes reach, each with a token of its own (64 if fewer do)
        const int j = lane < nblk ? -score_a(score_x(m, M, a.c)) : 1000;
        int Jb = 0;
#pragma unroll
        for (int step = 64; step > 0; step >>= 1) Jb += __builtin_popcountll(__ballot(j < Jb + step)) < kk ? step : 0;
        Jb = min(Jb, 64);
        for (int c0 = b0; c0 < b1; c0 += 64) {
            const int best = best_of(c0);
            uint64_t mask = __ballot(a.dbg.a ? best <= 64 : best <= min(Jb, 63));   // the export wants every token
            kept = b1 - b0 <= 64 && __builtin_popcountll(mask) <= kKeep;
            while (mask) {
                take(c0, mask);
                count(Jb);
            }
        }
        if (Jb < 64) {
            n_top = wave_read(wave_scan_add(n_top), 63);
            if (lane == 0) hist_s[wave][Jb] = n_top;
        }
    }
    __syncthreads();
    // ---- the cut, and the selected tokens of each kind in the waves before this one
    int tot = 0, before = 0;   // bucket `lane`: all waves / the waves before this one
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
        const int c = hist_s[v][lane];
        tot += c;
        before += v < wave ? c : 0;
    }
    // both running counts in one scan, sixteen bits each: neither is told apart above k' <= 64, in 64 buckets
    const int upto = wave_scan_add(min(tot, AKV_MAX_TOPK) | min(before, AKV_MAX_TOPK) << 16);
    const uint64_t reached = __ballot((upto & 0xFFFF) >= kk);
    const int J = reached ? __builtin_ctzll(reached) : 64;   // 64, the floor bucket, if none before it is the cut
    const int sum = J == 0 ? 0 : wave_read(upto, J - 1);      // of the buckets before the cut, none of which holds k' tokens
    const int fromcut = kk - (sum & 0xFFFF);
    int n_lt0 = sum >> 16;
    int n_eq0 = J < 64 ? wave_read(before, J) : min(b0 * kTB, len) - n_lt0;   // the cut in the floor bucket: all tokens before it are in buckets before it or in it
    // ---- pass 2.  Selected tokens go to their places in sel and score (place AKV_MAX_TOPK takes the others)
    auto emit = [&](int u, int i, float x, int pos, bool on) {
        pos = on ? pos : AKV_MAX_TOPK;
        ms.sel[pos] = blk[u] * kTB + lane * 4 + i;
        ms.phat[pos] = x;
    };
    auto place = [&] {
#pragma unroll
        for (int u = 0; u < kKeep; ++u) {
            if (u >= nb) break;   // uniform
            float x[4];
            int e[4], w_eq = 0, w_all = 0, n = 0;
            score4(u, x, e);
            if (!__ballot(max(max(e[0], e[1]), max(e[2], e[3])) >= -J)) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) w_eq += __builtin_popcountll(__ballot(e[i] == -J));
            if (n_eq0 >= fromcut || n_eq0 + w_eq <= fromcut) {   // the tokens of bucket J are all left out or all in: one kind
                const int least = n_eq0 >= fromcut ? 1 - J : -J;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint64_t on = __ballot(e[i] >= least);
                    n = __builtin_amdgcn_mbcnt_hi((uint32_t)(on >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)on, n));
                    w_all += __builtin_popcountll(on);
                }
                n += n_lt0 + min(n_eq0, fromcut);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    emit(u, i, x[i], n, e[i] >= least);
                    n += e[i] >= least;
                }
                n_lt0 += n_eq0 >= fromcut ? w_all : w_all - w_eq;
            } else {
                int j[4], n_lt, n_eq, w_lt;
#pragma unroll
                for (int i = 0; i < 4; ++i) j[i] = -e[i];
                mid_wave_order(j, J, n_lt, n_eq, w_lt, w_eq);
                n_lt += n_lt0;
                n_eq += n_eq0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    emit(u, i, x[i], n_lt + min(n_eq, fromcut), j[i] < J || (j[i] == J && n_eq < fromcut));
                    n_lt += j[i] < J;
                    n_eq += j[i] == J;
                }
                n_lt0 += w_lt;
            }
            n_eq0 += w_eq;
        }
    };
    if (kept && (all || J < 64)) {   // the blocks of pass 1, which are those up to the cut and perhaps more; the floor bucket may be in any block
        place();
    } else {
        for (int c0 = b0; c0 < b1; c0 += 64) {
            const int best = best_of(c0);
            uint64_t mask = __ballot(best <= J);
            while (mask) {
                if (n_eq0 >= fromcut) mask &= __ballot(best < J);   // blocks that could only add to the cut bucket
                if (!mask) break;
                take(c0, mask);
                place();
            }
        }
    }
    __syncthreads();
    if (tid < kk) {   // the weight: 2^x with a linear mantissa, the exponent floored at -64
        const float x = ms.phat[tid], fl = floorf(x);
        ms.phat[tid] = ldexpf(1.0f + (x - fl), score_a(x));
    }
    int ehat = 32767;
    mid_oest<NT>(a, bh, hq, kk, ms, ehat);
    if (stores) {
        const uint32_t mag = nt.store_k(a, sl, bh, d_new, true);
        if (mag > colmax) const_cast<uint16_t*>(a.colmax)[bh * kD + d_new] = (uint16_t)mag;
    }
    if (tid < kD) a.Ehat[hq * kD + tid] = ehat;
    if (tid == 0) a.M[hq] = M;
}

// Workgroup = kVWaves waves, one (sequence, KV head, chunk of a.vchunk tokens); wave w takes the batches of rows
// w, w + kVWaves, ... of the chunk.  Groups of four or eight query heads run v_rows_shared: every wave
// fetches and assembles its rows once, the rows pass through LDS, and the sums over rows for all heads of the group
// are matrix products on the matrix cores.
template <int G> constexpr bool v_shared() { return G >= kVWaves; }
template <int G, bool DEBUG>
__global__ __launch_bounds__(64 * kVWaves) void split_v_kernel(DecodeArgs a)
{
    constexpr bool SHARED = v_shared<G>();
    constexpr int KG = 2, RB = 8 * KG;                      // rows of a batch
    static_assert(RB == kSRows && (kVMinChunk % (RB * kVWaves)) == 0, "a chunk is whole rounds");
    // a chunk's partial sums are kCols vectors of four; the combining workgroup: a thread takes one of them over every kSub-th chunk
    constexpr int kCols = G * kD / 4, kSub = 64 * kVWaves / kCols;
    struct Private { union { float red[kVWaves][G][kD]; f32x4_t comb[kSub][kCols]; }; };
    struct Shared { union { VShare rows; f32x4_t comb[kSub][kCols]; }; };
    __shared__ __align__(16) std::conditional_t<SHARED, Shared, Private> lds_s;
    __shared__ float z_s[kVWaves][G];
    __shared__ VRuleShared rule_s;
    __shared__ int last_s;

    const int h = blockIdx.y, b = blockIdx.z, split = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cl = lane & 7;
    const int Hkv = a.s.Hkv, Hq = a.s.Hq, Ncap = a.s.Ncap;
    const int len = __builtin_amdgcn_readfirstlane((int)float_bits(a.tilemax[(size_t(b) * Hq + size_t(h) * G) * (Ncap / kMinUnit) + Ncap / kTB]));   // the attended length
    if (a.k_new && split == 0 && h == 0 && tid == 0) {   // fused append: nothing else of this kernel reads lens
        int32_t* const stored = const_cast<int32_t*>(a.lens) + b;
        if (*stored < Ncap) *stored += 1;
    }
    const int vchunk = a.vchunk;   // tokens per workgroup: a multiple of 64 chosen at launch
    const int c0 = split * vchunk;
    const size_t bh = size_t(b) * Hkv + h;
    const int nsplit = a.vslots;
    if (c0 >= len) {                                    // uniform: chunk beyond the sequence
        if (len == 0 && split == 0)                     // an empty sequence attends to nothing: zeros
            for (int idx = tid; idx < G * kD; idx += 64 * kVWaves)
                store_out(a, size_t(b) * Hq + size_t(h) * G + idx / kD, idx % kD, 0.0f);
        return;
    }

    // Rule 2 aligns to the smallest result exponent of the group.  Asked for in front of the rows; worked out (ready()) when the first
    // rows are on their way
    const size_t hq0 = size_t(b) * Hq + size_t(h) * G;
    int eg[G];
#pragma unroll
    for (int g = 0; g < G; ++g) eg[g] = a.Ehat[(hq0 + g) * kD + tid % kD];
    float Ml[SHARED ? G / 4 : 1];   // the global max of this lane's query heads (one load per lane: taken for all heads at once they went through scratch memory, a round trip each)
#pragma unroll
    for (int s = 0; s < (SHARED ? G / 4 : 1); ++s) Ml[s] = a.M[hq0 + 4 * s + lane % (SHARED ? 4 : G)];
    auto ready = [&](auto& vr) {
        if (tid < kD) {
            int e = eg[0];
#pragma unroll
            for (int g = 1; g < G; ++g) e = min(e, eg[g]);
            v_rule_store(rule_s, tid, e, a.guard_bits);
            if (a.dbg.Ehat && split == 0) a.dbg.Ehat[bh * kD + tid] = (int16_t)e;
        }
        lds_barrier();
        v_rule_load(rule_s, a.force_level, vr);
    };
    const __amdgpu_buffer_rsrc_t rs_o = make_rsrc(a.partO + bh * G * nsplit * kD, uint32_t(G) * uint32_t(nsplit) * kD * 4u);
    float* const part_z = a.partZ + bh * G * nsplit;
    // HI bytes fetched three or four batches ahead in the private mode (few waves per SIMD: each keeps more bytes in
    // flight), two in the shared mode (four waves per SIMD; three and four measured 1.5 % and 3 % slower;
    // where waves are few, four ahead with the decisions three ahead gains nothing: a round of a wave by itself is 2300 cycles of instructions).
    constexpr int DL = SHARED ? 2 : (G == 2 ? 4 : 3);
    if constexpr (SHARED) {
        VRule<4> vr;
        float acc[8], z[G / 4];
#pragma unroll
        for (int s = 0; s < G / 4; ++s) z[s] = 0.0f;
        v_rows_shared<G, DEBUG, DL>(a, b, h, c0 + wave * RB, vchunk / (RB * kVWaves), len, vr, Ml, acc, z, lds_s.rows, [&] { ready(vr); });
#pragma unroll
        for (int s = 0; s < G / 4; ++s) {   // over the lanes of the same query heads
            z[s] = wave_sum<4>(z[s]);
            if (lane < 4) z_s[wave][lane + 4 * s] = z[s];
        }
        // a result tile holds the high parts of the weights in its rows 0 .. G-1 and the low parts in rows G .. 2G-1:
        // lanes 16 * (G / 4) apart hold the two parts of one (query head, line).  A lane's four words are those of four query heads for
        // one line, and as such they go out: vector 128 (lane / 16) + line of the chunk
        f32x4_t part[2];
#pragma unroll
        for (int i = 0; i < 8; ++i) part[i / 4][i % 4] = (G == 4 ? add_lane16(acc[i]) : add_lane32(acc[i])) * (1.0f / kVWeightScale);
        if (lane < 4 * G) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
                buf_store_b128_agent(__builtin_bit_cast(u32x4_t, part[t]), rs_o, (uint32_t(split) * kCols + kD * uint32_t(lane >> 4) + uint32_t(32 * wave + 16 * t + (lane & 15))) * 16u);
        }
        __syncthreads();
    } else {
        VRule<> vr;
        float acc[G][16], z[G], sum[G][2];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            z[g] = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[g][i] = 0.0f;
        }
        const u32x4_t none[1][KG] = {};
        v_rows<G, KG, DEBUG, 0, DL, true>(a, b, h, c0 + wave * RB, RB * kVWaves, vchunk / (RB * kVWaves), len, vr, Ml[0], acc, z, none, false, nullptr, 0, [&] { ready(vr); });
        v_reduce_rows<G>(acc, z, sum);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            *reinterpret_cast<float2*>(&lds_s.red[wave][g][cl * 16 + row_lane_column(lane)]) = make_float2(sum[g][0], sum[g][1]);
            if (lane == 0) z_s[wave][g] = z[g];
        }
        __syncthreads();
        if (tid < kCols) {
            f32x4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int w = 0; w < kVWaves; ++w) o += *reinterpret_cast<const f32x4_t*>(&lds_s.red[w][0][4 * tid]);
            buf_store_b128_agent(__builtin_bit_cast(u32x4_t, o), rs_o, (uint32_t(split) * kCols + uint32_t(tid)) * 16u);
        }
    }
    if (tid < G) {
        float z = z_s[0][tid];
#pragma unroll
        for (int w = 1; w < kVWaves; ++w) z += z_s[w][tid];
        store_agent(&part_z[split * G + tid], z);
    }

    // ---- the workgroup that finishes last for this (sequence, KV head) combines the chunks -------------
    // out = sum_chunks O / sum_chunks Z: every chunk used the same global max, so nothing is rescaled.  All threads take part
    // with 16-byte loads, eight chunks each in flight, the weights' sums beside them; the round trips of stores, ticket and loads are
    // what is left.  (The waves' sums by exchanges in the vector ALU and straight to memory as the lanes hold them, Rule 2's constants by a
    // thread per channel, no trip through scratch memory for the maxima: B 1, 32/8, 1024 tokens 20.0 -> 18.4 us a call, 4096 24.2 -> 22.3, B 8, 32/8,
    // 32768 188 -> 182, B 4, 131072 346 -> 336.)
    const int used = (len + vchunk - 1) / vchunk;
    stores_done();
    __syncthreads();
    if (tid == 0) last_s = take_ticket(&a.vcount[bh]) == used - 1;
    __syncthreads();
    if (!last_s) return;
    const int c = tid % kCols, sub = tid / kCols;
    constexpr int kZ = 64 / G;   // chunks a wave's lanes take at a time: lane -> query head lane % G
    const __amdgpu_buffer_rsrc_t rs_z = make_rsrc(part_z, uint32_t(G) * uint32_t(used) * 4u);
    float zs = 0.0f;
    f32x4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int sp0 = 0; sp0 < used; sp0 += 8 * kSub) {   // eight chunks' words in flight; the additions stay in chunk order
        static_assert(kZ == 8 * kSub, "one word of the weights' sums per lane and turn");
        u32x4_t po[8];
        const float pz = bits_float(__builtin_amdgcn_raw_buffer_load_b32(rs_z, uint32_t((sp0 + lane / G) * G + lane % G) * 4u, 0, kAuxSc1));   // chunks past the last one: zeros
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int sp = sp0 + sub + i * kSub;
            po[i] = buf_load_b128_agent(rs_o, sp < used ? (uint32_t(sp) * kCols + uint32_t(c)) * 16u : kSkip);
        }
        zs += pz;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] += bits_float(po[i][k]);
    }
    zs = wave_sum<G>(zs);   // of query head lane % G
    if (kSub > 1) {
        lds_s.comb[sub][c] = o;
        __syncthreads();
    }
    if (sub == 0) {   // whole waves (kCols of 32, single heads: the lower half of one)
#pragma unroll
        for (int u = 1; u < kSub; ++u) o += lds_s.comb[u][c];
        // the sum of a query head's weights, from the lane that holds it: by a lane number and not from an array, whose index the compiler
        // would take through scratch memory
        auto z_of = [&](int g) { return bits_float((uint32_t)wave_read((int)float_bits(zs), g)); };
        if constexpr (SHARED) {   // four query heads of one line; whole waves have the same four
            const int quad = __builtin_amdgcn_readfirstlane(c / kD), d = line_channel(c % kD);
#pragma unroll
            for (int k = 0; k < 4; ++k) store_out(a, hq0 + 4 * quad + k, d, o[k] / z_of(4 * quad + k));
        } else {
            const int g = c / (kD / 4);
            const float z0 = z_of(0), z1 = z_of(G - 1), zk = g == 0 ? z0 : z1;
#pragma unroll
            for (int k = 0; k < 4; ++k) store_out(a, hq0 + g, (c % (kD / 4)) * 4 + k, o[k] / zk);
        }
    }
    if (tid == 0) store_agent(&a.vcount[bh], 0);   // ready for the next call
}

// Workgroups of split_v_kernel<G> per compute unit that the chunks are sized for: what the registers leave room for (single heads
// 117, groups of two 156; groups of four 104 and of eight 112, with 38 KB of LDS).
int split_v_workgroups_per_cu(int G) { return G == 2 ? 3 : 4; }

template <int G>
static hipError_t launch_split_g(const DecodeArgs& a, hipStream_t st, hipEvent_t k_done_event, hipEvent_t mid_event)
{
    const int tile = a.kshort ? kTB : kTB * kKWaves;   // tokens per workgroup of the K kernel
    const dim3 kgrid((a.max_len + tile - 1) / tile, a.s.Hkv, a.s.B), kblock(64 * kKWaves);
    if (a.kshort) hipLaunchKernelGGL(split_k_short_kernel<G>, kgrid, kblock, 0, st, a);
    else hipLaunchKernelGGL(split_k_kernel<G>, kgrid, kblock, 0, st, a);
    if (hipError_t e = hipGetLastError()) return e;
    if (k_done_event)
        if (hipError_t e = hipEventRecord(k_done_event, st)) return e;
    const int nt = a.max_len > 16 * kTB && long(a.s.B) * a.s.Hq <= compute_units() ? 1024 : 512;
    auto select = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(a.s.Hq, a.s.B), dim3(nt), 0, st, a); };
    if (a.k_new && a.k_late) nt == 1024 ? select(split_select_kernel<1024, true>) : select(split_select_kernel<512, true>);
    else nt == 1024 ? select(split_select_kernel<1024, false>) : select(split_select_kernel<512, false>);
    if (hipError_t e = hipGetLastError()) return e;
    if (mid_event)
        if (hipError_t e = hipEventRecord(mid_event, st)) return e;
    const dim3 vgrid((a.max_len + a.vchunk - 1) / a.vchunk, a.s.Hkv, a.s.B), vblock(64 * kVWaves);
    if (a.dbg.needV || a.dbg.appliedV || a.stats) hipLaunchKernelGGL((split_v_kernel<G, true>), vgrid, vblock, 0, st, a);
    else hipLaunchKernelGGL((split_v_kernel<G, false>), vgrid, vblock, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_decode_split(const DecodeArgs& a, hipStream_t st, hipEvent_t k_done_event, hipEvent_t mid_event)
{
    switch (a.s.Hq / a.s.Hkv) {
        case 1: return launch_split_g<1>(a, st, k_done_event, mid_event);
        case 2: return launch_split_g<2>(a, st, k_done_event, mid_event);
        case 4: return launch_split_g<4>(a, st, k_done_event, mid_event);
        case 8: return launch_split_g<8>(a, st, k_done_event, mid_event);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace akv
