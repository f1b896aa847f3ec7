// Decode attention, token-split path: the tokens of every (sequence, KV head) are spread over many
// workgroups (long contexts, few heads).  Three kernels:
//   K kernel          Rule 1 levels + q.K~, a 256-token block per wave, half of one, or a block per two waves;
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
    const int len = min(min(a.lens[b], Ncap), a.max_len);   // a hint below the true length: the tokens past it are left out, consistently in all kernels
    const int wave_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int blk = blockIdx.x * kKWaves + wave_u;
    if (blockIdx.x * kKWaves * kTB >= len) return;   // whole workgroup beyond the sequence (uniform)

    if (blockIdx.x == 0 && h == 0 && threadIdx.x == 0 && min(a.lens[b], Ncap) > a.max_len) atomicAdd(&a.flags[AKV_FLAG_MAXLEN], 1);
    k_levels<G>(a, b, h, ks, blockIdx.x == 0, len);
    if (blk * kTB < len) {                    // else this wave's block is beyond the sequence
        float tm[G];
        const u32x4_t zero4 = {0u, 0u, 0u, 0u};
        const u32x4_t none[6] = {zero4, zero4, zero4, zero4, zero4, zero4};
        float lg[G][4];
        const size_t hq0 = size_t(b) * Hq + size_t(h) * G;
        k_tile<G>(a, b, h, hq0, blk, len, ks, tm, none, false, lg, &kstage[wave_u][0]);
        if (lane == 0)
#pragma unroll
            for (int g = 0; g < G; ++g) a.tilemax[(hq0 + g) * (Ncap / kMinUnit) + blk] = tm[g];
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
    const int len = min(min(a.lens[b], Ncap), a.max_len);   // as in split_k_kernel
    const int wave_u = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int unit = blockIdx.x * kKWaves + wave_u;
    if (blockIdx.x * kTB >= len) return;   // whole workgroup beyond the sequence (uniform)
    KShortHi hi;
    k_short_hi(a, b, h, unit, len, hi);
    if (blockIdx.x == 0 && h == 0 && threadIdx.x == 0 && min(a.lens[b], Ncap) > a.max_len) atomicAdd(&a.flags[AKV_FLAG_MAXLEN], 1);
    const KPairLevels lv = k_pair_levels<G>(a, b, h, ks, in, unit == 0, len);
    const size_t hq0 = size_t(b) * Hq + size_t(h) * G;
    float best = -INFINITY;   // of head lane / (64 / G)
    if (unit * kSUnit < len) {                    // else this wave's unit is beyond the sequence
        float lg[G], m[G];
        k_short_tile<G>(a, b, h, unit, len, lv, hi, ks, &kstage[wave_u][0], lg);
        const int t = unit * kSUnit + lane;
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
        a.tilemax[(hq0 + threadIdx.x) * (Ncap / kMinUnit) + blockIdx.x] = m;
    }
}

// Mid step: one workgroup per (sequence, query head) does all of it -- the global max logit, the approximate top-k, O_est
// and the result exponents of its head.  It reads only the K blocks that can hold a selected token: every block maximum
// the K kernel left behind is itself a token, so the bucket Jb in which the running count of block maxima reaches k' is
// an upper bound of the cut bucket, and a block whose best token lies beyond Jb holds nothing that counts (fewer than k'
// blocks: all are read).  Each wave takes a contiguous range of the blocks, in token order:
//   pass 1  the histogram of its tokens in buckets <= Jb (LDS; the floor bucket is what is left of the range, uncounted);
//   cut     from the totals, and from the waves in front of it how many selected tokens precede its range;
//   pass 2  the blocks up to the cut once more (from L2), in order: ballots place the selected tokens.  A block whose best
//           token is in the cut bucket itself is passed over once enough tokens of that bucket have been seen.
// Bound by its chain of dependent round trips to memory (maxima, pass 1, pass 2, V rows), about a microsecond each, not by
// bytes; so a head has a workgroup of its own, with 32 blocks in flight in each pass.
// Measured on whole calls, against a pass over every logit (1024-token slices, histograms and candidates through memory)
// followed by one selecting workgroup per KV head: 198 -> 181 us (B 8, 32/8 heads, 32768 tokens), 301 -> 273 us (B 4, 32/8,
// up to 131072), 101 -> 80 us (B 3, 64/8, up to 13000); no call got slower.
// NT: 512 threads, or 1024 where every head can have a compute unit to itself and has more than 16 blocks (B 8, 32/8, 32768
// tokens 173.4 -> 171.6 us a call, B 3, 64/8, up to 13000 69.8 -> 68.9; with 512 heads of 33 blocks 283.3 -> 284.7, with 32 heads
// of 8 blocks 27.2 -> 28.0).
template <int NT>
__global__ __launch_bounds__(NT) void split_select_kernel(DecodeArgs a)
{
    constexpr int kWaves = NT / 64, kAhead = 32 / kWaves;   // kAhead: blocks of a wave in flight
    __shared__ MidShared ms;
    constexpr int kBest = 1024;
    __shared__ float red_s[kWaves], best_s[kBest];

    const int hq_i = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Hq = a.s.Hq, Hkv = a.s.Hkv, Ncap = a.s.Ncap;
    const int len = min(min(a.lens[b], Ncap), a.max_len);   // a hint below the true length: the tokens past it are left out, consistently in all kernels
    if (len <= 0) return;   // uniform: an empty sequence has no selection (the V kernel writes its zeros)
    const size_t hq = size_t(b) * Hq + hq_i, bh = size_t(b) * Hkv + hq_i / (Hq / Hkv);
    const int nblk = (len + kTB - 1) / kTB;
    const int kk = a.topk < len ? a.topk : len;
    const float* tm = a.tilemax + hq * (Ncap / kMinUnit);
    // the maxima are looked at up to four times, each a round trip in the chain: those of the first kBest blocks stay in LDS (B 1, 32/8,
    // 8192 tokens 34.8 -> 34.1 us a call, B 4 45.8 -> 45.0, others 0 to 0.6 %)
    auto block_max = [&](int i) { return i < kBest ? best_s[i] : tm[i]; };

    // ---- the global max logit (exact, order-free) and the bound of the cut
    float m = -INFINITY;
    for (int i = tid; i < nblk; i += NT) {
        const float bm = tm[i];
        if (i < kBest) best_s[i] = bm;
        m = fmaxf(m, bm);
    }
    m = wave_max(m);
    if (lane == 0) red_s[wave] = m;
    if (tid < kBuckets) ms.cnt[tid] = 0;
    for (int i = tid; i < kWaves * (kBuckets + 1); i += NT) (&ms.cntw[0][0])[i] = 0;
    __syncthreads();
    float M = red_s[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) M = fmaxf(M, red_s[w]);
    int Jb = 64;
    if (nblk >= kk) {   // uniform
        int n64 = 0;
        for (int i0 = 0; i0 < nblk; i0 += NT) mid_hist_add(ms.cnt, i0 + tid < nblk ? -score_a(score_x(block_max(i0 + tid), M, a.c)) : 1000, n64);
        __syncthreads();
        int below;
        mid_find_cut(ms.cnt[lane], kk, Jb, below);   // the floor bucket is not counted: 64 if none before it is
    }

    const int b0 = int((long long)nblk * wave / kWaves), b1 = int((long long)nblk * (wave + 1) / kWaves);   // the wave's blocks
    const __amdgpu_buffer_rsrc_t rs_lg = make_rsrc(a.logits + hq * Ncap, uint32_t(Ncap) * 4u);
    // bucket of the best token of block c0 + lane (1000 past the range)
    auto best_of = [&](int c0) { return c0 + lane < b1 ? -score_a(score_x(block_max(c0 + lane), M, a.c)) : 1000; };
    // takes up to kAhead blocks off the mask and asks for their logits (lane -> four consecutive tokens)
    auto fetch = [&](int c0, uint64_t& mask, int (&blk)[kAhead], u32x4_t (&w)[kAhead]) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            blk[u] = mask ? c0 + __builtin_ctzll(mask) : -1;
            mask &= mask - 1;
            w[u] = buf_load_b128(rs_lg, blk[u] >= 0 ? uint32_t(blk[u] * kTB + lane * 4) * 4u : kSkip);
        }
    };
    auto score4 = [&](int blk, const u32x4_t& w, float (&x)[4], int (&j)[4]) {
        const float lv[4] = {bits_float(w.x), bits_float(w.y), bits_float(w.z), bits_float(w.w)};
        const int t0 = blk * kTB + lane * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = score_x(lv[i], M, a.c);
            j[i] = t0 + i < len ? -score_a(x[i]) : 1000;
        }
    };
    // ---- pass 1.  Bucket Jb is counted in the lanes: where scores are flat nearly all tokens are in it, and LDS atomics of a whole
    // wave on one address take a cycle per lane (B 1, 32/8, 131072 tokens of equal scores: 214 -> 126 us a call; where scores spread, 0.2 to 0.9 % more).
    int n_top = 0;
    for (int c0 = b0; c0 < b1; c0 += 64) {
        const int best = best_of(c0);
        uint64_t mask = __ballot(a.dbg.a ? best <= 64 : best <= min(Jb, 63));   // the export wants every token
        while (mask) {
            int blk[kAhead];
            u32x4_t w[kAhead];
            fetch(c0, mask, blk, w);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (blk[u] < 0) continue;   // uniform
                float x[4];
                int j[4];
                score4(blk[u], w[u], x, j);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (j[i] <= Jb) {
                        if (j[i] == Jb) ++n_top;
                        else atomicAdd(&ms.cntw[wave][j[i]], 1);
                    }
                    if (j[i] <= 64 && a.dbg.a) a.dbg.a[hq * Ncap + blk[u] * kTB + lane * 4 + i] = (int8_t)(-j[i]);
                }
            }
        }
    }
    n_top = wave_read(wave_scan_add(n_top), 63);
    if (lane == 0 && Jb < 64) ms.cntw[wave][Jb] = n_top;   // the floor bucket stays uncounted
    __syncthreads();
    // ---- the cut, and the selected tokens of each kind in the waves before this one
    int tot = 0, before = 0;   // bucket `lane`: all waves / the waves before this one
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int c = ms.cntw[w][lane];
        tot += c;
        before += w < wave ? c : 0;
    }
    int J, below;
    mid_find_cut(tot, kk, J, below);
    const int fromcut = kk - below;
    int n_lt0 = wave_read(wave_scan_add(lane < J ? before : 0), 63);
    int n_eq0 = J < 64 ? wave_read(before, J) : min(b0 * kTB, len) - n_lt0;   // the cut in the floor bucket: all buckets before it are counted
    // ---- pass 2
    for (int c0 = b0; c0 < b1; c0 += 64) {
        const int best = best_of(c0);
        uint64_t mask = __ballot(best <= J);
        while (mask) {
            if (n_eq0 >= fromcut) mask &= __ballot(best < J);   // blocks that could only add to the cut bucket
            if (!mask) break;
            int blk[kAhead];
            u32x4_t w[kAhead];
            fetch(c0, mask, blk, w);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (blk[u] < 0) continue;   // uniform
                float x[4];
                int j[4], n_lt, n_eq, w_lt, w_eq;
                score4(blk[u], w[u], x, j);
                mid_wave_order(j, J, n_lt, n_eq, w_lt, w_eq);
                n_lt += n_lt0;
                n_eq += n_eq0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool is_lt = j[i] < J, is_eq = j[i] == J;
                    if (is_lt || (is_eq && n_eq < fromcut)) mid_emit(ms, n_lt + (n_eq < fromcut ? n_eq : fromcut), blk[u] * kTB + lane * 4 + i, x[i], j[i]);
                    n_lt += is_lt;
                    n_eq += is_eq;
                }
                n_lt0 += w_lt;
                n_eq0 += w_eq;
            }
        }
    }
    __syncthreads();
    int ehat = 32767;
    mid_oest<NT>(a, bh, hq, kk, ms, ehat);
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
    // the combining workgroup: a thread sums four neighbouring outputs over every kSub-th chunk
    constexpr int kCols = G * kD / 4, kSub = 64 * kVWaves / kCols;
    struct Private { union { float red[kVWaves][G][kD]; f32x4_t comb[kSub][kCols]; }; };
    struct Shared { union { VShare rows; float red[G][kD]; f32x4_t comb[kSub][kCols]; }; };   // the sums are laid down when the last round has been read
    __shared__ __align__(16) std::conditional_t<SHARED, Shared, Private> lds_s;
    __shared__ float z_s[kVWaves][G];
    __shared__ int ehat_s[kD];
    __shared__ int last_s;

    const int h = blockIdx.y, b = blockIdx.z, split = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane >> 3, cl = lane & 7;
    const int Hkv = a.s.Hkv, Hq = a.s.Hq, Ncap = a.s.Ncap;
    const int len = min(min(a.lens[b], Ncap), a.max_len);   // a hint below the true length: the tokens past it are left out, consistently in all kernels
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

    if (tid < kD) {   // Rule 2 aligns to the smallest result exponent of the group
        int e = 32767;
#pragma unroll
        for (int g = 0; g < G; ++g) e = min(e, a.Ehat[(size_t(b) * Hq + size_t(h) * G + g) * kD + tid]);
        ehat_s[tid] = e;
        if (a.dbg.Ehat && split == 0) a.dbg.Ehat[bh * kD + tid] = (int16_t)e;
    }
    float Mg[G];
#pragma unroll
    for (int g = 0; g < G; ++g) Mg[g] = a.M[size_t(b) * Hq + size_t(h) * G + g];
    __syncthreads();
    // HI bytes fetched three or four batches ahead in the private mode (few waves per SIMD: each keeps more bytes in
    // flight), two in the shared mode (four waves per SIMD; three and four measured 1.5 % and 3 % slower)
    constexpr int DL = SHARED ? 2 : (G == 2 ? 4 : 3);
    if constexpr (SHARED) {
        VRule<4> vr;
        v_rule_setup(ehat_s, a.guard_bits, a.force_level, vr);
        float acc[8], z[G / 4];
#pragma unroll
        for (int s = 0; s < G / 4; ++s) z[s] = 0.0f;
        v_rows_shared<G, DEBUG, DL>(a, b, h, c0 + wave * RB, vchunk / (RB * kVWaves), len, vr, Mg, acc, z, lds_s.rows);
#pragma unroll
        for (int s = 0; s < G / 4; ++s) {   // over the lanes of the same query heads
            for (int o = 4; o < 64; o <<= 1) z[s] += __shfl_xor(z[s], o);
            if (lane < 4) z_s[wave][lane + 4 * s] = z[s];
        }
        // a result tile holds the high parts of the weights in its rows 0 .. G-1 and the low parts in rows G .. 2G-1:
        // lanes 16 * (G / 4) apart hold the two parts of one (query head, line)
        float part[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) part[i] = (acc[i] + __shfl(acc[i], (lane + 4 * G) & 63)) * (1.0f / kVWeightScale);
        __syncthreads();   // every wave is done with the rows of the last round: the same LDS now takes the sums
        if (lane < 4 * G) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) lds_s.red[4 * (lane >> 4) + i][line_channel(32 * wave + 16 * t + (lane & 15))] = part[4 * t + i];
        }
    } else {
        VRule<> vr;
        v_rule_setup(ehat_s, a.guard_bits, a.force_level, vr);
        float acc[G][16], z[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            z[g] = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[g][i] = 0.0f;
        }
        const u32x4_t none[1][KG] = {};
        v_rows<G, KG, DEBUG, 0, DL, true>(a, b, h, c0 + wave * RB, RB * kVWaves, vchunk / (RB * kVWaves), len, vr, Mg, acc, z, none, false);
        v_reduce_rows<G>(acc, z);
        if (r == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 16; ++i) lds_s.red[wave][g][cl * 16 + i] = acc[g][i];
        }
        if (lane == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) z_s[wave][g] = z[g];
        }
    }
    __syncthreads();
    for (int idx = tid; idx < G * (kD + 1); idx += 64 * kVWaves) {
        const int g = idx / (kD + 1), d = idx % (kD + 1);
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kVWaves; ++w) {
            if (d == kD) s += z_s[w][g];
            else if constexpr (SHARED) s += w == 0 ? lds_s.red[g][d] : 0.0f;
            else s += lds_s.red[w][g][d];
        }
        const size_t hq = size_t(b) * Hq + size_t(h) * G + g;
        if (d < kD) store_agent(&a.partO[(hq * nsplit + split) * kD + d], s);
        else store_agent(&a.partZ[hq * nsplit + split], s);
    }

    // ---- the workgroup that finishes last for this (sequence, KV head) combines the chunks -------------
    // out = sum_chunks O / sum_chunks Z: every chunk used the same global max, so nothing is rescaled.  All threads take part
    // with 16-byte loads, eight chunks each in flight (one word per thread and output before: 5-7 us at the end of a call of
    // eight heads per group, now 4; the round trips of stores, ticket and loads are what is left).
    const int used = (len + vchunk - 1) / vchunk;
    stores_done();
    __syncthreads();
    if (tid == 0) last_s = take_ticket(&a.vcount[bh]) == used - 1;
    __syncthreads();
    if (!last_s) return;
    const size_t hq0 = size_t(b) * Hq + size_t(h) * G;
    const int c = tid % kCols, sub = tid / kCols, g_out = c / (kD / 4);
    const __amdgpu_buffer_rsrc_t rs_o = make_rsrc(a.partO + hq0 * nsplit * kD, uint32_t(G) * uint32_t(nsplit) * kD * 4u);
    f32x4_t o = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int sp0 = sub; sp0 < used; sp0 += 8 * kSub) {   // eight chunks' words in flight; the additions stay in chunk order
        u32x4_t po[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int sp = sp0 + i * kSub;
            po[i] = buf_load_b128_agent(rs_o, sp < used ? (uint32_t(g_out) * uint32_t(nsplit) + uint32_t(sp)) * (kD * 4u) + uint32_t(c % (kD / 4)) * 16u : kSkip);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] += bits_float(po[i][k]);
    }
    for (int g = wave; g < G; g += kVWaves) {   // the weights' sums: a wave per query head, lane -> chunks
        float zs = 0.0f;
        for (int sp = lane; sp < used; sp += 64) zs += load_agent(&a.partZ[(hq0 + g) * nsplit + sp]);
        for (int k = 1; k < 64; k <<= 1) zs += __shfl_xor(zs, k);
        if (lane == 0) z_s[0][g] = zs;
    }
    if (kSub > 1) lds_s.comb[sub][c] = o;
    __syncthreads();
    if (sub == 0) {
#pragma unroll
        for (int u = 1; u < kSub; ++u) o += lds_s.comb[u][c];
#pragma unroll
        for (int k = 0; k < 4; ++k) store_out(a, hq0 + g_out, (c % (kD / 4)) * 4 + k, o[k] / z_s[0][g_out]);
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
    if (a.max_len > 16 * kTB && long(a.s.B) * a.s.Hq <= compute_units()) hipLaunchKernelGGL(split_select_kernel<1024>, dim3(a.s.Hq, a.s.B), dim3(1024), 0, st, a);
    else hipLaunchKernelGGL(split_select_kernel<512>, dim3(a.s.Hq, a.s.B), dim3(512), 0, st, a);
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
