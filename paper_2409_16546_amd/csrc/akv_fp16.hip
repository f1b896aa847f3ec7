// The unquantised yardstick: decode attention on plain fp16 K, V [B][Hkv][Ncap][D]
// ("Runtime of AlignedKV": S = QK^T/sqrt(128), softmax, O = SV on 16-bit data).
// K and V of a chunk of tokens are read in one kernel with a softmax of its own (split-KV), since nothing has to be decided
// between the passes; the chunks are merged by a second small kernel.
#include <algorithm>
#include <cfloat>

#include "akv_common.h"

namespace akv {

constexpr int kFWaves = 4;
constexpr int kFTile = 32;                          // tokens a wave takes at a time
constexpr int kFMinChunk = kFTile * kFWaves;        // tokens per workgroup are a multiple of this

// Tokens per workgroup: about twelve workgroups per compute unit over the whole call (three are resident; single heads eight,
// groups of eight four, with two resident), so that ragged lengths even out, and not fewer than one tile per wave.  Timed with 4 / 8 / 12 / 16
// / 32 workgroups per unit: B 8, 32/8, up to 16000 ragged 77 / 78 / 61 / 65 / 73 us, B 8, 32/8, 32768 178 / 178 / 176 / 182 / 194;
// B 8, 64/8, 8192 58 / 66 / 66 / 84 / 84; B 8, 32/32, 4096 89 / 85 / 87 / 89 / 92.  By the capacity and not by a bound of the
// lengths, so that chunks add up in an order the bound does not change (even shares, fp16_even_kernel, in one that the lengths of
// the whole batch decide).
// Except: as many pairs as compute units, and a bound of at most 1024: one workgroup for the whole pair, no merge (chunks / one, us:
// 256 single heads 512 18.0/13.7, 1024 28.6/24.7, 512 of them 1024 47.5/46.3, a third full 26.0/18.4; 256 groups of four 1024
// 33.1/26.1; 384 single heads 1024, the one call behind, 37.5/39.1).
static int f_chunk(const akv_shape& s, int max_len)
{
    const int G = s.Hq / s.Hkv;
    const long pairs = long(s.B) * s.Hkv;
    auto whole = [](long n) { return (n + kFMinChunk - 1) / kFMinChunk * kFMinChunk; };
    if (pairs >= compute_units() && max_len <= 1024) return (int)whole(max_len);
    const long wgs = (G == 8 ? 4L : (G == 1 ? 8L : 12L)) * compute_units();
    return (int)std::min(1024L, std::max(long(kFMinChunk), whole(pairs * s.Ncap / wgs)));
}

// workgroups of a compute unit at a time
constexpr int f_resident(int G) { return G == 8 ? 2 : 3; }

constexpr int kFEvenSeqs = 64;   // sequences the even shares have a lane for

struct F16Plan { int chunk, workgroups; };   // tokens per workgroup; workgroups of fp16_even_kernel, or 0: chunks
// More chunks than one round of workgroups: even shares, where they are not cut by the pairs' ends too often.  Chunks / even, us, full and
// ragged (lengths a quarter to all of the bound): groups of four, 8 pairs 30000 40.5/31.3, 16 pairs 8192 21.3/20.1, 17.4/18.6; 32 pairs
// 5000 23.3/22.6, 19.4..20.6/18.9..19.8; 64 pairs 5000 38.2/35, 27..29/25..27; 88 pairs 8192 68.0/67.9, 46..49/44..47; 128 pairs 16384
// 182/170, 123..128/106..113; but of those that the line leaves to chunks 128 pairs 2048 34.0/36.9, 256 pairs 2048 53.7/56.7 (shares that
// begin anywhere).  Groups of eight, 4 pairs 30000 35.8/27.2, 18.6/20.1; 16 pairs 5000 22.2/20.3, 15.7..21.9/17.2..20.2; 32 pairs 2100
// 21.1/19.3, 15.6/17.2; 64 pairs 5000 44.8/38.4, 36..38/30; 128 pairs 8192 97.3/102, 77..82/66..70.  Short ragged calls lose up to 1.7 us
// where the chunks happen to come out even; the host knows a bound of the lengths only.  Single heads and groups of two lose (8 x 32 of
// 4096 88/94).
static F16Plan fp16_plan(const akv_shape& s, int max_len)
{
    const int G = s.Hq / s.Hkv, round = f_resident(G) * compute_units(), chunk = f_chunk(s, max_len);
    const long pairs = long(s.B) * s.Hkv;
    const bool even = ((G == 8 && max_len >= 32 * pairs) || (G == 4 && max_len >= 64 * pairs)) && s.B <= kFEvenSeqs && chunk < max_len && pairs * ((max_len + chunk - 1) / chunk) > round;
    return {chunk, even ? round : 0};
}

int fp16_path(const akv_shape& s, int max_len)
{
    const F16Plan p = fp16_plan(s, max_len);
    return p.workgroups ? 3 : (max_len <= p.chunk ? 1 : 2);
}

size_t fp16_workspace_bytes(const akv_shape& s)
{
    const size_t bhq = size_t(s.B) * s.Hq, ns = s.Ncap / kFMinChunk;
    return align256(bhq * ns * kD * sizeof(float)) + 2 * align256(bhq * ns * sizeof(float));   // partial sums, maxima, weights' sums
}

struct F16Args {
    akv_shape s;
    const uint16_t *k, *v, *q;
    const int32_t* lens;
    void* out;
    float c;   // scale * log2(e)
    int out_dtype, nsplit, max_len, chunk;   // nsplit: chunks there is room for per query head
    int turn_shift, turn_mask;               // which chunk a workgroup takes: launch_fp16_g
    int workgroups;                          // of fp16_even_kernel, or 0: chunks
    float *partO, *partM, *partZ;
};

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

// the value of the lane 16 / 32 further (mod the pairs of rows / halves) folded in: op over lanes with the same lane % 16, in all of them
template <typename F>
__device__ __forceinline__ float over_rows(float v, F op)
{
    const auto a = __builtin_amdgcn_permlane16_swap(float_bits(v), float_bits(v), false, false);
    v = op(bits_float(a[0]), bits_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(float_bits(v), float_bits(v), false, false);
    return op(bits_float(b[0]), bits_float(b[1]));
}

__device__ __forceinline__ int fp16_len(const F16Args& a, int b) { return max(min(min(a.lens[b], a.s.Ncap), a.max_len), 0); }

// What a workgroup of fp16_even_kernel takes, from the lengths of all sequences (at most 64 of them: a lane each).  A wave finds it out
// by itself, two rounds of scans over the lanes in front of its first load.
// Whole parts: every pair is cut into parts of `share` tiles, its last one shorter, and a workgroup takes one.  Taken where the even share,
// or one up to three tiles larger (one from 32 tiles on: 88 ragged pairs, groups of four, share 37, 81 us without, 88 with three more),
// makes no more parts than there are workgroups.  Groups of four: eight tiles and not five or six, as wide for the waves that have two and
// fewer parts to merge (6 / 8: 8 pairs of 16384 23.7/21.3, 16 of 8192 21.5/19.8, 40 of 3500 21.2/22.6; groups of eight, 5 / 8: 16 pairs
// of 5000 20.1/21.9).
// Else the tiles of all pairs are numbered through, sequence after sequence, and a workgroup takes the next `share` of them, which may
// be the end of one pair and the beginning of the next: two ranges one after the other, 4 to 6 us where one takes 8.  (Whole parts / these
// always / chunks, us, groups of eight: 64 pairs 2100 25.7/28.9/27.3, ragged 20.5/25.4/20.7; 32 pairs 5000 25.8/31.1/28.4, ragged
// 23.2/28.0/21.4; 64 pairs 8192 ragged 38.3/41.2/46.8; groups of four: 16 pairs 30000 47.1/49.7/53.8, 128 pairs 8192 90.7/95.1/98.1.)
// A pair has room for Ncap / 128 partial results: at least two, as capacities are multiples of 256, and at least ceil(n / 4) for its n
// tiles.  Whole parts are of four tiles and more, so at most ceil(n / 4).  Shares that begin anywhere are of eight and more: one part for
// one tile, else at most (n - 2) / share + 2 parts, which is two for up to nine tiles and at most ceil(n / 4) for more.
// m / d for 0 <= m < 2^21, d >= 1: (m + 1/2) / d lies at least 1 / (2 d) from a whole number, and the two roundings and the reciprocal's
// last place move it by less than (m + 1/2) / d * 2^-22.  (A sequence has fewer than 2^24 tokens, the descriptors' reach, so 2^19 tiles.)
__device__ __forceinline__ int small_quotient(int m, int d) { return int((float(m) + 0.5f) * __builtin_amdgcn_rcpf(float(d))); }
struct F16Tiles {
    int len, per, end;   // of sequence `lane`: its length, the places (whole parts, or tiles) of one of its pairs, those up to and with its last
    int share;
    bool whole;
    __device__ __forceinline__ F16Tiles(const F16Args& a)
    {
        const int lane = threadIdx.x & 63, Hkv = a.s.Hkv;
        len = lane < a.s.B ? fp16_len(a, lane) : 0;
        const int tiles = (len + kFTile - 1) / kFTile;
        end = wave_scan_add(tiles * Hkv);
        share = (wave_read(end, 63) + a.workgroups - 1) / a.workgroups;
        // the parts that four shares make, two counts to a word: a sequence adds at most one part a pair to its tiles over the share, so
        // that all of them are fewer than workgroups + 64
        const int least = share > 6 || a.s.Hq == 8 * Hkv ? max(share, 4) : (share > 4 ? 8 : 4), most = least + (least < 32 ? 3 : 1);
        int parts[4], sum[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) parts[k] = small_quotient(tiles + least + k - 1, least + k);
#pragma unroll
        for (int k = 0; k < 4; k += 2) sum[k / 2] = wave_scan_add(parts[k] | parts[k + 1] << 16);
        whole = false;
#pragma unroll
        for (int k = 3; k >= 0; --k) {
            const int upto = (k & 1) ? int(uint32_t(sum[k / 2]) >> 16) : sum[k / 2] & 0xFFFF;
            if (wave_read(upto, 63) * Hkv <= a.workgroups && least + k <= most) {   // uniform
                whole = true;
                share = least + k;
                per = parts[k];
                end = upto * Hkv;
            }
        }
        if (whole) return;
        per = tiles;
        share = max(share, 8);
    }
    __device__ __forceinline__ int before(int b) const { return b > 0 ? wave_read(end, b - 1) : 0; }   // b uniform
    __device__ __forceinline__ int sequence_of(int place) const { return __builtin_popcountll(__ballot(end <= place)); }
    // partial results of KV head h of sequence b
    __device__ __forceinline__ int parts_of(int b, int h) const
    {
        const int n = wave_read(per, b);
        if (whole) return n;
        const int first = before(b) + h * n;
        return n > 0 ? (first + n - 1) / share - first / share + 1 : 0;
    }
};

__device__ __forceinline__ void store_result(const F16Args& a, size_t at, float v)
{
    if (a.out_dtype == 0) reinterpret_cast<float*>(a.out)[at] = v;
    else reinterpret_cast<_Float16*>(a.out)[at] = (_Float16)v;
}

// Workgroup = 4 waves, one (sequence, KV head, chunk of tokens); each wave walks its quarter of the chunk by itself in tiles of
// 32 tokens with a running maximum, so that nothing waits at a barrier until the chunk's end.  Bound by memory; K and V
// tiles take turns in flight (8 to 16 KB per wave, loads of the next K tile behind those of this V tile).
//   logits   matrix product on the matrix cores, 16 tokens x 16 columns (the G query heads, the rest zero) x 32 channels:
//            a lane holds 16 bytes of one token's row per step, no exchange between lanes;
//   weights  2^((l - m) c) in binary32, through LDS to the lanes that hold the token's V row;
//   O        multiply-adds in binary32 on the vector ALU, 8 channels of a row per lane (8 G per 16 bytes: a fifth of the
//            time the bytes take at G = 4).
// Measured against one row of 16 lanes per token with shuffled sums: B 8, 32/8 heads, up to 16000 tokens 137 -> 65 us, 32768
// 241 -> 176; B 8, 64/8, 8192 110 -> 58; B 1, 32 heads, 1024 29 -> 13; single heads at 4096 and 8192 as before (memory).
// Error against 64 bits over these ranges 3e-7 .. 6e-7, as before (one running sum of the logits: a third more).
// ONE: the workgroup has the whole sequence and writes the result itself; else a partial result into place `split` of the pair.
// LONG: ranges may be long: rows are added four at a time in a sum of their own, so that the running sums are rounded a quarter as
// often (error against 64 bits over B 2..16, 700..16384 tokens, groups of four and eight 4.1e-7; one row at a time 4.3e-7, up to 5.5e-7 at
// 16 x 16384; chunks of at most 1024 tokens one row at a time 4.2e-7).
// t_begin, t_end: the wave's tokens; some wave of the workgroup has some.
template <int G>
struct F16Shared {
    alignas(16) float p[kFWaves][kFTile][G];
    float red[kFWaves][G][kD];
    float max[kFWaves][G], z[kFWaves][G];
};
template <int G, bool ONE, bool LONG>
__device__ __forceinline__ void fp16_range(const F16Args& a, int b, int h, int split, int t_begin, int t_end, int len, F16Shared<G>& sm)
{
    auto& p_s = sm.p;
    auto& red_s = sm.red;
    auto& max_s = sm.max;
    auto& z_s = sm.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, j = lane >> 4;   // logits: token n of 16 (then query head n), channels 8j .. 8j+7 of 32; V: row j of 4, channels 8n .. 8n+7
    const int Hkv = a.s.Hkv, Hq = a.s.Hq, Ncap = a.s.Ncap;
    const size_t bh = size_t(b) * Hkv + h, hq0 = size_t(b) * Hq + size_t(h) * G;
    // rows at or past len are out of range: zeros, nothing fetched
    const __amdgpu_buffer_rsrc_t rs_k = make_rsrc(a.k + bh * Ncap * kD, uint32_t(len) * (kD * 2u));
    const __amdgpu_buffer_rsrc_t rs_v = make_rsrc(a.v + bh * Ncap * kD, uint32_t(len) * (kD * 2u));
    u32x4_t kf[2][4], vf[8];
    auto fetch_k = [&](int t0) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) kf[s][kb] = buf_load_b128_nt(rs_k, t0 < t_end ? uint32_t(t0 + 16 * s + n) * (kD * 2u) + kb * 64 + j * 16 : kSkip);
    };
    auto fetch_v = [&](int t0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) vf[k] = buf_load_b128_nt(rs_v, t0 < t_end ? uint32_t(t0 + 4 * k + j) * (kD * 2u) + n * 16 : kSkip);
    };
    fetch_k(t_begin);
    fetch_v(t_begin);
    half8_t qf[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        u32x4_t w = {0u, 0u, 0u, 0u};
        if (n < G) w = *reinterpret_cast<const u32x4_t*>(a.q + (hq0 + n) * kD + kb * 32 + j * 8);
        qf[kb] = __builtin_bit_cast(half8_t, w);
    }
    // z, m_run: of query head n (lanes with n < G).  The maximum starts at the lowest finite number and not at minus infinity: a
    // logit of minus infinity (a key that must not be attended) then has weight zero also where a wave has seen no other yet.
    float acc[G][8], z = 0.0f, m_run = -FLT_MAX;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[g][i] = 0.0f;

#pragma unroll 1
    for (int t0 = t_begin; t0 < t_end; t0 += kFTile) {
        f32x4_t s[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f32x4_t part[4];   // 32 channels each, added pairwise: less rounding than one running sum through the matrix cores
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) part[kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, kf[u][kb]), qf[kb], f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            s[u] = (part[0] + part[1]) + (part[2] + part[3]);
        }
        fetch_k(t0 + kFTile);
        // lane: query head n, tokens 16 u + 4 j + i
        float m = -INFINITY;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (t0 + 16 * u + 4 * j + i >= t_end) s[u][i] = -INFINITY;
                m = fmaxf(m, s[u][i]);
            }
        m = over_rows(m, [](float x, float y) { return fmaxf(x, y); });
        if (__ballot(m > m_run)) {   // uniform; rare after the first tiles
            const float m_new = fmaxf(m, m_run), sc = __builtin_amdgcn_exp2f((m_run - m_new) * a.c);
            z *= sc;
            m_run = m_new;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float sg = bits_float(__builtin_amdgcn_readlane(float_bits(sc), g));
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[g][i] *= sg;
            }
        }
        float zt = LONG ? 0.0f : z;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float p = __builtin_amdgcn_exp2f((s[u][i] - m_run) * a.c);
                zt += p;
                if (n < G) p_s[wave][16 * u + 4 * j + i][n] = p;
            }
        z = LONG ? z + zt : zt;
        __builtin_amdgcn_wave_barrier();
        constexpr int kRows = LONG ? 4 : 1;
#pragma unroll
        for (int k0 = 0; k0 < 8; k0 += kRows) {
            float p[kRows][G];
#pragma unroll
            for (int k = 0; k < kRows; ++k)
#pragma unroll
                for (int g = 0; g < G; ++g) p[k][g] = p_s[wave][4 * (k0 + k) + j][g];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float t[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) t[i] = LONG ? 0.0f : acc[g][i];
#pragma unroll
                for (int k = 0; k < kRows; ++k) {
                    const uint32_t w[4] = {vf[k0 + k].x, vf[k0 + k].y, vf[k0 + k].z, vf[k0 + k].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        t[2 * i] = fmaf(p[k][g], lo_half(w[i]), t[2 * i]);
                        t[2 * i + 1] = fmaf(p[k][g], hi_half(w[i]), t[2 * i + 1]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[g][i] = LONG ? acc[g][i] + t[i] : t[i];
            }
        }
        fetch_v(t0 + kFTile);
    }

    // ---- the waves' sums, rescaled to the chunk's maximum
    auto add = [](float x, float y) { return x + y; };
    z = over_rows(z, add);
    if (lane < G) {
        max_s[wave][lane] = m_run;
        z_s[wave][lane] = z;
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float o = over_rows(acc[g][i], add);
            if (j == 0) red_s[wave][g][8 * n + i] = o;
        }
    __syncthreads();
    for (int idx = tid; idx < G * kD; idx += 64 * kFWaves) {
        const int g = idx / kD, d = idx % kD;
        float M = max_s[0][g];
#pragma unroll
        for (int w = 1; w < kFWaves; ++w) M = fmaxf(M, max_s[w][g]);
        float o = 0.0f, zs = 0.0f;
#pragma unroll
        for (int w = 0; w < kFWaves; ++w) {
            const float sc = __builtin_amdgcn_exp2f((max_s[w][g] - M) * a.c);
            o = fmaf(sc, red_s[w][g][d], o);
            zs = fmaf(sc, z_s[w][g], zs);
        }
        const size_t hq = hq0 + g;
        if (ONE) {
            store_result(a, hq * kD + d, o / zs);
        } else {
            a.partO[(hq * a.nsplit + split) * kD + d] = o;
            if (d == 0) {
                a.partM[hq * a.nsplit + split] = M;
                a.partZ[hq * a.nsplit + split] = zs;
            }
        }
    }
}

template <int G, bool ONE>
__global__ __launch_bounds__(64 * kFWaves) void fp16_kernel(F16Args a)
{
    __shared__ F16Shared<G> sm;
    const int h = blockIdx.y, b = blockIdx.z, split = blockIdx.x ^ (((b * a.s.Hkv + h) >> a.turn_shift) & a.turn_mask);
    const int len = fp16_len(a, b), c0 = split * a.chunk;
    if (c0 >= len) {
        if (ONE)   // an empty sequence attends to nothing: zeros
            for (int idx = threadIdx.x; idx < G * kD; idx += 64 * kFWaves) store_result(a, (size_t(b) * a.s.Hq + size_t(h) * G) * kD + idx, 0.0f);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), per = a.chunk / kFWaves;
    fp16_range<G, ONE, false>(a, b, h, split, c0 + wave * per, min(c0 + (wave + 1) * per, len), len, sm);
}

// More work than one round of workgroups: one round of them, each with as many tiles of 32 tokens as the others or fewer (F16Tiles).
// Chunks by the shape end in a last round that is nearly empty, all the more where lengths differ (times: fp16_plan).  Bound by memory: 5.8
// TB/s where lengths are ragged, 6.2 where they are equal.
template <int G>
__global__ __launch_bounds__(64 * kFWaves, f_resident(G)) void fp16_even_kernel(F16Args a)
{
    __shared__ F16Shared<G> sm;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const F16Tiles all(a);
    const int total = all.before(64), share = all.share;
    int place = blockIdx.x, place_end = min(place + 1, total);
    if (!all.whole) {
        place *= share;
        place_end = min(place + share, total);
    }
    if (place >= place_end) return;   // uniform
    for (int b = all.sequence_of(place);; b = all.sequence_of(place)) {
        const int len = wave_read(all.len, b), per = wave_read(all.per, b), first = place - all.before(b);
        int h, t0, n, part;   // tiles t0 .. t0 + n - 1 of (b, h) are its partial result `part`
        if (all.whole) {
            h = small_quotient(first, per);
            part = first - h * per;
            t0 = part * share;
            n = min(share, (len + kFTile - 1) / kFTile - t0);
            ++place;
        } else {
            h = first / per;
            t0 = first - h * per;
            n = min(place_end - place, per - t0);
            part = place / share - (place - t0) / share;
            place += n;
        }
        fp16_range<G, false, true>(a, b, h, part, (t0 + n * wave / kFWaves) * kFTile, min((t0 + n * (wave + 1) / kFWaves) * kFTile, len), len, sm);
        if (place >= place_end) break;
        __syncthreads();   // the LDS areas are written again
    }
}

// merge the chunks of one query head: rescale each to the global max (a wave holds 64 chunks' weights; 16 rows in flight)
__global__ __launch_bounds__(kD) void fp16_combine_kernel(F16Args a)
{
    __shared__ float w_s[kD];
    const int hq_i = blockIdx.x, b = blockIdx.y, d = threadIdx.x, lane = d & 63;
    const int len = fp16_len(a, b);
    const size_t hq = size_t(b) * a.s.Hq + hq_i;
    int used;
    if (a.workgroups) {   // uniform
        const F16Tiles all(a);
        used = all.parts_of(b, hq_i / (a.s.Hq / a.s.Hkv));
    } else {
        used = (len + a.chunk - 1) / a.chunk;
    }
    const float *pm = a.partM + hq * a.nsplit, *pz = a.partZ + hq * a.nsplit, *po = a.partO + hq * a.nsplit * kD + d;
    float M = -INFINITY;
    for (int s = lane; s < used; s += 64) M = fmaxf(M, pm[s]);
    M = wave_max(M);
    float o = 0.0f, zsum = 0.0f;
    for (int s0 = 0; s0 < used; s0 += kD) {   // uniform
        const int s = s0 + d;
        const float w = s < used ? __builtin_amdgcn_exp2f((pm[s] - M) * a.c) : 0.0f;
        if (s < used) zsum = fmaf(w, pz[s], zsum);
        w_s[d] = w;
        __syncthreads();
        const int lim = min(used - s0, kD);
        for (int i0 = 0; i0 < lim; i0 += 16) {
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = i0 + i < lim ? po[size_t(s0 + i0 + i) * kD] : 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) o = fmaf(i0 + i < lim ? w_s[i0 + i] : 0.0f, v[i], o);
        }
        __syncthreads();
    }
    __shared__ float z2_s[2];
    for (int k = 1; k < 64; k <<= 1) zsum += __shfl_xor(zsum, k);
    if (lane == 0) z2_s[d >> 6] = zsum;
    __syncthreads();
    store_result(a, hq * kD + d, used > 0 ? o / (z2_s[0] + z2_s[1]) : 0.0f);
}

template <int G>
static hipError_t launch_fp16_g(F16Args a, hipStream_t st)
{
    const dim3 grid((a.max_len + a.chunk - 1) / a.chunk, a.s.Hkv, a.s.B), block(64 * kFWaves);
    // Workgroups are dealt to the eight XCDs in turn, and inside an XCD to its four shader engines.  Where the chunks of a pair are
    // a multiple of two, four ... 32, the first chunks of all pairs would fall on 16, 8 ... one of the 32 engines; and where
    // sequences are shorter than their bound, those are the only ones with work.  So chunks change places inside groups of that
    // many, by pair: single heads 16 x 32, 1024 of room, 133 stored 27 -> 15 us.  (Pairs varying fastest instead: even there, but
    // full sequences 3..17 % slower.)
    const int two = __builtin_ctz(grid.x | 32u);
    a.turn_mask = (1 << two) - 1;
    a.turn_shift = 5 - two;
    if (grid.x == 1) {
        hipLaunchKernelGGL((fp16_kernel<G, true>), grid, block, 0, st, a);
        return hipGetLastError();
    }
    if constexpr (G >= 4) {
        if (a.workgroups) hipLaunchKernelGGL(fp16_even_kernel<G>, dim3(a.workgroups), block, 0, st, a);
    }
    if (!a.workgroups) hipLaunchKernelGGL((fp16_kernel<G, false>), grid, block, 0, st, a);
    if (hipError_t e = hipGetLastError()) return e;
    hipLaunchKernelGGL(fp16_combine_kernel, dim3(a.s.Hq, a.s.B), dim3(kD), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_fp16(const akv_shape& s, const uint16_t* k, const uint16_t* v, const int32_t* lens, const uint16_t* q,
                       void* out, float scale, int out_dtype, int max_len, void* ws, hipStream_t st)
{
    F16Args a;
    a.s = s; a.k = k; a.v = v; a.q = q; a.lens = lens; a.out = out;
    a.c = (float)((double)scale * 1.4426950408889634);
    a.out_dtype = out_dtype;
    a.nsplit = s.Ncap / kFMinChunk;
    a.max_len = max_len;
    const F16Plan plan = fp16_plan(s, max_len);
    a.chunk = plan.chunk;
    a.workgroups = plan.workgroups;
    const size_t bhq = size_t(s.B) * s.Hq;
    char* p = reinterpret_cast<char*>(ws);
    a.partO = reinterpret_cast<float*>(p);
    p += align256(bhq * a.nsplit * kD * sizeof(float));
    a.partM = reinterpret_cast<float*>(p);
    p += align256(bhq * a.nsplit * sizeof(float));
    a.partZ = reinterpret_cast<float*>(p);
    switch (s.Hq / s.Hkv) {
        case 1: return launch_fp16_g<1>(a, st);
        case 2: return launch_fp16_g<2>(a, st);   // a.workgroups is 0 for these two
        case 4: return launch_fp16_g<4>(a, st);
        case 8: return launch_fp16_g<8>(a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace akv
