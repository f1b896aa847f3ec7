// Append tokens into the split-plane cache and its inverse.
// "Dynamic Quantization": the cache keeps all 16 bits of every element, the first 8 / next 4 / last 4
// bits in separately contiguous planes; "Quantization of K-Cache": K_colmax is kept while storing.
#include "akv_append_plan.h"
#include "akv_common.h"
#include "akv_unpack_plan.h"

namespace akv {

static_assert(kPlanTB == kTB, "one block size");

// One workgroup per (sequence, KV head), 128 threads: thread d owns K channel d (so it is the only writer
// of that column's nibble bytes and of colmax[d]); threads 0..63 own the V nibble byte of channels 2d, 2d+1.
// flags[AKV_NFLAGS + b] counts the workgroups of sequence b that have read its length (zero between calls).
__global__ __launch_bounds__(128) void append_kernel(akv_cache c, const uint16_t* __restrict__ k_new,
                                                     const uint16_t* __restrict__ v_new,
                                                     const int32_t* __restrict__ n_new, int n)
{
    const int h = blockIdx.x, b = blockIdx.y, d = threadIdx.x;
    const int Hkv = c.shape.Hkv, Ncap = c.shape.Ncap;
    const int len = c.lens[b];
    int cnt = n_new ? n_new[b] : n;
    cnt = cnt < 0 ? 0 : (cnt > n ? n : cnt);
    if (len + cnt > Ncap) {   // the sequence is left unchanged and the refusal is counted
        if (h == 0 && d == 0) atomicAdd(&c.flags[AKV_FLAG_OVERFLOW], 1);
        return;
    }
    if (cnt == 0) return;
    const size_t bh = size_t(b) * Hkv + h;
    // The ticket is drawn as soon as both waves of this workgroup have read the length (each has taken the branches above on
    // it, then they meet at the barrier): its round trip then runs beside the loads and stores below instead of after them.
    // Whoever draws the last one moves the length at its end -- every wave of the sequence's heads has read the old one by
    // then, and nothing in this kernel reads the planes.
    __syncthreads();
    int ticket = -1;
    if (d == 0) ticket = atomicAdd(&c.flags[AKV_NFLAGS + b], 1);
    const uint16_t* kn = k_new + bh * n * kD;
    const uint16_t* vn = v_new + bh * n * kD;
    uint32_t cm = c.colmax[bh * kD + d];
    for (int i = 0; i < cnt; ++i) {
        const uint32_t mag = store_token(c.k_hi, c.k_mid, c.k_lo, c.v_hi, c.v_mid, c.v_lo, bh, Ncap, len + i, d,
                                         kn + size_t(i) * kD, vn + size_t(i) * kD);
        cm = mag > cm ? mag : cm;
    }
    c.colmax[bh * kD + d] = (uint16_t)cm;
    if (d == 0 && ticket == Hkv - 1) {
        c.flags[AKV_NFLAGS + b] = 0;
        c.lens[b] = len + cnt;
    }
}

// Bulk append (prefill, chunks): 2 S workgroups of 256 threads per (sequence, KV head, 256-token K block touched): S for the block's K,
// two of them 64 channels each, and S for its V, two of them 128 rows each (twice the workgroups with half the chain each: launch_append).
// Bound by memory (2 bytes in, 2 bytes out per element), so both keep all their
// loads in flight at once and store whole 16-byte pieces.
//   V: no transposition; a thread turns 16 channels of a row (32 bytes in) into 16 + 8 + 8 bytes of the three planes.
//   K: 64 channels at a time (one workgroup for all: the second half is in flight while the first is turned).  A thread holds 8 tokens x 8
//      channels (rows 128 bytes apart in lanes, whole lines) and turns them in registers with byte permutes into two HI words
//      and one MID and one LO word per channel, which go to LDS channel-major; from there they leave as 16-byte pieces of
//      the channel-major runs.  The 16-byte pieces of a channel's LDS row are permuted by the channel's octet, so that neither
//      side has bank conflicts.  A piece that the new tokens cover only partly (the ends of the range) is merged with the
//      bytes that are there: no other workgroup writes those channels of the block.
// K_colmax: two channels at a time by compare-and-swap on their word, at the very end, when nothing of the workgroup waits for
// it (all blocks of a head meet there: per channel and between the halves it had cost a third of the launch).  The length
// moves in a launch of its own behind this one (every workgroup reads the old one), or by ticket where the workgroups are few.  Plain loads and non-temporal stores measured best of the four combinations.
// B 16, 32 heads, 8192 tokens (2.1 GB in, 2.1 GB out): 1510 -> 800 us, 5.4 TB/s (a plain copy reaches 4.9); chunks of up to 777
// tokens onto 6 x 8 heads: 155 -> 17 us (partly covered blocks used to be walked token by token).
constexpr int kHalf = kD / 2;   // channels per turn

// K_colmax of two neighbouring channels
__device__ __forceinline__ void colmax_update(uint32_t* word, uint32_t mags)
{
    uint32_t old = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (uint32_t want = max_halves(old, mags); want != old; want = max_halves(old, mags)) {
        const uint32_t seen = atomicCAS(word, old, want);
        if (seen == old) break;
        old = seen;
    }
}

// the two nibble words of eight elements from their low bytes (x0: elements 0..3, x1: 4..7); element 2i in the low nibble of byte i
__device__ __forceinline__ void nibble_words(uint32_t x0, uint32_t x1, uint32_t& mid, uint32_t& lo)
{
    const uint32_t m0 = ((x0 >> 4) & 0x000F000Fu) | ((x0 >> 8) & 0x00F000F0u), m1 = ((x1 >> 4) & 0x000F000Fu) | ((x1 >> 8) & 0x00F000F0u);
    const uint32_t l0 = (x0 & 0x000F000Fu) | ((x0 >> 4) & 0x00F000F0u), l1 = (x1 & 0x000F000Fu) | ((x1 >> 4) & 0x00F000F0u);
    mid = __builtin_amdgcn_perm(m1, m0, 0x06040200u);
    lo = __builtin_amdgcn_perm(l1, l0, 0x06040200u);
}

// bits [from, to) of a word, in units of `bits` bits counted from the word's first token t
__device__ __forceinline__ uint32_t token_mask(int t, int t_lo, int t_hi, int bits)
{
    const int per = 32 / bits, from = min(max(t_lo - t, 0), per), to = min(max(t_hi - t, 0), per);
    return (uint32_t)((1ull << (to * bits)) - 1) & ~(uint32_t)((1ull << (from * bits)) - 1);
}
// 16 bytes of a plane that hold tokens t .. t + 128 / bits - 1 of a column: stored whole, or merged with what is there
__device__ __forceinline__ void store_piece(uint8_t* dst, u32x4_t v, int t, int t_lo, int t_hi, int bits)
{
    const int n = 128 / bits;
    if (t >= t_hi || t + n <= t_lo) return;
    u32x4_t* p = reinterpret_cast<u32x4_t*>(dst);
    if (t < t_lo || t + n > t_hi) {
        const u32x4_t old = *p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t m = token_mask(t + i * (n / 4), t_lo, t_hi, bits);
            v[i] = (old[i] & ~m) | (v[i] & m);
        }
    }
    __builtin_nontemporal_store(v, p);
}

template <int S>
__global__ __launch_bounds__(256) void append_block_kernel(akv_cache c, const uint16_t* __restrict__ k_new,
                                                           const uint16_t* __restrict__ v_new,
                                                           const int32_t* __restrict__ n_new, int n, int ticketed)
{
    __shared__ u32x4_t hi_s[kHalf][kTB / 16], mid_s[kHalf][kTB / 32], lo_s[kHalf][kTB / 32];
    __shared__ uint32_t max_s[4][kD / 2];
    const int h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int Hkv = c.shape.Hkv, Ncap = c.shape.Ncap, NB = Ncap / kTB;
    // A head's parts begin at another one in every head (append_part).  As they were / turned, us: 8 x 32 heads 600 tokens 50.9/39.8, 16 x 32
    // 100 46.5/33.3, 512 72.0/66.7; long sequences stream worse (16 x 32 8192 783/808 with one workgroup per side), and there few blocks are
    // empty.
    const AppendPart part = append_part<S>(blockIdx.x, gridDim.x, unsigned(b * Hkv + h));
    const int len = c.lens[b];
    int cnt = n_new ? n_new[b] : n;
    cnt = cnt < 0 ? 0 : (cnt > n ? n : cnt);
    if (cnt == 0) return;
    if (len + cnt > Ncap) {                     // the sequence is left unchanged
        if (ticketed && part.i == 0 && part.v == 0 && part.sub == 0 && h == 0 && tid == 0) atomicAdd(&c.flags[AKV_FLAG_OVERFLOW], 1);
        return;
    }
    // ticketed: every workgroup of the sequence draws one once all its waves have read the length (each has taken the branches
    // above on it, then they meet at the barrier), and looks at it on leaving.  In a sequence that takes nothing or is refused
    // no length moves and none draws.
    int ticket = -1;
    if (ticketed) {
        __syncthreads();
        if (tid == 0) ticket = atomicAdd(&c.flags[AKV_NFLAGS + b], 1);
    }
    auto leave = [&] {
        if (ticket == append_tickets(gridDim.x / (2 * S), Hkv, S) - 1) {   // the last: every wave of the sequence's workgroups has read the length
            c.flags[AKV_NFLAGS + b] = 0;
            c.lens[b] = len + cnt;
        }
    };
    const AppendBlock ab = append_block(len, cnt, part.i);
    const int blk = ab.blk, t_lo = ab.t_lo, t_hi = ab.t_hi;   // tokens of this block: [t_lo, t_hi)
    if (t_lo >= t_hi) {
        leave();
        return;
    }
    const size_t bh = size_t(b) * Hkv + h;
    const bool is_v = part.v;
    const int sub = part.sub;   // which rows of V, or channels of K
    // row i of the input is token len + i; rows outside the range are asked for out of range and read as zeros
    const __amdgpu_buffer_rsrc_t rs = make_rsrc((is_v ? v_new : k_new) + bh * n * kD, uint32_t(n) * (kD * 2u));

    if (is_v) {   // thread -> (row tid/8 + 32 i of the part, 16 channels)
        constexpr int kRows = 8 / S;
        const int cl = tid & 7, t_first = blk * kTB + sub * (32 * kRows) + (tid >> 3);
        u32x4_t x[kRows][2];
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int t = t_first + 32 * i;
            const uint32_t off = t >= t_lo && t < t_hi ? uint32_t(t - len) * (kD * 2u) + uint32_t(cl) * 32u : kSkip;
            x[i][0] = buf_load_b128(rs, off);
            x[i][1] = buf_load_b128(rs, off + 16);
        }
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int t = t_first + 32 * i;
            u32x4_t hi;
            uint32_t low[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {   // a word of the input: channels 2i (low half), 2i + 1
                const uint32_t w0 = x[i][k >> 1][2 * (k & 1)], w1 = x[i][k >> 1][2 * (k & 1) + 1];
                hi[k] = __builtin_amdgcn_perm(w1, w0, 0x07050301u);
                low[k] = __builtin_amdgcn_perm(w1, w0, 0x06040200u);
            }
            u32x2_t mid, lo;
            uint32_t m0, m1, l0, l1;
            nibble_words(low[0], low[1], m0, l0);
            nibble_words(low[2], low[3], m1, l1);
            mid = u32x2_t{m0, m1};
            lo = u32x2_t{l0, l1};
            if (t >= t_lo && t < t_hi) {
                const size_t row = bh * Ncap + t;
                __builtin_nontemporal_store(hi, reinterpret_cast<u32x4_t*>(c.v_hi + row * kD + cl * 16));
                __builtin_nontemporal_store(mid, reinterpret_cast<u32x2_t*>(c.v_mid + row * (kD / 2) + cl * 8));
                __builtin_nontemporal_store(lo, reinterpret_cast<u32x2_t*>(c.v_lo + row * (kD / 2) + cl * 8));
            }
        }
        leave();
        return;
    }

    const int lane = tid & 63, wave = tid >> 6;
    const int p = lane & 7, oct = wave * 8 + (lane >> 3);   // channels 8p .. 8p+7 of the half, tokens 8 oct .. 8 oct + 7 of the block
    constexpr int kTurns = 2 / S;   // halves this workgroup turns
    u32x4_t x[kTurns][8];
    auto fetch = [&](int turn) {
        const int half = turn + sub;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = blk * kTB + 8 * oct + i;
            x[turn][i] = buf_load_b128(rs, t >= t_lo && t < t_hi ? uint32_t(t - len) * (kD * 2u) + uint32_t(half) * kD + uint32_t(p) * 16u : kSkip);
        }
    };
    fetch(0);
    const size_t colbase = (bh * NB + blk) * kD;
#pragma unroll
    for (int turn = 0; turn < kTurns; ++turn) {
        const int half = turn + sub;
        if (turn + 1 < kTurns) fetch(turn + 1);
#pragma unroll
        for (int w = 0; w < 4; ++w) {   // channel pair 8p + 2w, 8p + 2w + 1
            uint32_t hi[2][2], low[2][2];   // [channel of the pair][tokens 0..3, 4..7]
            uint32_t mx = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t w0 = x[turn][4 * q][w], w1 = x[turn][4 * q + 1][w], w2 = x[turn][4 * q + 2][w], w3 = x[turn][4 * q + 3][w];
                const uint32_t ha = __builtin_amdgcn_perm(w1, w0, 0x07030501u), hb = __builtin_amdgcn_perm(w3, w2, 0x07030501u);
                const uint32_t la = __builtin_amdgcn_perm(w1, w0, 0x06020400u), lb = __builtin_amdgcn_perm(w3, w2, 0x06020400u);
                hi[0][q] = __builtin_amdgcn_perm(hb, ha, 0x05040100u);
                hi[1][q] = __builtin_amdgcn_perm(hb, ha, 0x07060302u);
                low[0][q] = __builtin_amdgcn_perm(lb, la, 0x05040100u);
                low[1][q] = __builtin_amdgcn_perm(lb, la, 0x07060302u);
                mx = max_halves(max_halves(mx, max_halves(w0 & 0x7FFF7FFFu, w1 & 0x7FFF7FFFu)), max_halves(w2 & 0x7FFF7FFFu, w3 & 0x7FFF7FFFu));
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int ch = 8 * p + 2 * w + e;
                uint32_t mid, lo;
                nibble_words(low[e][0], low[e][1], mid, lo);
                *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint32_t*>(&hi_s[ch][(oct >> 1) ^ p]) + 2 * (oct & 1)) = u32x2_t{hi[e][0], hi[e][1]};
                reinterpret_cast<uint32_t*>(&mid_s[ch][(oct >> 2) ^ p])[oct & 3] = mid;
                reinterpret_cast<uint32_t*>(&lo_s[ch][(oct >> 2) ^ p])[oct & 3] = lo;
            }
            for (int o = 8; o < 64; o <<= 1) mx = max_halves(mx, (uint32_t)__shfl_xor((int)mx, o));
            if (lane < 8) max_s[wave][turn * (kHalf / 2) + 4 * p + w] = mx;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // HI: (channel, 16 tokens)
            const int ch = (tid >> 4) + 16 * i, g = tid & 15;
            store_piece(c.k_hi + (colbase + half * kHalf + ch) * kTB + g * 16, hi_s[ch][g ^ (ch >> 3)], blk * kTB + g * 16, t_lo, t_hi, 8);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {   // MID, LO: (channel, 32 tokens)
            const int ch = (tid >> 3) + 32 * i, g = tid & 7;
            const size_t at = (colbase + half * kHalf + ch) * (kTB / 2) + g * 16;
            store_piece(c.k_mid + at, mid_s[ch][g ^ (ch >> 3)], blk * kTB + g * 32, t_lo, t_hi, 4);
            store_piece(c.k_lo + at, lo_s[ch][g ^ (ch >> 3)], blk * kTB + g * 32, t_lo, t_hi, 4);
        }
        if (turn + 1 < kTurns) __syncthreads();   // the LDS areas are written again
    }
    if (tid < kTurns * (kHalf / 2))   // last, when nothing of this workgroup waits for it any more
        colmax_update(reinterpret_cast<uint32_t*>(c.colmax + bh * kD) + sub * (kHalf / 2) + tid, max_halves(max_halves(max_s[0][tid], max_s[1][tid]), max_halves(max_s[2][tid], max_s[3][tid])));
    leave();
}

// behind the bulk append: the lengths move, refusals are counted
__global__ __launch_bounds__(256) void append_lens_kernel(akv_cache c, const int32_t* __restrict__ n_new, int n)
{
    for (int b = threadIdx.x; b < c.shape.B; b += 256) {
        const int len = c.lens[b];
        int cnt = n_new ? n_new[b] : n;
        cnt = cnt < 0 ? 0 : (cnt > n ? n : cnt);
        if (len + cnt <= c.shape.Ncap) c.lens[b] = len + cnt;
        else atomicAdd(&c.flags[AKV_FLAG_OVERFLOW], 1);
    }
}

hipError_t launch_append(const akv_cache& c, const uint16_t* k_new, const uint16_t* v_new, const int32_t* n_new, int n,
                         hipStream_t st)
{
    if (n == 0) return hipSuccess;
    // A few tokens: one workgroup per (sequence, KV head) walks them, a round trip to memory each; from there on a block at a
    // time, which moves whole 16-byte pieces of every channel for however few tokens.  Timed with 1000 tokens stored, walk / block,
    // us: 8 pairs 8 tokens 10.2/10.3, 15 13.1/10.5; 128 pairs 16 tokens 15.8/15.9, 256 18.6/19.4, 24 tokens 24.1/19.4; 512 pairs 8
    // tokens 25.6/30.2, 12 34.0/30.1; 1024 pairs 1 token 19.3/30.6, 4 41.9/50.3, 6 56.5/50.3; 3072 pairs 1 token 47/111, 6
    // 164/186, 8 207/186; 8192 pairs 1 token 165/278, 6 454/486, 8 622/487.
    const long pairs = long(c.shape.B) * c.shape.Hkv;
    if (n <= (pairs >= 3072 ? 6 : 5) || (n <= (pairs < 128 ? 15 : 16) && pairs * n <= 4608)) {
        hipLaunchKernelGGL(append_kernel, dim3(c.shape.Hkv, c.shape.B), dim3(128), 0, st, c, k_new, v_new, n_new, n);
    } else {
        // Two workgroups per block's K and two per its V where that is one round or two of them and a head has few blocks.  One / two, us with
        // the copy that sets the lengths: 1 x 8 heads 100 tokens 9.5/8.6, 8 x 8 100 14.6/11.5, 2 x 32 512 19.1/15.2, chunks of 777 onto 6 x
        // 8 19.0/15.8, 8 x 32 600 50.8/39.8, 16 x 32 100 44.9/33.3, 512 75.8/66.7, 16 x 8 3000 82.5/78.5, with K_colmax from zero 88/82.
        // Not beyond: 16 x 32 2048 (9216 workgroups of one) 197/200, and from zero all blocks of a head meet at its K_colmax, the more
        // of them the shorter they run: 1 x 32 8192 54/57, 16 x 32 8192 798/1012.
        const int blocks = append_grid_blocks(n);
        const int parts = blocks <= 16 && 2 * blocks * pairs <= 4096 ? 2 : 1;
        const dim3 grid(2 * parts * blocks, c.shape.Hkv, c.shape.B);
        // few workgroups move the length by ticket: a launch less, but tickets on one cache line cost more than the launch where they are
        // many.  Launch / tickets, two per side, us for the copy that sets the lengths and K_colmax cleared in front (where the launches set the
        // pace), and what the tickets cost in device time behind a long kernel: 256 workgroups 15.6/12.8, +0.4; 320 15.6/13.5, +0.8; 384
        // 15.5/14.2, +1.5; 480 15.2/15.2, +2.1; 640 15.7/18.7, +4.5.  One per side (the copy alone): 320 on one sequence 13.4/12.4, 384
        // 17.4/18.7.
        const bool ticketed = long(grid.x) * grid.y * grid.z <= 320;
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, c, k_new, v_new, n_new, n, ticketed ? 1 : 0); };
        if (parts == 2) launch(append_block_kernel<2>);
        else launch(append_block_kernel<1>);
        if (ticketed) return hipGetLastError();
        if (hipError_t e = hipGetLastError()) return e;
        hipLaunchKernelGGL(append_lens_kernel, dim3(1), dim3(256), 0, st, c, n_new, n);
    }
    return hipGetLastError();
}

// planes -> fp16 [B][Hkv][Ncap][D], the bulk append run backwards: a workgroup of 256 threads per 256-token block of K, and VP per
// block of V.  Bound by memory; K goes through LDS 64 channels at a time (16-byte pieces of the channel-major runs in, rows of 128
// bytes out), with the same placement as there.  V: sixteen lanes per row, so that a store covers whole lines (eight lanes with two
// stores each, and one workgroup per block of V as of K: 8 x 32 heads, 4096 tokens 235 -> 176 us, 6.1 TB/s; 4 x 8, 4096 30 -> 25).
// KP: workgroups per block of K, 1 or 0 (V alone).
template <int KP, int VP>
__global__ __launch_bounds__(256) void unpack_kernel(akv_cache c, uint16_t* __restrict__ k_out,
                                                     uint16_t* __restrict__ v_out)
{
    __shared__ u32x4_t hi_s[KP ? kHalf : 1][kTB / 16], mid_s[KP ? kHalf : 1][kTB / 32], lo_s[KP ? kHalf : 1][kTB / 32];
    const int tid = threadIdx.x;
    const size_t item = blockIdx.x / (KP + VP);   // (b * Hkv + h) * NB + blk: the token rows item * 256 .. + 255
    const int part = int(blockIdx.x % (KP + VP)) - KP;
    if (VP > 0 && part >= 0) {   // thread -> (row tid / 16 + 16 i of the part, 8 channels)
        constexpr int kRows = VP > 0 ? kTB / (VP > 0 ? VP : 1) / 16 : 1;
        const int cl = tid & 15;
        const size_t row0 = item * kTB + part * (16 * kRows) + (tid >> 4);
        u32x2_t hi[kRows];
        uint32_t mid[kRows], lo[kRows];
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const size_t row = row0 + 16 * i;
            hi[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(c.v_hi + row * kD + cl * 8));
            mid[i] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(c.v_mid + row * (kD / 2) + cl * 4));
            lo[i] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(c.v_lo + row * (kD / 2) + cl * 4));
        }
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            uint32_t w[4];
            assemble8(hi[i].x, hi[i].y, mid[i], lo[i], w);   // channels (0,2), (1,3), (4,6), (5,7)
            u32x4_t o;
            o.x = __builtin_amdgcn_perm(w[1], w[0], 0x05040100u);
            o.y = __builtin_amdgcn_perm(w[1], w[0], 0x07060302u);
            o.z = __builtin_amdgcn_perm(w[3], w[2], 0x05040100u);
            o.w = __builtin_amdgcn_perm(w[3], w[2], 0x07060302u);
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4_t*>(v_out + (row0 + 16 * i) * kD + cl * 8));
        }
        return;
    }
    if constexpr (KP > 0) {
    const int lane = tid & 63, wave = tid >> 6;
    const int p = lane & 7, oct = wave * 8 + (lane >> 3);   // channels 8p .. 8p+7 of the half, tokens 8 oct .. 8 oct + 7 of the block
    const size_t colbase = item * kD;
    u32x4_t hi[2][4], mid[2][2], lo[2][2];
    auto fetch = [&](int half) {
#pragma unroll
        for (int i = 0; i < 4; ++i) hi[half][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(c.k_hi + (colbase + half * kHalf) * kTB) + tid + 256 * i);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            mid[half][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(c.k_mid + (colbase + half * kHalf) * (kTB / 2)) + tid + 256 * i);
            lo[half][i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(c.k_lo + (colbase + half * kHalf) * (kTB / 2)) + tid + 256 * i);
        }
    };
    fetch(0);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        if (half == 0) fetch(1);
        else __syncthreads();   // the LDS areas have been read
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = (tid >> 4) + 16 * i;
            hi_s[ch][(tid & 15) ^ (ch >> 3)] = hi[half][i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ch = (tid >> 3) + 32 * i;
            mid_s[ch][(tid & 7) ^ (ch >> 3)] = mid[half][i];
            lo_s[ch][(tid & 7) ^ (ch >> 3)] = lo[half][i];
        }
        __syncthreads();
        u32x4_t o[8];   // token: the 8 channels
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            uint32_t e[2][4];   // channel of the pair: tokens (0,2), (1,3), (4,6), (5,7)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int ch = 8 * p + 2 * w + k;
                const u32x2_t hh = *reinterpret_cast<const u32x2_t*>(reinterpret_cast<const uint32_t*>(&hi_s[ch][(oct >> 1) ^ p]) + 2 * (oct & 1));
                assemble8(hh.x, hh.y, reinterpret_cast<const uint32_t*>(&mid_s[ch][(oct >> 2) ^ p])[oct & 3],
                          reinterpret_cast<const uint32_t*>(&lo_s[ch][(oct >> 2) ^ p])[oct & 3], e[k]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int t = (q & 1) + 4 * (q >> 1);   // first token of the pair (t, t + 2)
                o[t][w] = __builtin_amdgcn_perm(e[1][q], e[0][q], 0x05040100u);
                o[t + 2][w] = __builtin_amdgcn_perm(e[1][q], e[0][q], 0x07060302u);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            __builtin_nontemporal_store(o[i], reinterpret_cast<u32x4_t*>(k_out + (item * kTB + 8 * oct + i) * kD + half * kHalf + 8 * p));
    }
    }
}

hipError_t launch_unpack(const akv_cache& c, uint16_t* k_out, uint16_t* v_out, hipStream_t st)
{
    const UnpackPlan p = unpack_plan(size_t(c.shape.B) * c.shape.Hkv * (c.shape.Ncap / kTB), k_out != nullptr, v_out != nullptr);
    if (!p.workgroups) return hipErrorInvalidConfiguration;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)p.workgroups), dim3(256), 0, st, c, k_out, v_out); };
    if (!v_out) launch(unpack_kernel<1, 0>);
    else if (!k_out) p.v_parts == 8 ? launch(unpack_kernel<0, 8>) : (p.v_parts == 4 ? launch(unpack_kernel<0, 4>) : launch(unpack_kernel<0, 2>));
    else if (p.v_parts == 1) launch(unpack_kernel<1, 1>);
    else launch(unpack_kernel<1, 16>);
    return hipGetLastError();
}

// zero a buffer with 16-byte stores (a kernel rather than a memset node, so that a caller may capture it)
__global__ __launch_bounds__(256) void zero_kernel(uint4* __restrict__ p16, size_t n16, uint8_t* __restrict__ tail,
                                                   int ntail)
{
    const size_t stride = size_t(gridDim.x) * 256;
    for (size_t i = size_t(blockIdx.x) * 256 + threadIdx.x; i < n16; i += stride) p16[i] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st)
{
    if (bytes == 0) return hipSuccess;
    const size_t n16 = bytes / 16;   // buffers come from an allocator: 16-byte aligned
    size_t blocks = (n16 + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks);
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<uint4*>(p), n16,
                       reinterpret_cast<uint8_t*>(p) + n16 * 16, int(bytes - n16 * 16));
    return hipGetLastError();
}

// Plain streaming read (16 bytes per lane with the non-temporal hint, four loads in flight per lane): the read ceiling of the
// device that the roofline fractions of the other kernels are put beside.
__global__ __launch_bounds__(256) void stream_read_kernel(const uint4* __restrict__ p, size_t n16, uint32_t* sink)
{
    auto ld = [](const uint4* q) {   // non-temporal, as the decode kernels read the bytes they stream
        const u32x4_t w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(q));
        return make_uint4(w.x, w.y, w.z, w.w);
    };
    // 4-KB chunks (one per workgroup and step) in blocks of 1 MB that go to the XCDs in turn (workgroup L runs on XCD
    // L % 8): an XCD reads stretches, as in the decode kernels -- chunks dealt singly over the XCDs read 15 % slower
    constexpr size_t kCpb = 256;   // chunks per block
    const size_t nchunks = (n16 + 255) / 256, x = blockIdx.x % kXcds, per = gridDim.x / kXcds;
    auto at = [&](size_t n) { return (((n / kCpb) * kXcds + x) * kCpb + n % kCpb) * 256 + threadIdx.x; };   // vector of chunk n of this XCD
    const uint4 zero = make_uint4(0, 0, 0, 0);
    uint32_t acc = 0;
    for (size_t n = blockIdx.x / kXcds; (n / kCpb) * kXcds * kCpb < nchunks; n += 4 * per) {
        const size_t i0 = at(n), i1 = at(n + per), i2 = at(n + 2 * per), i3 = at(n + 3 * per);
        const uint4 a = i0 < n16 ? ld(p + i0) : zero, b = i1 < n16 ? ld(p + i1) : zero;
        const uint4 c = i2 < n16 ? ld(p + i2) : zero, d = i3 < n16 ? ld(p + i3) : zero;
        acc += a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w ^ c.x ^ c.y ^ c.z ^ c.w ^ d.x ^ d.y ^ d.z ^ d.w;
    }
    if (acc == 0x9E3779B9u) *sink = acc;   // keeps the loads alive; practically never taken
}

hipError_t launch_stream_read(const void* p, size_t bytes, uint32_t* sink, hipStream_t st)
{
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    size_t blocks = (n16 + 1023) / 1024;
    blocks = blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks);
    hipLaunchKernelGGL(stream_read_kernel, dim3(xcd_grid(blocks)), dim3(256), 0, st, reinterpret_cast<const uint4*>(p), n16, sink);
    return hipGetLastError();
}

}  // namespace akv
