// Precision-aligned weight GEMV (declared in include/akw.h): y = x W with the rows of W read at the precision
// Rule 1 assigns them from x and rowmax.  "Precision Alignment in Uncertainty Calculation" (A W = A (W_quant +- dW)),
// "A Framework for Aligning Precision" (Rule 1; an addend's bit width is its weight's), "Dynamic Quantization"
// (first 8 / first 12 / all 16 bits, the rest counts as 100...).
//
// One kernel.  A workgroup (8 waves) owns a strip of 128 columns x 512 rows; a wave owns 64 of those rows, as
// eight groups of 8 rows; lane -> row lane/8 of the group and the 16-column slice lane%8, so one 16-byte load per
// lane fetches the 128 contiguous HI bytes of each of 8 rows (the MID and LO bytes: 8 bytes per lane; a row whose
// level does not need a plane is asked for out of range and fetches nothing).  All of a wave's loads are in flight
// at once: the HI bytes go before anything is known about the levels.  Every workgroup derives the largest
// addend exponent of each activation row from x and rowmax itself (K products, from L2) -- cheaper than a launch
// of its own in front of a kernel that runs for a few microseconds.  One activation row is multiplied on the vector ALU, two
// to four by 4x4x4 matrix products (the weights stay where the lanes hold them; four fp16 rows of a column are two byte
// permutes).  The sums over the 8 row lanes meet in the vector ALU, the waves' sums in LDS, the slabs' sums (K/512 of them) in the workspace: the workgroup that draws
// the last ticket of a strip adds them in slab order, so the result does not depend on timing.
// Measured against multiply-adds for every activation row and row sums through lane exchange (1 / 2 / 4 rows, us a call, copies of
// the matrix over 768 MB in turn): 4096x4096 10.9 / 14.0 / 19.6 -> 10.6 / 11.7 / 12.8, 4096x11008 19.0 / 25.8 / 36.5 ->
// 17.9 / 22.7 / 25.0, 11008x4096 21.2 / 31.2 / 45.1 -> 20.2 / 25.8 / 28.3.
#include <cstdarg>

#include "../../include/akw.h"
#include "akv_common.h"

namespace akv {

constexpr int kWWaves = 8;                   // waves per workgroup
constexpr int kWThreads = 64 * kWWaves;
constexpr int kWCols = 128;                  // columns per workgroup: 16 per lane, 8 lanes per row
constexpr int kWGroups = 8;                  // groups of 8 rows per wave
constexpr int kWSlab = kWWaves * kWGroups * 8;   // rows per workgroup: 512
static_assert(AKW_MAX_B * kWCols <= kWThreads && kWSlab == kWThreads, "a thread per (activation row, column) and per slab row");

struct GemvArgs {
    int K, N, nslab;
    const uint8_t *hi, *mid, *lo;
    const uint16_t *rowmax, *x;
    float *y, *part;      // part: [nslab][B][N]
    int32_t* count;       // [column strips]
    int guard_bits, force_level;
    uint8_t* lvl_out;
};

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

// two fp16 magnitudes, each at least the smallest normal
__device__ __forceinline__ uint32_t at_least_smallest_normal(uint32_t w)
{
    typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, w), u16x2_t{0x0400, 0x0400}));
}

template <int B>
__global__ __launch_bounds__(kWThreads, 4) void gemv_kernel(GemvArgs a)   // two workgroups per compute unit at least
{
    __shared__ int pmax_s[B][kWWaves];   // bits of magnitudes: integer order
    __shared__ __align__(8) uint8_t lvl_s[kWWaves][8][kWGroups];                  // of row (group g, row lane r) of a wave
    __shared__ __align__(16) uint16_t xh[B == 1 ? 1 : 4][kWWaves][8][kWGroups];   // x of that row, as the matrix instruction takes it
    __shared__ __align__(16) float red_s[kWWaves][B][kWCols];
    __shared__ int last_s;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane >> 3, cl = lane & 7;
    const int strip = blockIdx.x, slab_i = blockIdx.y;
    const int K = a.K, N = a.N;
    const int col = strip * kWCols + cl * 16, k0 = (slab_i * kWWaves + wave) * kWGroups * 8;   // the wave's first row
    const bool lane_ok = col < N;                                   // N % 16 == 0: a lane is inside or outside as a whole

    const __amdgpu_buffer_rsrc_t rs_hi = make_rsrc(a.hi, uint32_t(K) * uint32_t(N));
    const __amdgpu_buffer_rsrc_t rs_mid = make_rsrc(a.mid, uint32_t(K) * uint32_t(N / 2));
    const __amdgpu_buffer_rsrc_t rs_lo = make_rsrc(a.lo, uint32_t(K) * uint32_t(N / 2));
    const __amdgpu_buffer_rsrc_t rs_rm = make_rsrc(a.rowmax, uint32_t(K) * 2u), rs_x = make_rsrc(a.x, uint32_t(B) * uint32_t(K) * 2u);

    // ---- x and rowmax of the first features, and of this thread's row of the slab.  In front of the weights: loads come back in the order
    // they were asked for, and a wave that has these waits for none of its HI bytes before it knows its levels and asks for MID / LO bytes.
    // Behind the weights they cost a round trip more.  us a call, 1 / 2 / 4 rows, behind -> in front: 4096x4096 10.7/11.6/12.7 ->
    // 9.7/10.5/10.7, 4096x11008 17.1/21.5/24.5 -> 16.1/19.3/20.8, 11008x4096 19.8/25.2/28.6 -> 18.4/22.5/24.2, 8192x28672 69.7/91.5/102.8 ->
    // 66.4/83.3/90.8.  (Only with as many of them as registers hold until the weights have been asked for: a loop that adds them up as they
    // come, in front of the weights, held the stream up.)
    constexpr int kPre = B == 1 ? 3 : 2;   // rounds of 4096 features
    const uint32_t nvec = uint32_t(K) / 8;
    u32x4_t rm_pre[kPre], x_pre[kPre][B];
    auto load_x = [&](uint32_t v, u32x4_t& rm, u32x4_t (&xv)[B]) {   // eight features; past the last: zeros
        rm = buf_load_b128(rs_rm, v < nvec ? v * 16 : kSkip);
#pragma unroll
        for (int b = 0; b < B; ++b) xv[b] = buf_load_b128(rs_x, v < nvec ? (uint32_t(b) * nvec + v) * 16 : kSkip);
    };
#pragma unroll
    for (int i = 0; i < kPre; ++i)
        if (i == 0 || i * kWThreads < (int)nvec) load_x(uint32_t(tid) + i * kWThreads, rm_pre[i], x_pre[i]);   // uniform
    const int g_row = lane >> 3, r_row = lane & 7, k_row = k0 + g_row * 8 + r_row;   // the row of the slab whose level this thread finds
    uint32_t r16_row = 0, x16_row[B];
#pragma unroll
    for (int b = 0; b < B; ++b) x16_row[b] = 0;
    if (k_row < K) {
        r16_row = a.rowmax[k_row];
#pragma unroll
        for (int b = 0; b < B; ++b) x16_row[b] = a.x[size_t(b) * K + k_row];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- the wave's HI bytes, before anything is known about the levels
    // K % 8 == 0: a group is inside or outside as a whole
    auto group_in = [&](int g) { return k0 + g * 8 < K; };
    const uint32_t lane_hi = lane_ok ? uint32_t(r) * uint32_t(N) + uint32_t(col) : kSkip, lane_low = uint32_t(r) * uint32_t(N / 2) + uint32_t(col / 2);
    u32x4_t H[kWGroups];
#pragma unroll
    for (int g = 0; g < kWGroups; ++g)
        H[g] = __builtin_amdgcn_raw_buffer_load_b128(rs_hi, group_in(g) ? lane_hi : kSkip, group_in(g) ? (k0 + g * 8) * N : 0, 0);
    __builtin_amdgcn_sched_barrier(0);

    // ---- Rule 1: largest addend exponent of every activation row, over all K input features (8 per thread and round)
    if (B > 1 && B < 4)   // activation rows that are not there
        for (int i = tid; i < (4 - B) * kWSlab; i += kWThreads) (&xh[B == 1 ? 0 : B][0][0][0])[i] = 0;
    // (the exponent of the largest product: one multiply and one maximum per product; a product that is not a number, of an infinite
    // weight and a zero, counts as larger than all, as its exponent says: the maximum that returns such an operand)
    float pmax[B];
#pragma unroll
    for (int b = 0; b < B; ++b) pmax[b] = 0.0f;
    auto products = [&](const u32x4_t& rm, const u32x4_t (&xv)[B]) {
        const uint32_t rw[4] = {at_least_smallest_normal(rm.x), at_least_smallest_normal(rm.y), at_least_smallest_normal(rm.z), at_least_smallest_normal(rm.w)};
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i)                             // exact products
                pmax[b] = __builtin_elementwise_maximum(pmax[b], __builtin_elementwise_maximum(fabsf(lo_half(xv[b][i]) * lo_half(rw[i])), fabsf(hi_half(xv[b][i]) * hi_half(rw[i]))));
    };
#pragma unroll
    for (int i = 0; i < kPre; ++i)
        if (i == 0 || i * kWThreads < (int)nvec) products(rm_pre[i], x_pre[i]);   // uniform
    for (uint32_t v = uint32_t(tid) + kPre * kWThreads; v < nvec; v += kWThreads) {
        u32x4_t rm, xv[B];
        load_x(v, rm, xv);
        products(rm, xv);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int m = wave_max_int((int)(float_bits(pmax[b]) & 0x7FFFFFFFu));
        if (lane == 0) pmax_s[b][wave] = m;
    }
    __syncthreads();
    {                                                               // thread -> row k_row: level and activations
        int level = 0;
#pragma unroll
        for (int b = 0; b < B; ++b) {
            int pm = pmax_s[b][0];
#pragma unroll
            for (int w = 1; w < kWWaves; ++w) pm = max(pm, pmax_s[b][w]);
            const int em = pm >> 23;
            const float P = half_bits_to_float(x16_row[b]) * half_bits_to_float(r16_row < 0x0400u ? 0x0400u : r16_row);   // rows at or past K: 0
            if (P != 0.0f) {
                const int l = level_for_mantissa_bits(10 + a.guard_bits - (em - float_exp_field(P)));
                level = l > level ? l : level;
            }
            xh[b][wave][r_row][g_row] = (uint16_t)x16_row[b];
        }
        if (a.force_level >= 0) level = a.force_level;
        lvl_s[wave][r_row][g_row] = (uint8_t)level;
        if (a.lvl_out && strip == 0 && k_row < K) a.lvl_out[k_row] = (uint8_t)level;
    }
    __builtin_amdgcn_wave_barrier();   // a wave's rows are its own: LDS serves its accesses in order

    // ---- the planes the levels ask for, then the multiply-adds
    u32x2_t M[kWGroups], L[kWGroups];
    const u32x2_t lv_w = *reinterpret_cast<const u32x2_t*>(&lvl_s[wave][r][0]);   // a byte per group
    auto lv = [&](int g) { return int((lv_w[g / 4] >> (8 * (g % 4))) & 0xFFu); };
#pragma unroll
    for (int g = 0; g < kWGroups; ++g) {
        const int need = lane_ok && group_in(g) ? lv(g) : 0, at = group_in(g) ? (k0 + g * 8) * (N / 2) : 0;
        M[g] = __builtin_amdgcn_raw_buffer_load_b64(rs_mid, need >= 1 ? lane_low : kSkip, at, 0);
        L[g] = __builtin_amdgcn_raw_buffer_load_b64(rs_lo, need >= 2 ? lane_low : kSkip, at, 0);
    }
    float acc[B][16];
    auto assemble = [&](int g, uint32_t (&pa)[4], uint32_t (&pb)[4]) {
        const uint32_t fill = fill_for_level(lv(g));
        assemble8_fill(H[g].x, H[g].y, M[g].x, L[g].x, fill, pa);   // columns 0..7 of the lane
        assemble8_fill(H[g].z, H[g].w, M[g].y, L[g].y, fill, pb);   // columns 8..15
    };
    const u32x4_t xa = *reinterpret_cast<const u32x4_t*>(&xh[B == 1 ? 0 : lane & 3][wave][r][0]);   // eight groups' rows, of activation row lane % 4
    if constexpr (B == 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[0][i] = 0.0f;
#pragma unroll
        for (int g = 0; g < kWGroups; ++g) {
            uint32_t pa[4], pb[4];
            assemble(g, pa, pb);
            const float v[16] = {lo_half(pa[0]), lo_half(pa[1]), hi_half(pa[0]), hi_half(pa[1]),
                                 lo_half(pa[2]), lo_half(pa[3]), hi_half(pa[2]), hi_half(pa[3]),
                                 lo_half(pb[0]), lo_half(pb[1]), hi_half(pb[0]), hi_half(pb[1]),
                                 lo_half(pb[2]), lo_half(pb[3]), hi_half(pb[2]), hi_half(pb[3])};
            const float xf = (g & 1) ? hi_half(xa[g / 2]) : lo_half(xa[g / 2]);
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][i] = fmaf(xf, v[i], acc[0][i]);
        }
    } else {
        // Two to four activation rows: sixteen 4x4x4 products per instruction.  A block is four lanes of one row lane r, its
        // four k are four groups' rows, its four columns one column of each of the four lanes, its four rows the activation
        // rows (those that are not there are zero): D[b] of the instruction for column i is this lane's acc[b][i].
        f32x4_t d[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < kWGroups / 4; ++q) {
            const half4_t x4 = __builtin_bit_cast(half4_t, u32x2_t{xa[2 * q], xa[2 * q + 1]});
            uint32_t p[4][8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t pa[4], pb[4];
                assemble(4 * q + i, pa, pb);
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    p[i][w] = pa[w];
                    p[i][4 + w] = pb[w];
                }
            }
#pragma unroll
            for (int w = 0; w < 8; ++w) {   // word w: columns c, c + 2
                const int c = 8 * (w >> 2) + 4 * ((w >> 1) & 1) + (w & 1);
                const u32x2_t lo = {__builtin_amdgcn_perm(p[1][w], p[0][w], 0x05040100u), __builtin_amdgcn_perm(p[3][w], p[2][w], 0x05040100u)};
                const u32x2_t hi = {__builtin_amdgcn_perm(p[1][w], p[0][w], 0x07060302u), __builtin_amdgcn_perm(p[3][w], p[2][w], 0x07060302u)};
                d[c] = __builtin_amdgcn_mfma_f32_4x4x4f16(x4, __builtin_bit_cast(half4_t, lo), d[c], 0, 0, 0);
                d[c + 2] = __builtin_amdgcn_mfma_f32_4x4x4f16(x4, __builtin_bit_cast(half4_t, hi), d[c + 2], 0, 0, 0);
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] = d[i][b];
    }

    // ---- sums: over the 8 row lanes in the vector ALU, over the waves in LDS, over the slabs in the workspace
#pragma unroll
    for (int b = 0; b < B; ++b) {
        float v[2];
        sum_row_lanes(acc[b], v);
        *reinterpret_cast<float2*>(&red_s[wave][b][cl * 16 + row_lane_column(lane)]) = make_float2(v[0], v[1]);
    }
    __syncthreads();
    const int nslab = a.nslab;
    const int c_out = strip * kWCols + (tid % kWCols), b_out = tid / kWCols;   // thread -> one (activation row, column)
    const bool mine = tid < B * kWCols && c_out < N;
    if (mine) {
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < kWWaves; ++w) sum += red_s[w][b_out][tid % kWCols];
        if (nslab == 1) a.y[size_t(b_out) * N + c_out] = sum;
        else store_agent(&a.part[(size_t(slab_i) * B + b_out) * N + c_out], sum);
    }
    if (nslab == 1) return;

    // ---- the workgroup that finishes last for this strip adds the slabs, in slab order
    stores_done();
    __syncthreads();
    if (tid == 0) last_s = take_ticket(&a.count[strip]) == nslab - 1;
    __syncthreads();
    if (!last_s) return;
    if (mine) {
        float sum = 0.0f;
        for (int s0 = 0; s0 < nslab; s0 += 8) {   // eight slabs' words in flight; the additions stay in slab order
            float p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                p[i] = s0 + i < nslab ? load_agent(&a.part[(size_t(s0 + i) * B + b_out) * N + c_out]) : 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += p[i];
        }
        a.y[size_t(b_out) * N + c_out] = sum;
    }
    if (tid == 0) store_agent(&a.count[strip], 0);   // ready for the next call
}

// W [K][N] fp16 -> planes and rowmax: one workgroup per row, a thread packs 16 columns at a time
__global__ __launch_bounds__(256) void pack_kernel(int K, int N, const uint16_t* __restrict__ W, uint8_t* hi, uint8_t* mid,
                                                   uint8_t* lo, uint16_t* rowmax)
{
    __shared__ uint32_t mx_s[4];
    const int k = blockIdx.x, tid = threadIdx.x;
    uint32_t mx = 0;
    for (int c = tid * 16; c < N; c += 256 * 16) {
        const uint4 a = *reinterpret_cast<const uint4*>(W + size_t(k) * N + c);
        const uint4 b = *reinterpret_cast<const uint4*>(W + size_t(k) * N + c + 8);
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};   // w[i] = columns 2i (low half), 2i+1 (high half)
        uint32_t h[4] = {0, 0, 0, 0}, m[2] = {0, 0}, l[2] = {0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t e = w[i] & 0xFFFFu, o = w[i] >> 16;
            h[i >> 1] |= ((e >> 8) | ((o >> 8) << 8)) << (16 * (i & 1));
            m[i >> 2] |= (((e >> 4) & 15u) | (((o >> 4) & 15u) << 4)) << (8 * (i & 3));
            l[i >> 2] |= ((e & 15u) | ((o & 15u) << 4)) << (8 * (i & 3));
            const uint32_t me = e & 0x7FFFu, mo = o & 0x7FFFu;
            mx = me > mx ? me : mx;
            mx = mo > mx ? mo : mx;
        }
        *reinterpret_cast<uint4*>(hi + size_t(k) * N + c) = make_uint4(h[0], h[1], h[2], h[3]);
        *reinterpret_cast<uint2*>(mid + size_t(k) * (N / 2) + c / 2) = make_uint2(m[0], m[1]);
        *reinterpret_cast<uint2*>(lo + size_t(k) * (N / 2) + c / 2) = make_uint2(l[0], l[1]);
    }
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t other = (uint32_t)__shfl_xor((int)mx, o);
        mx = other > mx ? other : mx;
    }
    if ((tid & 63) == 0) mx_s[tid >> 6] = mx;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) mx = mx_s[w] > mx ? mx_s[w] : mx;
        rowmax[k] = (uint16_t)mx;
    }
}

__global__ __launch_bounds__(256) void unpack_kernel(int K, int N, const uint8_t* __restrict__ hi, const uint8_t* __restrict__ mid,
                                                     const uint8_t* __restrict__ lo, uint16_t* W)
{
    const int k = blockIdx.x;
    for (int c = threadIdx.x * 2; c < N; c += 512) {
        const uint32_t m = mid[size_t(k) * (N / 2) + c / 2], l = lo[size_t(k) * (N / 2) + c / 2];
        const uint32_t h0 = hi[size_t(k) * N + c], h1 = hi[size_t(k) * N + c + 1];
        const uint32_t e = (h0 << 8) | ((m & 15u) << 4) | (l & 15u), o = (h1 << 8) | ((m >> 4) << 4) | (l >> 4);
        *reinterpret_cast<uint32_t*>(W + size_t(k) * N + c) = e | (o << 16);
    }
}

}  // namespace akv

namespace {

bool wshape_ok(int K, int N)
{
    return K >= 8 && K % 8 == 0 && K <= (1 << 20) && N >= 16 && N % 16 == 0 && (long long)K * N < (1LL << 31);
}
size_t align256(size_t x) { return (x + 255) / 256 * 256; }
bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }
size_t part_bytes(int K, int N)
{
    return align256(size_t((K + akv::kWSlab - 1) / akv::kWSlab) * AKW_MAX_B * size_t(N) * sizeof(float));
}
size_t count_bytes(int N) { return align256(size_t((N + akv::kWCols - 1) / akv::kWCols) * sizeof(int32_t)); }

akv_status check_weights(const akw_weights* w)
{
    if (!w) return akv::fail_msg(AKV_EINVAL, "weights is NULL");
    if (!wshape_ok(w->K, w->N))
        return akv::fail_msg(AKV_EINVAL, "bad shape: K=%d N=%d (need K %% 8 == 0, K <= 2^20, N %% 16 == 0, K*N < 2^31)", w->K, w->N);
    if (!w->hi || !w->mid || !w->lo || !w->rowmax) return akv::fail_msg(AKV_EINVAL, "weights has a NULL plane / rowmax pointer");
    if (!aligned16(w->hi) || !aligned16(w->mid) || !aligned16(w->lo) || !aligned16(w->rowmax))
        return akv::fail_msg(AKV_EINVAL, "the planes and rowmax must be 16-byte aligned");
    return AKV_OK;
}

}  // namespace

extern "C" {

akv_status akw_layout_sizes(int32_t K, int32_t N, akw_sizes* out)
{
    if (!out) return akv::fail_msg(AKV_EINVAL, "NULL argument");
    if (!wshape_ok(K, N)) return akv::fail_msg(AKV_EINVAL, "bad shape: K=%d N=%d (need K %% 8 == 0, K <= 2^20, N %% 16 == 0, K*N < 2^31)", K, N);
    out->hi = size_t(K) * N;
    out->mid = out->lo = size_t(K) * (N / 2);
    out->rowmax = size_t(K) * sizeof(uint16_t);
    out->workspace = part_bytes(K, N) + count_bytes(N);
    return AKV_OK;
}

akv_status akw_workspace_init(int32_t K, int32_t N, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!wshape_ok(K, N)) return akv::fail_msg(AKV_EINVAL, "bad shape: K=%d N=%d", K, N);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) || workspace_bytes < part_bytes(K, N) + count_bytes(N))
        return akv::fail_msg(AKV_EWORKSPACE, "workspace NULL, misaligned or smaller than %zu bytes", part_bytes(K, N) + count_bytes(N));
    if (hipError_t e = akv::launch_zero(static_cast<char*>(workspace) + part_bytes(K, N), count_bytes(N), static_cast<hipStream_t>(stream)))
        return akv::fail_msg(AKV_EHIP, "workspace init launch: %s", hipGetErrorString(e));
    return AKV_OK;
}

akv_status akw_pack(const akw_weights* w, const uint16_t* W, void* stream)
{
    if (akv_status st = check_weights(w)) return st;
    if (!W || !aligned16(W)) return akv::fail_msg(AKV_EINVAL, "W is NULL or not 16-byte aligned");
    hipLaunchKernelGGL(akv::pack_kernel, dim3(w->K), dim3(256), 0, static_cast<hipStream_t>(stream), w->K, w->N, W, w->hi, w->mid,
                       w->lo, w->rowmax);
    if (hipError_t e = hipGetLastError()) return akv::fail_msg(AKV_EHIP, "pack launch: %s", hipGetErrorString(e));
    return AKV_OK;
}

akv_status akw_unpack(const akw_weights* w, uint16_t* W_out, void* stream)
{
    if (akv_status st = check_weights(w)) return st;
    if (!W_out || !aligned16(W_out)) return akv::fail_msg(AKV_EINVAL, "W_out is NULL or not 16-byte aligned");
    hipLaunchKernelGGL(akv::unpack_kernel, dim3(w->K), dim3(256), 0, static_cast<hipStream_t>(stream), w->K, w->N, w->hi, w->mid,
                       w->lo, W_out);
    if (hipError_t e = hipGetLastError()) return akv::fail_msg(AKV_EHIP, "unpack launch: %s", hipGetErrorString(e));
    return AKV_OK;
}

akv_status akw_gemv(const akw_weights* w, const uint16_t* x, int32_t B, float* y, const akw_params* params, void* workspace,
                    size_t workspace_bytes, void* stream)
{
    if (akv_status st = check_weights(w)) return st;
    if (!x || !y) return akv::fail_msg(AKV_EINVAL, "x / y is NULL");
    if (!aligned16(x) || !aligned16(y)) return akv::fail_msg(AKV_EINVAL, "x and y must be 16-byte aligned");
    if (B < 1 || B > AKW_MAX_B) return akv::fail_msg(AKV_EINVAL, "B = %d out of range 1..%d", B, AKW_MAX_B);
    akw_params p = {0, -1, nullptr};
    if (params) p = *params;
    if (p.guard_bits < 0 || p.guard_bits > 12) return akv::fail_msg(AKV_EINVAL, "guard_bits = %d out of range 0..12", p.guard_bits);
    if (p.force_level < -1 || p.force_level > 2) return akv::fail_msg(AKV_EINVAL, "force_level = %d out of range -1..2", p.force_level);
    const size_t need = part_bytes(w->K, w->N) + count_bytes(w->N);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) || workspace_bytes < need)
        return akv::fail_msg(AKV_EWORKSPACE, "workspace NULL, misaligned or smaller than %zu bytes", need);
    akv::GemvArgs a;
    a.K = w->K; a.N = w->N;
    a.nslab = (w->K + akv::kWSlab - 1) / akv::kWSlab;
    a.hi = w->hi; a.mid = w->mid; a.lo = w->lo; a.rowmax = w->rowmax; a.x = x; a.y = y;
    a.part = static_cast<float*>(workspace);
    a.count = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + part_bytes(w->K, w->N));
    a.guard_bits = p.guard_bits; a.force_level = p.force_level; a.lvl_out = p.lvl_out;
    const dim3 grid((w->N + akv::kWCols - 1) / akv::kWCols, a.nslab), block(akv::kWThreads);
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (B) {
        case 1: hipLaunchKernelGGL(akv::gemv_kernel<1>, grid, block, 0, st, a); break;
        case 2: hipLaunchKernelGGL(akv::gemv_kernel<2>, grid, block, 0, st, a); break;
        case 3: hipLaunchKernelGGL(akv::gemv_kernel<3>, grid, block, 0, st, a); break;
        default: hipLaunchKernelGGL(akv::gemv_kernel<4>, grid, block, 0, st, a); break;
    }
    if (hipError_t e = hipGetLastError()) return akv::fail_msg(AKV_EHIP, "gemv launch: %s", hipGetErrorString(e));
    return AKV_OK;
}

}  // extern "C"
