// C ABI of the library (declared in include/akv.h): argument checks, workspace carving, launches.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "akv_common.h"

namespace {

thread_local char g_err[256] = "";

constexpr auto fail = &akv::fail_msg;   // one error record for every entry point of the library

bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

bool shape_ok(const akv_shape& s)
{
    return s.B > 0 && s.Hq > 0 && s.Hkv > 0 && s.D == akv::kD && s.Hq % s.Hkv == 0 && s.Hq / s.Hkv <= akv::kMaxG &&
           ((s.Hq / s.Hkv) & (s.Hq / s.Hkv - 1)) == 0 && s.Ncap > 0 && s.Ncap % AKV_TB == 0 && s.Ncap <= (1 << 22) &&
           size_t(s.B) * s.Hq * size_t(s.Ncap) < (size_t(1) << 40);
}

akv_status check_cache(const akv_cache* c)
{
    if (!c) return fail(AKV_EINVAL, "cache is NULL");
    if (!shape_ok(c->shape))
        return fail(AKV_EINVAL, "bad shape: B=%d Hq=%d Hkv=%d D=%d Ncap=%d (need D=128, Hq/Hkv a power of two <= 8, Ncap %% 256 == 0)",
                    c->shape.B, c->shape.Hq, c->shape.Hkv, c->shape.D, c->shape.Ncap);
    if (!c->k_hi || !c->k_mid || !c->k_lo || !c->v_hi || !c->v_mid || !c->v_lo || !c->colmax || !c->lens || !c->flags)
        return fail(AKV_EINVAL, "cache has a NULL plane / colmax / lens / flags pointer");
    if (!aligned16(c->k_hi) || !aligned16(c->k_mid) || !aligned16(c->k_lo) || !aligned16(c->v_hi) || !aligned16(c->v_mid) ||
        !aligned16(c->v_lo) || !aligned16(c->colmax) || reinterpret_cast<uintptr_t>(c->lens) % 4 || reinterpret_cast<uintptr_t>(c->flags) % 4)
        return fail(AKV_EINVAL, "cache planes and colmax must be 16-byte aligned, lens and flags 4-byte aligned");
    return AKV_OK;
}

akv_status hip_fail(hipError_t e, const char* what)
{
    return fail(AKV_EHIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace

namespace akv {
akv_status fail_msg(akv_status st, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}
int compute_units()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) cus = n;
        else cus = 256;
    }
    return cus;
}
}  // namespace akv

extern "C" {

int akv_version(void) { return 101; }

const char* akv_last_error(void) { return g_err; }

akv_status akv_layout_sizes(const akv_shape* shape, akv_sizes* out)
{
    if (!shape || !out) return fail(AKV_EINVAL, "NULL argument");
    if (!shape_ok(*shape))
        return fail(AKV_EINVAL, "bad shape: B=%d Hq=%d Hkv=%d D=%d Ncap=%d (need D=128, Hq/Hkv a power of two <= 8, Ncap %% 256 == 0)",
                    shape->B, shape->Hq, shape->Hkv, shape->D, shape->Ncap);
    const size_t e = size_t(shape->B) * shape->Hkv * size_t(shape->Ncap) * shape->D;   // elements of K (and of V)
    out->k_hi = e; out->k_mid = e / 2; out->k_lo = e / 2;
    out->v_hi = e; out->v_mid = e / 2; out->v_lo = e / 2;
    out->colmax = size_t(shape->B) * shape->Hkv * shape->D * sizeof(uint16_t);
    out->lens = size_t(shape->B) * sizeof(int32_t);
    out->flags = (AKV_NFLAGS + size_t(shape->B)) * sizeof(int32_t);
    out->workspace = akv::ws_layout(*shape).total;
    out->fp16_workspace = akv::fp16_workspace_bytes(*shape);
    return AKV_OK;
}

akv_status akv_cache_reset(const akv_cache* cache, void* stream)
{
    if (akv_status st = check_cache(cache)) return st;
    akv_sizes sz;
    akv_layout_sizes(&cache->shape, &sz);
    hipStream_t s = static_cast<hipStream_t>(stream);
    struct { void* p; size_t n; } bufs[] = {
        {cache->k_hi, sz.k_hi}, {cache->k_mid, sz.k_mid}, {cache->k_lo, sz.k_lo}, {cache->v_hi, sz.v_hi},
        {cache->v_mid, sz.v_mid}, {cache->v_lo, sz.v_lo}, {cache->colmax, sz.colmax}, {cache->lens, sz.lens},
        {cache->flags, sz.flags}};
    for (auto& bf : bufs) {
        if (hipError_t e = akv::launch_zero(bf.p, bf.n, s)) return hip_fail(e, "zero launch");
    }
    return AKV_OK;
}

akv_status akv_workspace_init(const akv_shape* shape, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!shape || !shape_ok(*shape)) return fail(AKV_EINVAL, "bad shape");
    const akv::WsLayout w = akv::ws_layout(*shape);
    if (!workspace || workspace_bytes < w.total)
        return fail(AKV_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace_bytes, w.total);
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(AKV_EWORKSPACE, "workspace is not 256-byte aligned");
    if (hipError_t e = akv::launch_zero(static_cast<char*>(workspace) + w.control, akv::align256(w.control_bytes),
                                        static_cast<hipStream_t>(stream)))
        return hip_fail(e, "zero launch");
    return AKV_OK;
}

akv_status akv_append(const akv_cache* cache, const uint16_t* k_new, const uint16_t* v_new, const int32_t* n_new,
                      int32_t n, void* stream)
{
    if (akv_status st = check_cache(cache)) return st;
    if (n < 0 || n > cache->shape.Ncap) return fail(AKV_EINVAL, "n = %d out of range 0..Ncap", n);
    if (n > 0 && (!k_new || !v_new)) return fail(AKV_EINVAL, "k_new / v_new is NULL");
    if (!aligned16(k_new) || !aligned16(v_new)) return fail(AKV_EINVAL, "k_new / v_new must be 16-byte aligned");
    if (hipError_t e = akv::launch_append(*cache, k_new, v_new, n_new, n, static_cast<hipStream_t>(stream)))
        return hip_fail(e, "append launch");
    return AKV_OK;
}

akv_status akv_check_capacity_sync(const akv_cache* cache, int32_t n, void* stream)
{
    if (akv_status st = check_cache(cache)) return st;
    if (n < 0) return fail(AKV_EINVAL, "n = %d is negative", n);
    const int B = cache->shape.B;
    std::vector<int32_t> lens(B);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (hipError_t e = hipMemcpyAsync(lens.data(), cache->lens, size_t(B) * sizeof(int32_t), hipMemcpyDeviceToHost, s)) return hip_fail(e, "hipMemcpyAsync");
    if (hipError_t e = hipStreamSynchronize(s)) return hip_fail(e, "hipStreamSynchronize");
    for (int b = 0; b < B; ++b)
        if (long(lens[b]) + n > cache->shape.Ncap)
            return fail(AKV_ECAPACITY, "sequence %d holds %d tokens: %d more exceed the capacity of %d", b, lens[b], n, cache->shape.Ncap);
    return AKV_OK;
}

akv_status akv_stream_read(const void* buf, size_t bytes, uint32_t* sink, void* stream)
{
    if (!buf || !sink) return fail(AKV_EINVAL, "buf / sink is NULL");
    if ((reinterpret_cast<uintptr_t>(buf) & 15) || (bytes & 15)) return fail(AKV_EINVAL, "buf and bytes must be multiples of 16");
    if (hipError_t e = akv::launch_stream_read(buf, bytes, sink, static_cast<hipStream_t>(stream)))
        return hip_fail(e, "stream read launch");
    return AKV_OK;
}

akv_status akv_unpack(const akv_cache* cache, uint16_t* k_out, uint16_t* v_out, void* stream)
{
    if (akv_status st = check_cache(cache)) return st;
    if (!k_out && !v_out) return AKV_OK;
    if (!aligned16(k_out) || !aligned16(v_out)) return fail(AKV_EINVAL, "k_out / v_out must be 16-byte aligned");
    if (hipError_t e = akv::launch_unpack(*cache, k_out, v_out, static_cast<hipStream_t>(stream)))
        return hip_fail(e, "unpack launch");
    return AKV_OK;
}

}  // extern "C"

// ---- the scratch of akv_decode_attention_static: one device array per GPU, never allocated or freed ------------
// In host code the array's name is only a handle: its device address is looked up per device and kept.
static __device__ __align__(256) unsigned char akv_static_scratch[AKV_STATIC_SCRATCH_BYTES];

namespace {

using akv::compute_units;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the static scratch array on the current device; on the first call on a device its control block
// is zeroed by a fill kernel on `s` (ordered in front of the decode kernels that follow on the same stream).
// Returns nullptr after recording the error text.
void* static_scratch_for_current_device(hipStream_t s)
{
    int dev = -1;
    if (hipError_t e = hipGetDevice(&dev)) { hip_fail(e, "hipGetDevice"); return nullptr; }
    if (dev < 0 || dev >= kMaxDevices) { fail(AKV_EHIP, "device ordinal %d out of range", dev); return nullptr; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(akv_static_scratch))) { hip_fail(e, "hipGetSymbolAddress"); return nullptr; }
        if (!ptr) { fail(AKV_EHIP, "hipGetSymbolAddress returned a null address"); return nullptr; }
        if (hipError_t e = akv::launch_zero(ptr, akv::kCtlReserve, s)) { hip_fail(e, "zero launch"); return nullptr; }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

// Head-per-workgroup or token-split kernels, when the caller leaves the choice to the library.  One head kernel
// workgroup occupies a compute unit, so `pairs` (sequence, KV head) pairs run in ceil(pairs / CUs) rounds of equal
// length: the path pays when there is one round and it is full enough for the length, or when the sequences are so short
// that the single launch outweighs idle units; for single query heads, which go two to a unit where there are more pairs than units, also
// with any number of them, as long as the logits of a pair fit its LDS, 12288 tokens (the token-split kernels write theirs to memory, and
// written bytes cost several times what read bytes cost).
// The host knows a bound of the lengths only (max_len, or the capacity), and sequences that are not full cost the token-split
// path more: its workgroups past the lengths are launched all the same, and those that have work fall on few XCDs.  A step (append and
// attention in one call) costs it more as well.  So the lines lie
// where the head kernel wins on attention over full sequences, or where it is behind by a few per cent there and ahead by more
// over sequences that are not full (a tenth of the bound counts too: there it is ahead nearly everywhere) and in steps.  Timed on MI355X
// over 8..256 pairs, bounds 128..11008, group sizes 1, 2, 4 (head / split, us: full, lengths a quarter to all of the bound, step, a tenth full):
//   single heads  64 pairs 256 16.5/16.3, 16.0/16.2, 20.4/19.1, 13.4/15.6; 64 pairs 512 18.1/17.7, 17.8/17.3, 22.0/20.6, 14.2/16.0, 80 pairs
//                 18.2/19.3, 18.0/19.1, 22.7/23.0, 14.2/17.9; 64 pairs 1024 20.9/20.5, 20.5/18.8, 24.5/24.3, 14.1/17.6, 80 pairs 21.3/22.1,
//                 20.5/21.6, 25.3/24.8, 14.2/19.5; 64 pairs 2048 31.2/25.3, 28.7/23.0, 33.3/28.9, 15.9/19.1, 128 pairs 32.8/30.2,
//                 30.6/28.7, 34.6/36.2, 16.2/26.2; 96 pairs 3072 38.4/34.5, 36.9/31.2, 41.6/36.9, 20.7/21.6, 128 pairs 39.7/39.1,
//                 37.2/34.5, 43.1/48.3, 20.8/23.3; 128 pairs 4096 49.7/48.3, 45.1/41.2, 54.0/60.4, 21.2/35.2, 144 pairs 50.6/56.8,
//                 45.7/48.1, 55.8/62.9, 21.2/28.8; 160 pairs 8192 103/96, 91/85, 107/108, 24/56, 176 pairs 105/107, 93/95, 110/119, 25/58;
//                 224 pairs 11008 155/167, 131/139, 161/178, 28/81
//   groups of 2   64 pairs 128 17.0/17.0, 16.8/16.9, 20.8/20.1, 15.7/16.3; 64 pairs 256 18.7/17.5, 18.3/17.3, 22.9/20.3, 16.4/16.8, 80 pairs
//                 18.8/20.7, 18.4/20.6, 23.5/23.8, 16.4/19.8; 64 pairs 512 20.7/18.9, 20.4/18.4, 25.0/22.4, 16.8/17.1, 80 pairs 20.9/21.5,
//                 20.6/21.3, 25.6/24.4, 16.9/20.2; 128 pairs 1024 26.5/25.4, 25.7/24.3, 33.3/31.8, 17.2/22.0, 160 pairs 26.7/30.0,
//                 26.0/29.1, 33.7/35.0, 17.3/26.3; 128 pairs 2048 37.2/33.7, 36.0/32.4, 42.3/40.7, 21.6/29.6, 160 pairs 37.5/41.0,
//                 36.7/38.6, 43.0/46.2, 21.8/35.2; 144 pairs 4096 66.1/63.7, 62.9/53.9, 72.7/70.2, 23.9/35.2, 160 pairs 67.1/69.0,
//                 63.3/59.0, 73.3/80.3, 24.3/48.1; 208 pairs 6144 110/112, 92/92, 115/125, 26/46; 240 pairs 8192 156/156, 135/136, 161/170,
//                 29/85
//   groups of 4   128 pairs 128 23.5/22.4, 23.5/22.2, 27.5/24.8, 21.9/21.2, 256 pairs 24.2/26.3, 23.9/26.3, 29.2/30.0, 22.0/24.4; 176 pairs
//                 512 29.5/27.9, 29.1/27.4, 34.5/35.0, 23.5/23.7, 224 pairs 29.7/30.5, 29.2/30.0, 34.8/37.4, 23.6/26.1; 192 pairs 1024
//                 35.8/33.8, 34.8/32.1, 44.6/40.9, 23.6/28.5, 208 pairs 35.9/38.2, 35.2/36.0, 45.3/44.9, 23.8/31.4; 144 pairs 2048
//                 53.2/44.3, 52.9/40.2, 59.8/51.8, 30.4/36.9, 192 pairs 54.0/49.9, 52.4/46.0, 60.4/63.7, 30.7/37.5; 208 pairs 4096 101/97,
//                 91/79, 107/110, 34/58, 256 pairs 108/106, 93/87, 114/121, 34/61; 256 pairs 6144 157/148, 132/114, 161/169, 37/78
// Single heads with more pairs than units, two to a unit up to 11264 tokens (full, lengths a quarter to all of the bound, step):
//   257 to 512    264 pairs 128 15.3/22.0, 14.9/21.6, 21.4/26.5, 384 19.3/25.5, 17.6/24.6, 24.4/29.1, 1024 32.3/33.8, 26.6/31.2, 36.4/49.3,
//                 2048 51.6/56.7, 41.6/47.6, 56.3/67.0, 3072 74.6/71.6, 62.6/60.8, 80.4/85.8, 4096 100.7/90.1, 80.4/77.0, 107/103; 320 pairs
//                 4096 104/97, 76/79, 111/114; 384 pairs 3072 82/87, 72/73, 91/104, 6144 160/156, 120/118, 169/175, 8192 211/201,
//                 166/169, 224/221; 448 pairs 8192 223/239, 172/203, 239/263, 11008 299/320, 230/251, 316/337; 512 pairs 512 24.0/30.7,
//                 22.8/29.0, 32.6/49.4, 2048 65.8/79.0, 48.5/67.2, 77/102, 8192 241/265, 183/222, 258/287
//   more          520 pairs 1024 50.3/57.3, 42.0/49.6, 62.2/75.0, 5000 196/195, 123/152, 214/210, 8192 311/305, 205/261, 332/326; 768 pairs
//                 1024 57.9/64.1, 50.9/52.5, 80.4/90.7, 4096 182/204, 127/166, 209/232; 1040 pairs 1024 86/90, 67/76, 112/125, 4096
//                 273/289, 193/237, 313/321, 8192 532/551, 376/467, 590/586; 1312 pairs 5000 403/430, 269/317, 470/455, 8192 640/673,
//                 472/569, 726/717; 2080 pairs 512 97/95, 84/83, 141/147, 1024 154/161, 120/130, 208/227, 8192 986/1042, 686/871,
//                 1129/1116; 4096 pairs 512 175/177, 152/151, 262/288, 2048 474/545, 332/436, 628/691.
//                 A block or two, not quite filled: 520 pairs 320 tokens 32.0/32.8, 29.2/30.4, 39.6/36.9; 640 pairs 128 26.8/27.8, 25.6/27.4,
//                 36.0/33.5, 384 32.5/35.5, 30.7/33.6, 43.0/44.8; 1040 pairs 128 39.6/38.8, 37.8/37.9, 50.8/51.0; 1792 pairs 256
//                 61.0/63.4, 58.2/60.6, 85.9/96.6; 2080 pairs 256 75.9/72.3, 72.1/68.9, 108/115, 448 97/94, 82/82, 133/125; 4096 pairs 256
//                 139/125, 130/119, 213/217, 384 160/157, 140/133, 240/239
// Longer ones run one after the other, and an idle part of the last round is shared by all rounds: 12288 tokens 384 pairs 320/296, 231/218,
// 512 368/383, 249/285, 544 475/457, 304/342, 768 543/573, 386/427, 896 671/686, 462/521, 1312 993/995, 669/735 (its step in an earlier
// state 5 per cent behind).
bool head_path_pays(long pairs, int G, int max_len)
{
    const long cus = compute_units(), rounds = (pairs + cus - 1) / cus;
    const double fill = double(pairs) / double(rounds * cus), last = double(pairs - (rounds - 1) * cus) / double(cus);   // of all rounds, of the last one
    if (rounds >= 2 && G != 1) return false;
    if (rounds == 2)
        return max_len <= 3072 || (max_len <= 4096 && fill >= 0.6) || (max_len <= 8192 && fill >= 0.75) || (max_len <= 11264 && fill >= 0.8) ||
               (max_len <= 12288 && fill >= 0.85);
    if (rounds > 2 && max_len <= 11264) return max_len > 448 || (pairs > 5 * cus / 2 && pairs <= 7 * cus);
    if (rounds > 2) return max_len <= 12288 && fill >= 0.83 && last >= 0.5;
    struct Rule { int len; double fill; };   // up to len tokens from this fill on
    static constexpr Rule g1[] = {{256, 0.0}, {1024, 0.3}, {2048, 0.25}, {3072, 0.5}, {4096, 0.53}, {8192, 0.65}, {12288, 0.85}},
                          g2[] = {{128, 0.0}, {512, 0.3}, {2048, 0.4}, {4096, 0.6}, {6144, 0.85}, {8192, 0.9}},
                          g4[] = {{128, 0.6}, {512, 0.7}, {1024, 0.8}, {2048, 0.6}, {4096, 0.85}, {6144, 0.97}};
    auto pays = [&](const Rule* r, int n) {
        for (int i = 0; i < n; ++i)
            if (max_len <= r[i].len) return fill >= r[i].fill;
        return false;
    };
    return G == 1 ? pays(g1, 7) : (G == 2 ? pays(g2, 6) : pays(g4, 6));
}

// decode attention, optionally preceded by the append of one token per sequence (k_new, v_new: [B][Hkv][D])
// static_scratch: the workspace is the library's own device array (akv_decode_attention_static)
akv_status decode_impl(const akv_cache* cache, const uint16_t* k_new, const uint16_t* v_new, const uint16_t* q, void* out,
                       const akv_params* params, void* workspace, size_t workspace_bytes, void* stream,
                       bool static_scratch = false)
{
    if (akv_status st = check_cache(cache)) return st;
    if (!q || !out) return fail(AKV_EINVAL, "q / out is NULL");
    if (!aligned16(q) || !aligned16(out) || !aligned16(k_new) || !aligned16(v_new))
        return fail(AKV_EINVAL, "q, out, k_new and v_new must be 16-byte aligned");
    akv_params p;
    std::memset(&p, 0, sizeof p);
    p.force_level = -1;
    if (params) p = *params;
    if (p.topk == 0) p.topk = 32;
    if (p.topk < 1 || p.topk > AKV_MAX_TOPK) return fail(AKV_EINVAL, "topk = %d out of range 1..%d", p.topk, AKV_MAX_TOPK);
    if (p.guard_bits < 0 || p.guard_bits > 12) return fail(AKV_EINVAL, "guard_bits = %d out of range 0..12", p.guard_bits);
    if (p.force_level < -1 || p.force_level > 2) return fail(AKV_EINVAL, "force_level = %d out of range -1..2", p.force_level);
    if (p.out_dtype != 0 && p.out_dtype != 1) return fail(AKV_EINVAL, "out_dtype = %d is neither 0 (f32) nor 1 (f16)", p.out_dtype);
    if (p.max_len < 0 || p.max_len > cache->shape.Ncap) return fail(AKV_EINVAL, "max_len = %d out of range 0..Ncap", p.max_len);
    if (!(p.scale == p.scale) || std::isinf(p.scale)) return fail(AKV_EINVAL, "scale is not finite");
    const akv::WsLayout w = akv::ws_layout(cache->shape, static_scratch);
    if (static_scratch) {
        if (w.total > AKV_STATIC_SCRATCH_BYTES || w.control_bytes > akv::kCtlReserve)
            return fail(AKV_EWORKSPACE, "this shape needs %zu bytes of scratch (%zu of control words); the static array holds %zu (%zu): "
                        "use akv_decode_attention with a workspace of the caller's", w.total, w.control_bytes,
                        size_t(AKV_STATIC_SCRATCH_BYTES), akv::kCtlReserve);
        hipStream_t s0 = static_cast<hipStream_t>(stream);
        workspace = static_scratch_for_current_device(s0);
        if (!workspace) return AKV_EHIP;   // the text has been recorded
        workspace_bytes = AKV_STATIC_SCRATCH_BYTES;
    }
    if (!workspace || workspace_bytes < w.total)
        return fail(AKV_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace_bytes, w.total);
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(AKV_EWORKSPACE, "workspace is not 256-byte aligned");
    if (p.stats && reinterpret_cast<uintptr_t>(p.stats) % 8) return fail(AKV_EINVAL, "stats must be 8-byte aligned");

    akv::DecodeArgs a;
    std::memset(&a, 0, sizeof a);
    a.s = cache->shape;
    a.k_hi = cache->k_hi; a.k_mid = cache->k_mid; a.k_lo = cache->k_lo;
    a.v_hi = cache->v_hi; a.v_mid = cache->v_mid; a.v_lo = cache->v_lo;
    a.colmax = cache->colmax; a.lens = cache->lens; a.q = q; a.out = out;
    a.flags = cache->flags;
    a.k_new = k_new;   // the kernels of either path store the new token themselves
    a.v_new = v_new;
    const double scale = p.scale > 0.0f ? (double)p.scale : 1.0 / std::sqrt((double)a.s.D);
    a.c = (float)(scale * 1.4426950408889634);
    a.topk = p.topk; a.guard_bits = p.guard_bits; a.force_level = p.force_level; a.out_dtype = p.out_dtype;
    a.max_len = p.max_len > 0 ? p.max_len : a.s.Ncap;
    {   // V kernel of the token-split path: one round of workgroups that fills the device -- the tokens of a
        // (sequence, KV head) pair are cut into as many chunks as there are resident workgroups per pair, so that
        // the fixed costs per workgroup (Rule 2 constants, pipeline start, partial results) are paid once per slot
        const int cus = compute_units();
        const int G = a.s.Hq / a.s.Hkv;
        const int per_cu = akv::split_v_workgroups_per_cu(G);
        const long pairs = long(a.s.B) * a.s.Hkv;
        const long per_pair = std::max(1L, long(cus) * per_cu / pairs);
        long chunk = (a.max_len + per_pair - 1) / per_pair;
        chunk = (chunk + 63) / 64 * 64;                       // whole batches of rows for every wave
        // few pairs of small capacity: chunks down to 128 tokens, at most 16 per pair (the workgroup that combines them pays
        // for each; this lower limit goes by the capacity, `chunk` by the bound of the lengths, which so may change the order of
        // the sums where there are more tokens than slots): 36.2 -> 31.9 us at 2048 tokens, 8 pairs of four heads; with 32 and
        // 64 chunks (4096, 8192 tokens) slower again
        long shortest = akv::kVChunk;
        if (pairs <= akv::kVFewPairs)
            shortest = std::min(shortest, std::max(long(akv::kVMinChunk), ((a.s.Ncap / akv::kVFewChunks + 63) / 64) * 64L));
        a.vslots = akv::v_slots(a.s);
        a.vchunk = int(std::max(shortest, chunk));
        // K kernel: a block per wave streams best where the device is full of waves; with few blocks per compute unit the time is one wave's
        // walk, and four waves share a block.  Both timed at 3 to 10 blocks per unit over 16 to 768 pairs, full, ragged (a quarter to all of
        // the bound) and a tenth full.  Four / one, us a call, 128 pairs:
        //   single heads     5 blocks 35.4/38.0, 32.1/35.0, 20.7/23.6; 6 38.6/40.6, 34.4/36.3, 23.2/25.0; 7 46.2/46.5, 38.0/39.8, 22.7/26.9; 8
        //                    50.8/48.1, 41.0/41.7, 35.9/35.6 (256 pairs, 7: 46.5/46.0; 8: 50.5/47.7, 44.4/41.3)
        //   groups of two    5 40.5/43.5, 36.4/40.3, 23.2/26.5; 6 45.2/46.4, 39.0/41.7, 25.7/27.8; 7 51.7/50.5, 41.4/43.5, 26.2/32.1
        //   groups of four   5 46.0/47.0, 38.4/43.4, 25.6/30.8; 6 51.2/49.6, 42.5/45.2, 29.0/32.5 (768 pairs, 6: 66.1/64.5, 61.1/60.4)
        //   groups of eight  5 55.3/58.9, 47.9/55.2, 32.2/37.8; 6 61.7/61.8, 52.3/57.2, 37.3/39.2; 7 69.9/68.2, 57.4/60.7, 36.1/47.3
        // Where full sequences are the slower ones the block stays with one wave.
        const long waves = pairs * ((a.max_len + akv::kTB - 1) / akv::kTB);
        a.kshort = waves <= (G == 4 ? 5L : 6L) * cus;
        // Workgroups go to the XCDs and their units in turn: where a pair has 64 or 128 of them the first blocks of all pairs meet on a few units, and
        // where sequences are far shorter than their bound those are the ones with work.  There the pairs begin at equal distances.  As they
        // were / turned, us, full, ragged, a tenth of the bound: 8 pairs 32768 single heads 37.8/37.7, 29.3/28.0, 22.6/19.9, groups of two
        // 41.4/41.4, 37.2/37.5, 26.4/23.0, of eight 51.8/51.8, 48.8/49.1, 33.1/25.7; 16 single heads 16384 36.0/36.0, 31.3/30.8, 23.0/20.4.
        // (Other counts lie differently from pair to pair by themselves: 64 pairs of four heads 5120, turned, 23.4 -> 26.1 a tenth full, 24
        // pairs of eight 13000 ragged 44.4 -> 45.2.)
        const long kgrid = (a.max_len + akv::kTB - 1) / akv::kTB;
        a.kturn = a.kshort && kgrid % 64 == 0 ? int(kgrid / pairs) : 0;
        // Fused append: the new token's K bytes are a line each for 128 channels in three planes.  Where the planes are more than the caches hold,
        // their lines leave the caches at any time among the K kernel's loads, and each turns the memory from reading to writing and back.  From
        // 32 blocks per compute unit on (0.5 GB of bounds) the selection kernel stores them, with the device nearly idle.  Stored by the K
        // kernel / the selection kernel, us a step, full and ragged: 128 single heads 32768 tokens 305.1/289.6, 213.6/213.4; 64 pairs of four
        // heads 32768 190.6/182.7, 146.2/146.8; 512 pairs of four 8192 418/398, 287/286; 1024 pairs of eight 4096 525/488, 399/381.  With fewer
        // blocks (256 single heads 6656 tokens 126.5/132.2, 98.2/101.8) and in more workgroups of shorter bounds (4096 single heads 512
        // 230/241) the K kernel is ahead.
        a.k_late = waves >= 32L * cus && a.max_len >= 4096;
        a.lg_nt = long(a.s.B) * a.s.Hq * a.max_len * long(sizeof(float)) >= (8L << 20);   // of one or two heads; figures: k_tile
    }
    char* ws = static_cast<char*>(workspace);
    a.logits = reinterpret_cast<float*>(ws + w.logits);
    a.tilemax = reinterpret_cast<float*>(ws + w.tilemax);
    a.M = reinterpret_cast<float*>(ws + w.M);
    a.Ehat = reinterpret_cast<int32_t*>(ws + w.Ehat);
    a.partO = reinterpret_cast<float*>(ws + w.partO);
    a.partZ = reinterpret_cast<float*>(ws + w.partZ);
    a.vcount = reinterpret_cast<int32_t*>(ws + w.control) + size_t(a.s.B) * a.s.Hkv;
    a.stats = p.stats;
    if (p.dbg) {
        a.dbg = *p.dbg;
        if (a.dbg.logits) a.logits = a.dbg.logits;   // same shape: the pass writes the export directly
    }
    if (p.path < 0 || p.path > 2) return fail(AKV_EINVAL, "path = %d out of range 0..2", p.path);
    if (p.path == 1 && !akv::head_path_supported(a.s))
        return fail(AKV_EINVAL, "path 1 (head per workgroup) needs Hq/Hkv <= 4");
    const bool head_path = p.path == 1 || (p.path == 0 && akv::head_path_supported(a.s) &&
                                           head_path_pays(long(a.s.B) * a.s.Hkv, a.s.Hq / a.s.Hkv, a.max_len));
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto ev = [&](int i) -> hipEvent_t { return p.events ? static_cast<hipEvent_t>(p.events[i]) : nullptr; };
    if (p.events)
        if (hipError_t e = hipEventRecord(ev(0), s)) return hip_fail(e, "hipEventRecord");
    if (head_path) {
        if (p.events)
            for (int i = 1; i < 4; ++i)
                if (hipError_t e = hipEventRecord(ev(i), s)) return hip_fail(e, "hipEventRecord");
        if (hipError_t e = akv::launch_decode_head(a, s)) return hip_fail(e, "decode (head path) launch");
    } else {
        if (p.events)
            if (hipError_t e = hipEventRecord(ev(1), s)) return hip_fail(e, "hipEventRecord");
        if (hipError_t e = akv::launch_decode_split(a, s, ev(2), ev(3))) return hip_fail(e, "decode (split path) launch");
    }
    if (p.events)
        if (hipError_t e = hipEventRecord(ev(4), s)) return hip_fail(e, "hipEventRecord");
    return AKV_OK;
}

}  // namespace

extern "C" {

akv_status akv_decode_attention(const akv_cache* cache, const uint16_t* q, void* out, const akv_params* params,
                                void* workspace, size_t workspace_bytes, void* stream)
{
    return decode_impl(cache, nullptr, nullptr, q, out, params, workspace, workspace_bytes, stream);
}

int32_t akv_decode_path(const akv_shape* shape, int32_t max_len)
{
    if (!shape || !shape_ok(*shape) || max_len < 0 || max_len > shape->Ncap) return 0;
    const int ml = max_len > 0 ? max_len : shape->Ncap;
    if (!(akv::head_path_supported(*shape) && head_path_pays(long(shape->B) * shape->Hkv, shape->Hq / shape->Hkv, ml))) return 2;
    return akv::head_logits_in_lds(*shape, ml) ? 3 : 1;
}

int32_t akv_fp16_path(const akv_shape* shape, int32_t max_len)
{
    if (!shape || !shape_ok(*shape) || max_len < 0 || max_len > shape->Ncap) return 0;
    return akv::fp16_path(*shape, max_len > 0 ? max_len : shape->Ncap);
}

akv_status akv_decode_attention_static(const akv_cache* cache, const uint16_t* q, void* out, const akv_params* params,
                                       void* stream)
{
    return decode_impl(cache, nullptr, nullptr, q, out, params, nullptr, 0, stream, true);
}

akv_status akv_append_decode_attention(const akv_cache* cache, const uint16_t* k_new, const uint16_t* v_new,
                                       const uint16_t* q, void* out, const akv_params* params, void* workspace,
                                       size_t workspace_bytes, void* stream)
{
    if (!k_new || !v_new) return fail(AKV_EINVAL, "k_new / v_new is NULL");
    return decode_impl(cache, k_new, v_new, q, out, params, workspace, workspace_bytes, stream);
}

akv_status akv_fp16_decode_attention(const akv_shape* shape, const uint16_t* k, const uint16_t* v, const int32_t* lens,
                                     const uint16_t* q, void* out, float scale, int32_t out_dtype, int32_t max_len,
                                     void* workspace, size_t workspace_bytes, void* stream)
{
    if (!shape || !shape_ok(*shape)) return fail(AKV_EINVAL, "bad shape");
    if (!k || !v || !lens || !q || !out) return fail(AKV_EINVAL, "NULL pointer argument");
    if (!aligned16(k) || !aligned16(v) || !aligned16(q) || !aligned16(out)) return fail(AKV_EINVAL, "k, v, q and out must be 16-byte aligned");
    if (out_dtype != 0 && out_dtype != 1) return fail(AKV_EINVAL, "out_dtype = %d is neither 0 (f32) nor 1 (f16)", out_dtype);
    if (max_len < 0 || max_len > shape->Ncap) return fail(AKV_EINVAL, "max_len = %d out of range 0..Ncap", max_len);
    const size_t need = akv::fp16_workspace_bytes(*shape);
    if (!workspace || workspace_bytes < need)
        return fail(AKV_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace_bytes, need);
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(AKV_EWORKSPACE, "workspace is not 256-byte aligned");
    const float sc = scale > 0.0f ? scale : (float)(1.0 / std::sqrt((double)shape->D));
    if (hipError_t e = akv::launch_fp16(*shape, k, v, lens, q, out, sc, out_dtype, max_len > 0 ? max_len : shape->Ncap,
                                        workspace, static_cast<hipStream_t>(stream)))
        return hip_fail(e, "fp16 attention launch");
    return AKV_OK;
}

}  // extern "C"
