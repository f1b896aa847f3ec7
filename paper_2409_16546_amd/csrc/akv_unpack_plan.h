// The launch of the unpack as plain arithmetic: workgroups of 256 threads per 256-token block of a (sequence, KV head).
#pragma once
#include <stddef.h>

namespace akv {

struct UnpackPlan {
    int k_parts, v_parts;   // workgroups per block of K (1, or 0 where K is not wanted) and per block of V
    size_t workgroups;      // 0: more than a launch can hold
};

// Both outputs: many short V workgroups between those of K keep reads and writes of the two mixed, but cost a launch that is over in a
// few rounds (one / sixteen per block of V, us: 256 blocks 13.7/15.4, 512 25.3/25.8, 1024 48.6/46.9, 2048 93/89, 4096 188/176, 8192
// 380/350).  A launch holds fewer than 2^32 threads: from 986896 blocks on (129 GB of cache) seventeen workgroups per block do not fit.
// V alone, one / two / four / eight per block: 256 blocks 7.5/7.5/7.5/7.6, 512 12.9/12.6/12.9/13.5, 4096 91/86/84/86.
inline UnpackPlan unpack_plan(size_t blocks, bool k, bool v)
{
    constexpr size_t kMost = 0xFFFFFFFFu / 256;   // workgroups of a launch
    const bool many = k && v && blocks >= 1024 && blocks * 17 <= kMost;
    const int k_parts = k ? 1 : 0, v_parts = !v ? 0 : (many ? 16 : (k ? 1 : 2));
    const size_t n = blocks * size_t(k_parts + v_parts);
    return {k_parts, v_parts, n <= kMost ? n : 0};
}

}  // namespace akv
