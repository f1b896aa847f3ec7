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
// V alone: a small call needs waves enough to fill the device, a large one fewer and longer workgroups (two / four / eight per block, us: 96
// blocks 3.7/3.7/3.2, 128 4.2/4.2/4.0, 144 5.6/4.8/4.4, 160 5.7/4.9/4.7, 168 5.8/4.9/5.2, 192 5.7/4.9/5.4, 224 6.3/6.2/6.1, 256
// 6.7/6.7/6.8, 512 11.2/11.2/11.6, 1024 21.6/22.0/21.9, 4096 83.8/82.8/83.2).
inline UnpackPlan unpack_plan(size_t blocks, bool k, bool v)
{
    constexpr size_t kMost = 0xFFFFFFFFu / 256;   // workgroups of a launch
    const bool many = k && v && blocks >= 1024 && blocks * 17 <= kMost;
    const int k_parts = k ? 1 : 0, v_parts = !v ? 0 : (k ? (many ? 16 : 1) : (blocks <= 160 ? 8 : (blocks <= 192 ? 4 : 2)));
    const size_t n = blocks * size_t(k_parts + v_parts);
    return {k_parts, v_parts, n <= kMost ? n : 0};
}

}  // namespace akv
