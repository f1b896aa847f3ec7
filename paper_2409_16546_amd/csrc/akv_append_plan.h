// The block append as plain arithmetic, for host and device: which tokens a workgroup of the launch stores, and how many
// workgroups have to have read a sequence's length before it may move.
#pragma once

#if defined(__HIPCC__)
#define AKV_HOST_DEVICE __host__ __device__
#else
#define AKV_HOST_DEVICE
#endif

namespace akv {

constexpr int kPlanTB = 256;   // tokens per K block

// blocks per head a launch for up to n tokens covers: from any place inside a block, n tokens touch at most this many
AKV_HOST_DEVICE inline int append_grid_blocks(int n) { return (n + kPlanTB - 2) / kPlanTB + 1; }

// block i of the launch for a sequence of len tokens that takes cnt more: tokens [t_lo, t_hi) of K block blk, none if t_lo >= t_hi
struct AppendBlock { int blk, t_lo, t_hi; };
AKV_HOST_DEVICE inline AppendBlock append_block(int len, int cnt, int i)
{
    const int blk = len / kPlanTB + i, lo = blk * kPlanTB, hi = lo + kPlanTB;
    return {blk, len > lo ? len : lo, len + cnt < hi ? len + cnt : hi};
}

// What workgroup x of `grid` = 2 S blocks of a head does: block i of the launch, K or V, and which of the S parts of that side (channels of K,
// rows of V).  Workgroups go to the XCDs in turn: were a head's parts always in the same order, those without tokens (the last block's,
// mostly) would leave the same XCDs idle where the parts are a multiple of two, four or eight.  So with S > 1 they begin at another one in
// every head (head: its number over the whole batch).
struct AppendPart { int i, v, sub; };
template <int S> AKV_HOST_DEVICE inline AppendPart append_part(unsigned x, unsigned grid, unsigned head)
{
    const unsigned turned = x + (S == 1 ? 0u : head % grid), part = turned < grid ? turned : turned - grid;
    return {int(part / (2 * S)), int(part & 1), S == 1 ? 0 : int(part >> 1) % S};
}

// Tickets of a sequence: one of every workgroup of the launch (`parts` each for K and V of each block of each head), also of those whose block
// the tokens do not touch.  Such a workgroup only knows so from the length: were the length to move before it has read it, it
// would find work that is not there.
AKV_HOST_DEVICE inline int append_tickets(int grid_blocks, int Hkv, int parts) { return 2 * parts * grid_blocks * Hkv; }

}  // namespace akv
