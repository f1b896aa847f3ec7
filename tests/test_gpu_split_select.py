"""GPU parity of the selection of the token-split path where it reads only part of the K blocks: 32 blocks and more, with the
cut in the first bucket (flat scores), in the middle, and in the floor bucket (peaked scores); block and wave edges.
The score exponents are not exported here: their export makes the kernel read every block."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import akv_oracle
    akv_oracle.build()
    import akv_testlib
    return akv_testlib


@pytest.mark.parametrize("topk", [1, 32, 64])
@pytest.mark.parametrize("cfg,G,scale,lens", [
    (1, 1, 0.0, [8192, 8193]),          # exactly 32 blocks, and one token in a block of its own
    (2, 2, 0.002, [16640, 8191]),       # flat: every token in the first buckets; 65 blocks (more than a ballot), 31.99
    (3, 4, 0.0, [20000, 9001]),         # peaked: the cut lies in the floor bucket, taken by position
    (4, 8, 0.02, [12288, 300]),
    (5, 1, 0.0, [33000, 16384]),
    (2, 4, 1e-6, [33000, 8200]),        # all but the best token in one bucket
])
def test_selection_matches_oracle(T, cfg, G, scale, lens, topk):
    from paper_2409_16546_amd import binding as A, workloads
    from oracle import akv_oracle as O
    print(f"split selection: cfg{cfg} G{G} scale {scale} lens {lens} topk {topk}", flush=True)
    w = workloads.make(cfg, B=2, Hq=G, Hkv=1, N=max(lens), seed=77 + G)
    Ncap = (max(lens) + 255) // 256 * 256
    oc = T.oracle_cache(w.k, w.v, lens, Ncap)
    r = O.decode_attention(oc, T.bits(w.q), topk=topk, scale=scale)
    gc = T.gpu_cache(w.k, w.v, lens, G, Ncap)
    dbg = A.DebugBuffers.allocate(gc, topk=topk, want_needV=False)
    dbg.a = None
    out = A.akv_decode_attention(gc, w.q.to(DEV), dbg=dbg, path=2, topk=topk, scale=scale)
    torch.cuda.synchronize()
    assert np.array_equal(dbg.sel.cpu().numpy(), r.sel)
    assert np.array_equal(dbg.oest.cpu().numpy().view(np.uint32), r.oest.view(np.uint32))
    assert np.array_equal(dbg.Ehat.cpu().numpy(), r.Ehat)
    bound = T.out_tolerance(r, lens, scale)
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - r.out).max(axis=2) <= bound)


def test_selection_of_more_than_1024_blocks(T):
    """More than 1024 blocks in a sequence: a wave's share is more than 64 of them, a ballot each.  Tokens of the later ones are selected, and one
    sequence ends with a block of a single token."""
    from paper_2409_16546_amd import binding as A, workloads
    from oracle import akv_oracle as O
    lens, topk, scale = [300000, 262145], 64, 0.02
    print(f"split selection: lens {lens}", flush=True)
    w = workloads.make(4, B=2, Hq=2, Hkv=1, N=max(lens), seed=78)
    w.k[1, :, 262144] = w.k[1, :, :262144].abs().amax(1) * w.q[1, 0].sign()        # the lone token has the largest score of a head
    Ncap = (max(lens) + 255) // 256 * 256
    oc = T.oracle_cache(w.k, w.v, lens, Ncap)
    r = O.decode_attention(oc, T.bits(w.q), topk=topk, scale=scale)
    assert (r.sel[0] >= 262144).any() and (r.sel[1, 0] == 262144).any()
    gc = T.gpu_cache(w.k, w.v, lens, 2, Ncap)
    dbg = A.DebugBuffers.allocate(gc, topk=topk, want_needV=False)
    dbg.a = None
    out = A.akv_decode_attention(gc, w.q.to(DEV), dbg=dbg, path=2, topk=topk, scale=scale)
    torch.cuda.synchronize()
    assert np.array_equal(dbg.sel.cpu().numpy(), r.sel)
    assert np.array_equal(dbg.oest.cpu().numpy().view(np.uint32), r.oest.view(np.uint32))
    assert np.array_equal(dbg.Ehat.cpu().numpy(), r.Ehat)
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - r.out).max(axis=2) <= T.out_tolerance(r, lens, scale))


@pytest.mark.parametrize("n", [700, 9000])
def test_selection_stays_in_range_on_infinite_keys(T, n):
    """One sequence holds infinities in K (its logits are infinite or not numbers: results unspecified), the other does not: the
    selection of the first still names stored tokens only, the second's result is that of finite data."""
    from paper_2409_16546_amd import binding as A, workloads
    print(f"split selection: infinite keys, {n} tokens", flush=True)
    w = workloads.make(3, B=2, Hq=4, Hkv=2, N=n, seed=5)
    Ncap = (n + 255) // 256 * 256
    q = w.q.to(DEV)
    good = A.akv_decode_attention(T.gpu_cache(w.k, w.v, [n, n], 4, Ncap), q, path=2)
    k = w.k.clone()
    k[0, :, ::3, ::5] = float("inf")
    k[0, :, 1::7, 2] = float("-inf")
    gc = T.gpu_cache(k, w.v, [n, n], 4, Ncap)
    dbg = A.DebugBuffers.allocate(gc, want_needV=False)
    dbg.a = None
    out = A.akv_decode_attention(gc, q, dbg=dbg, path=2)
    torch.cuda.synchronize()
    sel = dbg.sel.cpu().numpy()
    assert sel.min() >= 0 and sel.max() < n
    assert torch.equal(out[1], good[1])


def test_selection_of_many_heads(T):
    """More query heads than compute units: the selection runs with 512 threads per head (1024 in the cases above)."""
    from paper_2409_16546_amd import binding as A, workloads
    from oracle import akv_oracle as O
    B, Hkv, lens = 5, 64, [8300, 8192, 1, 4097, 6000]
    print(f"split selection: {B * Hkv} heads, lens {lens}", flush=True)
    w = workloads.make(3, B=B, Hq=Hkv, Hkv=Hkv, N=max(lens), seed=91)
    oc = T.oracle_cache(w.k, w.v, lens, 8448)
    r = O.decode_attention(oc, T.bits(w.q))
    gc = T.gpu_cache(w.k, w.v, lens, Hkv, 8448)
    dbg = A.DebugBuffers.allocate(gc, want_needV=False)
    dbg.a = None
    A.akv_decode_attention(gc, w.q.to(DEV), dbg=dbg, path=2)
    torch.cuda.synchronize()
    assert np.array_equal(dbg.sel.cpu().numpy(), r.sel) and np.array_equal(dbg.Ehat.cpu().numpy(), r.Ehat)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_token_split_with_four_blocks_per_unit(T, G):
    """1024 K blocks, four waves each: four workgroups of the K kernel to a compute unit.  More pairs than those the V kernel cuts into short
    chunks; ragged lengths down to one token."""
    from paper_2409_16546_amd import workloads
    lens = [2048, 1, 1027, 300]
    print(f"token-split path, four blocks per unit: G{G} lens {lens}", flush=True)
    w = workloads.make(2, B=4, Hq=32 * G, Hkv=32, N=2048, seed=500 + G)
    gc, oc, out, dbg, r = T.run_both(w.k, w.v, w.q, lens, path=2)
    T.assert_decode_equal(out, dbg, r, lens, G, f"four blocks per unit G{G}")


def test_token_split_with_one_wave_per_block_of_eight_heads(T):
    """Groups of eight, 128 pairs of 13 blocks: more than six blocks per compute unit; a wave of the K kernel takes a whole one for all eight heads."""
    from paper_2409_16546_amd import workloads
    lens = [3328, 1025, 256, 2817]
    print(f"token-split path, one wave per block: G8 lens {lens}", flush=True)
    w = workloads.make(3, B=4, Hq=256, Hkv=32, N=3328, seed=508)
    gc, oc, out, dbg, r = T.run_both(w.k, w.v, w.q, lens, path=2)
    T.assert_decode_equal(out, dbg, r, lens, 8, "one wave per block G8")


@pytest.mark.parametrize("G,lens", [(1, [1024, 129]), (2, [2048, 127]), (4, [4100, 128]), (8, [700, 385])])
def test_token_split_with_short_chunks(T, G, lens):
    """Few pairs of short sequences: chunks of the V kernel below 512 tokens (128, 128, 320 and 128 of them), lengths around 128."""
    from paper_2409_16546_amd import workloads
    print(f"token-split path, short chunks: G{G} lens {lens}", flush=True)
    w = workloads.make(4, B=2, Hq=2 * G, Hkv=2, N=max(lens), seed=600 + G)
    gc, oc, out, dbg, r = T.run_both(w.k, w.v, w.q, lens, path=2)
    T.assert_decode_equal(out, dbg, r, lens, G, f"short chunks G{G}")


@pytest.mark.parametrize("lens", [[1, 63, 64, 65], [255, 256, 257, 191], [0, 513, 128, 193]])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_token_split_with_four_waves_per_block(T, G, lens):
    """Few K blocks: the four waves of a workgroup take 64 tokens of its block each; lengths around the edges of waves and blocks."""
    from paper_2409_16546_amd import workloads
    print(f"token-split path, four waves per block: G{G} lens {lens}", flush=True)
    w = workloads.make(2, B=4, Hq=3 * G, Hkv=3, N=max(lens), seed=700 + G)
    gc, oc, out, dbg, r = T.run_both(w.k, w.v, w.q, lens, path=2, guard_bits=G % 3)
    T.assert_decode_equal(out, dbg, r, lens, G, f"four waves per block G{G}")


@pytest.mark.parametrize("G", [1, 2, 4])
def test_token_split_with_one_wave_per_block(T, G):
    """More than six K blocks per compute unit: a wave takes a whole one."""
    from paper_2409_16546_amd import workloads
    lens = [3328, 1, 2049, 300]
    print(f"token-split path, one wave per block: G{G} lens {lens}", flush=True)
    w = workloads.make(2, B=4, Hq=32 * G, Hkv=32, N=3328, seed=800 + G)
    gc, oc, out, dbg, r = T.run_both(w.k, w.v, w.q, lens, path=2)
    T.assert_decode_equal(out, dbg, r, lens, G, f"one wave per block G{G}")


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_token_split_with_six_blocks_per_unit(T, G):
    """Six K blocks per compute unit, the last count that goes to four waves each (groups of four: a wave each)."""
    from paper_2409_16546_amd import workloads
    lens = [3072, 3, 2049, 1281]
    print(f"token-split path, six blocks per unit: G{G} lens {lens}", flush=True)
    w = workloads.make(2, B=4, Hq=32 * G, Hkv=32, N=3072, seed=820 + G)
    gc, oc, out, dbg, r = T.run_both(w.k, w.v, w.q, lens, path=2)
    T.assert_decode_equal(out, dbg, r, lens, G, f"six blocks per unit G{G}")


@pytest.mark.parametrize("cfg,scale", [(3, 0.0), (2, 1e-6), (2, 0.01)])          # the cut in the floor bucket, in the first, between
@pytest.mark.parametrize("lens", [[16384, 16385, 4097], [5000, 129, 33]])
def test_selection_where_every_wave_reads_all_of_its_blocks(T, cfg, scale, lens):
    """Up to 64 blocks the sixteen waves read and keep all of them; one block more and they read those up to a bound."""
    from paper_2409_16546_amd import binding as A, workloads
    from oracle import akv_oracle as O
    print(f"split selection: cfg{cfg} scale {scale} lens {lens}", flush=True)
    w = workloads.make(cfg, B=3, Hq=2, Hkv=2, N=max(lens), seed=60 + cfg)
    Ncap = (max(lens) + 255) // 256 * 256
    r = O.decode_attention(T.oracle_cache(w.k, w.v, lens, Ncap), T.bits(w.q), topk=64, scale=scale)
    gc = T.gpu_cache(w.k, w.v, lens, 2, Ncap)
    dbg = A.DebugBuffers.allocate(gc, topk=64, want_needV=False)
    dbg.a = None
    A.akv_decode_attention(gc, w.q.to(DEV), dbg=dbg, path=2, topk=64, scale=scale)
    torch.cuda.synchronize()
    assert np.array_equal(dbg.sel.cpu().numpy(), r.sel) and np.array_equal(dbg.Ehat.cpu().numpy(), r.Ehat)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("Hkv,Ncap,lens,max_len", [
    (3, 1024, [0, 1, 63, 64, 255, 256, 1023, 1024], 0),          # four waves per block; the last sequence is full
    (3, 1024, [0, 511, 512, 513, 700, 1023, 767, 1024], 512),    # the new token at, behind and far behind the bound
    (40, 1280, [0, 255, 256, 1023, 1024, 1025, 1279, 1280], 0),  # 1600 blocks: a wave per block
    (40, 1280, [1100, 1101, 1102, 1150, 1200, 1024, 1279, 1280], 1101),
])
def test_token_split_step_is_append_then_attention(T, G, Hkv, Ncap, lens, max_len):
    """The token-split kernels store the new token themselves: cache, flags and result are those of an append followed by attention."""
    from paper_2409_16546_amd import binding as A, workloads
    print(f"token-split step: G{G} Hkv{Hkv} Ncap{Ncap} lens{lens} max_len{max_len}", flush=True)
    B = len(lens)
    w = workloads.make(2, B=B, Hq=Hkv * G, Hkv=Hkv, N=Ncap, seed=900 + G)
    gen = torch.Generator().manual_seed(G)
    kn, vn = ((torch.randn(B, Hkv, 1, 128, generator=gen) * 3).half().to(DEV) for _ in range(2))
    q = w.q.to(DEV)
    one, two = (T.gpu_cache(w.k, w.v, lens, Hkv * G, Ncap) for _ in range(2))
    for turn in range(2):   # an even place, then an odd one
        if turn:
            kn, vn = kn.flip(0).contiguous(), vn.flip(1).contiguous()
        out = A.akv_append_decode_attention(one, kn, vn, q, path=2, max_len=max_len)
        A.akv_append(two, kn, vn)
        ref = A.akv_decode_attention(two, q, path=2, max_len=max_len)
        torch.cuda.synchronize()
        for name in ("k_hi", "k_mid", "k_lo", "v_hi", "v_mid", "v_lo", "colmax", "lens", "flags"):
            assert torch.equal(getattr(one, name), getattr(two, name)), f"{name}, turn {turn}"
        assert torch.equal(out, ref)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("max_len", [0, 131072 + 5])                             # every token attended; tokens at and behind the bound
def test_token_split_step_of_many_blocks_is_append_then_attention(T, G, max_len):
    """From 32 blocks per compute unit on the selection kernel stores the new token's K bytes, the workgroups of a group's heads a share of the
    channels each: cache, flags and result are those of an append followed by attention."""
    from paper_2409_16546_amd import binding as A
    B, Hkv, Ncap, n = 9, 2, 262144, 1100
    lens = [0, 1, 255, 256, 1023, 70000, Ncap - 1, Ncap, 131072 + 4]
    print(f"token-split step of many blocks: G{G} max_len {max_len}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(G)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEV).half()
    k, v, q = randn(B, Hkv, n, 128), randn(B, Hkv, n, 128), randn(B, Hkv * G, 128)
    one, two = (A.Cache.allocate(B, Hkv * G, Hkv, 128, Ncap, DEV) for _ in range(2))
    for c in (one, two):
        A.akv_append(c, k, v, torch.tensor([min(x, n) for x in lens], dtype=torch.int32, device=DEV))
        c.lens.copy_(torch.tensor(lens, dtype=torch.int32))                      # rows of zeros behind the first 1100 tokens
    for turn in range(2):   # an even place, then an odd one
        kn, vn = randn(B, Hkv, 1, 128) * 9, randn(B, Hkv, 1, 128)
        out = A.akv_append_decode_attention(one, kn, vn, q, path=2, max_len=max_len)
        A.akv_append(two, kn, vn)
        ref = A.akv_decode_attention(two, q, path=2, max_len=max_len)
        torch.cuda.synchronize()
        for name in ("k_hi", "k_mid", "k_lo", "v_hi", "v_mid", "v_lo", "colmax", "lens", "flags"):
            assert torch.equal(getattr(one, name), getattr(two, name)), f"{name}, turn {turn}"
        assert torch.equal(out, ref)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_token_split_step_where_the_pairs_begin_at_equal_distances(T, G):
    """64 K blocks per pair, four waves per block: the workgroups of a pair begin with another block in every pair, and the one that stores
    the new token and the one that counts move with them."""
    from paper_2409_16546_amd import binding as A, workloads
    from oracle import akv_oracle as O
    B, Hkv, N, lens = 2, 3, 16384, [16384, 4099]
    print(f"token-split step, turned: G{G} lens {lens}", flush=True)
    w = workloads.make(2, B=B, Hq=Hkv * G, Hkv=Hkv, N=N, seed=1000 + G)
    oc, gc = T.oracle_cache(w.k, w.v, lens, N), T.gpu_cache(w.k, w.v, lens, Hkv * G, N)
    gen = torch.Generator().manual_seed(G)
    kn, vn = (torch.randn(B, Hkv, 1, 128, generator=gen).half() for _ in range(2))
    refused = O.append(oc, T.bits(kn), T.bits(vn), np.array([1] * B, np.int32))
    dbg = A.DebugBuffers.allocate(gc, want_needV=False)
    out = A.akv_append_decode_attention(gc, kn.to(DEV), vn.to(DEV), w.q.to(DEV), dbg=dbg, path=2)
    torch.cuda.synchronize()
    T.assert_cache_equal(gc, oc)
    T.assert_decode_equal(out, dbg, O.decode_attention(oc, T.bits(w.q)), oc.lens.tolist(), G, f"turned G{G}")
    assert refused == 1 and int(gc.flags.cpu()[A.AKV_FLAG_OVERFLOW]) == 1


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_token_split_step_with_one_wave_per_block(T, G):
    """1600 K blocks: a wave per block, and the one whose block the new token joins takes its values from the token's row.  Cache and decisions
    against the oracle; the new token is the first of a block, the last, between, at odd and even places, and refused."""
    from paper_2409_16546_amd import binding as A, workloads
    from oracle import akv_oracle as O
    B, Hkv, N, lens = 8, 40, 1280, [0, 255, 256, 1023, 1024, 1025, 1279, 1280]
    print(f"token-split step, one wave per block: G{G} lens {lens}", flush=True)
    w = workloads.make(2, B=B, Hq=Hkv * G, Hkv=Hkv, N=N, seed=1100 + G)
    oc, gc = T.oracle_cache(w.k, w.v, lens, N), T.gpu_cache(w.k, w.v, lens, Hkv * G, N)
    gen = torch.Generator().manual_seed(G)
    kn, vn = ((torch.randn(B, Hkv, 1, 128, generator=gen) * 3).half() for _ in range(2))
    refused = O.append(oc, T.bits(kn), T.bits(vn), np.array([1] * B, np.int32))
    dbg = A.DebugBuffers.allocate(gc, want_needV=False)
    out = A.akv_append_decode_attention(gc, kn.to(DEV), vn.to(DEV), w.q.to(DEV), dbg=dbg, path=2)
    torch.cuda.synchronize()
    T.assert_cache_equal(gc, oc)
    T.assert_decode_equal(out, dbg, O.decode_attention(oc, T.bits(w.q)), oc.lens.tolist(), G, f"step, one wave per block G{G}")
    assert refused == 1 and int(gc.flags.cpu()[A.AKV_FLAG_OVERFLOW]) == 1
