"""GPU parity of the head kernel where two workgroups share a compute unit: more (sequence, KV head) pairs than units, single heads, on both
sides of the bounds where half blocks end (1024 tokens) and where the logits of two workgroups stop fitting the LDS (11264)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("Ncap,B", [(1024, 65), (1280, 65), (11264, 65), (11520, 65), (1280, 131)])   # 131: more than two pairs per unit
def test_more_single_heads_than_units_match_oracle(Ncap, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import akv_oracle as O
    O.build()
    import akv_testlib as T
    from paper_2409_16546_amd import binding as A, workloads
    Hkv = 4
    print(f"head kernel: {B * Hkv} pairs, room for {Ncap}", flush=True)
    n = min(Ncap, 1280)
    w = workloads.make(2, B=B, Hq=Hkv, Hkv=Hkv, N=n, seed=Ncap)
    rng = np.random.default_rng(Ncap)
    lens = [int(x) for x in rng.integers(2, 330, size=B)]
    lens[:8] = [0, 1, n - 1, n, 511, 512, 513, 255]
    oc, gc = T.oracle_cache(w.k, w.v, lens, Ncap), T.gpu_cache(w.k, w.v, lens, Hkv, Ncap)
    if Ncap > n:                                     # up to the room: rows of zeros behind the tokens
        for b, x in ((3, Ncap - 1), (64, Ncap), (20, Ncap - 700)):
            lens[b] = x
        oc.lens[:] = lens
        gc.lens.copy_(torch.tensor(lens, dtype=torch.int32))
    dbg = A.DebugBuffers.allocate(gc, want_needV=False)
    out = A.akv_decode_attention(gc, w.q.to(DEV), dbg=dbg, path=1).clone()
    plain = A.akv_decode_attention(gc, w.q.to(DEV), path=1)
    torch.cuda.synchronize()
    assert torch.equal(plain, out)
    T.assert_decode_equal(out, dbg, O.decode_attention(oc, T.bits(w.q)), lens, 1, f"{B * Hkv} pairs, {Ncap}")
    gen = torch.Generator().manual_seed(Ncap)        # then one token more, fused; the full sequence refuses it
    kn, vn = (torch.randn(B, Hkv, 1, 128, generator=gen).half() for _ in range(2))
    refused = O.append(oc, T.bits(kn), T.bits(vn), np.array([1] * B, np.int32))
    out = A.akv_append_decode_attention(gc, kn.to(DEV), vn.to(DEV), w.q.to(DEV), dbg=dbg, path=1)
    torch.cuda.synchronize()
    T.assert_cache_equal(gc, oc)
    T.assert_decode_equal(out, dbg, O.decode_attention(oc, T.bits(w.q)), oc.lens.tolist(), 1, f"{B * Hkv} pairs, {Ncap}, step")
    assert refused == 1 and int(gc.flags.cpu()[A.AKV_FLAG_OVERFLOW]) == 1
