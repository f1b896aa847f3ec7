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
