"""GPU parity of the weight GEMV where two to four activation rows go through the matrix cores: the smallest shapes, ragged strips and
slabs, subnormal weights and activations (they must not be flushed), an activation row of zeros."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("B", [1, 2, 3, 4])
@pytest.mark.parametrize("K,N,tiny", [(8, 16, False), (520, 144, False), (64, 128, True), (1032, 272, True)])
def test_gemv_edges_match_oracle(K, N, tiny, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import akw_oracle as OW
    from paper_2409_16546_amd import binding as A, workloads
    OW.build()
    print(f"gemv edges: K{K} N{N} B{B} subnormal {tiny}", flush=True)
    bits = lambda t: np.ascontiguousarray(t.contiguous().view(torch.int16).numpy().view(np.uint16))
    wl = workloads.make_weights((K, N), B, outliers=2, seed=K + B)
    W, x = (wl.W.float() * 2.0 ** -16).half() if tiny else wl.W, (wl.x.float() * 2.0 ** -16).half() if tiny else wl.x
    if B > 2:
        x[1] = 0
    gw = A.Weights.allocate(K, N, DEV)
    A.akw_pack(gw, W.to(DEV))
    lvl = torch.empty(K, dtype=torch.uint8, device=DEV)
    y = A.akw_gemv(gw, x.to(DEV), lvl_out=lvl)
    torch.cuda.synchronize()
    r = OW.gemv(OW.pack(bits(W)), bits(x))
    assert np.array_equal(lvl.cpu().numpy(), r.lvl)
    # at most 19 + K/512 binary32 additions of a running sum no larger than S_n = sum |x w| (2^-24 of it each): below 1.3e-6
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - r.y) <= 1.3e-6 * r.abs_sum)


@pytest.mark.parametrize("B", [1, 2, 4])
def test_gemv_levels_with_infinite_weights_match_oracle(B):
    """An infinite weight makes its row's products infinite or, where the activation is zero, not a number; either has the largest
    exponent there is, so that the other rows are read at level 0.  Columns without the infinity stay finite."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import akw_oracle as OW
    from paper_2409_16546_amd import binding as A
    OW.build()
    print(f"gemv infinite weights: B{B}", flush=True)
    bits = lambda t: np.ascontiguousarray(t.contiguous().view(torch.int16).numpy().view(np.uint16))
    g = torch.Generator().manual_seed(B)
    K, N = 1040, 160
    W, x = torch.randn(K, N, generator=g).half(), torch.randn(B, K, generator=g).half()
    W[3, 5], W[700, 150] = float("inf"), float("-inf")
    for zeros in ([3, 700], [3], []):                       # both products are no numbers, one, none
        x[:, 3], x[:, 700] = 0.5, -0.25
        x[:, zeros] = 0
        gw = A.Weights.allocate(K, N, DEV)
        A.akw_pack(gw, W.to(DEV))
        lvl = torch.empty(K, dtype=torch.uint8, device=DEV)
        y = A.akw_gemv(gw, x.to(DEV), lvl_out=lvl).cpu().numpy().astype(np.float64)
        r = OW.gemv(OW.pack(bits(W)), bits(x))
        assert np.array_equal(lvl.cpu().numpy(), r.lvl)
        fin = np.isfinite(r.y)
        assert np.array_equal(np.isnan(y), np.isnan(r.y)) and np.array_equal(y[~fin & ~np.isnan(r.y)], r.y[~fin & ~np.isnan(r.y)])
        assert fin.sum() == B * (N - 2) and np.all(np.abs(y[fin] - r.y[fin]) <= 1.3e-6 * r.abs_sum[fin])


@pytest.mark.parametrize("B,K", [(1, 4104), (2, 4088), (4, 4104), (1, 8200), (3, 8192), (4, 8200), (1, 12288), (1, 12304), (2, 12304)])
def test_gemv_rounds_of_features_match_oracle(B, K):
    """The largest product is found 4096 features a round, the first rounds (three for one activation row, two for more) in flight together
    and the others one after the other: sizes at the edges of the rounds, the largest product in the last feature."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import akw_oracle as OW
    from paper_2409_16546_amd import binding as A, workloads
    OW.build()
    N = 144
    print(f"gemv rounds: K{K} N{N} B{B}", flush=True)
    bits = lambda t: np.ascontiguousarray(t.contiguous().view(torch.int16).numpy().view(np.uint16))
    wl = workloads.make_weights((K, N), B, outliers=2, seed=K + B)
    wl.x[:, K - 1] = 300.0
    gw = A.Weights.allocate(K, N, DEV)
    A.akw_pack(gw, wl.W.to(DEV))
    lvl = torch.empty(K, dtype=torch.uint8, device=DEV)
    y = A.akw_gemv(gw, wl.x.to(DEV), lvl_out=lvl)
    torch.cuda.synchronize()
    r = OW.gemv(OW.pack(bits(wl.W)), bits(wl.x))
    assert np.array_equal(lvl.cpu().numpy(), r.lvl)
    # 19 + K / 512 binary32 additions of a running sum no larger than S_n = sum |x w|, 2^-24 of it each
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - r.y) <= (19 + (K + 511) // 512) * 2.0 ** -24 * r.abs_sum)
