"""GPU parity of the fp16 decode attention at the edges of its tiles: every group size, lengths around a tile of 32 tokens, a wave's
and a workgroup's share, one chunk (the workgroup writes the result itself) and several (merged), fp16 output."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("Ncap,lens", [(256, [0, 1, 31, 32, 33, 127, 128, 129, 256]), (2816, [2816, 2785, 640, 129, 0])])
def test_fp16_attention_matches_textbook(G, Ncap, lens):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import akv_testlib as T
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A, workloads
    O.build()
    print(f"fp16 attention: G{G} Ncap {Ncap} lens {lens}", flush=True)
    B, Hkv = len(lens), 2
    w = workloads.make(2, B=B, Hq=G * Hkv, Hkv=Hkv, N=Ncap, seed=40 + G)
    lens = np.asarray(lens, np.int32)
    args = (w.k.to(DEV), w.v.to(DEV), torch.from_numpy(lens).to(DEV), w.q.to(DEV))
    out = A.akv_fp16_decode_attention(*args)
    first = A.akv_fp16_decode_attention(*args, max_len=128)                      # one chunk per sequence
    out16 = A.akv_fp16_decode_attention(*args, out=torch.empty_like(args[3]))
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    ref = O.fp16_attention(T.bits(w.k), T.bits(w.v), lens, T.bits(w.q))
    assert np.abs(got - ref).max() <= T.MAX_ABS and T.rel_l2(got, ref) <= T.REL_L2
    assert torch.equal(out16, out.to(torch.float16)) and not got[lens == 0].any()
    ref1 = O.fp16_attention(T.bits(w.k), T.bits(w.v), np.minimum(lens, 128), T.bits(w.q))
    got1 = first.cpu().numpy().astype(np.float64)
    assert np.abs(got1 - ref1).max() <= T.MAX_ABS and T.rel_l2(got1, ref1) <= T.REL_L2


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_fp16_minus_infinite_logits_have_weight_zero(G):
    """Keys of minus infinity (positive queries): the first tiles of a wave, whole shares and chunks, scattered tokens; a sequence of
    nothing else is not a number, as in the textbook form."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import akv_testlib as T
    from paper_2409_16546_amd import binding as A
    print(f"fp16 attention, minus infinity: G{G}", flush=True)
    g = torch.Generator().manual_seed(G)
    B, Hkv, N = 3, 2, 1024
    q = (torch.rand(B, Hkv * G, 128, generator=g) + 0.1).half()
    k, v = torch.randn(B, Hkv, N, 128, generator=g).half(), torch.randn(B, Hkv, N, 128, generator=g).half()
    k[0, :, :650] = float("-inf")              # whole chunks, then a share that begins with them
    k[1, :, 32:64, 5] = float("-inf")
    k[1, :, 300::7, 9] = float("-inf")
    k[2] = float("-inf")
    args = [t.to(DEV) for t in (k, v, torch.tensor([1024, 650, 700], dtype=torch.int32), q)]
    got = A.akv_fp16_decode_attention(*args).cpu().double()
    one = A.akv_fp16_decode_attention(*args, max_len=128).cpu().double()   # one chunk per sequence
    torch.cuda.synchronize()
    for out, lens in ((got, [1024, 650]), (one, [128, 128])):
        for b, n in enumerate(lens):
            kk, vv = (t[b, :, :n].double().repeat_interleave(G, 0) for t in (k, v))
            ref = torch.softmax((q[b].double()[:, None] * kk).sum(-1) / 128 ** 0.5, -1)[:, None] @ vv
            if out is one and b == 0:
                assert torch.isnan(out[b]).all()
            else:
                assert (out[b] - ref[:, 0]).abs().max() <= T.MAX_ABS and T.rel_l2(out[b].numpy(), ref[:, 0].numpy()) <= T.REL_L2
    assert torch.isnan(got[2]).all()


WALKS = [   # G, B, Hkv, Ncap, lens, kernels (akv_fp16_path)
    # chunks of 256 tokens, 32 per pair (64 of them where groups of four have more than 64 sequences): two tiles per wave; tails inside
    (1, 8, 8, 8192, [8192, 8191, 4100, 257, 225, 33, 0, 6000], 2),
    (2, 8, 8, 8192, [8192, 8095, 300, 256, 1, 5000, 7777, 2048], 2),
    (4, 65, 1, 6144, [6144, 6001, 161, 97, 3000, 129, 513, 1] * 8 + [0], 2),
    (8, 65, 2, 2048, [2048, 0, 0, 1, 33, 129, 2047, 384] * 8 + [77], 2),   # chunks of 384
    # even shares of a few tiles
    (4, 8, 8, 8192, [8000, 8192, 161, 97, 3000, 129, 513, 1], 3),
    (8, 8, 8, 4096, [4096, 4001, 224, 2049, 1000, 31, 4095, 300], 3),
    # as many pairs as compute units: one workgroup takes the whole pair, up to eight tiles per wave
    (1, 32, 8, 1024, [1024, 1023, 1000, 600, 257, 256, 33, 0] * 4, 1),
    (2, 32, 8, 768, [768, 767, 500, 385, 193, 192, 191, 1] * 4, 1),
    (4, 32, 8, 1024, [1024, 993, 900, 513, 255, 129, 97, 2] * 4, 1),
    (8, 32, 8, 512, [512, 480, 511, 300, 129, 128, 65, 0] * 4, 1),
    # more chunks (130) than the merge takes at a time
    (1, 1, 1, 16640, [16640], 2),
    (4, 1, 1, 16640, [16500], 2),
]


@pytest.mark.parametrize("G,B,Hkv,Ncap,lens,kernels", WALKS)
def test_fp16_walks_of_several_tiles_match_textbook(G, B, Hkv, Ncap, lens, kernels):
    """A wave's maximum rises late in the first sequence (its last tokens hold the largest keys), falls in the second, and wanders in
    the others: sums are rescaled, left as they are, and merged."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import akv_testlib as T
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A
    O.build()
    print(f"fp16 attention, several tiles: G{G} {B}x{Hkv} Ncap {Ncap}", flush=True)
    assert A.akv_fp16_path(B, Hkv * G, Hkv, 128, Ncap) == kernels
    g = torch.Generator().manual_seed(100 * G + B)
    q = torch.randn(B, Hkv * G, 128, generator=g).half()
    k, v = torch.randn(B, Hkv, Ncap, 128, generator=g).half(), torch.randn(B, Hkv, Ncap, 128, generator=g).half()
    ramp = torch.linspace(0.05, 2.0, Ncap)[:, None]
    k[0] *= ramp.half()
    if B > 1:
        k[1] *= ramp.flip(0).half()
    lens = np.asarray(lens, np.int32)
    got = A.akv_fp16_decode_attention(k.to(DEV), v.to(DEV), torch.from_numpy(lens).to(DEV), q.to(DEV)).cpu().numpy().astype(np.float64)
    ref = O.fp16_attention(T.bits(k), T.bits(v), lens, T.bits(q))
    assert np.abs(got - ref).max() <= T.MAX_ABS and T.rel_l2(got, ref) <= T.REL_L2
    assert not got[lens == 0].any()


EVEN = [   # G, B, Hkv, Ncap, lens, max_len
    (4, 2, 3, 32768, [32768, 31999], 0),                                  # whole parts of eight tiles
    (4, 2, 3, 32768, [32768, 20001], 20000),                              # the bound cuts both
    (4, 3, 2, 16640, [16640, 0, 40], 0),                                  # of four
    (8, 64, 1, 2048, [2048, 0, 0, 1, 33, 129, 2047, 0] * 8, 0),           # a lane per sequence, empty ones between
    (8, 64, 1, 8192, [8192, 1, 40, 8191, 0, 33, 5000, 64] * 8, 0),        # of twelve, most pairs shorter than one
    (8, 64, 1, 4096, [0] * 63 + [4096], 0),                               # hardly any work: most workgroups have no tile
    (4, 2, 3, 32768, [0, 0], 0),                                          # none at all
]


@pytest.mark.parametrize("G,B,Hkv,Ncap,lens,max_len", EVEN)
def test_fp16_even_shares_match_textbook(G, B, Hkv, Ncap, lens, max_len):
    """Head by head, to 2e-5: logits of magnitude up to 64 carry 64 * 2^-24 = 4e-6 into a weight, the sums less.  A tile that is left out,
    taken twice or merged into another head shows."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import akv_testlib as T
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A
    O.build()
    print(f"fp16 attention, even shares: G{G} {B}x{Hkv} Ncap {Ncap}", flush=True)
    assert A.akv_fp16_path(B, Hkv * G, Hkv, 128, Ncap, max_len) == 3
    g = torch.Generator().manual_seed(G + B)
    q = torch.randn(B, Hkv * G, 128, generator=g).half()
    k, v = torch.randn(B, Hkv, Ncap, 128, generator=g).half(), torch.randn(B, Hkv, Ncap, 128, generator=g).half()
    k *= torch.linspace(0.05, 2.0, Ncap)[:, None].half()
    lens = np.asarray(lens, np.int32)
    args = (k.to(DEV), v.to(DEV), torch.from_numpy(lens).to(DEV), q.to(DEV))
    out = A.akv_fp16_decode_attention(*args, max_len=max_len)
    got = out.cpu().numpy().astype(np.float64)
    ref = O.fp16_attention(T.bits(k), T.bits(v), np.minimum(lens, max_len) if max_len else lens, T.bits(q))
    err, size = np.linalg.norm(got - ref, axis=2), np.linalg.norm(ref, axis=2)
    assert np.all(err <= 2e-5 * size), (err / np.maximum(size, 1e-30)).max()
    assert not got[lens == 0].any()
    assert torch.equal(out, A.akv_fp16_decode_attention(*args, max_len=max_len))


CUTS = [   # G, B, Hkv, Ncap, lens, whole parts, tiles of a share
    (8, 64, 2, 4096, [4096 - (i * 1237) % 2048 for i in range(64)], False, 25),       # shares over the end of a pair
    (4, 24, 6, 9472, [[9472, 8000, 8100, 1, 8300, 0, 9001, 8500][i % 8] for i in range(24)], False, 38),   # ... of two sequences, empty ones between
    (8, 64, 3, 6144, [32 * (25, 13, 25)[i % 3] - (i * 5) % 32 for i in range(64)], False, 8),   # the smallest that begin anywhere
    (8, 64, 2, 4096, [[4096, 289, 300, 1, 0, 33, 2081, 4000][i % 8] for i in range(64)], True, 12),
    (8, 3, 1, 24576, [24576, 24001, 1], True, 4),                                     # the smallest whole ones
]


def _cut(G, Hkv, lens):
    """The share of tiles and whether pairs are cut into whole parts, as the rule has it (256 compute units)."""
    workgroups, tiles = 256 * (2 if G == 8 else 3), [(n + 31) // 32 for n in lens]
    even = -(-Hkv * sum(tiles) // workgroups)
    least = 8 if G == 4 and even in (5, 6) else max(even, 4)
    for share in range(least, least + (4 if least < 32 else 2)):
        if Hkv * sum(-(-t // share) for t in tiles) <= workgroups:
            return True, share
    return False, max(even, 8)


@pytest.mark.parametrize("G,B,Hkv,Ncap,lens,whole,share", CUTS)
def test_fp16_shares_that_span_pairs_and_whole_parts(G, B, Hkv, Ncap, lens, whole, share):
    """Head by head, to 2e-5 as above; a tile that is left out, taken twice or merged into another head shows."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import akv_testlib as T
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A
    O.build()
    print(f"fp16 attention, cuts: G{G} {B}x{Hkv} Ncap {Ncap}", flush=True)
    assert A.akv_fp16_path(B, Hkv * G, Hkv, 128, Ncap) == 3
    g = torch.Generator().manual_seed(G + B)
    most, lens = (max(lens) + 255) // 256 * 256, np.asarray(lens, np.int32)
    q = torch.randn(B, Hkv * G, 128, generator=g).half()
    k, v = torch.randn(B, Hkv, most, 128, generator=g).half(), torch.randn(B, Hkv, most, 128, generator=g).half()
    k *= torch.linspace(0.05, 2.0, most)[:, None].half()
    kd, vd = (torch.full((B, Hkv, Ncap, 128), float("nan"), dtype=torch.float16, device=DEV) for _ in range(2))      # past the lengths nothing is read
    for b in range(B):
        kd[b, :, :lens[b]], vd[b, :, :lens[b]] = k[b, :, :lens[b]].to(DEV), v[b, :, :lens[b]].to(DEV)
    args = (kd, vd, torch.from_numpy(lens).to(DEV), q.to(DEV))
    out = A.akv_fp16_decode_attention(*args)
    got = out.cpu().numpy().astype(np.float64)
    ref = O.fp16_attention(T.bits(k), T.bits(v), lens, T.bits(q))
    err, size = np.linalg.norm(got - ref, axis=2), np.linalg.norm(ref, axis=2)
    assert np.all(err <= 2e-5 * size), (err / np.maximum(size, 1e-30)).max()
    assert not got[lens == 0].any()
    assert torch.equal(out, A.akv_fp16_decode_attention(*args))
