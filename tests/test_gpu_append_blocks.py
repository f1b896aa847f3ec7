"""GPU parity of the block-wise append and of unpack at the edges of their tiles: ranges that begin and end inside a nibble byte,
a 16-byte piece, a 64-token wave or a block, onto planes that hold older tokens behind the length (they stay), ragged counts
with none and with a refusal; each output of unpack alone."""
import ctypes as C

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


@pytest.mark.parametrize("n,lens,counts", [
    (16, [0, 1, 255, 241], None),                    # inside one block, into the next, up to its end
    (33, [15, 16, 17, 480], [33, 0, 32, 33]),        # pieces of 16 and 32 tokens; the last one fits exactly no more (refused at 512)
    (256, [0, 256, 1, 255], None),                   # whole blocks and every split of one
    (257, [0, 255, 254, 63], [257, 257, 1, 200]),
    (300, [100, 212, 213, 31], None),                # 212 + 300 fills the capacity, 213 + 300 is refused
])
def test_append_blocks_match_oracle_and_leave_the_rest(T, n, lens, counts):
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A, workloads
    print(f"append blocks: n {n} lens {lens} counts {counts}", flush=True)
    B, Hkv, Ncap = len(lens), 3, 512
    k, v = workloads.edge_patterns(B, Hkv, Ncap + n, seed=n)
    full = [Ncap] * B
    oc = T.oracle_cache(k[:, :, :Ncap], v[:, :, :Ncap], full, Ncap)
    gc = T.gpu_cache(k[:, :, :Ncap], v[:, :, :Ncap], full, Hkv, Ncap)
    T.assert_cache_equal(gc, oc)
    oc.lens[:] = lens
    gc.lens.copy_(torch.tensor(lens, dtype=torch.int32))
    kn, vn = k[:, :, Ncap:].contiguous(), v[:, :, Ncap:].contiguous()
    n_new = np.array([n] * B if counts is None else counts, np.int32)
    refused = O.append(oc, T.bits(kn), T.bits(vn), n_new)
    A.akv_append(gc, kn.to(DEV), vn.to(DEV), torch.from_numpy(n_new).to(DEV) if counts is not None else None)
    torch.cuda.synchronize()
    T.assert_cache_equal(gc, oc)
    assert int(gc.flags.cpu()[A.AKV_FLAG_OVERFLOW]) == refused and not gc.flags.cpu()[A.AKV_NFLAGS:].any()
    # unpack: both outputs, and each alone
    ku, vu = A.akv_unpack(gc)
    k1, v1 = torch.zeros_like(ku), torch.zeros_like(vu)
    s, st = gc.struct(), torch.cuda.current_stream().cuda_stream
    assert A.lib().akv_unpack(C.byref(s), k1.data_ptr(), None, st) == A.AKV_OK
    assert A.lib().akv_unpack(C.byref(s), None, v1.data_ptr(), st) == A.AKV_OK
    torch.cuda.synchronize()
    full16 = lambda hi, mid, lo: (hi.astype(np.uint16) << 8) | (mid << 4) | lo
    vm, vl = (x.reshape(B, Hkv, Ncap, 64) for x in (oc.v_mid, oc.v_lo))
    nib = lambda x: np.stack([x & 15, x >> 4], axis=-1).reshape(*x.shape[:-1], -1).astype(np.uint16)
    assert np.array_equal(T.bits(vu), full16(oc.v_hi.reshape(B, Hkv, Ncap, 128), nib(vm), nib(vl)))
    kh = oc.k_hi.reshape(B, Hkv, Ncap // 256, 128, 256)
    km, kl = (nib(x.reshape(B, Hkv, Ncap // 256, 128, 128)) for x in (oc.k_mid, oc.k_lo))
    assert np.array_equal(T.bits(ku), full16(kh, km, kl).transpose(0, 1, 2, 4, 3).reshape(B, Hkv, Ncap, 128))
    assert torch.equal(k1.view(torch.int16), ku.view(torch.int16)) and torch.equal(v1.view(torch.int16), vu.view(torch.int16))


@pytest.mark.parametrize("B,Hkv,n", [(32, 32, 4), (32, 32, 6), (4, 32, 60)])
def test_append_of_few_tokens_for_many_heads(T, B, Hkv, n):
    """Enough (sequence, head) pairs that six tokens already go block by block and four do not; enough workgroups that the lengths of a
    block launch move in a launch of their own (the cases above draw tickets), with a refused sequence."""
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A, workloads
    Ncap = 256
    print(f"append blocks: {B * Hkv} pairs, {n} tokens", flush=True)
    k, v = workloads.edge_patterns(B, Hkv, 2 * n + 3, seed=9)
    lens = [i % 8 for i in range(B)]
    if n == 60:
        k, v = workloads.edge_patterns(B, Hkv, 200 + n, seed=9)
        lens = [0, 7, 196, 200]                      # 196 + 60 fills the capacity, 200 + 60 is refused
    m = max(lens)
    oc = T.oracle_cache(k[:, :, :m], v[:, :, :m], lens, Ncap)
    gc = T.gpu_cache(k[:, :, :m], v[:, :, :m], lens, Hkv, Ncap)
    kn, vn = k[:, :, m:m + n].contiguous(), v[:, :, m:m + n].contiguous()
    refused = O.append(oc, T.bits(kn), T.bits(vn), np.array([n] * B, np.int32))
    A.akv_append(gc, kn.to(DEV), vn.to(DEV))
    torch.cuda.synchronize()
    T.assert_cache_equal(gc, oc)
    assert int(gc.flags.cpu()[A.AKV_FLAG_OVERFLOW]) == refused == (1 if n == 60 else 0)


def _append_beside_busy_stream(T, Hkv, B, counts):
    """Appends of counts[0], counts[1], ... tokens, one after another onto empty sequences, while products on a second stream hold the
    compute units, so that workgroups of a launch start late and far apart; eight times, each against the oracle's cache."""
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A, workloads
    n = sum(counts)
    Ncap = (n + 255) // 256 * 256
    k, v = workloads.edge_patterns(B, Hkv, n, seed=n)
    oc = O.Cache.empty(B, Hkv, 128, Ncap)
    at, parts = 0, []
    for c in counts:
        kn, vn = k[:, :, at:at + c].contiguous(), v[:, :, at:at + c].contiguous()
        assert O.append(oc, T.bits(kn), T.bits(vn)) == 0
        parts.append((kn.to(DEV), vn.to(DEV)))
        at += c
    a = torch.randn(4096, 4096, device=DEV, dtype=torch.float16)
    y = torch.empty_like(a)
    side = torch.cuda.Stream()
    gcs = [A.Cache.allocate(B, Hkv, Hkv, 128, Ncap, DEV) for _ in range(8)]
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(60):
            torch.mm(a, a, out=y)
    for gc in gcs:
        for kn, vn in parts:
            A.akv_append(gc, kn, vn)
    torch.cuda.synchronize()
    for gc in gcs:
        T.assert_cache_equal(gc, oc)
        assert not gc.flags.cpu().numpy().any()


def test_block_append_beside_a_busy_stream(T):
    """The lengths move by ticket (256 workgroups); every launch but the third has workgroups whose block no token falls into."""
    print("append blocks: 200 tokens and more beside a busy stream", flush=True)
    _append_beside_busy_stream(T, 32, 2, [200, 40, 250, 16])


def test_walking_append_beside_a_busy_stream(T):
    """A few tokens per call: one workgroup of two waves per head, ticket drawn in front of the stores."""
    print("append: one to fifteen tokens beside a busy stream", flush=True)
    _append_beside_busy_stream(T, 8, 3, [1, 2, 15, 1, 1, 8, 3, 1, 15])


@pytest.mark.parametrize("B", [341, 342])            # 1023 and 1026 blocks: one workgroup per block of V, and sixteen
def test_unpack_of_many_blocks_gives_back_what_was_stored(T, B):
    from paper_2409_16546_amd import binding as A, workloads
    print(f"unpack: {3 * B} blocks", flush=True)
    k, v = (t.repeat(B, 1, 1, 1).to(DEV) for t in workloads.edge_patterns(1, 3, 256, seed=B))
    k[:, :, :, 5] = torch.arange(B, device=DEV)[:, None, None].half()      # a block that lands in another's place is seen
    v[:, :, :, 6] = torch.arange(256, device=DEV).half()
    gc = A.Cache.allocate(B, 3, 3, 128, 256, DEV)
    A.akv_append(gc, k, v)
    ku, vu = A.akv_unpack(gc)
    torch.cuda.synchronize()
    for got, want in ((ku, k), (vu, v)):
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("B,H", [(1, 1), (20, 8), (23, 7), (24, 8), (193, 1)])    # 1 and 160 blocks: eight workgroups each; 161 and 192: four; 193: two
def test_unpack_of_v_alone_gives_back_what_was_stored(T, B, H):
    from paper_2409_16546_amd import binding as A, workloads
    print(f"unpack of V: {H * B} blocks", flush=True)
    k, v = (t.repeat(B, 1, 1, 1).to(DEV) for t in workloads.edge_patterns(1, H, 256, seed=B))
    v[:, :, :, 5] = torch.arange(B, device=DEV)[:, None, None].half()      # a block or a row that lands in another's place is seen
    v[:, :, :, 6] = torch.arange(256, device=DEV).half()
    gc = A.Cache.allocate(B, H, H, 128, 256, DEV)
    A.akv_append(gc, k, v)
    out = torch.zeros(B * H * 256 + 1, 128, dtype=torch.float16, device=DEV)      # a row more than the tensor has
    s = gc.struct()
    assert A.lib().akv_unpack(C.byref(s), None, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == A.AKV_OK
    torch.cuda.synchronize()
    assert torch.equal(out[:-1].view(torch.int16), v.view(-1, 128).view(torch.int16)) and not out[-1].any()


@pytest.mark.parametrize("B,Hkv,n", [
    (25, 16, 256),                # two workgroups per side, the length by a launch
    (10, 4, 36), (41, 1, 36),     # 320 and 328 workgroups of two per side: the length by ticket, by a launch
    (32, 32, 60), (33, 32, 60),   # 4096 workgroups of one per side, the last with two; one more sequence
    (3, 3, 3841), (3, 3, 3842),   # 16 blocks, the last with two per side; 17, and the length by ticket
])
def test_append_with_one_and_two_workgroups_per_block_side(T, B, Hkv, n):
    """One workgroup takes all channels of a block's K, or two take half each, and two its V: ranges that begin inside a nibble byte, a
    piece and the second half of a block's rows, one refusal and one empty count."""
    from oracle import akv_oracle as O
    from paper_2409_16546_amd import binding as A, workloads
    Ncap = (n + 511) // 256 * 256
    print(f"append block sides: {B * Hkv} pairs, {n} tokens", flush=True)
    k, v = workloads.edge_patterns(B, Hkv, n, seed=n)
    lens = [(i * 37) % 256 for i in range(B)]
    lens[0], lens[1] = 129, Ncap - n + 1
    n_new = np.full(B, n, np.int32)
    if B > 3:
        lens[3], n_new[5], n_new[9] = 128, 0, n // 2
    oc, gc = O.Cache.empty(B, Hkv, 128, Ncap), A.Cache.allocate(B, Hkv, Hkv, 128, Ncap, DEV)
    oc.lens[:] = lens
    gc.lens.copy_(torch.tensor(lens, dtype=torch.int32))
    refused = O.append(oc, T.bits(k), T.bits(v), n_new)
    A.akv_append(gc, k.to(DEV), v.to(DEV), torch.from_numpy(n_new).to(DEV))
    torch.cuda.synchronize()
    T.assert_cache_equal(gc, oc)
    assert refused >= 1 and int(gc.flags.cpu()[A.AKV_FLAG_OVERFLOW]) == refused and not gc.flags.cpu()[A.AKV_NFLAGS:].any()
