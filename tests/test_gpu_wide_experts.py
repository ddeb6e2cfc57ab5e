"""More than 256 experts: the wide Top-K kernel (k <= 8 and k <= 16 lists, every
key kind), the MFMA Gram over 128-expert groups, the finalize split over rows
(also at 129 to 256 experts), and streams whose micro-batches share words.

Whole numbers only: signatures, distances and the loss sums equal the oracle's.
"""
import numpy as np
import pytest
import torch

from gpu_util import D_np, bits_np, loss_close, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_32398_amd as p

    p.lib()
    return p


def _check(dl, orc, x, k, bits, D, rec):
    F = orc.topk_signature(x, k)
    Dr = orc.hamming(F)
    np.testing.assert_array_equal(bits_np(bits, x.shape[0]), orc.pack(F))
    np.testing.assert_array_equal(D_np(D), Dr)
    loss_close(rec, orc.loss(Dr))


def _scores(syn, kind, E, N, dtype):
    if kind == "ties":
        return syn.int_ties(E, N, E, -2, 2, dtype)
    if kind == "buckets":  # fp32 values that differ only in their low 10 bits: every row ties in its bucket
        r = np.random.default_rng(E)
        return (np.float32(1.0).view(np.uint32) + r.integers(0, 1024, (N, E), dtype=np.uint32)).view(np.float32)
    x = syn.normal(E, N, E, dtype, mean=-9.0 if kind == "negative" else 0.0)
    if kind == "special":
        v = x if dtype == 0 else x.view(np.uint16)
        vals = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1e-40], dtype=np.float32)
        vals = vals if dtype == 0 else (vals.view(np.uint32) >> 16).astype(np.uint16)
        r = np.random.default_rng(E)
        m = r.random(v.shape) < 0.3
        v[m] = r.choice(vals, size=int(m.sum()))
    return x


# experts at the edges of tiles, chunks and groups; k at the edges of the lists
@pytest.mark.parametrize("E,k,dtype", [(257, 1, 0), (257, 16, 1), (288, 8, 1), (300, 9, 0), (384, 8, 0), (385, 12, 1),
                                       (512, 8, 1), (513, 16, 0), (1000, 7, 1), (1023, 9, 1), (1024, 8, 0),
                                       (1024, 16, 1)])
def test_wide_experts(dl, orc, syn, E, k, dtype):
    kinds = ["normal", "ties", "special", "negative"] + (["buckets"] if dtype == 0 else [])
    for kind, N in zip(kinds, (577, 130, 200, 65, 70)):
        print(f"[case] wide E={E} k={k} N={N} dtype={dtype} {kind}", flush=True)
        x = _scores(syn, kind, E, N, dtype)
        bits, D, out = dl.do_fused(to_dev(x), k, want_bits=True)
        torch.cuda.synchronize()
        _check(dl, orc, x, k, bits[0], D[0], dl.loss_records(out)[0])


@pytest.mark.parametrize("E,k,dtype", [(260, 6, 1), (520, 12, 0)])
def test_wide_layers_share_blocks(dl, orc, syn, E, k, dtype):
    # more half units than the launch has blocks, layers of a ragged token
    # count: blocks walk over segment ends with some waves idle
    L, N = 90, 2700
    x0 = _scores(syn, "normal", E, N, dtype)
    x = np.stack([np.roll(x0, l, axis=0) for l in range(L)])
    bits, D, out = dl.do_fused(to_dev(x), k, want_bits=True)
    torch.cuda.synchronize()
    for l in range(1, L):  # the same tokens in another order: the same distances
        assert torch.equal(D[l], D[0]), l
    for l in (0, 1, 64, L - 1):
        _check(dl, orc, x[l], k, bits[l], D[l], dl.loss_records(out)[l])
    w = bits_np(bits, N)
    assert np.array_equal(np.bitwise_count(w).sum(axis=2), np.broadcast_to(np.bitwise_count(w[0]).sum(axis=1), (L, E)))


@pytest.mark.parametrize("E,k,dtype,sizes", [(300, 8, 1, (64, 512, 1000, 7, 1)), (520, 10, 0, (100, 100, 700))])
def test_wide_stream(dl, orc, syn, E, k, dtype, sizes):
    s = dl.DoStream(E, k, sum(sizes))
    for epoch in range(2):  # the second over the stale words of the first
        xs = [syn.normal(7 + i + epoch, n, E, dtype) for i, n in enumerate(sizes)]
        s.reset()
        for x in xs:
            s.append(to_dev(x))
        D, out = s.finalize()
        torch.cuda.synchronize()
        _check(dl, orc, np.concatenate(xs), k, s.history(), D, dl.loss_records(out)[0])
    s.close()


@pytest.mark.parametrize("E,L", [(129, 3), (200, 2), (255, 1), (256, 5)])
def test_finalize_split_over_rows(dl, orc, syn, E, L):
    N, k = 700, 5
    x = np.stack([syn.normal(40 + l, N, E, 0) for l in range(L)])
    bits, D, out = dl.do_fused(to_dev(x), k, want_bits=True)
    D2 = dl.do_pairwise_hamming(bits, N)
    torch.cuda.synchronize()
    assert torch.equal(D, D2)
    for l in range(L):
        _check(dl, orc, x[l], k, bits[l], D[l], dl.loss_records(out)[l])
