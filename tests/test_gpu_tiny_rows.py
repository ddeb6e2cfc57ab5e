"""Rows below 16 bytes (1 to 3 fp32 or 1 to 7 bf16 experts), which every lane
selects from by itself, and rows of exactly one 16-byte piece, aligned or not:
random, tied and special scores, partial words, a stream whose micro-batches
share words, and both Gram kinds.

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


def _scores(syn, kind, E, N, dtype, seed):
    if kind == "ties":
        return syn.int_ties(seed, N, E, -1, 1, dtype)
    x = syn.normal(seed, N, E, dtype)
    if kind == "special":
        rng = np.random.default_rng(seed)
        for v in (0x0000, 0x8000, 0x7F80, 0xFF80, 0x7FC0, 0xFFFF, 0x0001, 0x8001):
            x[rng.random((N, E)) < 0.1] = v if dtype == 1 else np.uint32(v << 16).view(np.float32)
    return x


def _dev(x, shift):
    t = to_dev(x)
    buf = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
    v = buf[shift:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("E,dtype", [(1, 0), (2, 0), (3, 0), (4, 0), (1, 1), (2, 1), (3, 1), (5, 1), (7, 1), (8, 1)])
def test_tiny_rows(dl, orc, syn, E, dtype):
    for N, kind, shift in ((512, "normal", 0), (1217, "special", 0), (577, "special", 1), (65, "ties", 0), (1, "ties", 1)):
        for k in sorted({1, (E + 1) // 2, E}):
            print(f"[case] tiny E={E} k={k} N={N} dtype={dtype} {kind} shift={shift}", flush=True)
            x = _scores(syn, kind, E, N, dtype, E + N)
            fb, fD, fout = dl.do_fused(_dev(x, shift), k, want_bits=True)
            sb = dl.do_topk_signature(_dev(x, shift), k)
            torch.cuda.synchronize()
            F = orc.topk_signature(x, k)
            D = orc.hamming(F)
            np.testing.assert_array_equal(bits_np(fb, N)[0], orc.pack(F))
            assert torch.equal(fb, sb)
            np.testing.assert_array_equal(D_np(fD)[0], D)
            loss_close(dl.loss_records(fout)[0], orc.loss(D))


@pytest.mark.parametrize("E,dtype,gram", [(3, 0, 0), (3, 0, 1), (6, 1, 0), (8, 1, 0)])
def test_tiny_rows_stream(dl, orc, syn, E, dtype, gram):
    k, sizes = 2, (37, 1000, 64, 1, 5230)
    print(f"[case] tiny stream E={E} dtype={dtype} gram={gram}", flush=True)
    x = _scores(syn, "normal", E, sum(sizes), dtype, E)
    dl.set_option(dl.DO_OPT_GRAM, gram)
    try:
        h = dl.DoStream(E, k, sum(sizes))
        t = 0
        for n in sizes:
            h.append(to_dev(x[t:t + n]))
            t += n
        D, out = h.finalize()
        torch.cuda.synchronize()
    finally:
        dl.set_option(dl.DO_OPT_GRAM, 0)
    ref = orc.hamming(orc.topk_signature(x, k))
    np.testing.assert_array_equal(D_np(D).reshape(ref.shape), ref)
    loss_close(dl.loss_records(out)[0], orc.loss(ref))
