"""16-byte aligned rows of whole 16-byte pieces whose last 128-byte chunk is
partial: last chunks of one to seven pieces after none to seven full ones, on
random, tied, negative and special scores, partial words, several layers, a
stream whose micro-batches share words, and both Gram kinds.

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
        return syn.int_ties(seed, N, E, -3, 3, dtype)
    x = syn.normal(seed, N, E, dtype, mean=-6.0 if kind == "negative" else 0.0)
    if kind == "special":
        rng = np.random.default_rng(seed)
        for v in (0x0000, 0x8000, 0x7F80, 0xFF80, 0x7FC0, 0xFFFF, 0x0001, 0x8001):
            hit = rng.random((N, E)) < 0.02
            x[hit] = v if dtype == 1 else np.uint32(v << 16).view(np.float32)
    return x


# pieces of a row: 1 to 63, never a multiple of 8
CASES = [(e, 1) for e in (8, 16, 24, 40, 56, 72, 88, 120, 136, 160, 200, 248)] + \
        [(e, 0) for e in (4, 8, 12, 28, 36, 60, 100, 120, 132, 180, 216, 252)]


@pytest.mark.parametrize("E,dtype", CASES)
def test_piece_rows(dl, orc, syn, E, dtype):
    for N, kind, k in ((1024, "normal", 8), (513, "ties", 5), (65, "special", 8), (1217, "special", 2),
                       (320, "negative", 8), (1217, "normal", 1)):
        k = min(k, E)
        print(f"[case] pieces E={E} k={k} N={N} dtype={dtype} {kind}", flush=True)
        xs = [_scores(syn, kind, E, N, dtype, E + 7 * l) for l in range(2)]
        xd = to_dev(np.stack(xs))
        fb, fD, fout = dl.do_fused(xd, k, want_bits=True)
        sb = dl.do_topk_signature(xd, k)
        torch.cuda.synchronize()
        assert torch.equal(fb, sb)
        for l, x in enumerate(xs):
            F = orc.topk_signature(x, k)
            D = orc.hamming(F)
            np.testing.assert_array_equal(bits_np(fb, N)[l], orc.pack(F))
            np.testing.assert_array_equal(D_np(fD)[l], D)
            loss_close(dl.loss_records(fout)[l], orc.loss(D))


@pytest.mark.parametrize("E,dtype,gram", [(24, 1, 0), (72, 1, 1), (200, 1, 0), (100, 0, 0), (252, 0, 1)])
def test_piece_rows_stream(dl, orc, syn, E, dtype, gram):
    k, sizes = 6, (37, 1000, 64, 1, 523)
    print(f"[case] pieces stream E={E} dtype={dtype} gram={gram}", flush=True)
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
