"""Rows that do not fill 16-byte-aligned 128-byte chunks: every row length class
of the staging (one to eight 16-byte slots per row, a last chunk of one to eight
pieces, a last piece that repeats 2 to 14 bytes) and score buffers that start
off a 16-byte boundary, on random, tied and special scores.

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


def _shifted(x: np.ndarray, elems: int) -> torch.Tensor:
    """The scores on the device, `elems` elements past an allocation's start."""
    t = to_dev(x)
    buf = torch.empty(t.numel() + elems, dtype=t.dtype, device="cuda")
    v = buf[elems:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == elems * t.element_size() % 16
    return v


# (E, dtype): row bytes 16, 18, 34, 66, 128, 130, 142, 200, 258, 386, 510 (bf16); 16, 20, 36, 68, 132, 252, 260, 500, 1012 (fp32)
CASES = [(8, 1), (9, 1), (17, 1), (33, 1), (64, 1), (65, 1), (71, 1), (100, 1), (129, 1), (193, 1), (255, 1),
         (4, 0), (5, 0), (9, 0), (17, 0), (33, 0), (63, 0), (65, 0), (125, 0), (253, 0)]


@pytest.mark.parametrize("E,dtype", CASES)
def test_ragged_rows(dl, orc, syn, E, dtype):
    k = min(8, max(1, E // 2))
    for N, shift, kind in ((513, 0, "normal"), (1217, 1, "normal"), (65, 3, "ties"), (320, 1, "negative")):
        print(f"[case] ragged E={E} k={k} N={N} dtype={dtype} shift={shift} {kind}", flush=True)
        if kind == "ties":
            x = syn.int_ties(E, N, E, -3, 3, dtype)
        else:
            x = syn.normal(E, N, E, dtype, mean=-6.0 if kind == "negative" else 0.0)
        if kind == "normal":  # special values in the first and last element of some rows
            nan = np.float32(np.nan) if dtype == 0 else 0x7FC0
            inf = np.float32(np.inf) if dtype == 0 else 0x7F80
            x[0, E - 1], x[3, 0], x[N - 1, E - 1] = nan, inf, inf
        xd = _shifted(x, shift)
        fb, fD, fout = dl.do_fused(xd, k, want_bits=True)
        sb = dl.do_topk_signature(xd, k)
        torch.cuda.synchronize()
        F = orc.topk_signature(x, k)
        D = orc.hamming(F)
        np.testing.assert_array_equal(bits_np(fb, N)[0], orc.pack(F))
        assert torch.equal(fb, sb)
        np.testing.assert_array_equal(D_np(fD)[0], D)
        loss_close(dl.loss_records(fout)[0], orc.loss(D))
