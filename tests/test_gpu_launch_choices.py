"""Choices of a launch that follow from how many units a block gets.

Aligned fp32 rows whose next chunk's loads are issued together or spread over
the ranking, a choice by row length and units per block: 64 layers below and
above the two lines (2 units per block at 512-byte rows, 16 at 1,024-byte rows
without a Gram), and row lengths that never spread.

The layers repeat two distinct ones.

One layer on a block per unit or on half as many (up to 8 or odd experts, more
than 160 units).

Whole numbers only: equal to the oracle's.
"""
import numpy as np
import pytest
import torch

from gpu_util import D_np, bits_np, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_32398_amd as p

    p.lib()
    return p


# units per layer: 64 layers x 8 units are 2 per block of 256, 64 x 64 are 16
@pytest.mark.parametrize("E,units,gram", [(128, 8, True), (128, 9, True), (128, 9, False), (96, 9, True),
                                          (64, 9, True), (256, 64, False), (256, 65, False), (256, 9, True)])
def test_spread_loads(dl, orc, syn, E, units, gram):
    L, N, k = 64, 512 * units, 8
    print(f"[case] spread E={E} L={L} N={N} gram={gram}", flush=True)
    xs = [syn.normal(E + units + l, N, E, 0, mean=-0.5 * l) for l in range(2)]
    x = to_dev(np.stack(xs)).repeat(L // 2, 1, 1)
    if gram:
        bits, D, _ = dl.do_fused(x, k, want_bits=True)
    else:
        bits, D = dl.do_topk_signature(x, k), None
    torch.cuda.synchronize()
    assert all(torch.equal(bits[l], bits[l % 2]) for l in range(2, L))
    for l, xl in enumerate(xs):
        F = orc.topk_signature(xl, k)
        np.testing.assert_array_equal(bits_np(bits[l : l + 1], N)[0], orc.pack(F))
        if D is not None:
            assert all(torch.equal(D[m], D[l]) for m in range(l, L, 2))
            np.testing.assert_array_equal(D_np(D)[l], orc.hamming(F))


@pytest.mark.parametrize("E,dtype", [(3, 0), (8, 1), (53, 1), (255, 0), (64, 1)])
@pytest.mark.parametrize("units", [160, 161, 250])
def test_one_layer_blocks(dl, orc, syn, E, dtype, units):
    N, k = 512 * units - 100, min(E, 4)
    print(f"[case] one layer E={E} N={N} dtype={dtype}", flush=True)
    x = syn.normal(E + units, N, E, dtype)
    bits, D, _ = dl.do_fused(to_dev(x), k, want_bits=True)
    torch.cuda.synchronize()
    F = orc.topk_signature(x, k)
    np.testing.assert_array_equal(bits_np(bits, N)[0], orc.pack(F))
    np.testing.assert_array_equal(D_np(D)[0], orc.hamming(F))
