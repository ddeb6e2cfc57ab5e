"""The Gram of stored signatures up to 128 experts: one to four tiles of 32
experts, partial tiles, partial last units, odd expert counts (32-bit atomics),
more layers than blocks per layer and blocks that span layers.

Whole numbers only: distances equal the oracle's.
"""
import numpy as np
import pytest
import torch

from gpu_util import D_np, units_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_32398_amd as p

    p.lib()
    return p


@pytest.mark.parametrize("E", [2, 31, 32, 33, 64, 65, 96, 100, 127, 128, 129, 256])
@pytest.mark.parametrize("L,N", [(1, 64), (1, 513), (3, 4096), (7, 6400), (40, 3000)])
def test_gram_units(dl, orc, E, L, N):
    print(f"[case] gram units E={E} L={L} N={N}", flush=True)
    rng = np.random.default_rng(E + 1000 * L + N)
    F = rng.random((L, E, N)) < rng.random((L, E, 1))  # any density: a Gram takes any signatures
    words = np.stack([orc.pack(f.astype(np.uint8)) for f in F])
    bits = units_dev(words)
    if words.shape[-1] % 8:  # words past the signature hold anything
        bits[:, -1, :, words.shape[-1] % 8:] = -1
    D = dl.do_pairwise_hamming(bits, N)
    torch.cuda.synchronize()
    got = D_np(D)
    for l in range(L):
        f = F[l].astype(np.float64)
        c = f @ f.T
        n = np.diag(c)
        np.testing.assert_array_equal(got[l], (n[:, None] + n[None, :] - 2 * c).astype(np.uint32))
