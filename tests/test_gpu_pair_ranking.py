"""The bf16 ranking by pairs: chunks of 4 to 8 pieces, rows of one to four chunks,
with and without a repeated tail, on scores where a pair's two experts tie, sit
both in the Top-K or straddle its edge, and where a wave meets tokens with fewer
than eight positive scores (its first chunk is then ranked twice).

Whole numbers only: signatures and distances equal the oracle's.
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


def _bf16(x: np.ndarray) -> np.ndarray:
    return torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16).copy()


def _scores(kind: str, N: int, E: int) -> np.ndarray:
    rng = np.random.default_rng(E * 7 + N)
    x = rng.standard_normal((N, E)).astype(np.float32)
    if kind == "pairs":  # both experts of a pair alike up to a small step, often equal
        x[:, 1::2] = x[:, : E // 2 * 2 : 2] + rng.integers(-1, 2, (N, E // 2)) * np.float32(2.0**-7)
    elif kind == "few":  # 0 to 12 positive scores per token
        m = rng.integers(0, 13, N)
        x = -np.abs(x) - 1e-3
        for t in range(N):
            x[t, rng.permutation(E)[: m[t]]] *= -1
    elif kind == "equal":
        x[:] = rng.integers(-1, 2, (N, 1))
    elif kind == "special":
        b = _bf16(x)
        for v in (0x0000, 0x8000, 0x7F80, 0xFF80, 0x7FC0, 0xFFFF, 0x0001, 0x8001):
            b[rng.random((N, E)) < 0.02] = v
        return b
    return _bf16(x)


@pytest.mark.parametrize("E", [25, 32, 33, 64, 96, 100, 127, 128, 130, 192, 256])
@pytest.mark.parametrize("kind", ["normal", "pairs", "few", "equal", "special"])
def test_pair_ranking(dl, orc, E, kind):
    for N, k in ((512, 8), (577, 1), (640, 5)):
        print(f"[case] pairs E={E} k={k} N={N} {kind}", flush=True)
        x = _scores(kind, N, E)
        bits, D, _ = dl.do_fused(to_dev(x), k, want_bits=True)
        torch.cuda.synchronize()
        F = orc.topk_signature(x, k)
        np.testing.assert_array_equal(bits_np(bits, N)[0], orc.pack(F))
        np.testing.assert_array_equal(D_np(D)[0], orc.hamming(F))


@pytest.mark.parametrize("E", [8, 24, 32])
@pytest.mark.parametrize("k", [1, 2, 7, 8])
def test_one_chunk_fp32_rows(dl, orc, E, k):
    """fp32 rows of one chunk whose k-th score is negative, zero or special in some tokens."""
    for kind in ("normal", "few", "special"):
        x = (_scores(kind, 577, E).astype(np.uint32) << 16).view(np.float32)
        print(f"[case] one chunk fp32 E={E} k={k} {kind}", flush=True)
        bits, D, _ = dl.do_fused(to_dev(x), k, want_bits=True)
        torch.cuda.synchronize()
        F = orc.topk_signature(x, k)
        np.testing.assert_array_equal(bits_np(bits, 577)[0], orc.pack(F))
        np.testing.assert_array_equal(D_np(D)[0], orc.hamming(F))


@pytest.mark.parametrize("L,N", [(16, 8192), (33, 4096), (33, 1000), (64, 513), (70, 2048)])
def test_layer_partitions(dl, orc, L, N):
    """8, 16 and 32 schedule partitions, grids that they divide or not, two launches (70 layers)."""
    E, k = 64, 6
    x = np.stack([_scores("normal", N, E) if l % 5 else _scores("pairs", N, E) for l in range(L)])
    x[1::2] = np.roll(x[1::2], 3, axis=2)
    print(f"[case] partitions L={L} N={N}", flush=True)
    bits, D, _ = dl.do_fused(to_dev(x), k, want_bits=True)
    torch.cuda.synchronize()
    got, dist = bits_np(bits, N), D_np(D)
    for l in {0, 1, L // 2, L - 1}:
        F = orc.topk_signature(x[l], k)
        np.testing.assert_array_equal(got[l], orc.pack(F))
        np.testing.assert_array_equal(dist[l], orc.hamming(F))
    for l in range(2, L):  # the other layers repeat the first ones
        j = next(m for m in range(l + 1) if (m % 5 == 0) == (l % 5 == 0) and m % 2 == l % 2)
        np.testing.assert_array_equal(dist[l], dist[j])
