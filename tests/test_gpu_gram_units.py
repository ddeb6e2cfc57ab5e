"""The Gram of stored signatures up to 128 experts: one to four tiles of 32
experts, partial tiles, partial last units, odd expert counts (32-bit atomics).
test_gram_units holds fewer units than blocks (one unit per block; 97 to 128
experts then take the kernel of the wider routers); test_gram_many_units gives
every block more than the 12 units that its four waves and their three load
buffers take in one turn, in blocks that span layers; test_gram_long_layers
gives a block more units of one layer than its fp32 sums can count exactly.

Whole numbers only: distances equal the oracle's, or counts of the words.
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


@pytest.mark.parametrize("L,N", [(8, 500001), (61, 60001)])
@pytest.mark.parametrize("E", [31, 33, 64, 65, 96, 97, 127, 128])
def test_gram_many_units(dl, E, L, N):
    units = (N + 511) // 512
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert L * units > 12 * cus * (2 if E <= 64 else 1)
    assert L * units / (2 * cus) % units != 0
    print(f"[case] gram many units E={E} L={L} N={N}", flush=True)
    rng = np.random.default_rng(E + N)
    W = (N + 63) // 64
    words = rng.integers(0, 2**64, (L, E, W), dtype=np.uint64)
    words[:, 1::3] &= words[:, ::3][:, : words[:, 1::3].shape[1]]  # densities 1/2 and 1/4, overlapping
    words[:, :, -1] &= np.uint64((1 << (N % 64)) - 1)
    bits = units_dev(words)
    bits[:, -1, :, W % 8:] = -1  # words past the signature hold anything
    buf = torch.full((L * E * E + 1,), -1, dtype=torch.int32, device="cuda")
    D = buf[1:].view(L, E, E) if E % 2 else buf[:-1].view(L, E, E)  # odd counts: a matrix off 8 bytes
    dl.do_pairwise_hamming(bits, N, D=D)
    torch.cuda.synchronize()
    got = D_np(D)
    for l in {0, 1, L // 2, L - 2, L - 1} if E % 32 else range(L):
        for i in range(E):
            ref = np.bitwise_count(words[l, i] ^ words[l, i:]).sum(axis=1, dtype=np.uint32)
            np.testing.assert_array_equal(got[l, i, i:], ref)
            np.testing.assert_array_equal(got[l, i:, i], ref)
    assert int(buf[0 if E % 2 else -1]) == -1


def test_gram_long_layers(dl):
    """A block adds its counts after 32,767 units of a layer at the latest: an expert
    chosen by every token would pass 2^24 in fp32 otherwise (45,776 units per block)."""
    E, L, N = 2, 4, 3_000_000_000
    U = N // 512
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert N % 512 == 0 and L * U // (2 * cus) > 32768
    print(f"[case] gram long layers E={E} L={L} N={N}", flush=True)
    bits = torch.full((L, U, E, 8), -1, dtype=torch.int64, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    half = 0x0F0F0F0F0F0F0F0F  # 32 tokens of a word, else one
    counts = []
    for l in range(L):
        m = torch.rand((U, 8), generator=g, device="cuda") < 0.2 * (l + 1)
        bits[l, :, 1] = torch.where(m, half, 1)
        counts.append(8 * U + 31 * int(m.sum()))
    D = dl.do_pairwise_hamming(bits, N)
    torch.cuda.synchronize()
    got = D_np(D)
    for l in range(L):
        np.testing.assert_array_equal(got[l], np.array([[0, N - counts[l]], [N - counts[l], 0]], dtype=np.uint32))
