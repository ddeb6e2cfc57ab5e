"""Denormal scores keep their order in the oracle, in every one of its threads
and whichever of the oracle and the score generator is loaded first: loading
the generator must not change how the process treats denormals (it would turn
1e-40 into zero, which the Top-K then ties with the zeros of the row).

Each case runs in a process of its own, because such a change would outlive it.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASE = r"""
import sys
import numpy as np
import oracle, synth

def generate():
    synth.normal(1, 4096, 64, 0, threads=4)  # its threads start here

if sys.argv[1] == "generator":
    generate()
N, E = 997, 8
rng = np.random.default_rng(7)
x = np.array([0x00000000, 0x80000000, 0x000116C2, 0x800116C2, 0x00000001, 0x80000001, 0x3F800000, 0xBF800000],
             dtype=np.uint32)[rng.integers(0, 8, (N, E))]
# rank by the bit patterns alone: +0 and -0 alike, then the lower index
key = np.where(x >> 31 != 0, -(x & 0x7FFFFFFF).astype(np.int64), x.astype(np.int64))
order = np.argsort(-key, axis=1, kind="stable")
if sys.argv[1] == "oracle":
    oracle.topk_signature(x.view(np.float32), 2, 4)  # its threads start here
generate()
for threads in (1, 4, None):
    for k in (1, 2, 5):
        F = oracle.topk_signature(x.view(np.float32), k, threads) if threads else oracle.topk_signature(x.view(np.float32), k)
        ref = np.zeros((E, N), dtype=np.uint8)
        ref[order[:, :k].T, np.arange(N)] = 1
        assert np.array_equal(F.reshape(E, N), ref), (threads, k, int((F.reshape(E, N) != ref).sum()))
one = np.array([1e-40], dtype=np.float32)
assert one[0] != 0 and (one * np.float32(1)).view(np.uint32)[0] == one.view(np.uint32)[0]
"""


@pytest.mark.parametrize("first", ["generator", "oracle"])
def test_denormals_keep_their_order(first):
    r = subprocess.run([sys.executable, "-c", CASE, first], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
