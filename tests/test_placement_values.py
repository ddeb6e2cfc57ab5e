"""expert_rank takes any sequence whose entries int() takes, one rank per entry,
also where the sequence is raw memory (bytes)."""
import array

import numpy as np
import pytest
import torch

import paper_2609_32398_amd as dl

RANKS = [i % 2 for i in range(24)]  # as numbers, truth values and digits alike

CASES = dict(
    list=RANKS,
    tuple=tuple(RANKS),
    bytes=bytes(RANKS),
    bytearray=bytearray(RANKS),
    memoryview=memoryview(bytes(RANKS)),
    array_i=array.array("i", RANKS),
    array_b=array.array("b", RANKS),
    array_q=array.array("q", RANKS),
    int64=np.array(RANKS, dtype=np.int64),
    uint8=np.array(RANKS, dtype=np.uint8),
    float32=np.array(RANKS, dtype=np.float32),
    bool=np.array(RANKS, dtype=bool),
    tensor=torch.tensor(RANKS),
    bool_tensor=torch.tensor(RANKS, dtype=torch.bool),
    floats=[r + 0.5 for r in RANKS],
    strings=[str(r) for r in RANKS],
    digits="".join(map(str, RANKS)),
)


@pytest.mark.parametrize("name", CASES)
def test_placement_values(name):
    got = dl._rank_array(CASES[name], len(RANKS))
    assert got._length_ == len(RANKS) and list(got) == RANKS


def test_placement_values_wrap_as_before():
    """Entries outside int32 keep their low 32 bits; the library then rejects them as ranks."""
    assert list(dl._rank_array([0, 2**32 + 1, -1], 3)) == [0, 1, -1]
