"""REM scheduling on the device where its variants change: 32-bit and 64-bit
values (loads summing to just below and above 2^31, volumes up to 2^40 - 1),
register slots for 64 / 128 / 256 / 1,024 experts, ranks within and beyond one
wavefront, equal scores, and more replicas on one rank than a wavefront has lanes.

Whole numbers only: records, loads and volumes equal the oracle's.
"""
import random

import pytest
import torch

from oracle import rem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_32398_amd as p

    p.lib()
    return p


def _dev(x):
    return torch.tensor(x, dtype=torch.int64, device="cuda")


@pytest.mark.parametrize("E,R,D", [(5, 3, 2), (64, 64, 1), (65, 8, 3), (128, 65, 2), (129, 16, 4), (257, 64, 2),
                                   (1024, 130, 1)])
@pytest.mark.parametrize("scale", ["small", "edge", "wide", "equal"])
def test_allocate_and_dispatch(dl, E, R, D, scale):
    rng = random.Random(E * 131 + R)
    home = [rng.randrange(R) for _ in range(E)]
    Ts = []
    for l in range(3):
        if scale == "equal":
            T = [100] * E
        elif scale == "wide":
            T = [rng.randrange(1 << 40) for _ in range(E)]
        else:
            T = [int(rng.paretovariate(1.1) * 1000) if rng.random() < 0.9 else 0 for _ in range(E)]
        if scale == "edge":  # the loads sum to 2^31 - R - 1, 2^31 - R and 2^31 + 5
            T = [t % ((1 << 31) // E // 2) for t in T]
            T[0] += (1 << 31) + (-R - 1, -R, 5)[l] - sum(T)
        Ts.append(T)
    print(f"[case] rem E={E} R={R} D={D} {scale}", flush=True)
    m, n, lo, to = dl.do_rem_allocate(_dev(Ts), home, R, D)
    T1 = [[t * 3 // 4 + (7 if scale != "equal" else 0) for t in T] for T in Ts]
    r, nr, qo, t1 = dl.do_rem_dispatch(m, n, _dev(T1), home, R, D)
    torch.cuda.synchronize()
    got, routes = dl.rem_records(m, n), dl.rem_records(r, nr)
    for l, T in enumerate(Ts):
        base = [sum(T[e] for e in range(E) if home[e] == q) for q in range(R)]
        moves, L, left = rem.allocate(base, T, home, D)
        assert got[l] == moves and lo[l].tolist() == L and to[l].tolist() == left
        want, Q, left1 = rem.dispatch(moves, T1[l], home, R, D)
        assert routes[l] == want and qo[l].tolist() == Q and t1[l].tolist() == left1


def test_given_loads_apart_from_volumes(dl):
    # small loads with a volume beyond 32 bits, and the reverse
    home = [0, 0, 1, 2]
    for base, T in (([90, 10, 20], [1 << 33, 5, 6, 7]), ([1 << 39, 3, 1 << 38], [50, 60, 1, 2])):
        m, n, lo, to = dl.do_rem_allocate(_dev([T]), home, 3, 2, rank_load=_dev([base]))
        torch.cuda.synchronize()
        moves, L, left = rem.allocate(list(base), list(T), home, 2)
        assert dl.rem_records(m, n)[0] == moves and lo[0].tolist() == L and to[0].tolist() == left


def test_many_replicas_on_one_rank(dl):
    # 200 replicas on rank 0 (several per expert), so a step takes more than one round of lanes
    rng = random.Random(5)
    E, R, D = 40, 4, 3
    home = [1 + e % 3 for e in range(E)]
    T = [rng.randrange(50, 60) for _ in range(E)]
    reps = [(e % E, home[e % E], 0 if e < 200 else 1 + (home[e % E] % 3), 0) for e in range(230)]
    rec = [[a | (b << 32), c, 0] for a, b, c, _ in reps]
    r, nr, qo, _ = dl.do_rem_dispatch(_dev([rec]), torch.tensor([len(rec)], dtype=torch.int32, device="cuda"),
                                      _dev([T]), home, R, D)
    torch.cuda.synchronize()
    want, Q, _ = rem.dispatch([(a, b, c) for a, b, c, _ in reps], T, home, R, D)
    assert dl.rem_records(r, nr)[0] == want and qo[0].tolist() == Q


@pytest.mark.parametrize("E,R,D", [(8, 1, 50), (12, 3, 60), (40, 5, 17), (140, 70, 30)])
def test_more_passes_than_routes(dl, E, R, D):
    """The dispatch ends with the first pass that routes nothing: the passes after it would change nothing."""
    rng = random.Random(E + D)
    home = [e % R for e in range(E)]
    reps = [(e, home[e], rng.randrange(R)) for e in range(E) for _ in range(3)]
    rec = [[a | (b << 32), c, 0] for a, b, c in reps]
    T = [rng.randrange(1000) * (1 + 9 * (home[e] == 0)) for e in range(E)]
    r, nr, qo, t1 = dl.do_rem_dispatch(_dev([rec]), torch.tensor([len(rec)], dtype=torch.int32, device="cuda"),
                                       _dev([T]), home, R, D)
    torch.cuda.synchronize()
    want, Q, left = rem.dispatch(reps, T, home, R, D)
    assert len(want) < R * D
    assert dl.rem_records(r, nr)[0] == want and qo[0].tolist() == Q and t1[0].tolist() == left
