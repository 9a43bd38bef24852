"""The kernels on the CPU: arrival orders of atomics that a GPU may take and a
test there cannot ask for, against the oracle."""
import numpy as np
import pytest

import hip_on_host
import oracle
from oracle import validate
from paper_1205_1171_amd import workloads


def same(a, b):
    a, b = validate.canonical(a), validate.canonical(b)
    return a.shape == b.shape and bool((a == b).all())


def cone_with_interior(rng, rim, n):
    """An apex (smallest x, so it starts the first block) over a circle of `rim`
    points, then interior points: n in all."""
    r = 1 << 20
    t = np.linspace(0, 2 * np.pi, rim, endpoint=False)
    c = np.stack([r - rng.integers(0, 1000, rim), r * np.cos(t), r * np.sin(t)], 1).astype(np.int32)
    inner = workloads.ball(rng, n - rim - 1, r // 8)
    inner[:, 0] += r // 2
    return np.concatenate([[[-r, 3, 5]], c[rng.permutation(rim)], inner]).astype(np.int32)


# The host's bound on the points says lists by bins (2^17 points) or ranges (2^19),
# the device counts fewer and takes the atomics: the first event's place must
# be the one its atomic gave.  The rim's own hull is the whole hull.
@pytest.mark.parametrize("n,rim,seed", [(1 << 17, 4100, 1), (1 << 17, 4100, 2), (1 << 19, 5000, 1)])
def test_first_events_place(n, rim, seed):
    p = cone_with_interior(np.random.default_rng(seed), rim, n)
    want = oracle.hull(p[:rim + 1])
    for descending in (False, True):
        assert same(hip_on_host.hull(p, descending=descending, fill=0), want), descending
