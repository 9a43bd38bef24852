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
    for order in (0, 1, 2):
        assert same(hip_on_host.hull(p, order=order, fill=0), want), order


# The host's bound counts many merges at level 4, the device few: one of the two
# kernels launched for the level runs, also where level 4 is an LDS-staged one.
@pytest.mark.parametrize("lds_levels", ["3", "4"])
def test_level_runs_one_way(lds_levels, monkeypatch):
    monkeypatch.setenv("HULL_LDS_LEVELS", lds_levels)
    monkeypatch.setenv("HULL_WAVE_LEVEL", "-1")  # (lanes in lockstep without barriers)
    rng = np.random.default_rng(6)
    parts = [workloads.sphere(rng, 50 + k % 15, 1 << 20) for k in range(600)]
    parts += [workloads.sphere(rng, 5, 1 << 20) for _ in range(17000)]
    f, fo = hip_on_host.hull_batched(parts)
    for k in range(620):
        assert same(f[fo[k]:fo[k + 1]], oracle.hull(parts[k])), k


# A filter without room for its grid is an error (the sort would read a list that
# was never written), and every size that is sent to it has room.
def test_filter_room():
    rng = np.random.default_rng(2)
    assert hip_on_host.filter_rc(workloads.cube(rng, 300, 99)) == -5
    for n in (1024, 8193, 131071, 131072):
        assert hip_on_host.filter_rc(workloads.cube(rng, n, 99)) == 0


# Rows outside every cloud's offsets count to the first or the last cloud (so a
# batch's last cloud may be given by its first row alone).
@pytest.mark.parametrize("face_off", [[0, 100, 100], [0, 100, 260], [0, 0, 150], [40, 100, 260], [260, 260, 260]])
def test_adjacency_rows_past_the_offsets(face_off):
    rng = np.random.default_rng(7)
    faces = oracle.hull(workloads.sphere(rng, 132, 1 << 20))
    F = len(faces)
    assert F == 260
    # a cloud's rows are a surface with holes; its points: all for either cloud
    off = np.asarray(face_off, np.int64)
    cut = int(off[1])  # rows before it: the first cloud's
    want = np.full((F, 3), -1, np.int32)
    for rows in (range(0, cut), range(cut, F)):
        edge = {(int(faces[f][k]), int(faces[f][(k + 1) % 3])): f for f in rows for k in range(3)}
        for (a, b), f in edge.items():
            k = [int(v) for v in faces[f]].index(a)
            want[f, k] = edge.get((b, a), -1)
    for order in (0, 1, 2):
        st, adj, open_edges = hip_on_host.face_adjacency(
            faces, off, np.array([0, 132, 264], np.int64), order)
        assert st == 0 and (adj == want).all() and open_edges == (want < 0).sum()


def hubs(rng, n):
    """Two points of high degree side by side over a circle of n - 2 points."""
    r = 1 << 28
    t = np.linspace(0, 2 * np.pi, n, endpoint=False)
    p = np.stack([r - rng.integers(0, 1000, n), r * np.cos(t), r * np.sin(t)], 1)[rng.permutation(n)]
    p[n // 3], p[n // 2] = (-r, 3, 5), (-r + 9, -7, 11)
    return p.astype(np.int32)


# Lists of link changes as long as the movies, sorted by their workgroup: in LDS, and
# in global memory below and above the length that is sorted by rank.
@pytest.mark.parametrize("tile", ["11", "0"])
@pytest.mark.parametrize("n", [90, 700, 5000])
def test_points_of_high_degree(n, tile, monkeypatch):
    monkeypatch.setenv("HULL_TILE_LEVELS", tile)
    monkeypatch.setenv("HULL_SERIAL_LEVELS", "3")
    p = hubs(np.random.default_rng(n), n)
    want = oracle.hull(p)
    for order in (0, 1, 2):
        assert same(hip_on_host.hull(p, order=order), want)
