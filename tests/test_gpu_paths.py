"""GPU parity at the sizes where the kernels change path: edges of tiles and
ranges, remainders, the smallest and largest of a path's range."""
import numpy as np
import pytest

from oracle import volume_area as va
from paper_1205_1171_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def _fan_clouds(sizes, seed):
    """Clouds of given sizes with random (not convex) faces over all their
    points: the kernels take any face rows."""
    rng = np.random.default_rng(seed)
    P, F = [], []
    for m in sizes:
        P.append(workloads.noisy_sphere(rng, m) if m else np.zeros((0, 3), np.float32))
        F.append(rng.integers(0, m, size=(2 * m, 3)).astype(np.int32) if m >= 3
                 else np.zeros((0, 3), np.int32))
    return P, F


# one range exactly, one point more or less, the largest range-split cloud,
# one point above it (global atomics), empty and tiny clouds between
@pytest.mark.parametrize("sizes", [(4095, 4096, 4097), (0, 3, 0, 8192, 1, 5),
                                   (65536, 65537, 100)])
def test_volume_gradient_range_edges(sizes):
    import torch
    from paper_1205_1171_amd import hull
    P, F = _fan_clouds(sizes, sum(sizes))
    off = np.cumsum([0] + [len(p) for p in P]).astype(np.int64)
    foff = np.cumsum([0] + [len(f) for f in F]).astype(np.int64)
    H = len(sizes)
    gV = np.linspace(-1, 1, H).astype(np.float32) * 1e-5
    gA = np.linspace(1, 2, H).astype(np.float32)
    say("volume gradient", sizes)
    g = hull.volume_area_bwd(*(torch.from_numpy(x).cuda() for x in (
        np.concatenate(P), off, np.concatenate(F), foff, gV, gA))).cpu().numpy()
    for h in range(H):
        if len(F[h]) == 0:
            assert not g[off[h]:off[h + 1]].any()
            continue
        dV, dA = va.gradients(P[h], F[h])
        want = gV[h].astype(np.float64) * dV + gA[h].astype(np.float64) * dA
        got = g[off[h]:off[h + 1]]
        assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)


# an edge from a point to itself is its own twin; a third half-edge of an edge
# is an error whichever arrives last; a table of one slot group
@pytest.mark.parametrize("faces,want", [
    ([[0, 0, 1]], [[0, 0, 0]]),
    ([[0, 1, 2]], [[-1, -1, -1]]),
    ([[0, 1, 2], [2, 1, 0]], [[1, 1, 1], [1 - 1, 0, 0]]),
    ([[0, 1, 2], [1, 0, 3], [0, 1, 4]], None),
    ([[0, 0, 1], [0, 0, 2]], None)])
def test_adjacency_small_tables(faces, want):
    import torch
    from paper_1205_1171_amd import hull
    f = torch.tensor(faces, dtype=torch.int32, device="cuda")
    say("adjacency", faces)
    if want is None:
        with pytest.raises(hull.HullError):
            hull.face_adjacency(f)
        return
    adj, open_edges = hull.face_adjacency(f)
    assert adj.cpu().tolist() == want
    assert open_edges == sum(x < 0 for row in want for x in row)


# The time-segmented merges in LDS (every level up to 11, then none) with
# segments of the shortest length, of more steps than the counting pass notes
# and of whole movies; sizes at the edges of blocks and with ragged last blocks.
@pytest.mark.parametrize("seg", ["4", "16", "1000000"])
@pytest.mark.parametrize("tile", ["11", "0"])
def test_segment_walk_movies(monkeypatch, tile, seg):
    import oracle
    import torch
    from paper_1205_1171_amd import hull
    monkeypatch.setenv("HULL_SERIAL_LEVELS", "0")
    monkeypatch.setenv("HULL_TILE_LEVELS", tile)
    monkeypatch.setenv("HULL_WALK_SEGMENT", seg)
    rng = np.random.default_rng(5)
    # a cone: the apex is a neighbour of every rim point (one list as long as
    # the movie); lattices: every kind of tie; a curve whose points are all
    # vertices
    rim = workloads.sphere(rng, 600, 1 << 20)
    rim[:, 2] = 1000
    cone = np.concatenate([rim, [[3, 5, -(1 << 20)]]]).astype(np.int32)
    sets = [workloads.sphere(rng, n, 1 << 20) for n in (2, 3, 17, 255, 256, 257, 2047, 2049, 4100)]
    sets += [cone, workloads.lattice(rng, 700, 3), workloads.lattice(rng, 900, 20),
             workloads.moment_curve(), workloads.cube(rng, 3000, 1 << 29)]
    ws = hull.Workspace()
    for p in sets:
        p = np.ascontiguousarray(p)
        L = oracle.levels_for(len(p))
        x = torch.from_numpy(p).cuda()
        for run in (0, 1):
            for level in {L, L // 2 + 1}:
                say("segment walk", tile, seg, len(p), run, level)
                ev, bl, _ = hull.movies(x, run, level, ws=ws)
                want, wbl = oracle.level_movies(p, run, level)
                w = 1 << min(level, L)
                assert (bl[::w] == wbl).all()
                got = np.concatenate([ev[2 * s:2 * s + bl[s]] for s in range(0, len(p), w)])
                assert (got == want).all()


# Ragged sizes around powers of two: a trailing block waits in the buffer of
# its own last level, which is the merge's output buffer at every other level,
# on every strategy.
@pytest.mark.parametrize("serial,tile,wave", [("99", "0", "-1"), ("99", "0", "4"), ("3", "11", "-1"),
                                              ("0", "0", "-1")])
def test_trailing_blocks(monkeypatch, serial, tile, wave):
    import oracle
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    monkeypatch.setenv("HULL_SERIAL_LEVELS", serial)
    monkeypatch.setenv("HULL_TILE_LEVELS", tile)
    monkeypatch.setenv("HULL_WAVE_LEVEL", wave)
    rng = np.random.default_rng(8)
    ws = hull.Workspace()
    for n in [b + d for b in (64, 256, 1024, 2048) for d in (1, 2, 3, 7, 33, b // 2 + 1, b - 1)]:
        p = np.ascontiguousarray(workloads.sphere(rng, n, 1 << 20))
        say("trailing", serial, tile, wave, n)
        got = hull.hull_sync(torch.from_numpy(p).cuda(), ws=ws).cpu().numpy()
        a, b = validate.canonical(got), validate.canonical(oracle.hull(p))
        assert a.shape == b.shape and (a == b).all()


# Interior points taken out before the sort: the faces are those of all points.
# Shapes with many and few interior points, points on the facets and edges of
# a lattice hull, flat and thin clouds, one outlier, duplicates; sizes around the
# filter's smallest and its changes of grid.
@pytest.mark.parametrize("n", [1023, 1024, 1025, 8191, 8192, 131073])
def test_interior_filter(n):
    import oracle
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    rng = np.random.default_rng(n)
    r = 1 << 20
    ball = workloads.ball(rng, n, r)
    sets = {"ball": ball, "cube": workloads.cube(rng, n, r),
            "gaussian": workloads.gaussian(rng, n)}
    if n <= 8192:
        sets["sphere"] = workloads.sphere(rng, n, r)
        out = ball // 1024
        out[n // 2] = [r, -r, r // 2]
        thin = ball.copy()
        thin[:, 1] //= 1 << 18
        flat = ball.copy()
        flat[:, 2] = 7
        skew = ball // 64
        skew[:, 2] += 9 * skew[:, 0] - 5 * skew[:, 1]
        sets.update({"lattice": workloads.lattice(rng, n, 9), "outlier": out, "thin": thin,
                     "flat": flat, "skew": skew, "far": ball // 8 + (1 << 28),
                     "full": workloads.cube(rng, n, 1 << 29),
                     "corners": np.concatenate([workloads.cube_corners(r), ball[8:] // 2]),
                     "same": np.repeat(ball[:4], (n + 3) // 4, axis=0)[:n]})
    ws = hull.Workspace()
    for name, p in sets.items():
        p = np.ascontiguousarray(p, dtype=np.int32)
        for lower in (False, True) if n <= 1025 else (n % 2 == 0,):
            say("filter", n, name, lower)
            got = hull.hull_sync(torch.from_numpy(p).cuda(), lower_only=lower, ws=ws).cpu().numpy()
            a = validate.canonical(got)
            b = validate.canonical(oracle.hull(p, lower_only=lower))
            assert a.shape == b.shape and (a == b).all(), name
    p = (ball.astype(np.int64) * 512)
    p[:, 2] *= 1 << 12
    say("filter wide", n)
    a = validate.canonical(hull.hull_wide(torch.from_numpy(p).cuda()).cpu().numpy())
    assert (a == validate.canonical(oracle.hull_wide(p))).all()


# The filter of a batch: clouds at the edges of its three grids, clouds too small
# for it, empty ones, spheres that keep everything next to balls; eager and
# captured.
def test_batch_filter():
    import oracle
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    rng = np.random.default_rng(4)
    sizes = [0, 1, 2, 3, 255, 256, 257, 0, 2047, 2048, 2049, 8191, 8192, 8193, 1000, 30000, 0]
    parts = []
    for k, n in enumerate(sizes):
        make = [workloads.ball, workloads.sphere, workloads.cube][k % 3]
        parts.append(make(rng, n, 1 << 20) if n else np.zeros((0, 3), np.int32))
    parts[8][:, 2] = 5  # flat: nothing is interior
    parts[10] //= 1 << 17  # a lattice of many duplicates
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    x = torch.from_numpy(np.ascontiguousarray(np.concatenate(parts), dtype=np.int32)).cuda()
    say("batch filter eager")
    f, fo = hull.hull_batched_sync(x, off)
    bh = hull.BatchedHull(x, off)
    say("batch filter captured")
    bh.capture()
    for _ in range(3):
        bh.faces.zero_()
        bh.replay()
        g, go = bh.result()
        assert torch.equal(f, g) and torch.equal(fo, go)
    f, fo = f.cpu().numpy(), fo.cpu().numpy()
    for k, p in enumerate(parts):
        got = validate.canonical(f[fo[k]:fo[k + 1]])
        want = validate.canonical(oracle.hull(np.ascontiguousarray(p, dtype=np.int32))) if len(p) >= 3 \
            else np.zeros((0, 3))
        assert got.shape == want.shape and (got == want).all(), (k, len(p))


# Setup and sort in one launch: sizes at its changes of block size and chunk, equal
# x in one chunk and across chunks, the largest size and the first above it; the
# order itself through the movies' ranks.
@pytest.mark.parametrize("n", [1, 2, 3, 127, 128, 129, 512, 513, 1023, 4096, 4097, 8192, 8193])
def test_small_sort(n):
    import oracle
    import torch
    from paper_1205_1171_amd import hull
    rng = np.random.default_rng(n)
    for p in (workloads.cube(rng, n, 1 << 29), workloads.lattice(rng, n, 2),
              np.repeat(workloads.cube(rng, 1, 99), n, axis=0)):
        say("small sort", n)
        _, _, order = hull.movies(torch.from_numpy(np.ascontiguousarray(p)).cuda(), 0, 0)
        assert (order == oracle.sort_order(p)).all()
    p[n // 2, 1] = (1 << 29) + 1
    with pytest.raises(hull.HullError) as e:
        hull.hull_sync(torch.from_numpy(p).cuda()) if n > 2 else hull.movies(
            torch.from_numpy(p).cuda(), 0, 0)
    assert e.value.code == hull.HULL_ERANGE


# Lists built by ranges or bins of points (calls of many points), beside lists by global
# atomics (the small clouds one by one; the large ones by smaller bins): blocks of one range, one point more, several
# ranges and a ragged last one, clouds that end below the level and trailing
# blocks between others, lists long enough to be sorted (an apex over a circle), and
# a device-known number of points below and above the line; without tiles, also the
# ranges shorter than the widest, of one wave and more.
@pytest.mark.parametrize("big", [262144, 180000])
@pytest.mark.parametrize("tile", [None, "0"])
def test_lists_by_range(big, tile, monkeypatch):
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    rng = np.random.default_rng(big)
    t = np.linspace(0, 2 * np.pi, 9000, endpoint=False)
    r = 1 << 20
    cone = np.stack([r - rng.integers(0, 1000, 9000), r * np.cos(t), r * np.sin(t)], 1).astype(np.int32)
    cone[17] = (-r, 3, 5)
    parts = [workloads.sphere(rng, 4097, r), cone, workloads.sphere(rng, 8192, r), workloads.sphere(rng, 8193, r),
             workloads.sphere(rng, 300, r), workloads.sphere(rng, big, r), workloads.cube(rng, 20000, r),
             workloads.lattice(rng, 5000, 9), workloads.sphere(rng, 245771, r), workloads.sphere(rng, 7, r)]
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    x = torch.from_numpy(np.ascontiguousarray(np.concatenate(parts), dtype=np.int32)).cuda()
    want = []
    for k, p in enumerate(parts):
        say("lists by range: cloud", k, len(p))
        want.append(validate.canonical(hull.hull_sync(
            torch.from_numpy(np.ascontiguousarray(p, dtype=np.int32)).cuda()).cpu().numpy()))
    if tile:
        monkeypatch.setenv("HULL_TILE_LEVELS", tile)
    # (segments of 32 events leave no scratch for the bins)
    for sched in (None, hull.Schedule(0, 16, 0, -1), hull.Schedule(0, 32, 0, -1)):
        say("lists by range: batch", sched)
        f, fo = hull.hull_batched_sync(x, off, schedule=sched)
        f, fo = f.cpu().numpy(), fo.cpu().numpy()
        for k in range(len(parts)):
            got = validate.canonical(f[fo[k]:fo[k + 1]])
            assert got.shape == want[k].shape and (got == want[k]).all(), (k, len(parts[k]))


# The smaller bins beside lists by global atomics (segments of 32 events leave no
# scratch for bins; no tiles, so every level's lists differ): the first size that has them, one
# point fewer, both point types, a size that only the device knows.
@pytest.mark.parametrize("n", [131071, 131072, 150001])
def test_lists_by_small_bins(n, monkeypatch):
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    monkeypatch.setenv("HULL_TILE_LEVELS", "0")
    p = workloads.sphere(np.random.default_rng(n), n, 1 << 20)
    p[:9] //= 2  # interior points
    x = torch.from_numpy(p).cuda()
    off = np.array([0, n], np.int64)
    say("small bins: atomics", n)
    want = validate.canonical(hull.hull_batched_sync(x, off, schedule=hull.Schedule(0, 32, 0, -1))[0].cpu().numpy())
    say("small bins", n)
    bins = hull.hull_batched_sync(x, off, schedule=hull.Schedule(0, 4, 0, -1))[0]
    single = hull.hull_sync(x)
    for f in (bins, single, hull.hull_wide(x.to(torch.int64))):
        got = validate.canonical(f.cpu().numpy())
        assert got.shape == want.shape and (got == want).all()


# Calls whose size on the host says lists by bins or ranges and whose points left
# after the filter say atomics (a cone whose apex starts the first block and
# has a long list; the rim's own hull is the hull): single hulls of both point
# types and a batch.
@pytest.mark.parametrize("n,rim", [(1 << 17, 4100), (1 << 19, 5000)])
def test_few_points_left_of_many(n, rim):
    import oracle
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    from test_kernels_on_host import cone_with_interior
    rng = np.random.default_rng(rim)
    p = cone_with_interior(rng, rim, n)
    want = validate.canonical(oracle.hull(p[:rim + 1]))
    x = torch.from_numpy(p).cuda()
    for rep in range(3):
        for wide in (False, True):
            say("few points left", n, rep, wide)
            got = validate.canonical((hull.hull_wide(x.to(torch.int64)) if wide else hull.hull_sync(x)).cpu().numpy())
            assert got.shape == want.shape and (got == want).all()
    rims = [rim, 300, 4097, 2500]
    parts = [cone_with_interior(rng, m, n // 2 if m > 300 else 1000) for m in rims]
    off = np.cumsum([0] + [len(q) for q in parts]).astype(np.int64)
    say("few points left: batch", off[-1])
    f, fo = hull.hull_batched_sync(torch.from_numpy(np.concatenate(parts)).cuda(), off)
    f, fo = f.cpu().numpy(), fo.cpu().numpy()
    for k, q in enumerate(parts):
        got, want = validate.canonical(f[fo[k]:fo[k + 1]]), validate.canonical(oracle.hull(q[:rims[k] + 1]))
        assert got.shape == want.shape and (got == want).all(), k


# Level 4 with many merges by the host's bound and few by the device's, LDS-staged or
# not: many tiny clouds beside some of 50-64 points.
@pytest.mark.parametrize("lds_levels", ["3", "4"])
def test_many_tiny_clouds(lds_levels, monkeypatch):
    import oracle
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    monkeypatch.setenv("HULL_LDS_LEVELS", lds_levels)
    rng = np.random.default_rng(6)
    parts = [workloads.sphere(rng, 50 + k % 15, 1 << 20) for k in range(700)]
    parts += [workloads.sphere(rng, 5, 1 << 20) for _ in range(17000)]
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    say("many tiny clouds", lds_levels)
    f, fo = hull.hull_batched_sync(torch.from_numpy(np.concatenate(parts)).cuda(), off)
    f, fo = f.cpu().numpy(), fo.cpu().numpy()
    for k in range(720):
        got, want = validate.canonical(f[fo[k]:fo[k + 1]]), validate.canonical(oracle.hull(parts[k]))
        assert got.shape == want.shape and (got == want).all(), k


# Lists of link changes as long as the movies: in LDS, by atomics, by bins of both
# sizes and by ranges; the largest beside the lane-serial merges, which have no
# lists.
@pytest.mark.parametrize("n", [700, 9000, 140000, (1 << 19) + 5])
def test_points_of_high_degree(n, monkeypatch):
    import oracle
    import torch
    from oracle import validate
    from paper_1205_1171_amd import hull
    from test_kernels_on_host import hubs
    p = hubs(np.random.default_rng(n), n)
    x = torch.from_numpy(p).cuda()
    say("high degree", n)
    got = [validate.canonical(hull.hull_sync(x).cpu().numpy()),
           validate.canonical(hull.hull_wide(x.to(torch.int64)).cpu().numpy())]
    if n <= 9000:
        want = oracle.hull(p)
    else:
        say("high degree: lane-serial", n)
        monkeypatch.setenv("HULL_SERIAL_LEVELS", "99")
        monkeypatch.setenv("HULL_WAVE_LEVEL", "-1")
        want = hull.hull_sync(x).cpu().numpy()
    want = validate.canonical(want)
    for f in got:
        assert f.shape == want.shape and (f == want).all()


# The moment curve with exact coordinates: every face joins two neighbours to the
# first or the last point.
@pytest.mark.parametrize("half", [100, 1000, 16000])
def test_moment_curve_wide(half):
    import torch
    from paper_1205_1171_amd import hull
    t = np.arange(-half, half + 1, dtype=np.int64)
    n = len(t)
    i = np.arange(n - 1)
    want = np.sort(np.concatenate([np.stack([np.zeros(n - 2, np.int64), i[1:], i[1:] + 1], 1),
                                   np.stack([i[:-1], i[:-1] + 1, np.full(n - 2, n - 1)], 1)]), 1)
    say("moment curve", n)
    got = np.sort(hull.hull_wide(torch.from_numpy(np.stack([t, t * t, t * t * t], 1)).cuda()).cpu().numpy(), 1)
    assert (got[np.lexsort(got.T)] == want[np.lexsort(want.T)]).all()
