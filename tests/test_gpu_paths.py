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
