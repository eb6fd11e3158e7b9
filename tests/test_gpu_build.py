"""Trees at the edges of the build's tiles, blocks and level ranges, bit for bit against the oracle:
one and several sort tiles (8192 points), several chunks of tiles (32), blocks of 512 points, the
smallest and largest leaves, shallow trees, heavy duplicates and clusters deeper than the levels
that one workgroup aggregates."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _points(kind, n, rng):
    if kind == "cube":
        return rng.random((n, 3))
    if kind == "cluster":   # octaves around a corner: every level has few nodes
        return rng.random((n, 3)) * 2.0 ** -rng.integers(0, 20, (n, 1))
    if kind == "duplicates":   # a few places with many points each
        return rng.random((7, 3))[rng.integers(0, 7, n)]
    return np.c_[rng.random((n, 2)), np.zeros(n)]   # a plane


@pytest.mark.parametrize("kind,n,d,leaf,max_level", [
    ("cube", 1, 2, 8, 0), ("cube", 8, 2, 8, 0), ("cube", 9, 2, 8, 0), ("cube", 1023, 2, 1, 0), ("cube", 1024, 2, 8, 0),
    ("cube", 1025, 2, 64, 0), ("cube", 8191, 2, 8, 3), ("cube", 8192, 2, 1, 0), ("cube", 8193, 2, 8, 0),
    ("plane", 65537, 2, 8, 0), ("plane", 262145, 2, 8, 0), ("cube", 270001, 2, 3, 0), ("cube", 40000, 4, 8, 0),
    ("cube", 30001, 8, 8, 0), ("cluster", 20011, 2, 1, 0), ("cluster", 9001, 4, 8, 2), ("duplicates", 5000, 2, 8, 0),
    ("duplicates", 20000, 4, 64, 0), ("duplicates", 9999, 2, 8, 1),
])
def test_tree_edges_match_oracle(kind, n, d, leaf, max_level):
    from gpu_helpers import build_both, compare_trees
    rng = np.random.Generator(np.random.PCG64(n + d))
    src = _points(kind, n, rng).astype(np.float32)
    w = (rng.random(n) + 0.5).astype(np.float32)
    nrm = rng.standard_normal((n, 3)).astype(np.float32)
    gt, ot = build_both(src, w, nrm, d=d, leaf_size=leaf, max_level=max_level)
    compare_trees(gt, ot)


@pytest.mark.parametrize("n", [(1 << 21) + 12345, (1 << 24) + 700001])
def test_large_sort_is_stable(n):
    """Several chunks of 32 tiles, and chunks of more: codes sorted, ties in input order."""
    import paper_2506_02219_amd as P
    g = torch.Generator().manual_seed(2)
    src = (torch.randint(0, 64, (n, 3), generator=g).float() / 64.0).cuda()   # about eight points a cell
    a = P.sbh_build(src, torch.ones(n, device="cuda")).export()
    code = a["codes"].astype(np.int64)
    perm = a["perm"].astype(np.int64)
    assert np.array_equal(np.sort(perm), np.arange(n))
    step = np.diff(code)
    assert (step >= 0).all()
    assert (np.diff(perm)[step == 0] > 0).all()


@pytest.mark.parametrize("n", [8160, 20400])
@pytest.mark.parametrize("copies", [2, 16, 17])
@pytest.mark.parametrize("scale", [-17, -21])
def test_runs_of_equal_top_bits(n, copies, scale):
    """Groups of points that differ in the low bits of their codes alone: runs that one thread puts in
    order, the longest such run, and runs that take the passes over all bits."""
    from gpu_helpers import build_both, compare_trees
    rng = np.random.Generator(np.random.PCG64(n + copies))
    cells = (rng.permutation(64 ** 3)[:n // copies, None] // np.array([1, 64, 4096]) % 64 + 0.5) / 64.0
    src = (np.repeat(cells, copies, 0) + rng.integers(0, 16, (n // copies * copies, 3)) * 2.0 ** scale)
    src = src[rng.permutation(len(src))].astype(np.float32)
    w = np.ones(len(src), np.float32)
    gt, ot = build_both(src, w, None, d=2, leaf_size=8)
    compare_trees(gt, ot)


@pytest.mark.parametrize("n", [511, 512, 513])
@pytest.mark.parametrize("leaf,max_level", [(1, 0), (8, 0), (8, 1)])
def test_topology_block_edges(n, leaf, max_level):
    """One block of points and its neighbour, leaves that end in the next block among them."""
    from gpu_helpers import build_both, compare_trees
    rng = np.random.Generator(np.random.PCG64(n))
    src = rng.random((n, 3)).astype(np.float32)
    compare_trees(*build_both(src, np.ones(n, np.float32), src, d=2, leaf_size=leaf, max_level=max_level))
