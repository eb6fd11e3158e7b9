"""The per-query-stream walk where its selection and its swap take other branches: shallow trees whose
deepest children are large leaves, one-point leaves, a softening of zero (empty slots are skipped)
and of more (they add nothing), queries at the origin of the coordinates that empty slots hold."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [0.0, 1e-3])
@pytest.mark.parametrize("n,d,leaf,max_level", [(400, 2, 1, 0), (5000, 2, 8, 2), (5000, 2, 64, 0), (3000, 4, 8, 2),
                                                (3000, 4, 5, 0)])
def test_streams_match_oracle(n, d, leaf, max_level, eps):
    from gpu_helpers import build_both, check_sbh
    rng = np.random.Generator(np.random.PCG64(n + d))
    src = (rng.random((n, 3)) * 2 - 1).astype(np.float32)
    src[:, 2] = np.abs(src[:, 2]) ** 2   # a lopsided cloud: empty slots at every level
    w = (rng.random(n) + 0.5).astype(np.float32)
    q = (3 * rng.random((333, 3)) - 1.5).astype(np.float32)
    q[0] = 0.0
    gt, ot = build_both(src, w, d=d, leaf_size=leaf, max_level=max_level)
    check_sbh(gt, ot, q, 0, samples=2, seed=7, group=1, eps=eps)


@pytest.mark.parametrize("kernel", [0, 1, 2])
@pytest.mark.parametrize("d,samples", [(2, 1), (2, 3), (2, 32), (4, 1)])
def test_same_values_for_any_pool(d, samples, kernel):
    """Small launches give a wavefront fewer queries: a query's value is the same bit for bit."""
    import paper_2506_02219_amd as P
    rng = np.random.Generator(np.random.PCG64(9))
    n, nq = 9000, 140001 if samples < 32 else 9001
    src = torch.from_numpy(rng.random((n, 3)).astype(np.float32)).cuda()
    nrm = torch.from_numpy(rng.standard_normal((n, 3)).astype(np.float32)).cuda()
    q = torch.from_numpy((2 * rng.random((nq, 3)) - 0.5).astype(np.float32)).cuda()
    tree = P.sbh_build(src, torch.ones(n, device="cuda"), nrm, branching=d)
    whole = P.sbh_eval(tree, q, kernel, samples=samples, seed=3, group=1)
    for m in (33, 30001):   # streams are keyed by the query's index, so the first ones are the same
        part = P.sbh_eval(tree, q[:m].contiguous(), kernel, samples=samples, seed=3, group=1)
        assert torch.equal(whole[:m].view(torch.int32), part.view(torch.int32))


@pytest.mark.parametrize("d", [2, 4])
@pytest.mark.parametrize("eps", [1e-22, 1e-20, 1e-19, 1.08e-19, 1.2e-19])
def test_softening_with_a_subnormal_square(d, eps):
    """eps^2 below float32's smallest normal number (1.18e-38) is 0 to the hardware's square root: an empty
    slot, at the origin like the query, still adds nothing, and the values are those of eps = 0."""
    import paper_2506_02219_amd as P
    rng = np.random.Generator(np.random.PCG64(11))
    src = torch.from_numpy((rng.random((4000, 3)) + 0.5).astype(np.float32)).cuda()
    q = np.zeros((70, 3), np.float32)
    q[20:] = 1e-20 * rng.random((50, 3))
    tree = P.sbh_build(src, torch.ones(4000, device="cuda"), branching=d)
    got, want = (P.sbh_eval(tree, torch.from_numpy(q).cuda(), 0, samples=2, seed=7, group=1, eps=e) for e in (eps, 0.0))
    assert torch.isfinite(want).all()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
