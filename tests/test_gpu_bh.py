"""Barnes-Hut where its lists and leaves end: ragged tiles, cuts that fill a wavefront's part of the
next level's list and go on depth-first, leaves of up to 64 points, queries that take no part in the
vote, against the oracle's voted cut (and brute force for beta = infinity)."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cloud(n, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    src = rng.random((n, 3)).astype(np.float32)
    w = (rng.random(n) + 0.5).astype(np.float32)
    nrm = rng.standard_normal((n, 3)).astype(np.float32)
    return src, w, (nrm / np.linalg.norm(nrm, axis=1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("kernel", [0, 1, 2])
@pytest.mark.parametrize("n,d,leaf,nq,beta", [(9, 2, 8, 1, 2.0), (3000, 2, 1, 63, 0.3), (3000, 2, 64, 65, 3.0),
                                              (20000, 2, 8, 200, 6.0), (20000, 4, 8, 130, 6.0), (5000, 4, 5, 64, 0.7),
                                              (20000, 2, 8, 200, math.inf), (20000, 4, 8, 70, math.inf)])
def test_bh_matches_oracle(n, d, leaf, nq, beta, kernel):
    """(20,000 points at beta = 6 and infinity open more blocks a level than the lists hold.)"""
    from gpu_helpers import build_both, check_bh
    src, w, nrm = _cloud(n, n + d)
    q = (2 * np.random.Generator(np.random.PCG64(nq)).random((nq, 3)) - 0.5).astype(np.float32)
    gt, ot = build_both(src, w, nrm, d=d, leaf_size=leaf)
    check_bh(gt, ot, q, kernel, beta, alpha=20.0)


@pytest.mark.parametrize("d", [2, 4])
def test_bh_non_finite_queries_stay_out_of_the_vote(d):
    import paper_2506_02219_amd as P
    src, w, nrm = _cloud(8000, 4)
    rng = np.random.Generator(np.random.PCG64(9))
    q = (rng.random((128, 3)) + 2.0).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    tree = P.sbh_build(dev(src), dev(w), dev(nrm), branching=d)
    bad = q.copy()
    bad[5] = [np.nan, 0.5, 0.5]
    bad[70] = [0.5, np.inf, 0.5]
    keep = np.setdiff1d(np.arange(128), [5, 70])
    for kernel in (0, 1, 2):
        a = P.sbh_eval(tree, dev(q), kernel, beta=1.0, samples=0, alpha=5.0).cpu().numpy()
        b = P.sbh_eval(tree, dev(bad), kernel, beta=1.0, samples=0, alpha=5.0).cpu().numpy()
        assert np.isnan(b[[5, 70]]).all()
        # the others' cut can only be coarser by what queries 5 and 70 opened: every query here is far away
        assert np.allclose(a[keep], b[keep], rtol=1e-6, atol=0)


@pytest.mark.parametrize("d", [2, 4])
@pytest.mark.parametrize("kernel", [0, 1, 2])
@pytest.mark.parametrize("beta", [0.1, 0.3, 0.5, 2.0])
def test_same_values_for_any_number_of_wavefronts(d, kernel, beta):
    """Launches of 1,024 tiles and fewer, of up to 4,096, and of more take different numbers of wavefronts
    a tile; a query's value is the same bit for bit."""
    import paper_2506_02219_amd as P
    rng = np.random.Generator(np.random.PCG64(5))
    n, nq = 20000, 64 * 4200 - 17
    src = torch.from_numpy(rng.random((n, 3)).astype(np.float32)).cuda()
    nrm = torch.from_numpy(rng.standard_normal((n, 3)).astype(np.float32)).cuda()
    q = torch.from_numpy((2 * rng.random((nq, 3)) - 0.5).astype(np.float32)).cuda()
    tree = P.sbh_build(src, torch.ones(n, device="cuda"), nrm, branching=d)
    whole = P.sbh_eval(tree, q, kernel, beta=beta, samples=0)
    for size in (64 * 1024, 64 * 3000):
        parts = torch.cat([P.sbh_eval(tree, c, kernel, beta=beta, samples=0) for c in q.split(size)])
        assert torch.equal(whole.view(torch.int32), parts.view(torch.int32))
