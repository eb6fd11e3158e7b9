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
