"""The brute-force kernel at the edges of its tiles, shares and queries per lane, against a plain
float64 evaluation of Eq. (1).

Tolerances, in units u = 2^-53 (float64) or 2^-24 (float32): a term takes about a dozen roundings;
a sum of a tile's 64 terms, a wavefront's n / 1024 tiles and 16 partial sums takes at most
80 + n / 1024 + 16 more, each relative to the sum of the absolute terms; both sides are allowed
twice that.  A smooth distance is off by the sum's relative error / alpha and by the distances'
own four roundings, which enter through exp(-alpha r)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cloud(n, nq, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    s = rng.random((n, 3)).astype(np.float32)
    w = (rng.random(n) + 0.5).astype(np.float32)
    nm = rng.standard_normal((n, 3)).astype(np.float32)
    q = (2.0 * rng.random((nq, 3)) - 0.5).astype(np.float32)
    q[0] = s[-1]   # a source at the query
    return s, w, nm, q


def _reference(s, w, nm, q, kernel, eps, alpha):
    """(value, allowed absolute error in units of u) in float64."""
    s, w, nm, q = (a.astype(np.float64) for a in (s, w, nm, q))
    val, tol = np.empty(len(q)), np.empty(len(q))
    roundings = 2.0 * (12 + 80 + len(s) / 1024 + 16)
    for b in range(0, len(q), 4096):
        d = s[None] - q[b:b + 4096, None]
        r2 = (d * d).sum(-1)
        with np.errstate(divide="ignore", invalid="ignore"):
            if kernel == 0:
                t = w / np.sqrt(r2 + float(np.float32(eps)) ** 2)
                val[b:b + 4096], tol[b:b + 4096] = t.sum(1), roundings * t.sum(1)
            elif kernel == 1:
                t = np.where(r2 > 0, w * (nm * d).sum(-1) / (4 * np.pi * r2 * np.sqrt(r2)), 0.0)
                size = np.where(r2 > 0, w * (np.abs(nm * d)).sum(-1) / (4 * np.pi * r2 * np.sqrt(r2)), 0.0)
                val[b:b + 4096], tol[b:b + 4096] = t.sum(1), roundings * size.sum(1)
            else:
                r = np.sqrt(r2)
                m = r.min(1)
                f = (w * np.exp(-alpha * (r - m[:, None]))).sum(1)
                val[b:b + 4096] = m - np.log(f) / alpha
                tol[b:b + 4096] = roundings / alpha + 8.0 * r.max(1) + np.abs(np.log(f)) / alpha
    return val, tol


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kernel", [0, 1, 2])
@pytest.mark.parametrize("n,nq", [(1, 1), (63, 64), (64, 65), (65, 129), (1023, 3), (1024, 70), (1025, 7), (4161, 255),
                                  (97, 64 * 256 * 2 - 1), (66, 64 * 256 * 2), (66, 64 * 256 * 2 + 1),
                                  (33, 64 * 256 * 4 - 3), (70, 64 * 256 * 4 + 193)])
def test_brute_edges(n, nq, kernel, fp64):
    import paper_2506_02219_amd as P
    s, w, nm, q = _cloud(n, nq, 17 * n + nq)
    dev = lambda a: torch.from_numpy(a).cuda()
    out = P.sbh_brute(dev(s), dev(w), dev(nm), dev(q), kernel, eps=1e-3, alpha=20.0, fp64=fp64)
    got = out.cpu().numpy().astype(np.float64)
    val, tol = _reference(s, w, nm, q, kernel, 1e-3, 20.0)
    assert np.isfinite(got).all()
    off = np.abs(got - val) > tol * (2.0 ** -53 if fp64 else 2.0 ** -24)
    assert not off.any(), (np.nonzero(off)[0][:4], got[off][:4], val[off][:4])


@pytest.mark.parametrize("fp64", [False, True])
def test_brute_unsoftened_and_non_finite(fp64):
    """eps = 0: a source at the query is an infinite term; a non-finite query is NaN and leaves the others alone."""
    import paper_2506_02219_amd as P
    s, w, nm, q = _cloud(200, 70, 5)
    q[3] = [np.nan, 0.0, 0.0]
    q[4] = [np.inf, 0.0, 0.0]
    dev = lambda a: torch.from_numpy(a).cuda()
    for kernel in (0, 1, 2):
        got = P.sbh_brute(dev(s), dev(w), dev(nm), dev(q), kernel, eps=0.0, alpha=20.0, fp64=fp64).cpu().numpy()
        val, tol = _reference(s, w, nm, q, kernel, 0.0, 20.0)
        assert np.isnan(got[3:5]).all()
        rest = np.r_[1:3, 5:70]
        assert (np.abs(got[rest] - val[rest]) <= tol[rest] * (2.0 ** -53 if fp64 else 2.0 ** -24)).all()
        assert np.isposinf(got[0]) if kernel == 0 else np.isfinite(got[0])


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("bad", [(64, 128), (0, 64), (100, 101), (0, 200)])
def test_smooth_distance_of_nan_sources(bad, fp64):
    """A NaN source makes every smooth distance NaN, also where all of a wavefront's sources are."""
    import paper_2506_02219_amd as P
    s, w, nm, q = _cloud(200, 70, 6)
    s[bad[0]:bad[1], 1] = np.nan
    dev = lambda a: torch.from_numpy(a).cuda()
    got = P.sbh_brute(dev(s), dev(w), None, dev(q), 2, alpha=20.0, fp64=fp64).cpu().numpy()
    assert np.isnan(got).all()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("n", [1, 70, 1500])
def test_smooth_distance_at_infinite_sharpness(n, fp64):
    """alpha = infinity: the distance to the nearest source (three roundings)."""
    import paper_2506_02219_amd as P
    s, w, nm, q = _cloud(n, 70, 7)
    dev = lambda a: torch.from_numpy(a).cuda()
    got = P.sbh_brute(dev(s), dev(w), None, dev(q), 2, alpha=np.inf, fp64=fp64).cpu().numpy().astype(np.float64)
    r = np.sqrt(((s[None].astype(np.float64) - q[:, None].astype(np.float64)) ** 2).sum(-1)).min(1)
    assert (np.abs(got - r) <= 4 * r * (2.0 ** -53 if fp64 else 2.0 ** -24)).all()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("eps", [0.0, 1e-3])
def test_potential_of_infinitely_far_sources(eps, fp64):
    """A source at infinity, and every source under an infinite softening, adds 0 to the potential."""
    import paper_2506_02219_amd as P
    s, w, nm, q = _cloud(300, 70, 8)
    dev = lambda a: torch.from_numpy(a).cuda()
    near = np.ones(300, bool)
    near[[5, 64, 130]] = False
    s[5, 0], s[64], s[130, 2] = np.inf, -np.inf, -np.inf
    got = P.sbh_brute(dev(s), dev(w), None, dev(q), 0, eps=eps, fp64=fp64).cpu().numpy().astype(np.float64)
    val, tol = _reference(s[near], w[near], nm[near], q, 0, eps, 20.0)
    fin = np.isfinite(val)   # (without softening a source at the query is infinite)
    assert (np.abs(got[fin] - val[fin]) <= tol[fin] * (2.0 ** -53 if fp64 else 2.0 ** -24)).all()
    assert np.isposinf(got[~fin]).all()
    s[5, 1] = np.nan
    assert np.isnan(P.sbh_brute(dev(s), dev(w), None, dev(q), 0, eps=eps, fp64=fp64).cpu().numpy()).all()
    assert (P.sbh_brute(dev(s[near]), dev(w[near]), None, dev(q), 0, eps=np.inf, fp64=fp64).cpu().numpy() == 0.0).all()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kernel", [0, 1, 2])
@pytest.mark.parametrize("n,nq", [(64, 70001), (65, 100001), (500, 524289), (1500, 262145), (4161, 262145)])
def test_same_values_for_any_number_of_wavefronts(n, nq, kernel, fp64):
    """One, four and sixteen wavefronts share the sources, one to four queries a lane: a query's value is the
    same bit for bit."""
    import paper_2506_02219_amd as P
    s, w, nm, q = _cloud(n, nq, n)
    dev = lambda a: torch.from_numpy(a).cuda()
    src, qd = (dev(s), dev(w), dev(nm)), dev(q)
    whole = P.sbh_brute(*src, qd, kernel, alpha=20.0, fp64=fp64)
    as_int = torch.int64 if fp64 else torch.int32
    for first, m in ((0, 130), (nq - 40000, 40000)):
        part = P.sbh_brute(*src, qd[first:first + m].contiguous(), kernel, alpha=20.0, fp64=fp64)
        assert torch.equal(whole[first:first + m].view(as_int), part.view(as_int))
