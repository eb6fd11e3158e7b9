"""Training targets at the sizes where children pass between one wavefront and the whole workgroup,
and on paths cut short, against a float64 evaluation over the exported tree's points.

Tolerance: a target is r_c / sum r, r_c = |sum of the child's terms - the child's aggregate term|.
Every term takes at most about 20 float64 roundings and every sum at most log2-many more than its
length over 64, so r_c is off by at most e = 2^-53 (64 + n / 64) times the node's sum of absolute
terms on each side, a target by 2 (8 + 1) e / sum r, plus the final rounding to float32."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _term(p, w, dip, q, kernel, eps, alpha):
    d = p - q
    r2 = (d * d).sum(-1)
    with np.errstate(divide="ignore", invalid="ignore"):
        if kernel == 0:
            return w / np.sqrt(r2 + float(np.float32(eps)) ** 2)
        if kernel == 1:
            return np.where(r2 > 0, (dip * d).sum(-1) / (4 * np.pi * r2 * np.sqrt(r2)), 0.0)
    return w * np.exp(-alpha * np.sqrt(r2))


@pytest.mark.parametrize("kernel,eps", [(0, 1e-3), (0, 0.0), (1, 1e-3), (2, 1e-3)])
@pytest.mark.parametrize("n,side,depth", [(131072, 1.0, None), (40000, 1.0, 2), (17000, 0.02, None), (300, 1.0, 1)])
def test_targets_match_the_points(n, side, depth, kernel, eps):
    """Uniform cubes: 131,072 points give subdomains of about 16,384 whose children hold about 2,048."""
    import paper_2506_02219_amd as P
    rng = np.random.Generator(np.random.PCG64(n))
    src = (side * rng.random((n, 3))).astype(np.float32)
    if n == 17000:
        src[:5000] = src[0]   # one deepest cell with thousands of points
    w = (rng.random(n) + 0.5).astype(np.float32)
    nrm = rng.standard_normal((n, 3)).astype(np.float32)
    q = (side * (2 * rng.random((6, 3)) - 0.5)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()
    tree = P.sbh_build(dev(src), dev(w), dev(nrm))
    alpha = 5.0
    X, Tg, Cn, where = P.sbh_mlp_pairs(tree, dev(q), kernel, seed=3, max_depth=depth, eps=eps, alpha=alpha)
    Tg, Cn, where = Tg.cpu().numpy(), Cn.cpu().numpy(), where.cpu().numpy()
    a = tree.export()
    perm = a["perm"].astype(np.int64)
    pts, pw = src[perm].astype(np.float64), w[perm].astype(np.float64)
    dip = (w[:, None] * nrm)[perm].astype(np.float64)
    node_of = {(int(b), int(c)): i for i, (b, c) in enumerate(zip(a["begin"], a["count"]))}   # the deepest of equal ranges
    per_query = where.shape[0] // len(q)
    checked = 0
    for row in np.nonzero(where[:, 0] >= 0)[0]:
        qq = q[row // per_query].astype(np.float64)
        b, nt, level = int(where[row, 1]), int(where[row, 2]), int(where[row, 3])
        t = _term(pts[b:b + nt], pw[b:b + nt], dip[b:b + nt], qq, kernel, eps, alpha)
        cnt = Cn[row].astype(np.int64)
        assert cnt.sum() == nt
        r, lo = np.zeros(8), 0
        for c in range(8):
            if cnt[c]:
                i = node_of[(b + lo, int(cnt[c]))]
                while a["level"][i] > level + 1:
                    i = a["parent"][i]
                agg = a["agg"][i].astype(np.float64)
                r[c] = abs(t[lo:lo + cnt[c]].sum() - _term(agg[:3], agg[3], a["dip"][i, :3].astype(np.float64), qq, kernel, eps, alpha))
            lo += cnt[c]
        e = 2.0 ** -53 * (64 + nt / 64) * np.abs(t).sum()
        if r.sum() <= 100 * e:
            continue   # residuals below their own rounding
        off = np.abs(Tg[row] - r / r.sum())
        assert (off <= 18 * e / r.sum() + 2.0 ** -24).all(), (row, off.max(), 18 * e / r.sum())
        checked += 1
    assert checked >= 10
    assert (Tg[where[:, 0] < 0] == 0).all()


@pytest.mark.parametrize("kernel,eps", [(0, 1e-3), (0, 0.0), (1, 1e-3), (2, 1e-3)])
@pytest.mark.parametrize("n", [300, 40000, 150000])
def test_same_targets_for_any_number_of_wavefronts(n, kernel, eps):
    """Few and many queries take different numbers of wavefronts a path (40,000 points: children that the
    wavefronts share and others): a row's targets are the same bit for bit."""
    import paper_2506_02219_amd as P
    rng = np.random.Generator(np.random.PCG64(n))
    src = rng.random((n, 3)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    tree = P.sbh_build(dev(src), dev(rng.random(n) + 0.5), dev(rng.standard_normal((n, 3))))
    q = dev(2 * rng.random((600, 3)) - 0.5)
    whole = P.sbh_mlp_pairs(tree, q, kernel, seed=3, eps=eps, alpha=5.0)[1]
    for m in (5, 100):   # rows are keyed by the query's index, so the first ones are the same
        part = P.sbh_mlp_pairs(tree, q[:m].contiguous(), kernel, seed=3, eps=eps, alpha=5.0)[1]
        assert torch.equal(whole[:len(part)].view(torch.int32), part.view(torch.int32))
