"""Standalone mixed Laplace sums at structures that the rules of two walks both accept: at most 256 blocks
of 64 targets (short sums, 16 waves on 64 targets) and at least 32 bodies with 2.5e8 pairs (far tiles,
items of 256 targets), and at their neighbours that only one of them accepts.  Outputs are filled with NaN
before the call: every target has to be written.

Tolerance: 4 x the error of the float32 model (oracle/fp32_model.py) of the same sum on the same rows."""
import numpy as np
import pytest
import torch

from oracle import fp32_model as M
from oracle import mfs_oracle as O
from tests._helpers import rel_inf

pytestmark = pytest.mark.gpu


def _dev(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _points(sizes, m, n, seed):
    rg = np.random.default_rng(seed)
    nb = sum(sizes)
    side = int(np.ceil(nb ** (1 / 3)))
    cen = 2.5 * np.stack(np.unravel_index(np.arange(nb), (side,) * 3), axis=1).astype(float)

    def sphere(k, r):
        v = rg.standard_normal((k, 3))
        return r * v / np.linalg.norm(v, axis=1, keepdims=True)
    X, Y = np.repeat(cen, m, axis=0) + sphere(nb * m, 1.0), np.repeat(cen, n, axis=0) + sphere(nb * n, 0.7)
    geo = (np.concatenate([[0], np.cumsum(sizes)]), np.arange(nb + 1) * m, np.arange(nb + 1) * n)
    return geo, X, np.repeat(np.arange(nb), m), Y, np.repeat(np.arange(nb), n), rg


@pytest.mark.parametrize("skip", [True, False])
@pytest.mark.parametrize("sizes,m,n", [((32,), 512, 500), ((32,), 512, 480), ((32,), 513, 500), ((199,), 82, 84),
                                       ((40,), 409, 390), ((40, 40), 204, 400)])
def test_laplace_both_rules(sizes, m, n, skip):
    from paper_2409_04215_amd import mfs
    geo, X, tb, Y, sb, rg = _points(sizes, m, n, 51)
    q = rg.standard_normal(len(Y))
    out = torch.full((len(X),), float("nan"), dtype=torch.float64, device="cuda")
    mfs.p2p_laplace(*geo, _dev(X), _dev(Y), _dev(q), flags=mfs.SKIP_SAME_BODY if skip else 0, prec=mfs.MIXED, out=out)
    got = out.cpu().numpy()
    assert np.isfinite(got).all(), f"{np.isnan(got).sum()} of {len(got)} targets unwritten"
    ref_pts = M.ref_first_source(sum(sizes), sb, Y, tb, X)
    for s in range(len(sizes)):
        b0, b1 = geo[0][s], geo[0][s + 1]
        rows = np.unique(np.concatenate([rg.integers(b0 * m, b1 * m, 150), np.arange(b0 * m, b0 * m + 256, 37),
                                         np.arange(b1 * m - 256, b1 * m, 37), [b1 * m - 1]]))
        src = slice(b0 * n, b1 * n)
        model = {dt: M.pair_sum(O.LAPLACE, X[rows], tb[rows], Y[src], sb[src], q[src], ref_pts, skip, dt=dt)
                 for dt in (np.float32, np.float64)}
        bar = M.bar(rel_inf(model[np.float32], model[np.float64]))
        e = rel_inf(got[rows], model[np.float64])
        print(f"sizes={sizes} m={m} n={n} sys={s} skip={skip} err={e:.2e} bar={bar:.2e}")
        assert e <= bar


def test_laplace_strength_gradient_both_rules():
    """The strength gradient alone is the same sum with the roles of targets and sources swapped."""
    from paper_2409_04215_amd import mfs
    geo, X, tb, Y, sb, rg = _points((32,), 500, 512, 52)
    w = rg.standard_normal(len(X))
    grad = mfs.p2p_laplace_backward(*geo, _dev(X), _dev(Y), _dev(rg.standard_normal(len(Y))), _dev(w), want=("src",),
                                    flags=mfs.ACCUMULATE, prec=mfs.MIXED)[0].cpu().numpy()
    rows = np.unique(np.concatenate([rg.integers(0, len(Y), 200), np.arange(len(Y) - 256, len(Y), 37)]))
    ref_pts = M.ref_first_source(32, tb, X)
    model = {dt: M.pair_sum(O.LAPLACE, Y[rows], sb[rows], X, tb, w, ref_pts, False, dt=dt)
             for dt in (np.float32, np.float64)}
    e, bar = rel_inf(grad[rows], model[np.float64]), M.bar(rel_inf(model[np.float32], model[np.float64]))
    print(f"err={e:.2e} bar={bar:.2e}")
    assert e <= bar
