"""Mixed Laplace sums on the matrix cores (bodies far from a block of targets), at the sizes where
their walk begins, ends and has remainders: 31 / 32 bodies, whole and ragged tiles of 16 sources,
1024 / 1025 sources per body, too much padding, blocks of 256 targets cut short, systems below the
limit beside one above it, and values that are not finite.

Tolerance: 4 x the error of the float32 model (oracle/fp32_model.py) of the same sum on the same
rows, as in tests/test_gpu_p2p.py; the model takes the differences of the rounded coordinates, whose
rounding is no smaller than that of the expanded square."""
import numpy as np
import pytest
import torch

import mfs_workloads as W
from oracle import fp32_model as M
from oracle import mfs_oracle as O
from tests._helpers import rel_inf

pytestmark = pytest.mark.gpu


def _dev(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _suspension(sizes, n, m, seed, aspect=2.0):
    """Spheroids of n sources and m targets in systems of the given numbers of bodies."""
    rg = np.random.default_rng(seed)
    unit = np.ones(3)
    cen = [W.random_cluster(rg, p, unit, W.cube_side(p, unit), 0.1)[0] + 50.0 * s for s, p in enumerate(sizes)]
    nb = sum(sizes)
    return W.Workload("far", [W.spheroid_shape(1.0 / aspect, 1.0, n, m)], np.concatenate(cen),
                      np.stack([W.random_rotation(rg) for _ in range(nb)]), np.zeros(nb, np.int32),
                      np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64),
                      np.full(len(sizes), W.LAPLACE, np.int32), [rg.standard_normal(p) for p in sizes])


def _sum(geo, X, Y, q, flags, **kw):
    from paper_2409_04215_amd import mfs
    return mfs.p2p_laplace(*geo, _dev(X), _dev(Y), _dev(q), flags, mfs.MIXED, **kw).cpu().numpy()


@pytest.mark.parametrize("skip", [True, False])
@pytest.mark.parametrize("sizes,n,m", [
    ((31,), 400, 800), ((32,), 400, 800), ((32,), 320, 763), ((33,), 257, 1001), ((34,), 1024, 231),
    ((34,), 1025, 231), ((150,), 26, 601), ((150,), 20, 601), ((3, 40, 1, 33), 383, 409)])
def test_laplace_far_sizes(sizes, n, m, skip):
    from paper_2409_04215_amd import mfs
    wl = _suspension(sizes, n, m, 31)
    X, _ = wl.world_points("trg")
    Y, _ = wl.world_points("src")
    nb = wl.n_body
    tb, sb = np.repeat(np.arange(nb), m), np.repeat(np.arange(nb), n)
    rg = np.random.default_rng(32)
    X[m:2 * m] = X[2 * m:3 * m] * 0.999 + 0.001  # targets of one body beside another's surface
    q = rg.standard_normal(len(Y))
    geo = (wl.sys_body_ptr, np.arange(nb + 1) * m, np.arange(nb + 1) * n)
    got = _sum(geo, X, Y, q, mfs.SKIP_SAME_BODY if skip else 0)
    ref_pts = M.ref_first_source(nb, sb, Y, tb, X)
    for s in range(len(sizes)):
        b0, b1 = int(wl.sys_body_ptr[s]), int(wl.sys_body_ptr[s + 1])
        rows = np.unique(np.concatenate([rg.integers(b0 * m, b1 * m, 60), [b0 * m, b1 * m - 1],
                                         np.arange(m, m + 20) if s == 0 else []]).astype(int))
        src = slice(b0 * n, b1 * n)
        model = {dt: M.pair_sum(O.LAPLACE, X[rows], tb[rows], Y[src], sb[src], q[src], ref_pts, skip, dt=dt)
                 for dt in (np.float32, np.float64)}
        bar = M.bar(rel_inf(model[np.float32], model[np.float64]))
        e = rel_inf(got[rows], model[np.float64])
        print(f"sizes={sizes} n={n} m={m} sys={s} skip={skip} err={e:.2e} bar={bar:.2e}")
        assert e <= bar or (skip and b1 - b0 == 1 and not got[rows].any())


def test_laplace_far_accumulate_and_not_finite():
    from paper_2409_04215_amd import mfs
    n, m, nb = 389, 777, 33
    wl = _suspension((nb,), n, m, 33)
    X, _ = wl.world_points("trg")
    Y, _ = wl.world_points("src")
    q = np.random.default_rng(34).standard_normal(len(Y))
    geo = (wl.sys_body_ptr, np.arange(nb + 1) * m, np.arange(nb + 1) * n)
    base = _sum(geo, X, Y, q, mfs.SKIP_SAME_BODY)
    assert np.isfinite(base).all()
    twice = _sum(geo, X, Y, q, mfs.SKIP_SAME_BODY | mfs.ACCUMULATE, out=_dev(base))
    assert rel_inf(twice, 2 * base) <= 1e-15  # the same values, added in FP64
    own = slice(5 * m, 6 * m)
    others = np.ones(len(X), bool)
    others[own] = False
    for bad in (np.nan, np.inf):
        Xb = X.copy()
        Xb[7 * m + 3, 1] = bad
        got = _sum(geo, Xb, Y, q, mfs.SKIP_SAME_BODY)
        keep = np.arange(len(X)) != 7 * m + 3
        assert np.isnan(got[~keep]).all() if np.isnan(bad) else not np.isfinite(got[~keep]).any() or (got[~keep] == 0).all()
        assert rel_inf(got[keep], base[keep]) <= 1e-6  # the block's bodies take the other walk
        qb = q.copy()
        qb[5 * n + 17] = bad  # reaches every target but its own body's
        got = _sum(geo, X, Y, qb, mfs.SKIP_SAME_BODY)
        assert not np.isfinite(got[others]).any() and np.array_equal(got[own], base[own])
    Yb = Y.copy()
    Yb[5 * n + 17, 2] = np.nan
    got = _sum(geo, X, Yb, q, mfs.SKIP_SAME_BODY)
    assert np.isnan(got[others]).all() and np.isfinite(got[own]).all()


def test_laplace_far_plan():
    """matvec and adjoint of a mixed plan, its FP64 products beside them, and moved bodies."""
    from paper_2409_04215_amd import mfs
    wl = _suspension((34,), 385, 770, 35)
    pr = O.Problem.from_workload(wl)
    rg = np.random.default_rng(36)
    x, w = rg.standard_normal(pr.n_gamma), rg.standard_normal(pr.n_gamma)
    plan, plan64 = mfs.Plan.from_workload(wl, mfs.MIXED), mfs.Plan.from_workload(wl, mfs.FP64)
    ref = plan64.matvec(_dev(x)).cpu().numpy()
    y = plan.matvec(_dev(x)).cpu().numpy()
    rows = np.unique(rg.integers(0, pr.n_gamma, 100))
    bar = M.bar(rel_inf(M.matvec(pr, x, rows=rows), ref[rows]))
    e = rel_inf(y, ref)
    z = plan.matvec_adjoint(_dev(w)).cpu().numpy()
    gap = abs(w @ y - z @ x) / (np.linalg.norm(w) * np.linalg.norm(y))
    print(f"matvec err={e:.2e} bar={bar:.2e} adjoint gap={gap:.2e}")
    assert e <= bar and gap <= 2 * bar
    # the FP64 product of the mixed plan walks the general items
    assert rel_inf(plan.matvec(_dev(x), prec=mfs.FP64).cpu().numpy(), ref) <= 1e-12
    rot = np.stack([W.random_rotation(rg) for _ in range(wl.n_body)])
    plan.set_bodies(wl.centre * 1.1, rot)
    wl.centre, wl.rot = wl.centre * 1.1, rot
    fresh = mfs.Plan.from_workload(wl, mfs.MIXED)
    assert torch.equal(plan.matvec(_dev(x)), fresh.matvec(_dev(x)))
    for p in (plan, plan64, fresh):
        p.close()
