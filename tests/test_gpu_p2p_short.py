"""Short mixed pair sums in one launch (16 waves share the sources of a system) at the sizes where
the walk over bodies changes: one body and one source, more waves than sources, bodies without
sources or targets, more than 64 bodies (a wave's sources are found in blocks of 64), blocks of 64
targets cut short, several systems, and 256 / 257 blocks (the last that go this way and the first
that do not); and an output in the place of an input.

Tolerance: 4 x the error of the float32 model (oracle/fp32_model.py) of the same sum."""
import numpy as np
import pytest
import torch

from oracle import fp32_model as M
from oracle import mfs_oracle as O
from tests._helpers import rel_inf

pytestmark = pytest.mark.gpu


def _dev(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _points(sizes, n_trg, n_src, seed):
    """Bodies on a grid of unit spheres 2.5 apart; n_trg and n_src are cycled through over the bodies."""
    rg = np.random.default_rng(seed)
    nb = sum(sizes)
    side = int(np.ceil(nb ** (1 / 3)))
    cen = 2.5 * np.stack(np.unravel_index(np.arange(nb), (side,) * 3), axis=1).astype(float)
    nt = np.array([n_trg[b % len(n_trg)] for b in range(nb)])
    ns = np.array([n_src[b % len(n_src)] for b in range(nb)])
    tb, sb = np.repeat(np.arange(nb), nt), np.repeat(np.arange(nb), ns)

    def sphere(k, r):
        v = rg.standard_normal((k, 3))
        return r * v / np.linalg.norm(v, axis=1, keepdims=True)
    X, Y = cen[tb] + sphere(len(tb), 1.0), cen[sb] + sphere(len(sb), 0.7)
    geo = (np.concatenate([[0], np.cumsum(sizes)]), np.concatenate([[0], np.cumsum(nt)]),
           np.concatenate([[0], np.cumsum(ns)]))
    return geo, X, tb, Y, sb, rg


@pytest.mark.parametrize("kind", [O.STOKES, O.LAPLACE])
@pytest.mark.parametrize("skip", [True, False])
@pytest.mark.parametrize("sizes,n_trg,n_src", [
    ((1,), (1,), (1,)), ((2,), (65,), (3,)), ((4,), (600,), (300,)), ((5,), (63, 0, 64), (40, 17, 0)),
    ((130,), (7,), (5, 0)), ((65,), (3,), (2,)), ((1, 3, 2), (130,), (77,)), ((32,), (512,), (20,)),
    ((33,), (512,), (20,)), ((2,), (90,), (257,))])
def test_short_sums(sizes, n_trg, n_src, skip, kind):
    from paper_2409_04215_amd import mfs
    geo, X, tb, Y, sb, rg = _points(sizes, n_trg, n_src, 41)
    s = rg.standard_normal((len(Y), 3) if kind == O.STOKES else len(Y))
    f = mfs.p2p_stokes if kind == O.STOKES else mfs.p2p_laplace
    args = [*geo, _dev(X), _dev(Y), _dev(s)]
    flags = mfs.SKIP_SAME_BODY if skip else 0
    got = f(*args, flags=flags, prec=mfs.MIXED).cpu().numpy()
    ref_pts = M.ref_first_source(sum(sizes), sb, Y, tb, X)
    for y in range(len(sizes)):
        b0, b1 = geo[0][y], geo[0][y + 1]
        t, q = slice(geo[1][b0], geo[1][b1]), slice(geo[2][b0], geo[2][b1])
        model = {dt: M.pair_sum(kind, X[t], tb[t], Y[q], sb[q], s[q], ref_pts, skip, dt=dt)
                 for dt in (np.float32, np.float64)}
        if not model[np.float64].any():  # nothing to add up
            assert not got[t].any()
            continue
        bar = M.bar(rel_inf(model[np.float32], model[np.float64]), 6e-8)
        e = rel_inf(got[t], model[np.float64])
        print(f"kind={kind} sizes={sizes} sys={y} skip={skip} err={e:.2e} bar={bar:.2e}")
        assert e <= bar
    base = rg.standard_normal(got.shape)
    more = f(*args, flags=flags | mfs.ACCUMULATE, prec=mfs.MIXED, out=_dev(base)).cpu().numpy()
    assert np.array_equal(more, base + got)


@pytest.mark.parametrize("kind", [O.STOKES, O.LAPLACE])
def test_output_in_place_of_the_strengths(kind):
    from paper_2409_04215_amd import mfs
    geo, X, tb, Y, sb, rg = _points((4,), (120,), (120,), 43)
    s = rg.standard_normal((len(Y), 3) if kind == O.STOKES else len(Y))
    f = mfs.p2p_stokes if kind == O.STOKES else mfs.p2p_laplace
    apart = f(*geo, _dev(X), _dev(Y), _dev(s), prec=mfs.MIXED).cpu().numpy()
    buf = _dev(s)
    f(*geo, _dev(X), _dev(Y), buf, prec=mfs.MIXED, out=buf)
    # both errors are those of FP32 sums of the same terms
    assert rel_inf(buf.cpu().numpy(), apart) <= 1e-6


@pytest.mark.parametrize("skip", [True, False])
@pytest.mark.parametrize("n_src", [1, 3, 255, 256, 257, 300])
@pytest.mark.parametrize("bodies,n_trg", [(3, 5483), (5, 3290)])
def test_stokes_sources_through_lds(bodies, n_trg, n_src, skip):
    """258 blocks of 64 targets: 774 work items take their sources through LDS, 1290 by scalar loads; quarters of a
    body of one source, of none, and on both sides of the run of 64."""
    from paper_2409_04215_amd import mfs
    geo, X, tb, Y, sb, rg = _points((bodies,), (n_trg,), (n_src,), 45)
    s = rg.standard_normal((len(Y), 3))
    got = mfs.p2p_stokes(*geo, _dev(X), _dev(Y), _dev(s), flags=mfs.SKIP_SAME_BODY if skip else 0,
                         prec=mfs.MIXED).cpu().numpy()
    ref_pts = M.ref_first_source(bodies, sb, Y, tb, X)
    rows = np.unique(np.concatenate([rg.integers(0, len(X), 200), [0, len(X) - 1]]))
    model = {dt: M.pair_sum(O.STOKES, X[rows], tb[rows], Y, sb, s, ref_pts, skip, dt=dt) for dt in (np.float32, np.float64)}
    bar = M.bar(rel_inf(model[np.float32], model[np.float64]), 6e-8)
    e = rel_inf(got[rows], model[np.float64])
    print(f"bodies={bodies} n_src={n_src} skip={skip} err={e:.2e} bar={bar:.2e}")
    assert e <= bar
