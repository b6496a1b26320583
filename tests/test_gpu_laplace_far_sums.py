"""What a mixed Laplace sum with far tiles carries in FP32: never more than one body's sources, and for a
body near the targets never more than a quarter of it, as the walk without far tiles.

Two sets of very large strengths at the same points cancel: between bodies that lie at the same place, and
between the first and the third quarter of one body.  Every set is added to FP64 by itself, so the two
cancel there exactly (the same points, the opposite strengths) and the sum errs as the sum of the other
strengths does; a value carried in FP32 past them loses 2^-24 of their size.

Tolerance: 4 x the error of the float32 model (oracle/fp32_model.py) of the sum of the other strengths."""
import numpy as np
import pytest
import torch

from oracle import fp32_model as M
from oracle import mfs_oracle as O
from tests._helpers import rel_inf

pytestmark = pytest.mark.gpu

BODIES, N, TRG = 120, 100, 200  # 2.9e8 pairs, 375 blocks of 64 targets, 7 tiles of 16 sources a body
LARGE = 1e4


def _dev(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _cloud(seed, same=None):
    rg = np.random.default_rng(seed)
    cen = 3.0 * np.stack(np.unravel_index(np.arange(BODIES), (5,) * 3), axis=1).astype(float)

    def sphere(k, r):
        v = rg.standard_normal((BODIES, k, 3))
        return r * v / np.linalg.norm(v, axis=2, keepdims=True)
    src, trg = cen[:, None] + sphere(N, 0.7), cen[:, None] + sphere(TRG, 1.0)
    if same:
        src[same[1]] = src[same[0]]
    return rg, trg.reshape(-1, 3), src.reshape(-1, 3)


def _check(rg, X, Y, small, large, rows):
    from paper_2409_04215_amd import mfs
    geo = ([0, BODIES], np.arange(BODIES + 1) * TRG, np.arange(BODIES + 1) * N)
    got = mfs.p2p_laplace(*geo, _dev(X), _dev(Y), _dev(small + large), flags=0, prec=mfs.MIXED).cpu().numpy()
    tb, sb = np.repeat(np.arange(BODIES), TRG), np.repeat(np.arange(BODIES), N)
    ref_pts = M.ref_first_source(BODIES, sb, Y, tb, X)
    model = {dt: M.pair_sum(O.LAPLACE, X[rows], tb[rows], Y, sb, small, ref_pts, False, dt=dt)
             for dt in (np.float32, np.float64)}
    e, bar = rel_inf(got[rows], model[np.float64]), M.bar(rel_inf(model[np.float32], model[np.float64]))
    print(f"err={e:.2e} bar={bar:.2e}")
    assert e <= bar


@pytest.mark.parametrize("first,second", [(60, 61), (60, 64), (3, 116)])
def test_bodies_cancel(first, second):
    rg, X, Y = _cloud(71, same=(first, second))
    small = rg.standard_normal(BODIES * N)
    large = np.zeros((BODIES, N))
    large[first] = LARGE * rg.standard_normal(N)
    large[second] = -large[first]
    small.reshape(BODIES, N)[[first, second]] = 0.0
    _check(rg, X, Y, small, large.reshape(-1), np.unique(rg.integers(0, BODIES * TRG, 300)))


def test_quarters_cancel():
    b = 57
    rg, X, Y = _cloud(72)
    Y[b * N + 50] = Y[b * N]
    small = rg.standard_normal((BODIES, N))
    small[b, :25] = 0.0  # alone with the first large strength in the first quarter
    small[b, 49:75] = 0.0  # and with the second one in the third, and in a lane of the tiles
    large = np.zeros((BODIES, N))
    large[b, 0], large[b, 50] = LARGE, -LARGE
    rows = np.unique(np.concatenate([np.arange(b * TRG, (b + 1) * TRG), rg.integers(0, BODIES * TRG, 100)]))
    _check(rg, X, Y, small.reshape(-1), large.reshape(-1), rows)
