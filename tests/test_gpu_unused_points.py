"""Standalone calls whose body arrays name more bodies than the systems use (a subset of the systems over
the full point arrays): the points of the bodies left out stay zero, whatever the memory of the new output
held before, and the others are the sums of the systems given."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, M_, BODIES, USED = 40, 90, 6, 4  # the systems use the first 4 of 6 bodies


def _dev(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _stale(*shapes):
    """Leaves blocks of these shapes, filled with NaN, to the allocator's next requests of their sizes."""
    torch.cuda.synchronize()
    blocks = [torch.full(s, float("nan"), dtype=torch.float64, device="cuda") for s in shapes for _ in range(3)]
    torch.cuda.synchronize()
    del blocks


def _calls():
    from paper_2409_04215_amd import mfs
    rg = np.random.default_rng(61)
    cen = 3.0 * np.arange(BODIES)[:, None] * np.array([1.0, 0.3, 0.1])

    def sphere(k, r):
        v = rg.standard_normal((BODIES * k, 3))
        return np.repeat(cen, k, axis=0) + r * v / np.linalg.norm(v, axis=1, keepdims=True)
    X, Y, nv = _dev(sphere(M_, 1.0)), _dev(sphere(N, 0.7)), _dev(rg.standard_normal((BODIES * M_, 3)))
    f, q = _dev(rg.standard_normal((BODIES * N, 3))), _dev(rg.standard_normal(BODIES * N))
    w3, w1 = _dev(rg.standard_normal((BODIES * M_, 3))), _dev(rg.standard_normal(BODIES * M_))
    geo = ([0, 2, USED], np.arange(BODIES + 1) * M_, np.arange(BODIES + 1) * N)
    used = (geo[0], geo[1][:USED + 1], geo[2][:USED + 1])
    return geo, used, {
        "p2p_laplace": lambda g, **k: mfs.p2p_laplace(*g, X, Y, q, **k),
        "p2p_stokes": lambda g, **k: mfs.p2p_stokes(*g, X, Y, f, **k),
        "p2p_stokes_noalloc": lambda g, **k: mfs.p2p_stokes_noalloc(*g, X, Y, f, **k),
        "p2p_stokes_pressure": lambda g, **k: mfs.p2p_stokes_pressure(*g, X, Y, f, **k),
        "p2p_stokes_traction": lambda g, **k: mfs.p2p_stokes_traction(*g, X, nv, Y, f, **k),
        "p2p_laplace_gradient": lambda g, **k: mfs.p2p_laplace_gradient(*g, X, Y, q, **k),
        "p2p_laplace_backward": lambda g, **k: mfs.p2p_laplace_backward(*g, X, Y, q, w1, **k),
        "p2p_stokes_backward": lambda g, **k: mfs.p2p_stokes_backward(*g, X, Y, f, w3, **k)}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", ["p2p_laplace", "p2p_stokes", "p2p_stokes_noalloc", "p2p_stokes_pressure",
                                  "p2p_stokes_traction", "p2p_laplace_gradient", "p2p_laplace_backward",
                                  "p2p_stokes_backward"])
def test_points_of_bodies_left_out_are_zero(name, prec):
    geo, used, calls = _calls()
    want = calls[name](used, prec=prec)  # shorter body arrays: the outputs are larger than the structure
    _stale((BODIES * M_,), (BODIES * M_, 3), (BODIES * N,), (BODIES * N, 3))
    got = calls[name](geo, prec=prec)
    for g, r in zip(got if isinstance(got, tuple) else (got,), want if isinstance(want, tuple) else (want,)):
        per = M_ if len(g) == BODIES * M_ else N
        assert torch.count_nonzero(g[USED * per:]).item() == 0, f"{name}: points past the structure hold old values"
        assert torch.equal(g, r)
