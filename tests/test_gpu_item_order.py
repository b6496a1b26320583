"""Work items in order of their work, counted by amount (at most 256 different amounts) or sorted (more): a
target's sum does not depend on where its item stands, so a batch gives the same bits with its systems in
another order."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _dev(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("systems,same", [(7, True), (60, True), (60, False), (300, False)])
def test_order_of_systems(systems, same, prec):
    from paper_2409_04215_amd import mfs
    rg = np.random.default_rng(191)
    n_body = rg.integers(1, 6, systems)
    X, Y, f, nt, ns = [], [], [], [], []
    for s in range(systems):
        m, n = (130, 40) if same else rg.integers(65, 400, 2)
        cen = 3.0 * np.arange(n_body[s])[:, None] * np.array([1.0, 0.2, 0.1])
        X.append(np.repeat(cen, m, axis=0) + rg.standard_normal((n_body[s] * m, 3)) * 0.3 + 1.0)
        Y.append(np.repeat(cen, n, axis=0) + rg.standard_normal((n_body[s] * n, 3)) * 0.1)
        f.append(rg.standard_normal((n_body[s] * n, 3)))
        nt.append(np.full(n_body[s], m))
        ns.append(np.full(n_body[s], n))

    def run(order):
        cat = lambda a: np.concatenate([a[s] for s in order])  # noqa: E731
        ptr = lambda a: np.concatenate([[0], np.cumsum(a)])  # noqa: E731
        out = mfs.p2p_stokes(ptr(n_body[order]), ptr(cat(nt)), ptr(cat(ns)), _dev(cat(X)), _dev(cat(Y)), _dev(cat(f)),
                             prec=prec, out=torch.full((len(cat(X)), 3), float("nan"), dtype=torch.float64, device="cuda"))
        return dict(zip(order, torch.split(out, [len(X[s]) for s in order])))
    a, b = run(np.arange(systems)), run(np.arange(systems)[::-1])
    for s in range(systems):
        assert torch.isfinite(a[s]).all() and torch.equal(a[s], b[s]), s
