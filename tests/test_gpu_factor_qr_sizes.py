"""QR set-up at the sizes where its kernels change: rows at and beside the
multiples of 512 (rows per thread of the register-resident steps), at and
beyond 2560 (the last size they take), columns at and beside the panel width
16, and single panels.  The S_L^+ apply of a QR plan against the oracle's, with
the bar of tests/test_gpu_factor_qr.py (4 x the error of an independent FP64 QR
in oracle/fp32_model.py)."""
import numpy as np
import pytest
import torch
from scipy.linalg import solve_triangular

import mfs_workloads as W
from oracle import fp32_model as M
from oracle import mfs_oracle as O
from tests._helpers import rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,m", [
    (W.LAPLACE, 1, 1), (W.LAPLACE, 15, 20), (W.LAPLACE, 16, 511), (W.LAPLACE, 17, 512), (W.LAPLACE, 32, 513),
    (W.LAPLACE, 33, 1024), (W.LAPLACE, 40, 1025), (W.LAPLACE, 47, 2048), (W.LAPLACE, 49, 2049), (W.LAPLACE, 64, 2560),
    (W.LAPLACE, 31, 2561), (W.STOKES, 5, 171), (W.STOKES, 16, 853), (W.STOKES, 11, 854), (W.STOKES, 200, 220)])
def test_qr_sizes(kind, n, m):
    from paper_2409_04215_amd import mfs
    wl = W.small_cluster(2, kind, n, m, seed=171)
    pr = O.Problem.from_workload(wl)
    g = W.random_vector(pr.n_gamma, 172)
    ref = np.concatenate([pr.pinv_apply(k, pr.gblock(g, k)) for k in range(wl.n_body)])
    bar = M.bar(rel_inf(M.precond_apply(pr, g, qr=True, dt=np.float64), ref))
    plan = mfs.Plan.from_workload(wl, mfs.FP64, factorization=mfs.FACTOR_QR)
    got = plan.precond_apply(torch.tensor(g, dtype=torch.float64, device="cuda"), 0, mfs.FP64).cpu().numpy()
    plan.close()
    e = rel_inf(got, ref)
    print(f"kind={kind} n={n} m={m} err={e:.2e} bar={bar:.2e}")
    assert e <= bar


@pytest.mark.parametrize("n,m", [(513, 1025), (1025, 1537), (1537, 2560), (2049, 2560)])
def test_qr_many_columns(n, m):
    """Columns at the edges of the rows per thread of R^-1: the strengths from S_L c on one body, with the bar of a
    float64 Householder QR and explicit R^-1 (4 x its error)."""
    from paper_2409_04215_amd import mfs
    wl = W.small_cluster(1, W.LAPLACE, n, m, seed=173)
    pr = O.Problem.from_workload(wl)
    S = pr.one_body_matrix(wl.shapes[0].trg, wl.shapes[0].src, np.zeros(3))  # S_L
    c = W.random_vector(n, 174)
    g = S @ c
    q, r = np.linalg.qr(S)
    own = solve_triangular(r, np.eye(n)) @ (q.T @ g)
    plan = mfs.Plan.from_workload(wl, mfs.FP64, factorization=mfs.FACTOR_QR)
    got = plan.precond_apply(torch.tensor(g, dtype=torch.float64, device="cuda"), 0, mfs.FP64).cpu().numpy()
    plan.close()
    e, bar = rel_inf(got, c), M.bar(rel_inf(own, c))
    print(f"n={n} m={m} err={e:.2e} bar={bar:.2e}")
    assert e <= bar
