"""mfs_plan_autotune times the shape that the plan has beside its own list: two bodies with one source split
are one launch, where every listed shape (1024 items and more) cuts their sources in two and adds the
slices in a second launch."""
import numpy as np
import pytest
import torch

import mfs_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [W.STOKES, W.LAPLACE])
def test_autotune_keeps_a_faster_shape_of_the_plan(kind):
    from paper_2409_04215_amd import mfs
    wl = W.small_cluster(2, kind, 20, 60, seed=181)
    plan = mfs.Plan.from_workload(wl, mfs.MIXED)
    plan.set_launch(1, 1)
    g = torch.tensor(np.random.default_rng(182).standard_normal(plan.n_gamma), dtype=torch.float64, device="cuda")
    before = plan.matvec(g)
    tpl, items, ms = plan.autotune(mfs.MIXED, reps=50)
    print(f"kind={kind} targets per lane {tpl}, work items {items}, {ms * 1e3:.1f} us")
    assert (tpl, items) == (1, 1)
    assert torch.equal(plan.matvec(g), before)
    plan.close()
