"""The correction of CG passes that evaluate q again, against passes that store q.

At four cells per lane a 3-D FP32 grid without missing data evaluates q again
and adds to its correction in pairs: the last pass of an outer step adds, and
every second one before it, two terms each (pass 1 one).  At two cells per
lane the plan stores q and every pass adds one term.  Both do the same
arithmetic per cell and differ in the order of their FP64 sums only, so after
a few outer steps the fields agree to FP32 rounding of the scalars (bar 1e-5
of RMS(P)); a term lost, doubled or taken with another pass's alpha is off by
the size of the term.

Iteration counts: both parities, one pass (no pair), the first pair alone.
Segments of one, two, three and more planes per wave, short of and past the
loop's three register sets (pass 0's five); few blocks (every block sums the partials) and
more than 1024 (finalize kernel); rows of one and of two windows."""

import pytest
import torch

import synth
from gpu_common import DEV, announce, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("iters", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("dims,seg", [((40, 23, 17), 4), ((40, 23, 17), 1), ((36, 12, 21), 5), ((36, 12, 21), 32),
                                      ((260, 9, 11), 2), ((64, 130, 130), 2)])
def test_correction_in_pairs(dims, seg, iters):
    import paper_2311_16935_amd as pi

    announce("correction in pairs", dims, seg, iters)
    w = synth.random_small(61, 3, dims, anisotropic=True, mask_frac=0.0)
    g = [x.to(DEV, torch.float32).contiguous() for x in w.grads]
    plan = pi.Plan(w.dims, w.spacing, inner_iters=iters)
    pi.pi_set_tile(plan.handle, seg, 4)
    assert pi.pi_get_cg_recompute(plan.handle) == 1
    a = plan.solve(g, tol=0.0, max_iter=4, check=False)
    pi.pi_set_tile(plan.handle, seg, 2)
    assert pi.pi_get_cg_recompute(plan.handle) == 0
    b = plan.solve(g, tol=0.0, max_iter=4, check=False)
    assert a.info["inner_iters_total"] == b.info["inner_iters_total"]
    A, B = a.P.double(), b.P.double()
    err = float((A - B).abs().max() / B.square().mean().sqrt())
    print(f"pairs {dims} {seg} {iters}: {err:.2e}")
    assert err <= 1e-5, err
    plan.close()
