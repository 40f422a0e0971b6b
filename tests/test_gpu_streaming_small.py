"""Small grids whose plans ask for a tile, so that they stream: what only the
streaming solve has, on sizes that the chip takes by default -- the batched work
list that drops finished instances and captures its graph again, and the
correction buffer of an inner solve that ends after its first pass."""

import numpy as np
import pytest
import torch

import synth
from gpu_common import DEV, announce, np_, oracle_for, rel_maxabs, requires_gpu
from oracle.solve import fixed_point, residual_momentum
from test_gpu_variant_early_stop import _cos_mode

pytestmark = [pytest.mark.gpu, requires_gpu]


def _streams(pi, plan):
    pi.pi_set_tile(plan.handle, pi.pi_get_tile(plan.handle), 0)
    return plan


@pytest.mark.parametrize("noalloc", [False, True])
def test_batched_work_list_drops_finished_instances(noalloc):
    """A large instance that finishes early (zero source, or a loose tolerance)
    leaves the work list; the one still running, and the early one, return what
    their own solves return, bit for bit."""
    import paper_2311_16935_amd as pi

    announce("streaming work list", noalloc)
    big = synth.random_small(35, 2, (256, 256), mask_frac=0.0)
    small = synth.random_small(36, 3, (24, 17, 13), mask_frac=0.1)
    plans = [_streams(pi, pi.Plan(w.dims, w.spacing, mask=w.mask)) for w in (big, small)]
    grads = [[x.to(DEV, torch.float32).contiguous() for x in w.grads] for w in (big, small)]
    single = plans[1].solve(grads[1], tol=1e-9, max_iter=100000)
    for g0, tol0 in (([torch.zeros_like(x) for x in grads[0]], 1e-6), (grads[0], 0.3)):
        rc, Ps, infos = pi.solve_batched(plans, [g0, grads[1]], tol=[tol0, 1e-9], max_iter=100000, noalloc=noalloc)
        assert rc == 0, infos
        assert infos[0]["outer_iters"] < infos[1]["outer_iters"] == single.info["outer_iters"]
        # one instance of two can leave while the other runs: one rebuild
        assert infos[0]["worklist_rebuilds"] == infos[1]["worklist_rebuilds"] == 1, infos
        assert torch.equal(torch.nan_to_num(Ps[1], nan=7.0), torch.nan_to_num(single.P, nan=7.0))
        assert torch.equal(Ps[0], plans[0].solve(g0, tol=tol0, max_iter=100000).P)
    for p in plans:
        p.close()


def test_inner_solve_ending_after_its_first_pass():
    """The start and the preconditions of the test of the same name in
    test_gpu_variant_early_stop.py: two outer steps, of two and one inner
    iterations.  The buffer still holds the first step's correction then and
    must not be added again."""
    import paper_2311_16935_amd as pi

    nx, ny = 40, 32
    announce("variant early stop, streaming", (nx, ny))
    w = synth.random_small(7, 2, (nx, ny), anisotropic=False, mask_frac=0.0)
    sys_ = oracle_for(w)
    S = sys_.source([g.numpy() for g in w.grads])
    Pstar = fixed_point(sys_, S)
    rms = np.sqrt(np.mean(Pstar**2))
    P0 = Pstar + rms * (_cos_mode(nx, ny, 1, 0) + 0.7 * _cos_mode(nx, ny, 0, 1) + 1e-6 * _cos_mode(nx, ny, 3, 2))
    plan = _streams(pi, pi.Plan(w.dims, w.spacing, fp64=True, fixed_point=True, inner_iters=2))
    res = plan.solve([x.to(DEV, torch.float64) for x in w.grads], P=torch.from_numpy(sys_.to_grid(P0)).to(DEV), tol=1e-4,
                     max_iter=50, warm_start=True)
    assert res.status == pi.PI_OK, res.info
    assert res.info["outer_iters"] == 2 and res.info["inner_iters_total"] == 3, res.info
    got = np_(res.P).ravel()
    assert abs(residual_momentum(sys_, S, got) - res.info["eps_R"]) <= 1e-4 * res.info["eps_R"]
    assert rel_maxabs(got, Pstar) < 1e-5
    plan.close()
