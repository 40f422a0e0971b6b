"""pi_autotune on plans that are solved on the chip: it picks the tile of the
operator applies, which still stream, and leaves the solve where it is."""

import pytest
import torch

import synth
from gpu_common import DEV, announce, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _apply_us(pi, plan, x, y):
    """Shortest of ten runs of 40 applies."""
    best = 1e30
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(10):
        a.record()
        for _ in range(40):
            plan.apply(pi.PI_OP_M, x, y)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 40 * 1e3)
    return best


def test_applies_take_the_best_tile():
    """128^3: the default tile takes a quarter longer than the best one; after
    autotuning an apply is within 15 % of the best tile of a sweep."""
    import paper_2311_16935_amd as pi

    announce("autotune on chip: apply")
    dims = (128, 128, 128)
    x = torch.randn(tuple(reversed(dims)), device=DEV)
    y = torch.empty_like(x)
    plan = pi.Plan(dims, (1.0,) * 3)
    plan.autotune(reps=10)
    tuned = _apply_us(pi, plan, x, y)
    want = y.clone()
    sweep = {}
    for vw in (1, 2, 4):
        for m in (2, 4, 8, 16, 32):
            pi.pi_set_tile(plan.handle, m, vw)
            sweep[(m, vw)] = _apply_us(pi, plan, x, y)
            assert torch.equal(y, want)
    print(f"tuned {tuned:.2f} us, best of the sweep {min(sweep.values()):.2f}")
    assert tuned <= 1.15 * min(sweep.values()), (tuned, sweep)
    plan.close()


@pytest.mark.parametrize("dims,kw", [((300, 200), dict(fp64=True)), ((197, 131), dict(cell_centered=True)),
                                     ((40, 36, 28), dict(fixed_point=True)), ((1, 5), {}), ((2, 2, 2), {})])
def test_the_solve_stays_on_the_chip(dims, kw):
    """The same field bit for bit before and after (a streaming FP64 solve adds
    its sums in another order), and from a second plan with the cached tile."""
    import paper_2311_16935_amd as pi

    announce("autotune on chip: solve", dims, kw)
    w = synth.random_small(71, len(dims), dims, anisotropic="cell_centered" not in kw, mask_frac=0.0)
    g = [t.to(DEV, torch.float64 if kw.get("fp64") else torch.float32).contiguous() for t in w.grads]
    plan, plan2 = (pi.Plan(w.dims, w.spacing, **kw) for _ in range(2))
    before = plan.solve(g, tol=0.0, max_iter=5, check=False)
    m = plan.autotune(reps=3)
    assert m == pi.pi_get_tile(plan.handle) and plan2.autotune(reps=3) == m
    for p in (plan, plan2):
        after = p.solve(g, tol=0.0, max_iter=5, check=False)
        assert torch.equal(before.P, after.P) and before.info["inner_iters_total"] == after.info["inner_iters_total"]
        p.close()


def test_plans_of_one_shape_on_and_off_the_chip_keep_tiles_of_their_own():
    """FP64: without a mask on the chip, with one streaming.  Each takes a tile
    that was timed for it; the streaming plan's solve is the same at any tile."""
    import paper_2311_16935_amd as pi

    announce("autotune: two routes of one shape")
    w = synth.random_small(72, 2, (260, 131), mask_frac=0.1)
    g = [t.to(DEV, torch.float64).contiguous() for t in w.grads]
    chip = pi.Plan(w.dims, w.spacing, fp64=True)
    stream = pi.Plan(w.dims, w.spacing, mask=w.mask, fp64=True)
    ref = stream.solve(g, tol=1e-6, max_iter=100000)
    chip.autotune(reps=3)
    stream.autotune(reps=3)
    got = stream.solve(g, tol=1e-6, max_iter=100000)
    assert got.status == pi.PI_OK and abs(got.info["outer_iters"] - ref.info["outer_iters"]) <= 2
    for p in (chip, stream):
        p.close()
