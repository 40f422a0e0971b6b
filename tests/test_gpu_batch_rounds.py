"""How often finished grids leave a batch whose grids are solved on the chip
(pi_info.worklist_rebuilds), on batches whose rounds are known: each launch
counts the different numbers of passes after which some of its grids ended,
and the last grid of the call is not counted.  1024^2 takes all of the
device's workgroups, so two of them never run together."""

import pytest
import torch

import synth
from gpu_common import DEV, announce, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

BATCHES = [  # (dims, inner iterations (None: default), zero source) of each grid, times one leaves early
    ([((1024, 1024), None, False)] * 2, 1),
    ([((1024, 1024), None, False)] * 3, 2),
    ([((64, 64), None, False)] * 2, 0),
    ([((64, 64), 4, False), ((64, 64), 6, False)], 1),
    ([((64, 64), 4, False), ((64, 64), 6, False), ((64, 64), 4, True)], 2),
    ([((1024, 1024), None, True), ((64, 64), None, False)], 1),
    ([((1024, 1024), None, False), ((64, 64), None, False), ((48, 60), None, False)], 1),
    ([((64, 64), None, False), ((2080, 2080), None, False)], 1),  # the second streams
]


@pytest.mark.parametrize("grids,leaves", BATCHES, ids=[str(i) for i in range(len(BATCHES))])
@pytest.mark.parametrize("noalloc", [False, True])
def test_grids_that_leave_a_batch_are_counted(grids, leaves, noalloc):
    import paper_2311_16935_amd as pi

    announce("batch rounds", grids, noalloc)
    ws = [synth.random_small(31, 2, d, mask_frac=0.0) for d, _, _ in grids]
    plans = [pi.Plan(w.dims, w.spacing, inner_iters=k) for w, (_, k, _) in zip(ws, grids)]
    grads = [[(torch.zeros_like(x) if zero else x).to(DEV, torch.float32).contiguous() for x in w.grads]
             for w, (_, _, zero) in zip(ws, grids)]
    rc, Ps, infos = pi.solve_batched(plans, grads, tol=0.0, max_iter=3, check=False, noalloc=noalloc)
    for (_, _, zero), P, info in zip(grids, Ps, infos):
        assert info["outer_iters"] == (0 if zero else 3)
        assert info["worklist_rebuilds"] == leaves, infos
        assert bool(torch.isfinite(P).all())
    for p in plans:
        p.close()
