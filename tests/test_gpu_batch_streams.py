"""A batch of more mid-size grids than the chip takes faster streams, as one
whose plans ask for a tile does: same fields bit for bit, same counts, through
both entry points; a few of the same grids are solved on the chip and return
what their own solves return."""

import pytest
import torch

import synth
from gpu_common import DEV, announce, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("fp64", [False, True])
def test_many_mid_size_grids_stream_and_few_do_not(fp64):
    import paper_2311_16935_amd as pi

    announce("batch that streams", fp64)
    dtype, steps, n = (torch.float64 if fp64 else torch.float32), 6, 320
    ws = [synth.random_small(300 + i, 2, (101, 101), mask_frac=0.0) for i in range(8)]
    # FP64 plans with a mask stream by themselves: these have none
    plans = [pi.Plan(w.dims, w.spacing, fp64=fp64) for _ in range(n // 8) for w in ws]
    grads = [[x.to(DEV, dtype).contiguous() for x in ws[i % 8].grads] for i in range(n)]

    def run(k, noalloc=False):
        Ps = [torch.full(p.shape, 3.0, dtype=dtype, device=DEV) for p in plans[:k]]
        rc, Ps, infos = pi.solve_batched(plans[:k], grads[:k], Ps, tol=0.0, max_iter=steps, check=False,
                                         noalloc=noalloc)
        assert rc == pi.PI_ERR_NOT_CONVERGED
        return Ps, [(i["outer_iters"], i["inner_iters_total"], i["status"]) for i in infos], infos

    singles = [p.solve(g, tol=0.0, max_iter=steps, check=False) for p, g in zip(plans[:8], grads[:8])]
    few, _, _ = run(8)
    for one, P in zip(singles, few):
        assert torch.equal(one.P, P)
    many, counts, infos = run(n)
    many_na, counts_na, _ = run(n, noalloc=True)
    assert infos[0]["worklist_rebuilds"] == 0  # on the chip, 19 rounds
    for p in plans:
        pi.pi_set_tile(p.handle, pi.pi_get_tile(p.handle), 0)
    tiled, counts_t, _ = run(n)
    assert counts == counts_t == counts_na
    assert all(torch.equal(a, b) and torch.equal(a, c) for a, b, c in zip(many, tiled, many_na))
    for P, one in zip(many[:8], singles):
        err = float((P - one.P).abs().max()) / float(one.P.square().mean().sqrt())
        assert err <= (1e-12 if fp64 else 1e-5), err  # bars of the on-chip against the streaming solve
    for p in plans:
        p.close()
