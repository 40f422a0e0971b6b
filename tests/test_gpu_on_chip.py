"""The on-chip solve against the streaming kernels, through the C interface.

A plan at its default tile solves grids of up to a few million cells on the
chip; after pi_set_tile asks for a tile, the same plan streams.  Both run
Algorithm 1 with the same arithmetic per cell and differ in the order of
their FP64 sums only, so after a number of outer steps the FP32 fields must
agree to FP32 rounding of the scalars carried through those steps (bar 1e-5
of RMS(P)), FP64 ones to FP64 rounding (bar 1e-12), with the same counts.

Sizes: one box with and without lanes to spare, single rows and columns,
partial boxes, more than 64 boxes (sums in two hops), more than one ring cell
per lane, the largest grid, and every number of cells per lane."""

import pytest
import torch

import synth
from gpu_common import DEV, announce, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

CASES = [  # ndim, dims, mask fraction, fp64, fixed-point variant, outer steps
    (2, (64, 64), 0.0, False, False, 30),
    (2, (1, 70), 0.0, False, False, 30),
    (2, (301, 1), 0.0, False, False, 30),
    (2, (101, 97), 0.1, False, False, 30),
    (2, (257, 130), 0.1, False, False, 30),
    (2, (1025, 517), 0.05, False, False, 15),
    (2, (1500, 1100), 0.05, False, False, 8),
    (2, (2048, 2048), 0.0, False, False, 4),
    (2, (300, 200), 0.1, False, True, 1),
    (2, (130, 91), 0.0, True, False, 30),
    (2, (700, 650), 0.0, True, False, 10),
    (3, (5, 3, 2), 0.0, False, False, 10),
    (3, (40, 23, 17), 0.1, False, False, 20),
    (3, (17, 64, 65), 0.0, False, False, 20),
    (3, (100, 90, 80), 0.05, False, False, 8),
    (3, (127, 128, 126), 0.0, False, False, 4),
    (3, (66, 34, 35), 0.0, False, True, 1),
    (3, (64, 65, 63), 0.0, True, False, 10),
]


@pytest.mark.parametrize("ndim,dims,frac,fp64,variant,steps", CASES)
def test_on_chip_solve_follows_the_streaming_one(ndim, dims, frac, fp64, variant, steps):
    import paper_2311_16935_amd as pi

    announce("on chip", dims, frac, fp64, variant)
    w = synth.random_small(91, ndim, dims, anisotropic=False, mask_frac=frac)
    g = [x.to(DEV, torch.float64 if fp64 else torch.float32).contiguous() for x in w.grads]
    plan = pi.Plan(w.dims, w.spacing, mask=w.mask, fp64=fp64, fixed_point=variant)
    tile = pi.pi_get_tile(plan.handle)
    chip = plan.solve(g, tol=0.0, max_iter=steps, check=False)
    again = plan.solve(g, tol=0.0, max_iter=steps, check=False)
    assert torch.equal(torch.nan_to_num(chip.P, nan=7.0), torch.nan_to_num(again.P, nan=7.0))
    pi.pi_set_tile(plan.handle, tile, 0)
    stream = plan.solve(g, tol=0.0, max_iter=steps, check=False)
    for k in ("outer_iters", "inner_iters_total", "status", "components"):
        assert chip.info[k] == stream.info[k], k
    a, b = torch.nan_to_num(chip.P).double(), torch.nan_to_num(stream.P).double()
    assert torch.equal(torch.isnan(chip.P), torch.isnan(stream.P))
    rms = float(b.square().mean().sqrt())
    err = float((a - b).abs().max()) / max(rms, 1e-300)
    print(f"on chip {dims}: {err:.2e}")
    assert err <= (1e-12 if fp64 else 1e-5), err
    plan.close()


def test_batch_of_on_chip_and_streamed_grids_returns_the_single_solves():
    """Grids solved on the chip (more workgroups in all than the device holds
    at once), one that streams, and a zero source, in one call."""
    import paper_2311_16935_amd as pi

    announce("batch of both kinds")
    ws = [synth.random_small(92 + i, 2, d, mask_frac=0.05) for i, d in
          enumerate([(900, 800), (640, 500), (64, 60), (1000, 300), (333, 222)])]
    ws.append(synth.random_small(99, 3, (256, 130, 130), mask_frac=0.0))
    plans = [pi.Plan(w.dims, w.spacing, mask=w.mask) for w in ws]
    grads = [[x.to(DEV, torch.float32).contiguous() for x in w.grads] for w in ws]
    grads[4] = [torch.zeros_like(x) for x in grads[4]]
    for noalloc in (False, True):
        P0 = [torch.full(p.shape, 3.0, dtype=torch.float32, device=DEV) for p in plans]
        rc, Ps, infos = pi.solve_batched(plans, grads, P0, tol=0.0, max_iter=12, check=False, noalloc=noalloc)
        assert rc == pi.PI_ERR_NOT_CONVERGED
        for i, (p, g, P) in enumerate(zip(plans, grads, Ps)):
            if i == 5:
                continue  # the streamed grid's passes store q in a batch
            one = p.solve(g, tol=0.0, max_iter=12, check=False)
            assert one.info["outer_iters"] == infos[i]["outer_iters"] and one.status == infos[i]["status"], i
            assert torch.equal(torch.nan_to_num(P, nan=7.0), torch.nan_to_num(one.P, nan=7.0)), i
        assert infos[5]["outer_iters"] == 12 and infos[4]["outer_iters"] == 0
        assert float(Ps[5].abs().max()) > 0 and infos[0]["worklist_rebuilds"] >= 1
    for p in plans:
        p.close()


CELL_CASES = [  # dims, mask fraction, fp64, fixed-point variant, outer steps
    ((64, 64), 0.0, False, False, 30),
    ((1, 40), 0.0, False, False, 20),
    ((3, 2), 0.0, False, False, 5),
    ((101, 97), 0.1, False, False, 30),
    ((260, 131), 0.1, False, False, 30),
    ((1025, 517), 0.05, False, False, 12),
    ((2047, 2040), 0.03, False, False, 3),
    ((300, 200), 0.1, False, True, 1),
    ((130, 91), 0.0, True, False, 30),
    ((600, 500), 0.0, True, False, 8),
]


@pytest.mark.parametrize("dims,frac,fp64,variant,steps", CELL_CASES)
def test_on_chip_cell_centred_solve_follows_the_streaming_one(dims, frac, fp64, variant, steps):
    """The nine-point stencils: ring corners from diagonal boxes, and weights by ring code."""
    import paper_2311_16935_amd as pi

    announce("on chip cell-centred", dims, frac, fp64, variant)
    w = synth.random_small(93, 2, dims, anisotropic=False, mask_frac=frac)
    g = [x.to(DEV, torch.float64 if fp64 else torch.float32).contiguous() for x in w.grads]
    plan = pi.Plan(w.dims, w.spacing, mask=w.mask, fp64=fp64, fixed_point=variant, cell_centered=True)
    tile = pi.pi_get_tile(plan.handle)
    chip = plan.solve(g, tol=0.0, max_iter=steps, check=False)
    pi.pi_set_tile(plan.handle, tile, 0)
    stream = plan.solve(g, tol=0.0, max_iter=steps, check=False)
    for k in ("outer_iters", "inner_iters_total", "status", "components"):
        assert chip.info[k] == stream.info[k], k
    a, b = torch.nan_to_num(chip.P).double(), torch.nan_to_num(stream.P).double()
    assert torch.equal(torch.isnan(chip.P), torch.isnan(stream.P))
    err = float((a - b).abs().max()) / max(float(b.square().mean().sqrt()), 1e-300)
    print(f"on chip cell-centred {dims}: {err:.2e}")
    assert err <= (1e-12 if fp64 else 1e-5), err
    plan.close()
