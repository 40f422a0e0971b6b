"""A closed plan gives back all the device memory it took.

Plans of every kind (streaming CG with its ping-pong vectors, BiCGStab, on
the chip, cell-centred, FP64, with missing data and several groups) are made
and closed; after a first round, which sets up what the process keeps (queues,
the cooperative launch), the device's free memory must be the same after every
further round, to less than the smallest vector of any of these plans."""

import pytest
import torch

from gpu_common import announce, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

ROUNDS = 4


def _split_mask(dims):
    """Two groups: a column of missing cells between them."""
    m = torch.ones(tuple(reversed(dims)), dtype=torch.uint8)
    m[..., dims[0] // 2] = 0
    return m


@pytest.mark.parametrize("dims,kw,masked", [
    ((160, 160, 160), {}, False),
    ((160, 160, 161), {}, True),
    ((160, 160, 160), dict(bicgstab=True), False),
    ((2048, 1024), {}, False),
    ((2048, 1024), dict(cell_centered=True), True),
    ((1500, 1400), dict(fp64=True), True),
    ((1024, 1024), dict(fp64=True, fixed_point=True), False),
], ids=["stream3d", "stream3d_masked", "bicgstab", "chip2d", "chip_cell", "stream_fp64", "chip_fp64"])
def test_closed_plans_leave_no_device_memory_behind(dims, kw, masked):
    import paper_2311_16935_amd as pi

    announce("plan memory", dims, kw)
    mask = _split_mask(dims) if masked else None

    def free_after_a_plan():
        plan = pi.Plan(dims, (1.0,) * len(dims), mask=mask, **kw)
        held = plan.workspace_bytes
        plan.close()
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0], held

    free_after_a_plan()
    first, held = free_after_a_plan()
    cells = dims[0] * dims[1] * (dims[2] if len(dims) == 3 else 1)
    assert held > 10 * cells
    for k in range(ROUNDS):
        now, _ = free_after_a_plan()
        assert first - now < 4 * cells, (k, first - now)
