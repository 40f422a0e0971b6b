"""Host checks of the boxes of cell-centred grids on the chip (set_resident,
res_ring, res_lds and res_boxes in csrc/pi_resident.h, compiled for the host; no
GPU is used): the ring has the box's four corners besides its faces and fits one
cell per lane, lanes without a ring cell have a place to write, and the table of
weights and neighbour bits by ring code starts behind the box and q, on a
multiple of 16 bytes, and ends inside the LDS."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstring>
#include "pi_resident.h"
int main() {
  std::printf("%d %d %d %d %d\n", pi::kResLds, pi::kResBlock, pi::kResSpare, pi::kResMaxPat, pi::kResMaxWg);
  const int sides[] = {1, 2, 3, 5, 16, 31, 64, 65, 97, 128, 257, 386, 512, 1000, 1023, 2000, 2047, 2048, 2049, 65536};
  for (int fp64 = 0; fp64 < 2; ++fp64)
    for (int cus : {1, 256})
      for (int npat : {0, 2, 25, 600, 1200, 4096})
        for (int nx : sides)
          for (int ny : sides) {
            pi::Inst in;
            std::memset(&in, 0, sizeof in);
            in.ndim = 2, in.nx = nx, in.ny = ny, in.nz = 1, in.nm = ny;
            in.ncell = (long long)nx * ny;
            in.cc = 1;
            in.res_npat = npat;
            if (in.ncell >= (1ll << 31)) continue;
            pi::set_resident(in, fp64, cus);
            const bool on = in.res_nwg > 0;
            std::printf("%d %d %d %d %d  %d %d %d %d %d %d  %d %d %lld %lld\n", fp64, cus, npat, nx, ny, in.res_nwg, in.res_n,
                        in.res_tx, in.res_g, in.res_r, in.res_bx, on ? pi::res_ring(in) : 0, on ? in.res_tab : 0,
                        on ? (long long)pi::res_lds(in, fp64) : 0ll, on ? (long long)pi::res_boxes(in, fp64) : 0ll);
          }
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("cell")
    src, exe = d / "cell.hip", d / "cell"
    src.write_text(PROGRAM)
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-I",
                        os.path.join(ROOT, "paper_2311_16935_amd", "csrc"), "-o", str(exe), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120, check=True).stdout.splitlines()
    return [tuple(int(v) for v in ln.split()) for ln in out]


def test_cell_centred_boxes_meet_what_the_kernel_relies_on(rows):
    lds_max, block, spare, max_pat, max_wg = rows[0]
    used = {}
    for fp64, cus, npat, nx, ny, nwg, n, tx, g, r, bx, ring, tab, lds, boxes in rows[1:]:
        case = (fp64, cus, npat, nx, ny)
        if npat == 0:
            assert nwg == 0, case  # too many codes to number
        if nwg == 0:
            continue
        used[npat] = used.get(npat, 0) + 1
        tm, t = g * r, 8 if fp64 else 4
        bm = nwg // bx
        assert nwg == bx * bm and nwg <= min(cus, max_wg), case
        assert tx * bx >= nx > tx * (bx - 1) and tm * bm >= ny > tm * (bm - 1), case
        assert tx * g <= block and 1 <= r <= n and n in ((4, 8) if fp64 else (4, 8, 16)), case
        # one ring cell per lane, corners last; their places and the spare ones in 16 bits
        assert ring == 2 * (tx + tm) + 4 <= block, case
        cells = (tx + 2) * (tm + 2) + spare
        assert cells <= 65536 and r * block <= 16384, case
        # P in FP64, or p and every lane's q, then the table
        assert boxes >= max(8 * cells, t * (cells + block * r)), case
        assert tab == boxes and tab % 16 == 0 and tab - max(8 * cells, t * (cells + block * r)) < 16, case
        assert lds == tab + npat * (8 * t + 1) <= lds_max, case
    assert max_pat == 4096 and all(used.get(k, 0) > 50 for k in (2, 25, 600)), used


def test_more_ring_codes_leave_less_room(rows):
    """The tables of more codes take LDS from the boxes: a grid may need more
    workgroups with them, or not fit, never the other way round."""
    nwg = {r[:5]: r[5] for r in rows[1:]}
    lost = 0
    for (fp64, cus, npat, nx, ny), w in nwg.items():
        if npat > 2 and w:
            assert nwg[(fp64, cus, 2, nx, ny)] > 0
        if npat == 4096 and not w and nwg[(fp64, cus, 2, nx, ny)]:
            lost += 1
    assert lost > 0
    assert nwg[(0, 256, 600, 2048, 2048)] == 256 and nwg[(0, 256, 25, 2049, 2049)] == 0
