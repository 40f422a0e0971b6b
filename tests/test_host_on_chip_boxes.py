"""Host checks of the boxes the on-chip solve cuts a grid into (set_resident in
csrc/pi_resident.h): the header's own function is compiled for the host and
run over grids of every kind; no GPU is used.

What the kernel relies on: the boxes cover the grid and every box holds a
cell of it, at most one workgroup per CU (256), at most 1024 lanes with at
most as many cells each as the kernel is compiled for, a ring of at most 1024
cells in 2-D and 3072 in 3-D (one and three per lane), tile places that fit 16
bits, and the LDS limit."""

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
  const int side2[] = {1, 2, 3, 5, 16, 31, 64, 65, 97, 101, 128, 257, 386, 512, 1000, 1023, 2000, 2048, 2049, 4096, 65536};
  const int side3[] = {1, 2, 7, 17, 24, 33, 64, 97, 127, 128, 129, 200, 500};
  auto one = [&](int nd, int nx, int ny, int nz, int fp64, int cus) {
    pi::Inst in;
    std::memset(&in, 0, sizeof in);
    in.ndim = nd;
    in.nx = nx;
    in.ny = ny;
    in.nz = nz;
    in.ncell = (long long)nx * ny * nz;
    in.nm = nd == 3 ? nz : ny;
    if (in.ncell >= (1ll << 31)) return;
    pi::set_resident(in, fp64, cus);
    std::printf("%d %d %d %d %d %d  %d %d %d %d %d %d %d %d  %d %lld\n", nd, nx, ny, nz, fp64, cus, in.res_nwg, in.res_n,
                in.res_tx, in.res_ty, in.res_g, in.res_r, in.res_bx, in.res_by, in.res_nwg ? pi::res_ring(in) : 0,
                in.res_nwg ? (long long)pi::res_lds(in, fp64) : 0ll);
  };
  for (int fp64 = 0; fp64 < 2; ++fp64)
    for (int cus : {1, 256}) {
      for (int nx : side2)
        for (int ny : side2) one(2, nx, ny, 1, fp64, cus);
      for (int nx : side3)
        for (int ny : side3)
          for (int nz : side3) one(3, nx, ny, nz, fp64, cus);
    }
  return 0;
}
"""


@pytest.fixture(scope="module")
def boxes(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("boxes")
    src, exe = d / "boxes.hip", d / "boxes"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_2311_16935_amd", "csrc")
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-I", inc, "-o", str(exe), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120, check=True).stdout.splitlines()
    return [tuple(int(v) for v in ln.split()) for ln in out]


def test_boxes_meet_what_the_kernel_relies_on(boxes):
    used = 0
    for nd, nx, ny, nz, fp64, cus, nwg, n, tx, ty, g, r, bx, by, ring, lds in boxes:
        if nwg == 0:
            continue
        used += 1
        case = (nd, nx, ny, nz, fp64, cus)
        nm = nz if nd == 3 else ny
        ty_, by_ = (ty, by) if nd == 3 else (1, 1)
        tm = g * r
        bm = nwg // (bx * by_)
        assert nwg == bx * by_ * bm and nwg <= min(cus, 256), case
        for side, t, b in ((nx, tx, bx), (ny if nd == 3 else 1, ty_, by_), (nm, tm, bm)):
            assert t * b >= side and t * (b - 1) < side, case
        assert tx * ty_ * g <= 1024 and 1 <= r <= n, case
        assert n in ((4, 8) if fp64 else (4, 8, 16)) if nd == 2 else n in ((4,) if fp64 else (4, 8)), case
        assert ring == 2 * (tx * ty_ + (tx * tm if nd == 3 else 0) + ty_ * tm), case
        assert ring <= (3072 if nd == 3 else 1024), case
        tile = (tx + 2) * ((ty + 2) if nd == 3 else 1) * (tm + 2)
        assert tile <= 65536 and r * 1024 <= 16384, case
        t = 8 if fp64 else 4
        assert lds == max(8 * tile, t * (tile + 1024 * r)) and lds <= 150 * 1024, case
    assert used > 500


def test_which_grids_are_solved_on_the_chip(boxes):
    nwg = {b[:6]: b[6] for b in boxes}
    assert nwg[(2, 64, 64, 1, 0, 256)] == 1
    assert nwg[(2, 2048, 2048, 1, 0, 256)] == 256  # 4 M cells at 16 per lane fill the device
    assert nwg[(2, 2049, 2049, 1, 0, 256)] == 0
    assert 0 < nwg[(3, 128, 128, 128, 0, 256)] <= 256
    assert nwg[(3, 200, 200, 200, 0, 256)] == 0
    assert nwg[(2, 1000, 1000, 1, 0, 1)] == 0  # without cooperative launches: one box only
