"""Host checks of where a batch's grids are solved (batch_routes in
csrc/pi_resident.h, compiled for the host; no GPU is used): batches of many
mid-size grids stream, whose boxes for the chip hold one cell per lane, and all
others keep the chip.  Both sides of every line drawn here were measured; the
times are milliseconds of 24 outer steps on the chip and streamed."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <array>
#include <cstdio>
#include <cstring>
#include "pi_resident.h"
// the plan's default walk (set_walk) and inner iterations
static pi::Inst grid(int nx, int ny, int nz, int fp64, int cc, int cus, long max_iter, int opl) {
  pi::Inst in;
  std::memset(&in, 0, sizeof in);
  in.ndim = nz > 1 ? 3 : 2;
  in.nx = nx, in.ny = ny, in.nz = nz;
  in.ncell = (long long)nx * ny * nz;
  in.nm = nz > 1 ? nz : ny;
  in.cc = cc;
  in.res_npat = cc ? 25 : 0;
  in.inner_op = opl;
  in.vw = nx % 4 == 0 ? 4 : nx % 2 == 0 && !cc ? 2 : 1;
  in.nxs = (nx + 64 * in.vw - 1) / (64 * in.vw);
  const long strips = (long)in.nxs * (nz > 1 ? ny : 1);
  const long segs = std::max(1l, 8192 / strips);
  in.mseg = (int)std::min<long>(in.nm, std::max(4l, (in.nm + segs - 1) / segs));
  in.nseg = (in.nm + in.mseg - 1) / in.mseg;
  in.nblocks = (int)((strips * in.nseg + 3) / 4);
  int lg = 0, side = std::max({nx, ny, nz});
  while ((1 << lg) < side) ++lg;
  in.inner_iters = opl ? std::min(4096, std::max(32, 4 * side))
                       : nz > 1 ? std::min(24, std::max(4, 3 * lg - 12)) : std::min(32, std::max(4, 4 * lg - 24));
  in.max_iter = max_iter;
  in.gen = cc ? 0 : 1;
  pi::set_resident(in, fp64, cus);
  return in;
}
int main() {
  int nx, ny, nz, n, fp64, cc, opl, cus, ex, ey, ez;
  long max_iter;
  // sides of one range (a fixed sequence), so that all lane widths occur
  uint64_t r = 12345;
  auto draw = [&](int lo, int hi) {
    r = r * 6364136223846793005ull + 1442695040888963407ull;
    return lo + (int)((r >> 33) % (uint64_t)(hi - lo + 1));
  };
  for (auto &m : {std::array<int, 3>{300, 64, 256}, {200, 100, 500}, {64, 128, 1024}}) {
    std::vector<pi::Inst> b;
    for (int i = 0; i < m[0]; ++i) {
      const int x = draw(m[1], m[2]), y = draw(m[1], m[2]);
      b.push_back(grid(x, y, 1, 0, 0, 256, 24, 0));
    }
    pi::batch_routes(b, false, 256, 4096);
    int chip = 0;
    for (auto &i : b) chip += i.res_nwg > 0;
    std::printf("%d 0 %d\n", m[0], chip);
  }
  while (std::scanf("%d %d %d %d %d %d %d %d %ld %d %d %d", &nx, &ny, &nz, &n, &fp64, &cc, &opl, &cus, &max_iter, &ex,
                    &ey, &ez) == 12) {
    std::vector<pi::Inst> b(n, grid(nx, ny, nz, fp64, cc, cus, max_iter, opl));
    if (ex) b.push_back(grid(ex, ey, ez, fp64, cc, cus, max_iter, opl));
    const int fits = b[0].res_nwg > 0, extra = ex && b.back().res_nwg > 0;
    pi::batch_routes(b, fp64, cus, 4096);
    int chip = 0;
    for (auto &i : b) chip += i.res_nwg > 0;
    std::printf("%d %d %d\n", fits, extra, chip);
  }
}
"""

# (dims, grids, fp64, cell-centred, variant), one more grid or None: on the chip?
CASES = [
    ((101, 101, 1), 400, 0, 0, 0, None, False),   # 10.7 and 7.0
    ((101, 101, 1), 24, 0, 0, 0, None, True),     # 1.0 and 1.8
    ((128, 128, 1), 300, 0, 0, 0, None, False),   # 10.9 and 6.9
    ((200, 199, 1), 300, 0, 0, 0, None, False),   # 35.9 and 24.5
    ((200, 199, 1), 30, 0, 0, 0, None, True),     # 3.7 and 4.5
    ((256, 256, 1), 250, 0, 0, 0, None, False),   # 41.9 and 25.2
    ((300, 200, 1), 300, 0, 0, 0, None, False),   # 77.5 and 53.0
    ((302, 210, 1), 300, 0, 0, 0, None, False),   # 72.4 and 50.2
    ((1000, 30, 1), 300, 0, 0, 0, None, False),   # 91.3 and 30.7
    ((1000, 30, 1), 10, 0, 0, 0, None, True),     # 3.8 and 4.9
    ((30, 1000, 1), 300, 0, 0, 0, None, True),    # 43.1 and 63.2
    ((800, 700, 1), 30, 0, 0, 0, None, False),    # 53.3 and 47.9
    ((400, 300, 1), 130, 0, 0, 0, None, True),    # 32.5 and 36.7
    ((500, 400, 1), 80, 0, 0, 0, None, True),     # 22.3 and 38.5
    ((1000, 1000, 1), 16, 0, 0, 0, None, True),   # 29.1 and 44.3
    ((64, 64, 1), 512, 0, 0, 0, None, True),      # 2.4 and 9.5
    ((48, 48, 1), 1000, 0, 0, 0, None, True),     # 4.7 and 16.9
    ((32, 32, 32), 200, 0, 0, 0, None, True),     # 20.1 and 27.9
    ((64, 64, 64), 60, 0, 0, 0, None, True),      # 14.0 and 49.2
    ((128, 128, 128), 16, 0, 0, 0, None, True),   # 35.9 and 88.2
    ((101, 101, 1), 300, 1, 0, 0, None, False),   # 8.6 and 7.1
    ((300, 200, 1), 200, 1, 0, 0, None, True),    # 59.4 and 65.9
    ((64, 64, 64), 30, 1, 0, 0, None, True),      # 10.6 and 36.7
    ((300, 200, 1), 200, 0, 1, 0, None, True),    # 58.5 and 72.2
    ((500, 400, 1), 60, 0, 1, 0, None, True),     # 20.1 and 37.7
    ((300, 200, 1), 100, 0, 0, 1, None, False),   # one outer step: 85.4 and 78.8
    ((32, 32, 32), 100, 0, 0, 1, None, True),     # one outer step: 11.0 and 17.1
    ((64, 64, 1), 1, 0, 0, 0, None, True),
    ((2048, 2048, 1), 1, 0, 0, 0, None, True),
    ((101, 101, 1), 4, 0, 0, 0, (256, 256, 256), True),     # beside a grid that streams anyway
    ((300, 200, 1), 300, 0, 0, 0, (256, 256, 256), False),
]


def routes(tmp_path, cases, steps=24):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "routes.hip", tmp_path / "routes"
    src.write_text(PROGRAM)
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-I",
                        os.path.join(ROOT, "paper_2311_16935_amd", "csrc"), "-o", str(exe), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    lines = []
    for (nx, ny, nz), n, fp64, cc, opl, extra, cus in cases:
        e = extra or (0, 0, 0)
        lines.append(f"{nx} {ny} {nz} {n} {fp64} {cc} {opl} {cus} {1 if opl else steps} {e[0]} {e[1]} {e[2]}")
    out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, timeout=120, check=True)
    return [tuple(int(v) for v in ln.split()) for ln in out.stdout.splitlines()]


def test_batches_go_where_they_are_faster(tmp_path):
    got = routes(tmp_path, [c[:6] + (256,) for c in CASES])
    # uneven 2-D batches: 300 of 64..256 a side (26.2 and 20.5), 200 of 100..500 (43 and 54), 64 of 128..1024 (43 and 83)
    assert got[:3] == [(300, 0, 0), (200, 0, 200), (64, 0, 64)]
    for (dims, n, fp64, cc, opl, extra, chip), (fits, extra_fits, on_chip) in zip(CASES, got[3:]):
        case = (dims, n, fp64, cc, opl, extra)
        assert fits == 1, case
        assert on_chip == (n + extra_fits if chip else 0), case


def test_short_calls_do_not_pay_for_a_graph(tmp_path):
    """Few outer steps: the capture of the streaming graph costs more than the rounds on the chip."""
    cases = [((101, 101, 1), 24), ((300, 200, 1), 8), ((64, 64, 1), 1), ((64, 64, 1), 200), ((200, 199, 1), 30),
             ((1000, 1000, 1), 4), ((101, 101, 1), 100)]  # at 0 steps 0.3 and 0.7, 0.3 and 0.9, 0.2 and 0.6 ms, ...
    for steps in (0, 1, 2, 5):
        got = routes(tmp_path, [c + (0, 0, 0, None, 256) for c in cases], steps)[3:]
        assert [g[2] for g in got] == [c[1] for c in cases], steps


def test_a_grid_that_fits_no_device_is_left_for_the_rounds_to_report(tmp_path):
    """No CUs: nothing is decided (and nothing loops)."""
    assert routes(tmp_path, [((64, 64, 1), 3, 0, 0, 0, None, 0)])[3:] == [(0, 0, 0)]
