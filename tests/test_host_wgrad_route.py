"""Host check of which kernel takes a 3x3x3 weight gradient (wgrad_boxes_pay in
csrc/pi_conv.h, compiled for the host; no GPU is used): the boxes where they are
full enough, the general kernel for thin and tiny grids.  Times in microseconds
of the general kernel and of the boxes were measured for each."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include "pi_conv.h"
int main() {
  long n, d, h, w, cin, cout;
  while (std::scanf("%ld %ld %ld %ld %ld %ld", &n, &d, &h, &w, &cin, &cout) == 6) {
    const long P = n * d * h * w;
    const long chunk = std::max(2048l, ((P + 255) / 256 + 31) / 32 * 32);
    auto padded = [&](long ry) { return (d + 32 / ry - 1) / (32 / ry) * (32 / ry) * ((h + ry - 1) / ry * ry); };
    const long ry = padded(16) <= padded(8) ? 16 : 8, rz = 32 / ry;
    const long boxes = n * ((d + rz - 1) / rz) * ((h + ry - 1) / ry) * ((w + 7) / 8);
    std::printf("%d\n", (int)pu::wgrad_boxes_pay(boxes, P, (int)((P + chunk - 1) / chunk), (int)cin, (int)cout));
  }
}
"""

CASES = [  # grid, channels, boxes?
    ((4, 64, 64, 64), (64, 32), True),    # 1900, 170
    ((4, 64, 64, 64), (4, 32), True),     # 1941, 109
    ((4, 33, 33, 33), (32, 32), True),    # 348, 64
    ((1, 16, 16, 16), (32, 32), True),    # 110, 42
    ((4, 8, 8, 8), (32, 32), True),       # 110, 39
    ((1, 8, 8, 8), (256, 256), True),     # 40, 24
    ((4, 8, 8, 8), (256, 256), True),     # 122, 46
    ((1, 12, 12, 12), (32, 32), True),    # 94, 56
    ((1, 10, 9, 11), (32, 32), True),     # 56, 49
    ((1, 1, 64, 64), (32, 32), True),     # 109, 68
    ((1, 1, 256, 256), (256, 256), True),  # 1851, 543
    ((1, 64, 64, 3), (32, 32), True),     # 110, 96
    ((2, 40, 3, 40), (64, 64), True),     # 112, 86
    ((1, 64, 64, 2), (256, 256), True),   # 283, 144
    ((1, 64, 64, 1), (32, 32), False),    # 110, 257
    ((1, 64, 1, 64), (32, 32), False),    # 110, 251
    ((1, 64, 64, 2), (32, 32), False),    # 109, 135
    ((1, 64, 64, 1), (256, 256), False),  # 183, 265
    ((1, 100, 3, 3), (32, 32), False),    # 53, 102
    ((8, 1, 9, 9), (32, 32), False),      # 40, 67
    ((1, 5, 17, 9), (32, 32), False),     # 45, 55
    ((16, 4, 4, 4), (32, 32), False),     # 58, 66
    ((64, 2, 2, 2), (32, 32), False),     # 33, 240
    ((4, 2, 2, 2), (256, 256), False),    # 22, 31
    ((1, 2, 2, 4000), (128, 64), False),  # 138, 248
    ((1, 128, 128, 1), (64, 64), False),  # 122, 260
    ((1, 1000, 3, 3), (256, 256), False),  # 292, 393: 320 workgroups take two turns
    ((1, 3, 3, 1000), (256, 256), True),  # 293, 202
    ((1, 1, 1, 1), (32, 32), False),
]


def test_weight_gradients_go_to_the_faster_kernel(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "route.hip", tmp_path / "route"
    src.write_text(PROGRAM)
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-I",
                        os.path.join(ROOT, "paper_2311_16935_amd", "csrc"), "-o", str(exe), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, g + c)) for g, c, _ in CASES),
                         capture_output=True, text=True, timeout=60, check=True)
    for (grid, ch, want), got in zip(CASES, out.stdout.split(), strict=True):
        assert int(got) == want, (grid, ch)
