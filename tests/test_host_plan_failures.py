"""pi_plan when a HIP call fails, on the CPU: a program that brings its own
hipMalloc, hipMemcpy and so on (host memory, counted; the n-th allocation or
copy fails) calls the library's pi_plan and pi_plan_destroy.  Whatever fails,
no plan comes back, nothing stays allocated, and the status tells memory from
other errors; a plan that is made and destroyed leaves nothing either."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2311_16935_amd")

PROGRAM = r"""
#include <hip/hip_runtime_api.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>
#include "pi.h"
static std::map<void *, size_t> held;
static int mallocs, copies, fail_malloc = -1, fail_copy = -1, bad_frees;
static hipError_t alloc(void **p, size_t n) {
  *p = nullptr;
  if (mallocs++ == fail_malloc) return hipErrorOutOfMemory;
  *p = std::calloc(1, n);
  held[*p] = n;
  return hipSuccess;
}
static hipError_t release(void *p) {
  if (!p) return hipSuccess;
  if (!held.erase(p)) {
    ++bad_frees;
    return hipErrorInvalidValue;
  }
  std::free(p);
  return hipSuccess;
}
extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return alloc(p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return alloc(p, n); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostFree(void *p) { return release(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  if (copies++ == fail_copy) return hipErrorInvalidValue;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 1;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipLaunchCooperativeKernel(const void *, dim3, dim3, void **, unsigned, hipStream_t) { return hipSuccess; }
}
struct Case {
  int nd;
  int64_t dims[3];
  uint32_t flags;
  int mask;
};
int main() {
  const Case cases[] = {{3, {40, 36, 30}, 0, 0},
                        {2, {90, 70, 1}, PI_CELL_CENTERED, 1},
                        {2, {90, 70, 1}, PI_CELL_CENTERED, 0},
                        {2, {90, 70, 1}, PI_FP64, 1},
                        {3, {256, 160, 110}, 0, 0},
                        {2, {64, 64, 1}, PI_INNER_BICGSTAB, 1}};
  const double h[3] = {1, 1, 1};
  int n = 0;
  for (const Case &c : cases) {
    std::vector<uint8_t> m((size_t)(c.dims[0] * c.dims[1] * c.dims[2]), 1);
    for (int64_t y = 0; y < c.dims[1]; ++y) m[y * c.dims[0] + c.dims[0] / 2] = 0;  // two groups
    auto run = [&](int fm, int fc) {
      mallocs = copies = bad_frees = 0;
      fail_malloc = fm;
      fail_copy = fc;
      const size_t before = held.size();
      pi_plan_t p = nullptr;
      const int rc = pi_plan(c.nd, c.dims, h, c.mask ? m.data() : nullptr, c.flags, &p);
      const int made = p != nullptr;
      if (p) pi_plan_destroy(p);
      std::printf("%d %d %d %d %d %d %d\n", n, fm, fc, rc, made, (int)held.size() - (int)before, bad_frees);
      return std::make_pair(mallocs, copies);
    };
    run(-1, -1);  // sets up what the process keeps
    const auto calls = run(-1, -1);
    for (int k = 0; k < calls.first; ++k) run(k, -1);
    for (int k = 0; k < calls.second; ++k) run(-1, k);
    ++n;
  }
}
"""


def test_a_plan_that_fails_leaves_nothing_and_says_why(tmp_path):
    import paper_2311_16935_amd as pi  # the library is built

    rocm = "/opt/rocm"
    if not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("HIP headers not available")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    # the program's own definitions come before the runtime's in symbol lookup
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-rdynamic", "-I", os.path.join(rocm, "include"), "-I",
           os.path.join(ROOT, "include"), str(src), "-o", str(exe), pi.LIB_PATH, f"-Wl,-rpath,{PKG}",
           f"-Wl,-rpath,{rocm}/lib", f"-Wl,-rpath-link,{rocm}/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    rows = [[int(v) for v in ln.split()] for ln in out.stdout.splitlines()]
    fails = 0
    for case, fm, fc, rc, made, left, bad in rows:
        what = (case, fm, fc, rc)
        assert left == 0 and bad == 0, (what, left, bad)
        if fm < 0 and fc < 0:
            assert rc == pi.PI_OK and made, what
            continue
        fails += 1
        assert not made, what
        assert rc in ((pi.PI_ERR_OOM,) if fm >= 0 else (pi.PI_ERR_DEVICE, pi.PI_ERR_OOM)), what
    assert fails > 100
    # cell-centred plans (cases 1 and 2): the mask's copy, then the ring codes' copies
    # (the codes to the host; numbers, weights and neighbour bits back)
    for case in (1, 2):
        status = {fc: rc for c, _, fc, rc, *_ in rows if c == case and fc >= 0}
        assert [status[k] for k in range(5)] == [pi.PI_ERR_DEVICE] * 5, status
