"""Host checks of the on-chip solve's exchange (csrc/pi_resident.h): the
header's own functions are compiled for the host; no GPU is used."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(tmp_path, name, program):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / f"{name}.hip", tmp_path / name
    src.write_text(program)
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-I",
                        os.path.join(ROOT, "paper_2311_16935_amd", "csrc"), "-o", str(exe), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120, check=True).stdout
    return [[int(v) for v in ln.split()] for ln in out.splitlines()]


TAGS = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include "pi_resident.h"
int main() {
  for (uint32_t t : {0u, 1u, 2u, 0x7fffffffu, 0xfffffff0u}) {
    for (int i = 0; i < 40; ++i) {
      std::printf("%u %u\n", t, pi::res_next_tag(t));
      t = pi::res_next_tag(t);
    }
  }
}
"""


def test_tags_alternate_between_the_buffers_also_where_they_wrap(tmp_path):
    """A workgroup overwrites a buffer two synchronisations after it was
    written: neighbouring tags must differ in parity, and no tag may be 0,
    which the cleared buffers hold."""
    steps = run_host(tmp_path, "tags", TAGS)
    assert any(t == 0xFFFFFFFF for t, _ in steps)
    for t, n in steps:
        assert n != 0 and (t ^ n) & 1 == 1, (t, n)
    # tags near each other are distinct: a buffer never holds the tag that is awaited next
    for i in range(len(steps) - 3):
        if i % 40 < 37:
            assert len({s[1] for s in steps[i:i + 3]}) == 3


LATE = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstring>
#include "pi_resident.h"
int main() {
  pi::Inst in;
  std::memset(&in, 0, sizeof in);
  in.res_words = 1234;
  for (int done = 0; done < 2; ++done)
    for (int status : {0, 3, 4, 5})
      for (unsigned long long word : {0ull, 1ull}) {
        pi::State st;
        std::memset(&st, 0, sizeof st);
        st.done = done;
        st.status = status;
        st.outer = 7;
        const int late = pi::res_late(st, word);
        std::printf("%d %d %d %d %d %d %lld %lld\n", done, status, (int)word, late, st.done, st.status,
                    (long long)st.outer, (long long)pi::res_late_word(in));
      }
}
"""


def test_a_workgroup_that_gave_up_waiting_decides_the_status(tmp_path):
    """Whatever the workgroup that holds the state has stored, a late
    workgroup's word ends the solve with PI_ERR_DEVICE; without one nothing
    changes.  The word lies behind the exchange words of both parities."""
    rows = run_host(tmp_path, "late", LATE)
    assert len(rows) == 16
    for done, status, word, late, done1, status1, outer, at in rows:
        assert late == word and outer == 7 and at == 2 * 1234
        assert (done1, status1) == ((1, 6) if word else (done, status))


ADMIT = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include "pi_resident.h"
int main() {
  const int wg[] = {200, 100, 60, 56, 1, 256};
  for (int max_wg : {256, 100, 1, 0})
    for (int first = -1; first < 6; ++first) {
      std::vector<int64_t> todo, on;
      int used = 0;
      for (int i = 0; i < 6; ++i) (i == first ? on : todo).push_back(i);
      const bool ok = pi::res_admit(todo, on, max_wg, [&](int64_t i) { return wg[i]; });
      for (int64_t i : on) used += wg[i];
      std::printf("%d %d %d %d %d %d\n", max_wg, first, (int)ok, used, (int)on.size(), (int)todo.size());
    }
}
"""


def test_a_batch_whose_grids_do_not_fit_the_device_ends(tmp_path):
    """Grids go onto the chip in order as far as they fit; where none fits and
    none runs, that is said, so that the loop over the rounds ends."""
    rows = {(m, f): r for m, f, *r in run_host(tmp_path, "admit", ADMIT)}
    assert rows[(256, -1)] == [1, 256, 2, 4]  # 200 and 56: 100 and 60 would not fit beside the first
    assert rows[(256, 5)] == [1, 256, 1, 5]   # one that fills the device
    assert rows[(256, 2)] == [1, 217, 4, 2]   # beside a running one of 60: 100, 56 and 1
    assert rows[(100, -1)] == [1, 100, 1, 5]
    assert rows[(1, -1)] == [1, 1, 1, 5]
    assert rows[(0, -1)] == [0, 0, 0, 6]
    for (m, f), (ok, used, n_on, n_todo) in rows.items():
        assert n_on + n_todo == 6 and ok == (n_on > 0)
