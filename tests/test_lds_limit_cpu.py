"""The LDS limit of a kernel is raised on every device that launches it (host logic).

A host program built from the library's header records which devices the setting is made on:
once each, whatever the order of the launches, again after a failure, and from several threads at
once without a device left out. No GPU is needed.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_06640_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

PROGRAM = r"""
#include "lds_limit.hpp"
#include <cstdio>
#include <thread>
#include <vector>
using seis::PerDevice;
int main() {
  int bad = 0;
  {
    PerDevice p;
    std::vector<int> made(100, 0);
    auto on = [&](int d, hipError_t st) { return p.ensure(d, [&] { ++made[d]; return st; }); };
    bad += on(3, hipErrorInvalidValue) != hipErrorInvalidValue;  // not kept
    for (int i = 0; i < 2; ++i)
      for (int d : {0, 1, 3, 63}) bad += on(d, hipSuccess) != hipSuccess;
    bad += made[0] != 1 || made[1] != 1 || made[3] != 2 || made[63] != 1 || made[2] != 0;
    bad += on(2, hipErrorOutOfMemory) != hipErrorOutOfMemory;
    for (int i = 0; i < 2; ++i) bad += on(70, hipSuccess) != hipSuccess;  // beyond the record: every time
    bad += made[70] != 2;
  }
  {
    PerDevice p;
    std::atomic<int> made[8] = {};
    std::vector<std::thread> t;
    for (int d = 0; d < 8; ++d)
      t.emplace_back([&, d] {
        for (int i = 0; i < 100; ++i) (void)p.ensure(d, [&] { ++made[d]; return hipSuccess; });
      });
    for (auto& x : t) x.join();
    for (auto& m : made) bad += m != 1;
  }
  std::printf("violations %d\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_once_on_every_device(tmp_path):
    src, exe = tmp_path / "lds_check.cpp", tmp_path / "lds_check"
    src.write_text(PROGRAM)
    build = subprocess.run([HIPCC, "-O1", "-std=c++17", f"-I{CSRC}", "-x", "hip", "--offload-arch=gfx950", str(src),
                            "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "violations 0" in run.stdout, run.stdout + run.stderr


def test_every_kernel_with_more_than_the_default_uses_it():
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".hpp", ".cpp")) and name != "lds_limit.hpp":
            with open(os.path.join(CSRC, name)) as f:
                assert "MaxDynamicSharedMemorySize" not in f.read(), name
