"""The limit of a kernel's dynamic LDS belongs to the kernel on one device: a process that uses a second device has to raise
it there as well.  The helper that every launch goes through, built for the host against a HIP runtime of this file's own that
counts what it is asked."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_09026_amd", "csrc")
PROGRAM = r"""
#include "lds_limit.h"
#include <cstdio>
static int device, asked;
static hipError_t answer = hipSuccess;
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute a, int bytes) {
  if (a != hipFuncAttributeMaxDynamicSharedMemorySize || bytes != 81920) return hipErrorInvalidValue;
  ++asked;
  return answer;
}
static unsigned long done;
static int on(int d) {                       // how often the runtime is asked by one launch there, or -1
  device = d; asked = 0;
  return mg::raise_lds_limit(&done, 81920, done) == hipSuccess ? asked : -1;
}
int main() {
  int n[10], i = 0;
  n[i++] = on(0); n[i++] = on(0);            // once
  n[i++] = on(3); n[i++] = on(3); n[i++] = on(0);
  answer = hipErrorInvalidValue;
  n[i++] = on(5);                            // refused: reported, and asked again
  answer = hipSuccess;
  n[i++] = on(5); n[i++] = on(63);
  n[i++] = on(64); n[i++] = on(64);          // past the bits: every time
  for (int k = 0; k < i; ++k) printf("%d ", n[k]);
}
"""


def test_limit_is_raised_on_every_device(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                           "-o", str(exe), str(src)])
    assert subprocess.check_output([str(exe)], text=True).split() == "1 0 1 0 0 -1 1 1 1 1".split()


def test_no_launch_raises_it_by_itself():
    """Kernels with rings of several sizes set the attribute on every launch; all others go through the helper."""
    direct = [f for f in sorted(os.listdir(CSRC)) if f.endswith((".hip", ".h"))
              and "hipFuncSetAttribute(" in open(os.path.join(CSRC, f)).read()]
    assert direct == ["attention_mfma.hip", "lds_limit.h"]
