"""The once-per-kernel LDS reservation, compiled for the host against a stand-in for the runtime call."""
import os
import subprocess

from paper_2411_01075_amd import build

PROGRAM = r"""
#include "reserve_lds.h"
#include <cassert>
#include <cstdarg>
#include <map>

std::map<const void*, int> reserved;
int calls = 0, failures = 0;
extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int bytes) {
  ++calls;
  if (failures > 0) { --failures; return hipErrorInvalidValue; }
  reserved[f] = bytes;
  return hipSuccess;
}
int cephalo::fail(int code, const char*, ...) { return code; }

int touched = 0;
void narrow(int i) { touched += i; }        // three kernels of one signature
void wide(int i) { touched -= i; }
void refused(int i) { touched *= i; }

int main() {
  using cephalo::reserve_lds;
  assert(reserve_lds<narrow>("test", 32768) == CEPHALO_OK);
  assert(reserve_lds<wide>("test", 131072) == CEPHALO_OK);
  assert(reserved[(const void*)narrow] == 32768 && reserved[(const void*)wide] == 131072);
  assert(reserve_lds<narrow>("test", 32768) == CEPHALO_OK && calls == 2);      // once
  failures = 1;                                                                // a failure is reported and tried again
  assert(reserve_lds<refused>("test", 65536) == CEPHALO_EHIP && reserved.count((const void*)refused) == 0);
  assert(reserve_lds<refused>("test", 65536) == CEPHALO_OK && reserved[(const void*)refused] == 65536 && calls == 4);
  return 0;
}
"""


def test_every_kernel_gets_its_own_reservation(tmp_path):
    src, exe = tmp_path / "reserve.cpp", tmp_path / "reserve"
    src.write_text(PROGRAM)
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + build.CSRC, str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True)


def test_no_other_reservation():
    """The attribute is set in one place."""
    found = [f for f in sorted(os.listdir(build.CSRC)) if f.endswith((".hip", ".h")) and "hipFuncSetAttribute(" in open(os.path.join(build.CSRC, f)).read()]
    assert found == ["reserve_lds.h"]
