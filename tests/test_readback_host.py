"""The small read-backs of csrc/readback.h on the CPU, against a HIP runtime of a
few functions that copies only when its event is polled: a call that returns
between the two halves of a read-back must not leave its copy to land in the
mailbox that the thread's next call reads."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

PROGRAM = r"""
#include "readback.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace {
struct { void* dst = nullptr; const void* src; size_t n; int polls; } pending;
bool record_fails = false;
int synchronized = 0;
void land() {
  if (pending.dst) memcpy(pending.dst, pending.src, pending.n);
  pending.dst = nullptr;
}
}  // namespace
extern "C" {
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(&pending);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (pending.dst) { puts("a copy is still pending"); exit(2); }
  pending.dst = d, pending.src = s, pending.n = n, pending.polls = 0;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) {
  return record_fails ? hipErrorUnknown : hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) {
  if (++pending.polls < 3) return hipErrorNotReady;
  land();
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { ++synchronized; land(); return hipSuccess; }
}

int main() {
  using namespace optima;
  const int one = 1, two = 2;
  int got = 0;
  if (read_back(&got, &one, sizeof got, nullptr) != hipSuccess || got != 1) return 3;
  {  // a launch between the halves fails
    PendingReadBack p;
    if (p.begin(&one, sizeof one, nullptr) != hipSuccess) return 4;
  }
  if (pending.dst) return 5;
  if (read_back(&got, &two, sizeof got, nullptr) != hipSuccess || got != 2) return 6;
  record_fails = true;
  if (read_back(&got, &one, sizeof got, nullptr) == hipSuccess || !synchronized || pending.dst)
    return 7;
  if (read_back(&got, &one, kMailboxBytes + 1, nullptr) != hipErrorInvalidValue) return 8;
  puts("ok");
  return 0;
}
"""


@pytest.mark.slow
def test_an_unfinished_read_back_waits_for_its_copy(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not installed")
    src, obj, exe = (str(tmp_path / n) for n in ("t.hip", "t.o", "t"))
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-fPIC",
                    "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2512_13886_amd", "csrc"), "-c", src, "-o", obj],
                   check=True, timeout=300)
    subprocess.run(["g++", obj, "-o", exe, "-lpthread"], check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.returncode, r.stdout)
