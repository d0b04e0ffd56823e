"""moc_graph_upload when memory runs out (csrc/moc_graph.hip): the source's host part, compiled for the CPU against a
small stand-in for the HIP runtime whose allocations, like operator new, fail at a chosen call.  No GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2304_14463_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include "moc_internal.h"

static long new_left = -1, dev_left = -1, new_live = 0, dev_live = 0;   // calls until one fails; allocations in use
void* operator new(size_t n) {
  if (new_left >= 0 && new_left-- == 0) throw std::bad_alloc();
  ++new_live;
  return malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { if (p) { --new_live; free(p); } }
void operator delete(void* p, size_t) noexcept { operator delete(p); }

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = 160 * 1024;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  if (dev_left >= 0 && dev_left-- == 0) return hipErrorOutOfMemory;
  ++dev_live;
  *p = malloc(n);
  return hipSuccess;
}
hipError_t hipFree(void* p) { if (p) { --dev_live; free(p); } return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) { memcpy(to, from, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes*, const void*) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
}
int moc_node_stride(int C) { return C <= 2 ? C : 1; }
int moc_eval_lds_bytes(int, int, int, int) { return 1; }
bool moc_eval_shape(int n, int m, int, int* nt, int* per_lane, int* used) {
  *nt = 64;
  *per_lane = *used = (m + 63) / 64 + 1;
  return n > 0;
}
int moc_eval_prepare(const moc_graph* g) {
  int per_cu = 0;
  return moc_kernel_occupancy(g, &per_cu, 64, 64, false, &per_cu);
}
int moc_eval_static_setup(int) { return MOC_OK; }

int main() {
  const int32_t in_ptr[] = {0, 0, 1, 3, 5, 7}, in_idx[] = {0, 0, 1, 1, 2, 3, 3}, size[] = {1, 2, 3, 4, 5}, dur[] = {1, 1, 1, 1, 1};
  long first = 1;   // the first handle of the process leaves a list of prepared kernels
  for (int which = 0; which < 2; ++which)
    for (long k = 0;; ++k) {
      long& left = which ? dev_left : new_left;
      const long before_new = new_live;
      moc_graph* g = nullptr;
      left = k;
      const int rc = moc_graph_upload(5, in_ptr, in_idx, size, dur, 10, 2, &g);
      const bool all = left >= 0;   // no call failed
      left = -1;
      if (rc == MOC_OK) {           // (a sort does without the buffer it is refused)
        moc_graph_free(g);
        if (dev_live != 0 || new_live - before_new > first) return printf("%ld device and %ld host allocations left by a handle\n", dev_live, new_live - before_new), 1;
        first = 0;
        if (!all) continue;
        printf("%s: %ld calls\n", which ? "device" : "host", k);
        break;
      }
      if (rc != MOC_ENOMEM || g != nullptr) return printf("code %d at %ld\n", rc, k), 1;
      if (dev_live != 0 || new_live - before_new != 0) return printf("%s call %ld: %ld device and %ld host allocations left\n", which ? "device" : "host", k, dev_live, new_live - before_new), 1;
    }
  return 0;
}
"""


def test_nothing_is_left_behind_when_memory_runs_out(tmp_path):
    (tmp_path / "upload.hip").write_text(PROGRAM)
    flags = ["--offload-host-only", "-fPIC", "-O1", "-std=c++17", "-Wno-unused-result", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    for name, source in (("main", tmp_path / "upload.hip"), ("graph", os.path.join(CSRC, "moc_graph.hip"))):
        subprocess.run(["hipcc", *flags, "-c", "-o", str(tmp_path / f"{name}.o"), str(source)], check=True)
    subprocess.run(["g++", "-o", str(tmp_path / "upload"), str(tmp_path / "main.o"), str(tmp_path / "graph.o")], check=True)
    proc = subprocess.run([str(tmp_path / "upload")], capture_output=True, text=True, timeout=60)
    assert proc.returncode == 0, proc.stdout + proc.stderr
    calls = dict(line.split(": ") for line in proc.stdout.splitlines())
    assert int(calls["host"].split()[0]) > 10 and int(calls["device"].split()[0]) >= 9
