"""The opt-in for more than 64 KB of dynamic LDS, on the host with a stand-in runtime that keeps it per
kernel and device: every device of a process gets its own, calls are made only where a size exceeds the
device's largest, a failed one is made again, and threads never leave less than the largest size."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <assert.h>
#include <stdio.h>
#include <chrono>
#include <map>
#include <thread>
#include <utility>
#include <vector>
#include "hq_lds.h"

static thread_local int device = 0;
static std::mutex mu;
static std::map<std::pair<const void*, int>, int> attribute;
static int calls = 0;
static hipError_t result = hipSuccess;

extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int v) {
  std::this_thread::sleep_for(std::chrono::microseconds(1000 - v % 1000));  // smaller sizes take longer
  std::lock_guard<std::mutex> lock(mu);
  ++calls;
  if (result == hipSuccess) attribute[{f, device}] = v;
  return result;
}

static void launch(const void* f, int bytes, hq_lds_granted& g) {
  assert(hq_allow_lds(f, bytes, g) == 0);
  std::lock_guard<std::mutex> lock(mu);
  if (bytes > 65536) assert((attribute[{f, device}]) >= bytes);
}

int main() {
  static hq_lds_granted g, h, t;
  int k1, k2, k3;
  launch(&k1, 65536, g);
  assert(calls == 0);
  for (int dev : {0, 1, 0, 7, 1, 63, 64, 64}) {
    device = dev;
    launch(&k1, 100000, g);
    launch(&k1, 70000, g);
    launch(&k2, 120000, h);
  }
  assert(calls == 2 * 4 + 2 * 3);  // once per kernel and device 0, 1, 7 and 63, each time past the table
  device = 0;
  launch(&k1, 100001, g);
  result = hipErrorInvalidValue;
  assert(hq_allow_lds(&k1, 150000, g) == result);
  result = hipSuccess;
  launch(&k1, 150000, g);
  for (int rep = 0; rep < 40; ++rep) {
    std::vector<std::thread> th;
    for (int i = 0; i < 8; ++i)
      th.emplace_back([&, i] { device = i & 1; launch(&k3, 66000 + 1000 * rep + 100 * ((i * 5 + rep) % 8), t); });
    for (auto& x : th) x.join();
    for (int i = 0; i < 8; ++i)
      assert((attribute[{&k3, i & 1}]) >= 66000 + 1000 * rep + 100 * ((i * 5 + rep) % 8));
  }
  puts("ok");
}
"""


def test_opt_in_per_device(tmp_path):
    src, exe = tmp_path / "lds.cpp", tmp_path / "lds"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2606_23406_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True, timeout=120)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout == "ok\n"
