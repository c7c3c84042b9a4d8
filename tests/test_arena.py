"""The arena a batch's buffers come from, on the host with a device of limited
size: buffers cut from blocks are aligned and never overlap, and what fits one by
one fits (the owner starts again with exact requests where blocks did not)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "chap_internal.h"
#include <cstdio>
#include <map>

static size_t g_room = 0, g_used = 0;
static std::map<void*, size_t> g_live;
static char* g_next = (char*)0x100000;
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  n = (n + 4095) / 4096 * 4096;
  if (g_used + n > g_room) return hipErrorOutOfMemory;
  *p = g_next;
  g_next += n;
  g_used += n;
  g_live[*p] = n;
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
  g_used -= g_live.at(p);
  g_live.erase(p);
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError(void) { return hipSuccess; }

int main() {
  int bad = 0, again = 0;
  for (size_t n : {3000, 40000, 333333, 420000, 520001, 700000, 840000, 1000003}) {
    // a walk's buffers: four points, the tabu list, rows, records, a trace
    const size_t sizes[] = {8 * n, 8 * n, 8 * n, 8 * n, 4 * n, 8 * n, 192, 9600, 32 * n / 200, 544, 4 * n, n};
    const int walks = n < 50000 ? 400 : 60;
    size_t exact = 0;
    for (size_t z : sizes) exact += (z + 4095) / 4096 * 4096;
    exact *= walks;
    for (double room : {1.0, 1.02, 1.1}) {
      g_room = (size_t)(exact * room);
      chap::DeviceArena A;
      A.chunk = (size_t)32 << 20;
      auto fill = [&]() {
        std::map<char*, size_t> got;
        for (int w = 0; w < walks; ++w)
          for (size_t z : sizes) {
            char* p = nullptr;
            if (A.alloc(&p, z) != hipSuccess) return false;
            if ((size_t)p % 256) ++bad;
            auto after = got.lower_bound(p);
            if (after != got.end() && p + z > after->first) ++bad;
            if (after != got.begin() && std::prev(after)->first + std::prev(after)->second > p) ++bad;
            got[p] = z;
          }
        return true;
      };
      bool ok = fill();
      if (!ok && A.retry_exact()) {
        ++again;
        ok = fill();
      }
      bad += ok && !A.retry_exact() ? 0 : 1;
      printf("n=%zu room %.2f: %s, used %.3f\n", n, room, ok ? "fits" : "DOES NOT FIT", (double)g_used / exact);
    }
  }
  if (again == 0) ++bad;  // some of these need the second attempt
  return (bad || !g_live.empty()) ? 1 : 0;
}
"""


@pytest.mark.skipif(not shutil.which(HIPCC), reason="needs hipcc")
def test_batch_buffers_fit(tmp_path):
    src, exe = tmp_path / "arena.hip", tmp_path / "arena"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2605_05086_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0, out.stdout
