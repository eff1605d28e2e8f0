"""The reductions' and the integration's vector load (load_vec) reads the values
asked for and nothing past them: compiled for the host and run on arrays that
end where a page without access begins."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

SOURCE = r"""
#include <stdio.h>
#include <sys/mman.h>
#include <unistd.h>
#include "mr_internal.h"

template <typename T, int V>
__attribute__((noinline)) void load(const T* p, T* o) { mr::load_vec<T, V>(p, o); }

template <typename T, int V>
int check() {
  const long page = sysconf(_SC_PAGESIZE);
  char* m = (char*)mmap(nullptr, 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (m == (char*)MAP_FAILED || mprotect(m + page, page, PROT_NONE) != 0) return 1;
  T* p = (T*)(m + page) - V;
  for (int q = 0; q < V; ++q) p[q] = T(q + 1);
  T o[V];
  printf("case load_vec %d bytes x %d\n", (int)sizeof(T), V);
  fflush(stdout);
  load<T, V>(p, o);
  int bad = 0;
  for (int q = 0; q < V; ++q) bad += o[q] != T(q + 1);
  munmap(m, 2 * page);
  return bad;
}

int main() {
  const int bad = check<float, 1>() + check<float, 2>() + check<float, 3>() + check<float, 4>() + check<double, 1>() +
                  check<double, 2>() + check<double, 3>() + check<double, 4>();
  if (!bad) printf("loads ok\n");
  return bad;
}
"""


def test_load_vec_reads_nothing_past_its_values(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("needs hipcc")
    src, exe = tmp_path / "load_vec.hip", str(tmp_path / "load_vec")
    src.write_text(SOURCE)
    # (no optimisation: the host's vectoriser would pick loads of its own)
    cmd = [HIPCC, "-O0", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_1805_03426_amd", "csrc"), str(src), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "loads ok" in r.stdout, (r.returncode, r.stdout[-200:])
