"""The host's table builders when threads or memory run out (no GPU needed).

A small C++ program includes a builder and lets the n-th allocation of the calling thread fail, for
every n: the builder has to return (false, or true where it could do without), never to end the
process.  A second program lets no thread be started: the tables are the same.
"""
import os
import subprocess

import numpy as np
import pytest

import oracle

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_05341_amd", "csrc")

MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include <new>
#include <vector>
static thread_local long g_left = -1;  // allocations of this thread until one fails (-1: none does)
static void *get(size_t n) {
  if (g_left >= 0 && g_left-- == 0) throw std::bad_alloc();
  void *p = malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void *operator new(size_t n) { return get(n); }
void *operator new[](size_t n) { return get(n); }
void operator delete(void *p) noexcept { free(p); }
void operator delete[](void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
void operator delete[](void *p, size_t) noexcept { free(p); }
#include BUILDER
using namespace dd;
static bool build(const std::vector<int32_t> &sh, int nd, int nc, std::vector<uint32_t> *out) {
#ifdef QUADS
  QuadTables t;
  const QuadShifts qs = {sh.data(), nc, 1, 1, nd, nc};
  const bool ok = build_quad_tables(qs, 32, &t);
#else
  GroupTables t;
  const bool ok = build_group_tables(sh.data(), nd, nc, 8, 150000016, &t);
#endif
  g_left = -1;
  *out = t.data;
  return ok;
}
int main(int, char **argv) {
  const int nd = atoi(argv[1]), nc = atoi(argv[2]);
  std::vector<int32_t> sh((size_t)nd * nc);
  if (fread(sh.data(), 4, sh.size(), stdin) != sh.size()) return 2;
  std::vector<uint32_t> want, got;
  if (!build(sh, nd, nc, &want)) return 3;
  int failed = 0;
  for (long n = 0; n < 60; ++n) {
    g_left = n;
    if (!build(sh, nd, nc, &got)) ++failed;
    else if (got != want) return 4;
  }
  printf("%d failed, %zu words\n", failed, want.size());
  return 0;
}
"""
NO_THREADS = r"""
#include <pthread.h>
#include <errno.h>
extern "C" int pthread_create(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *) { return EAGAIN; }
"""


@pytest.mark.parametrize("threads", [True, False])
@pytest.mark.parametrize("builder", ["group_tables.cpp", "quad_tables.cpp"])
def test_builders_return_without_memory_or_threads(builder, threads, tmp_path):
    src = tmp_path / "m.cpp"
    src.write_text((NO_THREADS if not threads else "") + MAIN)
    exe = str(tmp_path / "m")
    flags = ["-DQUADS"] if builder.startswith("quad") else []
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, '-DBUILDER="%s"' % builder, *flags, str(src), "-o", exe],
                   check=True)
    n_dm, n_chan = 520, 512  # several blocks, several threads
    s = np.ascontiguousarray(oracle.shift_table(n_chan, 1500.0, 300.0 / n_chan, 64e-6, 0.0, 0.1, n_dm), dtype=np.int32)
    r = subprocess.run([exe, str(n_dm), str(n_chan)], input=s.tobytes(), capture_output=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    print(r.stdout.decode())
