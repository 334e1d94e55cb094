"""The quad kernel's tables, executed word by word on the CPU (no GPU needed).

A small C++ program includes the library's table builder, runs every record and sum entry the
way the kernel does (every LDS access checked) and compares the outputs, bit for bit, with
the float sums row by row in the same order, forward and adjoint.
"""
import os
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2311_05341_amd", "csrc")

SIM = r"""
#include "quad_tables.cpp"
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
using namespace dd;
#define CHECK(c) do { if (!(c)) { printf("FAILED line %d: %s\n", __LINE__, #c); return 1; } } while (0)
static const int64_t kRowLen = 1400;
static float x(int64_t k, int64_t t) {  // zeros outside the row
  if (t < 0 || t >= kRowLen) return 0.0f;
  uint64_t h = (uint64_t)k * 0x9E3779B97F4A7C15ull + (uint64_t)t * 0xD1342543DE82EF95ull;
  h ^= h >> 29; h *= 0xBF58476D1CE4E5B9ull; h ^= h >> 32;
  return (float)(int32_t)(h & 0xFFFFFF) * 1.37e-7f - 1.0f;
}
int main(int argc, char **argv) {
  const int n_dm = atoi(argv[1]), n_chan = atoi(argv[2]), adj = atoi(argv[3]), rows = atoi(argv[4]);
  std::vector<int32_t> sh((size_t)n_dm * n_chan);
  if (fread(sh.data(), 4, sh.size(), stdin) != sh.size()) return 2;
  const QuadShifts qs = {sh.data(), adj ? 1 : n_chan, adj ? n_chan : 1, adj ? -1 : 1, adj ? n_chan : n_dm,
                         adj ? n_dm : n_chan};
  QuadTables t;
  if (guess_quad_cost(qs, rows) >= 1e300) { printf("refused\n"); return 0; }
  if (!build_quad_tables(qs, rows, &t)) { printf("refused\n"); return 0; }
  const uint32_t *D = t.data.data();
  const int R = rows / kQuadWaves, nq = (qs.n_rows + 3) / 4, W = 2 * kQuadSetBytes / 4;
  CHECK(t.rows == rows && t.n_blk == (qs.n_out + rows - 1) / rows && t.n_quads % 2 == 0 && t.n_quads >= nq);
  CHECK(2 * kQuadSetBytes <= 160 * 1024);
  for (int b = 0; b < t.n_blk; ++b) {
    const int t0 = (b % 3) * kQuadWin;
    std::vector<float> lds(W), part(rows * kQuadWin, 0.0f), tot(rows * kQuadWin, 0.0f);
    std::vector<int> built(W, -1);
    QuadBlock qb;
    memcpy(&qb, D + b * (sizeof qb / 4), sizeof qb);
    const uint32_t *steps = D + qb.step_first;
    CHECK(qb.step_first + qb.n_steps * kQuadStepWords <= t.sum_off);
    int quad = 0;
    size_t rec[kQuadWaves];
    for (int w = 0; w < kQuadWaves; ++w) rec[w] = (size_t)qb.rec_first[w] * kQuadRecWords;
    for (int s = 0; s < (int)qb.n_steps; ++s) {
      const uint32_t *st = steps + s * kQuadStepWords;
      CHECK((int)st[0] == quad && st[1] >= 1 && (int)st[1] * (R / 2) <= 64);
      for (int w = 0; w < kQuadWaves; ++w) {
        int task = -1, start[4], done = 0;
        for (bool last = false; !last; rec[w] += kQuadRecWords) {
          CHECK(rec[w] + 4 * kQuadRecWords <= t.op_off);  // the kernel loads three records ahead
          const uint32_t *r = D + rec[w];
          last = r[0] & kQuadLast;
          const size_t oo = t.op_off + (size_t)(r[0] & ~kQuadLast) * kQuadOpWords;
          CHECK(oo + kQuadOpWords <= t.sum_off);
          const uint32_t *op = D + oo;
          const int stride = op[0] & 0x7FFF, k0 = 64 * quad_lane_words(rows) * (int)(r[1] & 0xFFFF);
          const int words = std::min(stride - k0, 64 * quad_lane_words(rows));
          uint32_t dst = r[1] >> 16;
          for (int q = 0; q < kQuadOps; ++q) {
            const uint32_t kind = op[1] >> (4 * q);
            const int c = kind & 3;
            if (c == 0 && words) task = (int)(op[0] >> 15), done = 0;
            start[c] = t0 + k0 + (int)op[2] + (int)(op[3 + q / 2] >> (16 * (q % 2)) & 0xFFFF);
            CHECK(start[c] >= t0 + qb.lo && start[c] + 64 * quad_lane_words(rows) <= t0 + qb.hi);
            CHECK(!words || !(kind & kQuadNone) == (4 * (int)(op[0] >> 15) + c < qs.n_rows));
            done |= 1 << c;
            if (!(kind & kQuadWrite)) continue;
            CHECK(done == 15 && words > 0 && task == (int)(op[0] >> 15) && task >= quad && task < quad + (int)st[1]);
            for (int i = 0; i < words; ++i) {
              const uint32_t a = dst + i;
              CHECK(a < (uint32_t)W && (int)(a * 4 / kQuadSetBytes) == (s & 1) && built[a] != s);
              built[a] = s;
              float v = x(4 * task, start[0] + i);
              for (int e = 1; e < 4; ++e) v += 4 * task + e < qs.n_rows ? x(4 * task + e, start[e] + i) : 0.0f;
              lds[a] = v;
            }
            dst += (uint32_t)stride;
          }
        }
      }
      for (int q = 0; q < (int)st[1]; ++q, ++quad)
        for (int d = 0; d < rows; ++d) {
          const size_t e = (((size_t)b * kQuadWaves + d / R) * t.n_quads + quad) * R + d % R;
          CHECK(t.sum_off + e / 2 + 64 <= t.data.size());
          const uint32_t a = D[t.sum_off + e / 2] >> (16 * (e & 1)) & 0xFFFF;
          CHECK(a + kQuadWin <= (uint32_t)W);
          for (int i = 0; i < kQuadWin; ++i) {
            CHECK(built[a + i] == s);
            float &p = part[d * kQuadWin + i];
            p += lds[a + i];
            if (quad % 8 == 7 || quad == nq - 1) tot[d * kQuadWin + i] += p, p = 0.0f;
          }
        }
    }
    CHECK(quad == nq);
    for (int w = 0; w < kQuadWaves; ++w) CHECK(D[rec[w]] == kQuadLast && !D[rec[w] + 2] && !D[t.op_off] && !D[t.op_off + 1]);  // two idle records end each stream
    for (int d = 0; d < rows && b * rows + d < qs.n_out; ++d)
      for (int i = 0; i < kQuadWin; ++i) {
        float want = 0, pt = 0;
        for (int k = 0; k < 4 * nq; k += 4) {
          float v = 0;
          for (int c = 0; c < 4; ++c) {
            const int o = b * rows + d;
            const float y = k + c < qs.n_rows
                                ? x(k + c, t0 + i + qs.sign * (int64_t)sh[o * qs.out_stride + (k + c) * qs.row_stride]) : 0.0f;
            v = c ? v + y : y;
          }
          pt += v;
          if (k / 4 % 8 == 7 || k / 4 == nq - 1) want += pt, pt = 0;
        }
        CHECK(!memcmp(&want, &tot[d * kQuadWin + i], 4));
      }
  }
  printf("ok\n");
  return 0;
}
"""


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    d = tmp_path_factory.mktemp("quad_sim")
    src = d / "sim.cpp"
    src.write_text(SIM)
    exe = str(d / "sim")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, str(src), "-o", exe], check=True)
    return exe


def _run(sim, shift, adjoint, rows):
    s = np.ascontiguousarray(shift, dtype=np.int32)
    r = subprocess.run([sim, str(s.shape[0]), str(s.shape[1]), str(int(adjoint)), str(rows)], input=s.tobytes(),
                       capture_output=True, timeout=300)
    assert r.returncode == 0, r.stdout.decode()
    return r.stdout.decode().strip()


# single rows and outputs, a partial last quad and block, one step and many, no delay at all,
# sums of more than one chunk, delays in no order
@pytest.mark.parametrize("rows", [32, 64])
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("args", [(1, 1, 0.0, 1.0), (7, 3, 0.0, 2.0), (130, 33, 0.0, 0.0), (203, 77, 3.0, 0.5),
                                  (256, 65, 50.0, 0.1), (512, 40, 0.0, 0.25)])
def test_tables_sum_rows_in_order(sim, args, adjoint, rows):
    n_chan, n_dm, start, step = args
    s = oracle.shift_table(n_chan, 1500.0, 300.0 / n_chan, 256e-6, start, step, n_dm)
    assert _run(sim, s, adjoint, rows) == "ok"
    if n_chan == 256:
        mixed = s[:, np.random.default_rng(2).permutation(n_chan)[:64]]
        assert _run(sim, mixed[:, :8], adjoint, rows) in ("ok", "refused")


def test_wide_spreads_are_refused(sim):
    s = oracle.shift_table(64, 190.0, 70.0 / 64, 327.68e-6, 0.0, 2.0, 64)
    for adjoint in (False, True):
        assert _run(sim, s, adjoint, 64) == "refused"
