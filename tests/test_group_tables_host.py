"""The group-sum kernel's tables, executed word by word on the CPU (no GPU needed).

A small C++ program includes the library's table builder, runs every record and sum entry the
way the kernel does (with every LDS access, window read and 16-bit sum checked) and compares
the outputs with the plain channel sum, over plans at the edges of what the tables accept.
"""
import os
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2311_05341_amd", "csrc")

SIM = r"""
#include "group_tables.cpp"
#include <stdio.h>
#include <stdlib.h>
using namespace dd;
#define CHECK(c) do { if (!(c)) { printf("FAILED line %d: %s\n", __LINE__, #c); return 1; } } while (0)
static uint32_t x(uint32_t c, int64_t t, uint32_t m) {
  uint64_t h = (uint64_t)c * 0x9E3779B97F4A7C15ull + (uint64_t)t * 0xD1342543DE82EF95ull;
  h ^= h >> 29; h *= 0xBF58476D1CE4E5B9ull; h ^= h >> 32;
  return (h & 7) == 0 ? m : (uint32_t)(h >> 8) % (m + 1);  // the largest value often
}
int main(int argc, char **argv) {
  const int n_dm = atoi(argv[1]), n_chan = atoi(argv[2]), bits = atoi(argv[3]);
  const uint32_t packed_max = bits == 16 ? 0 : (1u << bits) - 1, m = packed_max ? packed_max : 65535;
  const int kGrpRows = group_rows(bits), kSumWords = group_sum_words(bits);
  const int64_t pitch = 150000016;  // offsets far past 32 bits
  std::vector<int32_t> sh((size_t)n_dm * n_chan);
  if (fread(sh.data(), 4, sh.size(), stdin) != sh.size()) return 2;
  GroupTables t;
  if (!build_group_tables(sh.data(), n_dm, n_chan, bits, pitch, &t)) { printf("refused\n"); return 0; }
  CHECK(t.lds_bytes <= 2 * kGrpSetBytes && 2 * kGrpSetBytes + kGrpZeroBytes + kGrpTrashBytes <= 160 * 1024);
  const uint32_t *D = t.data.data();
  CHECK(!memcmp(D, &t.head, sizeof t.head));
  const int64_t total = (int64_t)t.data.size();
  for (int b = 0; b < t.n_blk; ++b) {
    const GroupBlock *gb = (const GroupBlock *)(D + kGrpHeadWords) + b;
    const int halves = packed_max ? 2 : 1;
    std::vector<int64_t> lds[2];
    const uint32_t zero = 2 * kGrpSetBytes;
    std::vector<int> step_of(zero / 4 + kGrpWin, -1);
    for (int h = 0; h < halves; ++h) lds[h].assign(zero / 4 + kGrpWin, 0);
    std::vector<int64_t> out[2], acc[2];
    for (int h = 0; h < halves; ++h) out[h].assign(kGrpRows * kGrpWin, 0), acc[h].assign(kGrpRows * kGrpWin, 0);
    uint32_t pos[kGrpWaves] = {};
    for (int step = 0; step < (int)gb->n_steps; ++step) {
      for (int wave = 0; wave < kGrpWaves; ++wave) {
        std::vector<int64_t> P[2], S[2];
        int phase = -1;
        for (bool last = false; !last;) {
          const int64_t ro = t.head.rec_off + ((int64_t)gb->rec_first[wave] + pos[wave]++) * kGrpRecWords;
          CHECK(ro + 4 * kGrpRecWords <= t.head.op_off);  // the kernel loads three records ahead
          const uint32_t *r = D + ro;
          last = (r[1] & kRecLast) != 0;
          const int lanes = (int)(r[1] >> 8) & 255, k0 = (int)(r[1] >> 16), n = 4 * lanes;
          CHECK(lanes <= 63 && k0 % kGrpChunk == 0);
          if (r[1] & kRecStart)
            for (int h = 0; h < halves; ++h) P[h].assign(n, 0), S[h].assign(n, 0);
          uint32_t slot = r[2];
          const int64_t oo = t.head.op_off + (int64_t)r[0] * kGrpBlockWords;
          CHECK(oo + kGrpBlockWords <= t.head.sum_off);
          const uint32_t *o = D + oo;
          const int64_t base = (int64_t)((uint64_t)o[1] << 32 | o[0]);
          for (int q = 0; q < kGrpOps; ++q) {
            const uint32_t w = o[2 + q / 4] >> (8 * (q % 4)) & 255;
            int64_t off = base + o[4 + q];
            const int64_t c = (off + pitch / 2) / pitch;  // rows are longer than any delay here
            off -= c * pitch;
            const int64_t s = off * 8 / bits + (w & 3);
            CHECK(off % (bits == 4 ? 2 : 4) == 0 && (bits != 16 || !(w & 2)));
            CHECK(c >= 0 && c < n_chan && off * 8 / bits >= t.head.lo && s + k0 + kGrpChunk + 8 <= t.head.hi);
            const bool move = (w & kOpMove) != 0;
            if (!(w & (kOpMove | kOpAdd))) { CHECK(!(w & kOpWrite)); continue; }
            CHECK(lanes > 0 && (int)P[0].size() == n && move == !(w & kOpAdd));
            for (int h = 0; h < halves; ++h)
              for (int k = 0; k < n; ++k) {
                const int64_t a = x(c, s + k0 + k + h * kGrpWin, m), u = x(c, s + 1 + k0 + k + h * kGrpWin, m);
                (move ? P : S)[h][k] += !move ? a : w & kOpDown ? a - u : u - a;
                if (!move && (w & kOpFold)) P[h][k] += S[h][k], S[h][k] = 0;
              }
            if (!move) {  // adds are folded in phase by phase before a pattern is written
              if (phase < 0) phase = (int)(w & 3);
              CHECK(phase == (int)(w & 3));
              if (w & kOpFold) phase = -1;
            }
            // a move stores P in the row at hand whether it is finished or not
            CHECK(!move || slot + 4 * n <= (uint32_t)t.lds_bytes);
            CHECK(!move || slot / kGrpSetBytes == (uint32_t)(step & 1));
            if (w & kOpWrite) {
              CHECK(phase < 0 && slot % 16 == 0 && slot + 4 * n <= (uint32_t)t.lds_bytes);
              CHECK(slot / kGrpSetBytes == (uint32_t)(step & 1) && (slot + 4 * n - 1) / kGrpSetBytes == (uint32_t)(step & 1));
              for (int k = 0; k < n; ++k) {
                CHECK(step_of[slot / 4 + k] != step);  // no word is built twice in a step
                step_of[slot / 4 + k] = step;
                for (int h = 0; h < halves; ++h) lds[h][slot / 4 + k] = P[h][k];
              }
              slot += r[3];
            }
          }
        }
      }
      int pair = 0;
      for (bool last = false; !last; ++pair) {
        const int R = group_rows_per_wave(bits);
        CHECK(pair < kGrpStepPairs);
        uint32_t marks = 0;
        for (int d = 0; d < kGrpRows; ++d) {
          const int64_t eo = t.head.sum_off + gb->sum_first + ((int64_t)step * kGrpWaves + d / R) * kSumWords + pair * 2 * R;
          CHECK(eo - pair * 2 * R + 64 <= total);
          if (d == 0) marks = D[eo] & ~kSumOffset;
          CHECK((D[eo] & ~kSumOffset) == marks);  // every wave sees the same marks
          for (int half = 0; half < 2; ++half) {
            const uint32_t e = D[eo + half * R + d % R];
            CHECK((half == 0 && d % R == 0) || !(e & ~kSumOffset));
            const uint32_t o = e & kSumOffset;
            CHECK(o == zero || (o % 4 == 0 && o + 4 * kGrpWin <= (uint32_t)t.lds_bytes));
            for (int k = 0; k < kGrpWin; ++k) {
              CHECK(o == zero || step_of[o / 4 + k] == step);  // built for this step
              for (int h = 0; h < halves; ++h) {
                acc[h][d * kGrpWin + k] += lds[h][o / 4 + k];
                if (packed_max) CHECK(lds[h][o / 4 + k] >= 0 && acc[h][d * kGrpWin + k] <= 65535);
              }
            }
          }
        }
        last = (marks & kSumLast) != 0;
        if (!packed_max || (marks & kSumFlush))
          for (int h = 0; h < halves; ++h)
            for (int i = 0; i < kGrpRows * kGrpWin; ++i) out[h][i] += acc[h][i], acc[h][i] = 0;
      }
    }
    for (int h = 0; h < halves; ++h)
      for (int64_t v : acc[h]) CHECK(v == 0);  // the last group flushes
    for (int wave = 0; wave < kGrpWaves; ++wave) {  // one idle record ends each stream
      const int64_t ro = t.head.rec_off + ((int64_t)gb->rec_first[wave] + pos[wave]) * kGrpRecWords;
      CHECK(ro + 4 * kGrpRecWords <= t.head.op_off && D[ro] == 0 && D[ro + 1] == kRecLast);
    }
    for (int d = 0; d < kGrpRows && b * kGrpRows + d < n_dm; ++d)
      for (int h = 0; h < halves; ++h)
        for (int k = 0; k < kGrpWin; k += 7) {
          int64_t want = 0;
          const int32_t *row = &sh[(size_t)(b * kGrpRows + d) * n_chan];
          for (int c = 0; c < n_chan; ++c) want += x(c, (int64_t)k + h * kGrpWin + row[c], m);
          CHECK(out[h][d * kGrpWin + k] == want);
        }
  }
  printf("ok\n");
  return 0;
}
"""


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    d = tmp_path_factory.mktemp("group_sim")
    src = d / "sim.cpp"
    src.write_text(SIM)
    exe = str(d / "sim")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, str(src), "-o", exe], check=True)
    return exe


def _run(sim, shift, bits):
    s = np.ascontiguousarray(shift, dtype=np.int32)
    r = subprocess.run([sim, str(s.shape[0]), str(s.shape[1]), str(bits)], input=s.tobytes(),
                       capture_output=True, timeout=300)
    assert r.returncode == 0, r.stdout.decode()
    return r.stdout.decode().strip()


def _table(n_chan, band, dm_start, dm_step, n_dm, f_high=1500.0, t_us=64.0):
    return oracle.shift_table(n_chan, f_high, band / n_chan, t_us * 1e-6, dm_start, dm_step, n_dm)


# 8-bit, 4-bit and 16-bit sums; DM blocks with a tail, single rows and channels, bands that end in
# a partial group, spreads from none to more than a pattern row holds
@pytest.mark.parametrize("bits", [8, 4, 16])
@pytest.mark.parametrize("args", [
    (1, 20.0, 0.0, 1.0, 1), (3, 30.0, 0.0, 2.0, 33), (64, 300.0, 0.0, 0.0, 5), (203, 182.7, 3.0, 0.77, 77),
    (257, 300.0, 300.0, 0.1, 64), (1000, 300.0, 0.0, 0.25, 40), (1024, 300.0, 900.0, 1.0, 32), (2048, 300.0, 0.0, 2.0, 33), (4096, 300.0, 0.0, 0.1, 32)])
def test_tables_sum_every_channel_once(sim, args, bits):
    assert _run(sim, _table(*args), bits) == "ok"


@pytest.mark.parametrize("bits", [8, 16])
def test_unordered_frequencies_and_wide_spreads(sim, bits):
    """Delays that are not monotone in the channel (windows may start before the tile), and a
    plan whose rows spread over more samples than a pattern row holds: refused."""
    rng = np.random.default_rng(5)
    s = _table(96, 300.0, 0.0, 0.03, 50)
    assert _run(sim, s[:, rng.permutation(96)], bits) == "ok"
    wide = _table(64, 70.0, 0.0, 0.5, 32, f_high=190.0, t_us=327.68)
    assert (wide[31] - wide[0]).max() > 3024
    assert _run(sim, wide, bits) == "refused"
