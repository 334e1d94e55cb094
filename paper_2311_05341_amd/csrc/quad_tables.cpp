// Host tables of the shared quad sums: see quad_tables.h.
#include "quad_tables.h"

#include <string.h>

#include <algorithm>
#include <climits>
#include <new>

#include "run_parts.h"

namespace dd {
namespace {

constexpr int kMaxOutputs = 64;

struct Pattern {
  int32_t r[3];
};

struct Quad {
  int32_t base = 0;   // least delay of the first row
  int words = 0, n_pat = 0;
  int32_t u[kMaxOutputs];      // delay of the first row less base
  int pat_of[kMaxOutputs];
  Pattern pat[kMaxOutputs];
  int chunks(int rows) const { return (words + 64 * quad_lane_words(rows) - 1) / (64 * quad_lane_words(rows)); }
  int bytes() const { return 4 * words * n_pat; }
};

// Modelled clocks of a quad: its sums read from LDS at 32 words a clock, its operations
// (instructions issued; the start of a second part of the patterns included), and its
// share of a step's barrier.  On 1024 ch x 131900 x 512 DMs (2 to 3 patterns) and 1024 ch
// x 2^17 x 1024 DMs (6): 1990 and 2640, measured 2000 and 2520.
double quad_cost(const Quad &q, int rows, double reloads) {
  return rows * kQuadWin / 32.0 + (14.0 + 4.0 * quad_lane_words(rows)) * q.chunks(rows) * (6.0 + reloads) + 250.0;
}

bool same(const Pattern &a, const Pattern &b) { return a.r[0] == b.r[0] && a.r[1] == b.r[1] && a.r[2] == b.r[2]; }
int changes(const Pattern &a, const Pattern &b) {
  return (a.r[0] != b.r[0]) + (a.r[1] != b.r[1]) + (a.r[2] != b.r[2]);
}

// Outputs past the last repeat it.  false: the sums do not fit.
bool fill_quad(const QuadShifts &sh, int blk, int rows, int k, Quad *q) {
  int64_t lo = INT32_MAX, hi = INT32_MIN;
  q->n_pat = 0;
  int last = 0;
  for (int d = 0; d < rows; ++d) {
    int32_t s[4];
    sh.quad(std::min(blk * rows + d, sh.n_out - 1), k, s);
    const Pattern p = {{s[1] - s[0], s[2] - s[0], s[3] - s[0]}};
    const auto r = std::minmax({0, p.r[0], p.r[1], p.r[2]});
    if ((int64_t)r.second - r.first > 32767) return false;  // (a block's windows: see task_ops)
    if (!q->n_pat || !same(p, q->pat[last])) {
      for (last = 0; last < q->n_pat && !same(p, q->pat[last]);) ++last;
      if (last == q->n_pat) q->pat[q->n_pat++] = p;
    }
    q->pat_of[d] = last;
    q->u[d] = s[0];
    lo = std::min<int64_t>(lo, s[0]);
    hi = std::max<int64_t>(hi, s[0]);
  }
  q->base = (int32_t)lo;
  if (hi - lo + kQuadWin + 63 > kQuadSetBytes / 4) return false;
  q->words = ((int)(hi - lo) + kQuadWin + 63) / 64 * 64;
  for (int d = 0; d < rows; ++d) q->u[d] -= q->base;
  return q->bytes() <= kQuadSetBytes;
}

// Order the patterns so that successive ones differ in few rows.
void order_patterns(Quad *q, int rows) {
  int place[kMaxOutputs];
  Pattern out[kMaxOutputs];
  bool used[kMaxOutputs] = {};
  int cur = 0;
  for (int i = 0; i < q->n_pat; ++i) {
    used[cur] = true;
    place[cur] = i;
    out[i] = q->pat[cur];
    int next = -1, best = INT_MAX;
    for (int k = 0; k < q->n_pat; ++k)
      if (!used[k] && changes(q->pat[cur], q->pat[k]) < best) best = changes(q->pat[cur], q->pat[k]), next = k;
    cur = next;
  }
  std::copy_n(out, q->n_pat, q->pat);
  for (int d = 0; d < rows; ++d) q->pat_of[d] = place[q->pat_of[d]];
}

struct Task {
  int run, chunk;
};

// A run of a quad's patterns [p0, p1): its records, first operation block.
struct Run {
  int quad, p0, p1;
  size_t recs, op0;
};

struct Op {
  uint32_t kind;
  int32_t start;
};

// How many operation blocks build patterns [p0, p1): four rows, then each change of a row.
size_t run_blocks(const Quad &q, int p0, int p1) {
  int ops = 4;
  for (int p = p0 + 1; p < p1; ++p) ops += changes(q.pat[p - 1], q.pat[p]);
  return (size_t)(ops + kQuadOps - 1) / kQuadOps;
}

// Append these operation blocks, of quad k.
void run_ops(const Quad &q, int k, int p0, int p1, int n_rows, std::vector<uint32_t> *out) {
  Op ops[4 + 3 * kMaxOutputs];
  size_t n_ops = 0;
  for (int p = p0; p < p1; ++p) {
    const int32_t *r = q.pat[p].r;
    if (p == p0) ops[n_ops++] = {0, 0};
    for (uint32_t c = 1; c < 4; ++c)
      if (p == p0 || r[c - 1] != q.pat[p - 1].r[c - 1]) ops[n_ops++] = {c, r[c - 1]};
    ops[n_ops - 1].kind |= kQuadWrite;
  }
  for (size_t o = 0; o < n_ops; o += kQuadOps) {
    int32_t least = INT32_MAX;
    for (size_t e = o; e < std::min(o + kQuadOps, n_ops); ++e) least = std::min(least, ops[e].start);
    uint32_t w[kQuadOpWords] = {(uint32_t)k << 15 | (uint32_t)q.words, 0, (uint32_t)(q.base + least), 0, 0};
    for (size_t e = 0; e < kQuadOps; ++e) {  // spare operations repeat the last window
      const bool spare = o + e >= n_ops;
      const Op &op = ops[spare ? n_ops - 1 : o + e];
      w[1] |= (spare ? op.kind & 3 : op.kind) << (4 * e);
      if (4 * k + (int)(op.kind & 3) >= n_rows) w[1] |= kQuadNone << (4 * e);
      w[3 + e / 2] |= (uint32_t)(op.start - least) << (16 * (e % 2));
    }
    out->insert(out->end(), w, w + kQuadOpWords);
  }
}

struct Block {
  bool ok = false;
  double records = 0;  // QuadTables
  int64_t lo = 0, hi = 64 * quad_lane_words(32);  // (an idle record reads the tile's first samples)
  std::vector<uint32_t> rec[kQuadWaves], steps, ops;  // operation blocks numbered from 1 (0: the idle one)
};

// One block's steps, records and operation blocks, and its entries of sums[n_blk][wave]
// [nqp][outputs of a wave].
void build_block(const QuadShifts &sh, int b, int rows, int nqp, uint16_t *sums, Block *out) {
  Block &B = *out;
  const int per_wave = rows / kQuadWaves, nq = (sh.n_rows + 3) / 4;
  std::vector<Quad> quads(nq);
  B.ops.assign(kQuadOpWords, 0);
  for (int k = 0; k < nq; ++k) {
    if (!fill_quad(sh, b, rows, 4 * k, &quads[k])) return;  // (B.ok stays false)
    const Quad &q = quads[k];
    order_patterns(&quads[k], rows);
    for (int p = 0; p < q.n_pat; ++p) {
      const auto r = std::minmax({0, q.pat[p].r[0], q.pat[p].r[1], q.pat[p].r[2]});
      B.lo = std::min<int64_t>(B.lo, (int64_t)q.base + r.first);
      B.hi = std::max<int64_t>(B.hi, (int64_t)q.base + r.second + q.chunks(rows) * 64 * quad_lane_words(rows));
    }
  }
  std::vector<Run> runs, best_runs;
  std::vector<Task> todo, best;
  std::vector<int> wave, best_wave;
  size_t best_load = 0, best_simd = 0;
  for (int i = 0; i < nq;) {
    const uint32_t set = (B.steps.size() / kQuadStepWords & 1) * kQuadSetBytes;
    int j = i, bytes = 0;
    while (j < nq && j < i + kQuadStep && bytes + quads[j].bytes() <= kQuadSetBytes) bytes += quads[j++].bytes();
    // Tasks: each chunk of each quad, its patterns in as many runs as leave the busiest
    // wave the fewest records; the longest first to the wave with the fewest.
    best_load = SIZE_MAX;
    bool more = true;  // a quad has patterns left for another split
    for (int split = 1; more && split <= 4; ++split) {
      more = false;
      runs.clear();
      todo.clear();
      wave.clear();
      for (int k = i; k < j; ++k) {
        const int n = std::min(split, quads[k].n_pat);
        more |= quads[k].n_pat > split;
        for (int s = 0; s < n; ++s) {
          const int p0 = quads[k].n_pat * s / n, p1 = quads[k].n_pat * (s + 1) / n;
          for (int c = 0; c < quads[k].chunks(rows); ++c) todo.push_back({(int)runs.size(), c});
          runs.push_back({k, p0, p1, run_blocks(quads[k], p0, p1), 0});
        }
      }
      std::stable_sort(todo.begin(), todo.end(),
                       [&](const Task &x, const Task &y) { return runs[x.run].recs > runs[y.run].recs; });
      size_t load[kQuadWaves] = {}, simd[4] = {}, total = 0;
      for (const Task &x : todo) {
        const int w = (int)(std::min_element(load, load + kQuadWaves) - load);
        load[w] += runs[x.run].recs;
        simd[w & 3] += runs[x.run].recs;
        total += runs[x.run].recs;
        wave.push_back(w);
      }
      const size_t v = kQuadWaves * *std::max_element(load, load + kQuadWaves) + total;
      if (v < best_load) {
        best_load = v;
        best_simd = *std::max_element(simd, simd + 4);
        best.swap(todo);
        best_wave.swap(wave);
        best_runs.swap(runs);
      }
    }
    B.records += (double)best_simd;
    for (Run &r : best_runs) {
      r.op0 = B.ops.size() / kQuadOpWords;
      run_ops(quads[r.quad], r.quad, r.p0, r.p1, sh.n_rows, &B.ops);
    }
    uint32_t slot[kQuadStep], at = set / 4;
    for (int k = i; k < j; ++k) {
      const Quad &q = quads[k];
      slot[k - i] = at;
      for (int d = 0; d < rows; ++d)
        sums[(((size_t)b * kQuadWaves + d / per_wave) * nqp + k) * per_wave + d % per_wave] =
            (uint16_t)(at + q.pat_of[d] * q.words + q.u[d]);
      at += (uint32_t)q.bytes() / 4;
    }
    B.steps.push_back((uint32_t)i);
    B.steps.push_back((uint32_t)(j - i));
    for (int w = 0; w < kQuadWaves; ++w) {
      std::vector<uint32_t> &rec = B.rec[w];
      const size_t mark = rec.size();
      for (size_t x = 0; x < best.size(); ++x) {
        if (best_wave[x] != w) continue;
        const Run &y = best_runs[best[x].run];
        const Quad &q = quads[y.quad];
        const int chunk = 64 * quad_lane_words(rows) * best[x].chunk;
        uint32_t dst = slot[y.quad - i] + (uint32_t)(y.p0 * q.words + chunk);
        for (size_t k = 0; k < y.recs; ++k) {
          const size_t o = y.op0 + k;
          rec.push_back((uint32_t)o);
          rec.push_back(dst << 16 | (uint32_t)best[x].chunk);
          for (int e = 0; e < kQuadOps; ++e)
            if (B.ops[o * kQuadOpWords + 1] >> (4 * e) & kQuadWrite) dst += (uint32_t)q.words;
        }
      }
      if (rec.size() == mark) rec.resize(mark + kQuadRecWords, 0);
      rec[rec.size() - kQuadRecWords] |= kQuadLast;
    }
    i = j;
  }
  for (auto &r : B.rec) {  // nothing is built during the last step; then the windows of one more record are loaded
    r.resize(r.size() + 2 * kQuadRecWords, 0);
    r[r.size() - 2 * kQuadRecWords] |= kQuadLast;
  }
  B.ok = true;
}

}  // namespace

double guess_quad_cost(const QuadShifts &sh, int rows) {
  const int n_blk = (sh.n_out + rows - 1) / rows;
  double c = 0;
  Quad q;
  for (int b : {n_blk / 2, n_blk - 1})
    for (int k = 0; k < sh.n_rows; k += 4) {
      if (!fill_quad(sh, b, rows, k, &q)) return 1e300;
      c += quad_cost(q, rows, 1.3 * (q.n_pat - 1));
    }
  return 0.5 * c * n_blk;
}

bool build_quad_tables(const QuadShifts &sh, int rows, QuadTables *t) {
  *t = QuadTables();
  const int n_blk = (sh.n_out + rows - 1) / rows, per_wave = rows / kQuadWaves, nq = (sh.n_rows + 3) / 4;
  const int nqp = (nq + 1) / 2 * 2;
  if (nq >= 1 << 17) return false;
  try {
    std::vector<Block> blocks(n_blk);
    std::vector<uint16_t> sums((size_t)n_blk * kQuadWaves * nqp * per_wave, 0);
    const int nthr = (int)std::min<int64_t>({kMaxParts, n_blk, std::max<int64_t>(1, (int64_t)n_blk * nq / 64),
                                             std::max(1u, std::thread::hardware_concurrency())});
    uint8_t failed[kMaxParts] = {};
    run_parts(nthr, [&](int k) {
      try {
        for (int b = k; b < n_blk; b += nthr) build_block(sh, b, rows, nqp, sums.data(), &blocks[b]);
      } catch (const std::bad_alloc &) {
        failed[k] = 1;
      }
    });
    for (uint8_t f : failed)
      if (f) return false;
    for (const Block &B : blocks) {
      if (!B.ok) return false;
      t->records += B.records;
      t->max_records = std::max(t->max_records, B.records);
    }
    size_t n_steps = 0, n_recs = 0, n_ops = kQuadOpWords;
    for (const Block &B : blocks) {
      n_steps += B.steps.size();
      n_ops += B.ops.size() - kQuadOpWords;
      for (const auto &r : B.rec) n_recs += r.size();
    }
    const size_t s0 = (size_t)n_blk * (sizeof(QuadBlock) / 4), r0 = (s0 + n_steps + 1) / 2 * 2;
    const size_t o0 = r0 + n_recs + 4 * kQuadRecWords;  // records are loaded ahead
    const size_t u0 = o0 + n_ops;
    const size_t total = u0 + sums.size() / 2 + 64;     // a wave loads 64 words of sums
    if (total >= ((size_t)1 << 31)) return false;
    t->data.assign(total, 0);
    size_t so = s0, ro = r0, oo = 0;
    for (int b = 0; b < n_blk; ++b) {
      QuadBlock qb;
      if (blocks[b].lo != (int32_t)blocks[b].lo || blocks[b].hi != (int32_t)blocks[b].hi) return false;
      qb.lo = (int32_t)blocks[b].lo;
      qb.hi = (int32_t)blocks[b].hi;
      qb.step_first = (uint32_t)so;
      qb.n_steps = (uint32_t)(blocks[b].steps.size() / kQuadStepWords);
      std::copy(blocks[b].steps.begin(), blocks[b].steps.end(), t->data.begin() + so);
      so += blocks[b].steps.size();
      for (int w = 0; w < kQuadWaves; ++w) {
        qb.rec_first[w] = (uint32_t)(ro / kQuadRecWords);
        std::vector<uint32_t> &rec = blocks[b].rec[w];
        for (size_t i = 0; i < rec.size(); i += kQuadRecWords)
          if (rec[i] & ~kQuadLast) rec[i] += (uint32_t)oo;
        std::copy(rec.begin(), rec.end(), t->data.begin() + ro);
        ro += rec.size();
      }
      std::copy(blocks[b].ops.begin() + kQuadOpWords, blocks[b].ops.end(), t->data.begin() + o0 + (oo + 1) * kQuadOpWords);
      oo += blocks[b].ops.size() / kQuadOpWords - 1;
      memcpy(&t->data[(size_t)b * (sizeof qb / 4)], &qb, sizeof qb);
    }
    for (size_t i = 0; i < sums.size(); i += 2) t->data[u0 + i / 2] = sums[i] | (uint32_t)sums[i + 1] << 16;
    t->rows = rows;
    t->n_blk = n_blk;
    t->n_quads = nqp;
    t->op_off = (uint32_t)o0;
    t->sum_off = (uint32_t)u0;
  } catch (const std::bad_alloc &) {
    return false;
  }
  return true;
}

}  // namespace dd
