// Host tables of the group-sum kernel: see group_tables.h.
#include "group_tables.h"

#include <string.h>

#include <algorithm>
#include <climits>
#include <new>

#include "run_parts.h"

namespace dd {
namespace {

constexpr int kMaxGroup = 12;   // channels per group
constexpr int kGroupStep = 4;   // group sizes are multiples of this (the last group of the band aside)
constexpr int kSizes = kMaxGroup / kGroupStep;
constexpr uint32_t kZeroRow = 2 * kGrpSetBytes;  // LDS offset of the row of zeros

struct Group {
  int c0 = 0, g = 0;
  int words = 0;                   // words of a pattern row (a multiple of 4)
  int n_pat = 0;
  uint8_t slot_of[kGrpMaxRows] = {};  // pattern of each DM row, in path order
  std::vector<int32_t> r;          // [n_pat][g] relative delays, in path order
  int base = 0;
  int lds() const { return n_pat * words * 4; }
};

struct Block {
  std::vector<uint32_t> rec[kGrpWaves];  // operation blocks numbered from 1 (0: the idle one)
  std::vector<uint32_t> ops;
  std::vector<uint32_t> sum;
  int n_steps = 0;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  std::vector<int> split;     // group lengths, in steps of channels, found in a first pass
  double cost = 0, work = 0;  // GroupTables
  int lds = 0;
  bool ok = true;
};

// Instructions that one chunk of a group's partial sums costs a wave.
constexpr double kCostAdd = 13, kCostMove = 23, kCostFold = 12, kCostWrite = 4, kCostRecord = 40;
// Weight of all waves' work against the busiest wave's where a step's work is split.
constexpr double kCostShared = 1.0, kCostCrowd = 3.0;

// Modelled clocks of a group with n_pat patterns over rows of `words` words: its
// LDS time (4 bytes per word written once and per window word read) and its
// instructions on 4 SIMDs, the larger in full.  A group that takes more than a
// fifth of an LDS set leaves a step too few parts for all waves.
double group_cost(int rows, int g, int n_pat, int words, double steps) {
  const int chunks = (words + kGrpChunk - 1) / kGrpChunk;
  const double bytes = 4.0 * n_pat * words;
  const double lds = (bytes + 4.0 * rows * kGrpWin) / 110.0;
  double build = chunks * (kCostAdd * g + 3 * kCostFold + kCostMove * steps + kCostWrite * n_pat +
                           kCostRecord * (g + steps + 4) / kGrpOps);
  build *= 1.0 + kCostCrowd * std::max(0.0, bytes / (0.2 * kGrpSetBytes) - 1.0);
  const double sum = rows * 18.0;
  return std::max(lds, build + sum) + 0.2 * std::min(lds, build + sum) + 40.0;
}

double guess_steps(int n_pat) { return n_pat - 1 + 0.04 * n_pat * n_pat; }

// How many of h[0..rows) differ, without branches on them (rows go back and forth between a
// few patterns: a search costs a mispredicted branch each): every row against the one `back`
// rows before it, for every `back`.  Before the first row stands a value that none has but by
// an accident, which only makes a worse split.
int distinct(const uint32_t *h, int rows) {
  typedef uint32_t Four __attribute__((vector_size(16)));
  uint32_t w[2 * kGrpMaxRows];
  memset(w, 0xA5, rows * sizeof *w);
  memcpy(w + rows, h, rows * sizeof *w);
  Four seen[kGrpMaxRows / 4] = {};
  for (int back = 1; back < rows; ++back)
    for (int k = back / 4; k < rows / 4; ++k) {
      Four x, y;
      memcpy(&x, w + rows + 4 * k, sizeof x);
      memcpy(&y, w + rows + 4 * k - back, sizeof y);
      seen[k] |= (Four)(x == y);
    }
  int n = 0;
  for (int k = 0; k < rows / 4; ++k)
    for (int e = 0; e < 4; ++e) n += seen[k][e] == 0;
  return n;
}

// Fill in a group's patterns and the path over them.
void fill_group(const int32_t *sh, int rows, Group *G) {
  const int g = G->g;
  const int32_t *s0 = sh + (size_t)G->c0 * rows;
  int first[kGrpMaxRows], cls[kGrpMaxRows], n = 0;
  for (int d = 0; d < rows; ++d) {
    auto same = [&](int e) {  // row e follows the same pattern
      for (int c = 1; c < g; ++c) {
        const int32_t *s = s0 + (size_t)c * rows;
        if (s[d] - s0[d] != s[e] - s0[e]) return false;
      }
      return true;
    };
    int k = 0;
    if (d && same(d - 1)) {
      k = cls[d - 1];
    } else {
      while (k < n && !same(first[k])) ++k;
      if (k == n) first[n++] = d;
    }
    cls[d] = k;
  }
  std::vector<int32_t> pat((size_t)n * g);
  int start = 0;
  int64_t best = INT64_MAX;
  for (int k = 0; k < n; ++k) {
    int64_t sum = 0;
    for (int c = 0; c < g; ++c) {
      pat[(size_t)k * g + c] = s0[(size_t)c * rows + first[k]] - s0[first[k]];
      sum += pat[(size_t)k * g + c];
    }
    if (sum < best) best = sum, start = k;
  }
  // nearest-neighbour path in the number of one-sample moves
  bool used[kGrpMaxRows] = {};
  int place[kGrpMaxRows];
  G->r.resize((size_t)n * g);
  int cur = start;
  for (int i = 0; i < n; ++i) {
    used[cur] = true;
    place[cur] = i;
    std::copy_n(&pat[(size_t)cur * g], g, &G->r[(size_t)i * g]);
    int next = -1;
    int64_t bd = INT64_MAX;
    for (int k = 0; k < n; ++k) {
      if (used[k]) continue;
      int64_t dist = 0;
      for (int c = 0; c < g; ++c) dist += std::abs((int64_t)pat[(size_t)k * g + c] - pat[(size_t)cur * g + c]);
      if (dist < bd) bd = dist, next = k;
    }
    cur = next;
  }
  G->n_pat = n;
  for (int d = 0; d < rows; ++d) G->slot_of[d] = (uint8_t)place[cls[d]];
}

struct Input {
  const int32_t *shift;
  int n_dm, n_chan, bits;
  int64_t pitch;
  uint32_t sample_max() const { return bits == 16 ? 0 : (1u << bits) - 1; }
};

struct Op {
  int32_t s, c;
  uint32_t flags;
};

// The operations that build some of a group's patterns, as operation blocks.
struct Part {
  int words, chunks;
  uint32_t slot;     // LDS address of its first pattern's row
  uint32_t block0;   // first operation block
  std::vector<int> rows;  // rows written by each block
};

// Append `ops` as operation blocks.  Spare operations of the last one repeat its
// first window and do nothing.
void emit_ops(const Input &in, const std::vector<Op> &ops, Block *b, Part *part) {
  const int per_load = in.bits == 16 ? 2 : 4;  // samples
  for (size_t i = 0; i < ops.size(); i += kGrpOps) {
    int64_t off[kGrpOps], base = INT64_MAX;
    for (int q = 0; q < kGrpOps; ++q) {
      const Op &op = ops[i + q < ops.size() ? i + q : i];
      off[q] = op.c * in.pitch + ((int64_t)op.s & ~(int64_t)(per_load - 1)) * in.bits / 8;
      base = std::min(base, off[q]);
      b->lo = std::min<int64_t>(b->lo, op.s - 3);
      b->hi = std::max<int64_t>(b->hi, (int64_t)op.s + part->chunks * kGrpChunk + 12);
    }
    part->rows.push_back(0);
    uint32_t words[kGrpBlockWords] = {(uint32_t)base, (uint32_t)(base >> 32)};
    for (int q = 0; q < kGrpOps; ++q) {
      if (off[q] - base > kGrpMaxOffset) b->ok = false;
      words[4 + q] = (uint32_t)(off[q] - base);
      if (i + q >= ops.size()) continue;
      const uint32_t kind = ops[i + q].flags | (uint32_t)(ops[i + q].s & (per_load - 1));
      words[2 + q / 4] |= kind << (8 * (q % 4));
      if (kind & kOpWrite) ++part->rows.back();
    }
    b->ops.insert(b->ops.end(), words, words + kGrpBlockWords);
  }
}

// A run of patterns [p0, p1) of a group, by its counts: what make_part will find.
struct Run {
  int group, p0, p1, chunks;
  double cost;  // of one chunk
};

Run count_run(const Input &in, const Group &G, int group, int p0, int p1) {
  const int g = G.g, per_load = in.bits == 16 ? 2 : 4;
  uint32_t phases = 0;
  int64_t moves = 0;
  for (int c = 0; c < g; ++c) phases |= 1u << ((G.base + G.r[(size_t)p0 * g + c]) & (per_load - 1));
  for (size_t k = (size_t)p0 * g; k < (size_t)(p1 - 1) * g; ++k) moves += std::abs((int64_t)G.r[k + g] - G.r[k]);
  const int64_t blocks = (g + moves + kGrpOps - 1) / kGrpOps;
  const double cost = kCostRecord * (double)blocks + kCostAdd * g + kCostFold * __builtin_popcount(phases) +
                      kCostMove * (double)moves + kCostWrite * (p1 - p0);
  return {group, p0, p1, (G.words + kGrpChunk - 1) / kGrpChunk, cost};
}

// Patterns [p0, p1) of a group: the first one's adds, phase by phase, then moves.
Part make_part(const Input &in, const Group &G, int p0, int p1, uint32_t slot0, Block *b) {
  const int g = G.g, per_load = in.bits == 16 ? 2 : 4;
  Part part = {};
  part.words = G.words;
  part.chunks = (G.words + kGrpChunk - 1) / kGrpChunk;
  part.slot = slot0 + (uint32_t)(p0 * G.words * 4);
  part.block0 = (uint32_t)(b->ops.size() / kGrpBlockWords) + 1;
  std::vector<Op> ops;
  for (int m = 0; m < per_load; ++m) {
    const size_t n = ops.size();
    for (int c = 0; c < g; ++c) {
      const int32_t s = G.base + G.r[(size_t)p0 * g + c];
      if ((s & (per_load - 1)) == m) ops.push_back({s, G.c0 + c, kOpAdd});
    }
    if (ops.size() > n) ops.back().flags |= kOpFold;
  }
  ops.back().flags |= kOpWrite;
  for (int p = p0 + 1; p < p1; ++p) {
    const int32_t *from = &G.r[(size_t)(p - 1) * g], *to = &G.r[(size_t)p * g];
    for (int c = 0; c < g; ++c) {
      for (int32_t v = from[c]; v < to[c]; ++v) ops.push_back({G.base + v, G.c0 + c, kOpMove});
      for (int32_t v = from[c]; v > to[c]; --v) ops.push_back({G.base + v - 1, G.c0 + c, kOpMove | kOpDown});
    }
    ops.back().flags |= kOpWrite;
  }
  emit_ops(in, ops, b, &part);
  return part;
}

// Records of one chunk of a part for wave stream `rec`.
void emit_chunk(const Part &part, int chunk, std::vector<uint32_t> *rec) {
  const int k0 = chunk * kGrpChunk, lanes = std::min(63, (part.words - k0 + 3) / 4);
  uint32_t slot = part.slot + 4u * (uint32_t)k0;
  for (size_t i = 0; i < part.rows.size(); ++i) {
    rec->push_back(part.block0 + (uint32_t)i);
    rec->push_back((i == 0 ? kRecStart : 0) | (uint32_t)lanes << 8 | (uint32_t)k0 << 16);
    rec->push_back(slot);
    rec->push_back((uint32_t)part.words * 4);
    slot += (uint32_t)(part.rows[i] * part.words * 4);
  }
}

void end_step(std::vector<uint32_t> *rec, size_t mark) {
  if (rec->size() == mark) rec->resize(mark + kGrpRecWords, 0);  // nothing to do in the step: an idle record
  (*rec)[rec->size() - kGrpRecWords + 1] |= kRecLast;
}

void build_block(const Input &in, int blk, bool cost_only, Block *b) {
  const int n_chan = in.n_chan, rows = group_rows(in.bits), per_wave = group_rows_per_wave(in.bits);
  const size_t sum_words = group_sum_words(in.bits);
  const uint32_t sample_max = in.sample_max();
  // delays of the block's rows, channel by channel; rows past the last repeat it
  std::vector<int32_t> sh((size_t)n_chan * rows);
  for (int c0 = 0; c0 < n_chan; c0 += 16)  // (a cache line of each row at a time)
    for (int d = 0; d < rows; ++d) {
      const int32_t *row = in.shift + (size_t)std::min(blk * rows + d, in.n_dm - 1) * n_chan;
      for (int c = c0; c < std::min(n_chan, c0 + 16); ++c) sh[(size_t)c * rows + d] = row[c];
    }
  auto words_of = [&](int c) {
    const int32_t *s = &sh[(size_t)c * rows];
    return (int)std::min<int64_t>(((int64_t)kGrpWin + s[rows - 1] - s[0] + 3) / 4 * 4, INT_MAX);
  };
  // Split the band into groups of least modelled time (dynamic programming over
  // the multiples of kGroupStep).
  const int np = (n_chan + kGroupStep - 1) / kGroupStep;
  std::vector<int> len;
  len.swap(b->split);
  std::vector<double> cost(len.empty() ? np + 1 : 0, 1e300);
  const bool known = !len.empty();
  if (!known) {
    len.assign(np + 1, 0);
    cost[0] = 0;
  }
  for (int p = 0; p < np && !known; ++p) {
    if (cost[p] >= 1e300) continue;
    const int c0 = p * kGroupStep;
    const int words = words_of(c0);
    if (words > kGrpMaxWords) continue;
    const int32_t *s0 = &sh[(size_t)c0 * rows];
    uint32_t h[kGrpMaxRows] = {};  // of each row's pattern (two patterns of one hash only make a worse split)
    for (int k = 1; k <= kSizes && p + k <= np; ++k) {
      const int lo = std::max(c0 + 1, c0 + (k - 1) * kGroupStep), hi = std::min(n_chan, c0 + k * kGroupStep);
      for (int c = lo; c < hi; ++c) {
        const int32_t *s = &sh[(size_t)c * rows];
        for (int d = 0; d < rows; ++d)
          h[d] = (h[d] << 5) + h[d] + (uint32_t)(s[d] - s0[d]);
      }
      const int n = distinct(h, rows);
      if ((int64_t)n * words * 4 > kGrpSetBytes) break;
      const double v = cost[p] + group_cost(rows, hi - c0, n, words, guess_steps(n));
      if (v < cost[p + k]) cost[p + k] = v, len[p + k] = k;
      if (n > rows * 7 / 8) break;
    }
  }
  if (!known && cost[np] >= 1e300) {
    b->ok = false;
    return;
  }
  if (!known) b->cost = cost[np];
  if (cost_only) {
    b->split.swap(len);
    return;
  }
  std::vector<Group> groups;
  for (int p = np; p > 0; p -= len[p]) {
    Group G;
    G.c0 = (p - len[p]) * kGroupStep;
    G.g = std::min(n_chan, p * kGroupStep) - G.c0;
    G.words = words_of(G.c0);
    G.base = sh[(size_t)G.c0 * rows];
    groups.push_back(std::move(G));
  }
  std::reverse(groups.begin(), groups.end());
  for (Group &G : groups) {
    fill_group(sh.data(), rows, &G);
    if (G.lds() > kGrpSetBytes) {
      b->ok = false;
      return;
    }
  }
  // Steps: as many groups as fit in one LDS set, at most 2 * kGrpStepPairs.  A group is
  // built in one or more parts (runs of its patterns), each chunk of a part by one
  // wave: the longest first to the wave with the least work, with as many parts
  // as make the busiest wave's work least.
  int64_t acc = 0;  // channels since the last flush of the 16-bit sums
  for (size_t i = 0; i < groups.size(); ++b->n_steps) {
    const uint32_t set = (uint32_t)(b->n_steps & 1) * kGrpSetBytes;
    size_t j = i;
    int bytes = 0;
    while (j < groups.size() && j < i + 2 * kGrpStepPairs && bytes + groups[j].lds() <= kGrpSetBytes) bytes += groups[j++].lds();
    b->lds = std::max(b->lds, (int)set + bytes);
    struct Task {
      int run, chunk;
    };
    double best = 1e300, best_simd = 0;
    std::vector<Run> runs, best_runs;
    std::vector<int> wave, best_wave;
    std::vector<Task> tasks, best_tasks;
    bool more = true;  // a group has patterns left for another split
    for (int split = 1; more && split <= 4 && (split == 1 || 4 * best_tasks.size() < 3 * kGrpWaves); ++split) {
      more = false;
      runs.clear();
      tasks.clear();
      wave.clear();
      for (size_t q = i; q < j; ++q) {
        const Group &G = groups[q];
        const int n = std::min(split, G.n_pat);
        more |= G.n_pat > split;
        for (int k = 0; k < n; ++k) runs.push_back(count_run(in, G, (int)q, G.n_pat * k / n, G.n_pat * (k + 1) / n));
      }
      for (size_t k = 0; k < runs.size(); ++k)
        for (int c = 0; c < runs[k].chunks; ++c) tasks.push_back({(int)k, c});
      std::stable_sort(tasks.begin(), tasks.end(),
                       [&](const Task &x, const Task &y) { return runs[x.run].cost > runs[y.run].cost; });
      double load[kGrpWaves] = {}, simd[4] = {}, total = 0;
      for (const Task &t : tasks) {  // (waves w, w + 4, ... share a SIMD)
        int w = 0;
        for (int k = 1; k < kGrpWaves; ++k)
          if (load[k] < load[w] || (load[k] == load[w] && simd[k & 3] < simd[w & 3])) w = k;
        load[w] += runs[t.run].cost;
        simd[w & 3] += runs[t.run].cost;
        total += runs[t.run].cost;
        wave.push_back(w);
      }
      const double cost = *std::max_element(load, load + kGrpWaves) + kCostShared * total / kGrpWaves;
      if (cost < best) {
        best = cost;
        best_simd = *std::max_element(simd, simd + 4);
        best_runs.swap(runs);
        best_tasks.swap(tasks);
        best_wave.swap(wave);
      }
    }
    b->work += best_simd;
    std::vector<Part> parts;
    uint32_t at = set;
    for (size_t k = 0; k < best_runs.size(); ++k) {
      const Run &r = best_runs[k];
      if (k && best_runs[k - 1].group != r.group) at += (uint32_t)groups[best_runs[k - 1].group].lds();
      parts.push_back(make_part(in, groups[r.group], r.p0, r.p1, at, b));
    }
    size_t mark[kGrpWaves];
    for (int w = 0; w < kGrpWaves; ++w) mark[w] = b->rec[w].size();
    for (size_t k = 0; k < best_tasks.size(); ++k)
      emit_chunk(parts[best_tasks[k].run], best_tasks[k].chunk, &b->rec[best_wave[k]]);
    for (int w = 0; w < kGrpWaves; ++w) end_step(&b->rec[w], mark[w]);
    const size_t sm = b->sum.size();
    b->sum.resize(sm + kGrpWaves * sum_words, kZeroRow);
    uint32_t slot = set;
    for (size_t q = i; q < j; ++q) {
      const Group &G = groups[q];
      const size_t pair = (q - i) / 2, half = (q - i) % 2;
      uint32_t marks = 0;
      acc += G.g;
      if (half == 1 || q + 1 == j) {
        int64_t next = 0;
        for (size_t k = q + 1; k < std::min(groups.size(), q + 3); ++k) next += groups[k].g;
        if (sample_max && (!next || (acc + next) * sample_max > 65535)) marks |= kSumFlush, acc = 0;
        if (q + 1 == j) marks |= kSumLast;
      }
      for (int d = 0; d < rows; ++d) {
        uint32_t *e = &b->sum[sm + (size_t)(d / per_wave) * sum_words + pair * 2 * per_wave];
        const int32_t u = sh[(size_t)G.c0 * rows + d] - G.base;
        uint32_t &dst = e[half * per_wave + d % per_wave];
        dst = (dst & ~kSumOffset) | (slot + 4u * (uint32_t)(G.slot_of[d] * G.words + u));
        if (d % per_wave == 0) e[0] |= marks;
      }
      slot += (uint32_t)G.lds();
    }
    i = j;
  }
  for (auto &r : b->rec) end_step(&r, r.size());  // nothing is built during the last step
}

}  // namespace

bool build_group_tables(const int32_t *shift, int n_dm, int n_chan, int bits, int64_t pitch_bytes, GroupTables *t,
                        double max_cost, double max_work) {
  static_assert(sizeof(GroupBlock) == 72, "device layout");
  static_assert(kMaxGroup * 255 <= 65535, "a group's packed sums fit 16 bits");
  *t = GroupTables();
  const int n_blk = (n_dm + group_rows(bits) - 1) / group_rows(bits);
  const Input in = {shift, n_dm, n_chan, bits, pitch_bytes};
  try {
    std::vector<Block> blocks(n_blk);
    const int64_t work = (int64_t)n_blk * n_chan;
    const int nthr = (int)std::min<int64_t>({kMaxParts, n_blk, std::max<int64_t>(1, work / 512),
                                             std::max(1u, std::thread::hardware_concurrency())});
    // Blocks `first`, `first` + step, ... as run by up to nthr threads; false on bad_alloc.
    auto build = [&](int first, int step, bool cost_only) {
      uint8_t failed[kMaxParts] = {};
      const int count = (n_blk - first + step - 1) / step;
      const int n = (int)std::min<int64_t>({nthr, count, std::max<int64_t>(1, (int64_t)count * n_chan / 512)});
      run_parts(n, [&](int k) {
        try {
          for (int b = first + k * step; b < n_blk; b += n * step)
            if (!blocks[b].n_steps) build_block(in, b, cost_only, &blocks[b]);
        } catch (const std::bad_alloc &) {
          failed[k] = 1;
        }
      });
      for (uint8_t f : failed)
        if (f) return false;
      return true;
    };
    if (max_cost > 0) {  // plans that are far from it: the costs of all blocks, or of two where that takes longer, tell
      const int mid = (n_blk - 1) / 2, step = n_blk <= nthr ? 1 : n_blk - 1 - mid;
      const int first = n_blk <= nthr ? 0 : mid;
      if (!build(first, step, true)) return false;
      double cost = 0;
      for (int b = first; b < n_blk; b += step) {
        if (!blocks[b].ok) return false;
        cost += blocks[b].cost;
      }
      if (n_blk <= nthr ? cost > max_cost : 0.5 * n_blk * cost > 1.2 * max_cost) return false;
    }
    if (max_work > 0 && n_blk > nthr) {  // and the instructions of one
      Block &mid = blocks[(n_blk - 1) / 2];
      build_block(in, (n_blk - 1) / 2, false, &mid);
      if (!mid.ok || mid.work > 1.3 * max_work) return false;
    }
    if (!build(0, 1, false)) return false;
    size_t recs = 0, ops = kGrpBlockWords, sums = 0;
    t->head.lo = 0;  // the idle operation block loads the tile's own samples of channel 0
    t->head.hi = kGrpChunk + 12;
    for (const Block &b : blocks) {
      if (!b.ok) return false;
      for (const auto &r : b.rec) recs += r.size();
      sums += b.sum.size();
      ops += b.ops.size();
      t->head.lo = std::min(t->head.lo, b.lo);
      t->head.hi = std::max(t->head.hi, b.hi);
      t->cost += b.cost;
      t->work += b.work;
      t->max_work = std::max(t->max_work, b.work);
      t->lds_bytes = std::max(t->lds_bytes, b.lds);
    }
    if (max_cost > 0 && t->cost > max_cost) return false;
    t->n_blk = n_blk;
    t->head.rec_off = (kGrpHeadWords + (int64_t)n_blk * (int64_t)(sizeof(GroupBlock) / 4) + 63) / 64 * 64;
    t->head.op_off = (t->head.rec_off + (int64_t)recs + 4 * kGrpRecWords + 63) / 64 * 64;  // records are loaded ahead
    t->head.sum_off = (t->head.op_off + (int64_t)ops + 63) / 64 * 64;
    const int64_t total = t->head.sum_off + (int64_t)sums + 64;  // a wave loads 64 entries
    if (total >= ((int64_t)1 << 31)) return false;
    t->data.assign((size_t)total, 0);
    memcpy(t->data.data(), &t->head, sizeof t->head);
    struct Place {
      size_t rec, op, sum;  // words
    };
    std::vector<Place> place(n_blk);
    size_t ro = 0, oo = kGrpBlockWords, so = 0;
    for (int b = 0; b < n_blk; ++b) {
      place[b] = {ro, oo, so};
      for (const auto &r : blocks[b].rec) ro += r.size();
      oo += blocks[b].ops.size();
      so += blocks[b].sum.size();
    }
    const int ncopy = total >= (int64_t)1 << 20 ? nthr : 1;
    run_parts(ncopy, [&](int k) {
      for (int b = k; b < n_blk; b += ncopy) {
        GroupBlock g = {};
        Place at = place[b];
        const uint32_t op0 = (uint32_t)(at.op / kGrpBlockWords) - 1;  // the block's operation blocks count from 1
        for (int w = 0; w < kGrpWaves; ++w) {
          std::vector<uint32_t> &r = blocks[b].rec[w];
          for (size_t i = 0; i < r.size(); i += kGrpRecWords)
            if (r[i]) r[i] += op0;
          g.rec_first[w] = (uint32_t)(at.rec / kGrpRecWords);
          std::copy(r.begin(), r.end(), t->data.begin() + t->head.rec_off + at.rec);
          at.rec += r.size();
        }
        std::copy(blocks[b].ops.begin(), blocks[b].ops.end(), t->data.begin() + t->head.op_off + at.op);
        g.sum_first = (uint32_t)at.sum;
        g.n_steps = (uint32_t)blocks[b].n_steps;
        std::copy(blocks[b].sum.begin(), blocks[b].sum.end(), t->data.begin() + t->head.sum_off + at.sum);
        memcpy(&t->data[kGrpHeadWords + (size_t)b * (sizeof g / 4)], &g, sizeof g);
        blocks[b] = Block();
      }
    });
  } catch (const std::bad_alloc &) {
    return false;
  }
  return true;
}

}  // namespace dd
