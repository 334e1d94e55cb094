// Host tables of the float kernel that shares sums of four rows (quad_f32.hip), for the
// forward transform and the adjoint.  Plain C++, no device code.
//
// Float sums have one fixed order: rows in quads, ((x0 + x1) + x2) + x3, the quads of 32
// rows in order into a partial, the partials in order.  A quad's sum for output o is
//   P_r(t + sh(o, k)) = sum_c X(k + c, t + sh(o, k) + r_c),  r_c = sh(o, k + c) - sh(o, k),
// and the outputs of a block share few delay patterns r (neighbouring outputs differ by
// much less than a sample of delay between neighbouring rows).  So each pattern's sums
// are computed once, over the range of words that the block's outputs read, and every output
// adds one word per quad and sample: the same additions in the same order as row by row.
#pragma once

#include <stdint.h>

#include <vector>

namespace dd {

constexpr int kQuadWin = 512;     // samples per tile
constexpr int kQuadWaves = 16;    // each builds its part of the next step's sums and adds up its outputs
// Words per lane of a pattern's sums that one record builds (what registers are left
// beside the outputs' sums).
constexpr int quad_lane_words(int rows) { return rows == 64 ? 4 : 6; }
constexpr int kQuadSetBytes = (160 * 1024 - 64) / 2 / 64 * 64;  // LDS: two sets, one step's sums each
constexpr int kQuadStep = 16;     // quads per step, at most
constexpr int kQuadOps = 4;       // operations per record
constexpr int kQuadRecWords = 2, kQuadOpWords = 5;
constexpr int kQuadStepWords = 2;

// A wave builds by records of 4 operations.  An operation takes a new window of one of a
// quad's rows; the one that completes a pattern stores the pattern's sums.  A record: 0: its
// operation block, kQuadLast; 1: LDS word of the next pattern's sums << 16 | chunk (of 64 *
// quad_lane_words of the sums' words).  An operation block: 0: quad << 15 | words from one
// pattern's sums to the next; 1: the operations' kinds, 4 bits each: the row of the quad,
// kQuadWrite, kQuadNone; 2: the least of its windows' first samples (relative to the tile's
// first); 3-4: theirs relative to that, 16 bits each.  A quad's first block takes all four
// rows.  The sums' words are a multiple of 64.
constexpr uint32_t kQuadLast = 1u << 31;  // the wave's last record of the step
constexpr uint32_t kQuadWrite = 4;
constexpr uint32_t kQuadNone = 8;  // a row past the last: zeros

struct QuadBlock {
  uint32_t rec_first[kQuadWaves];  // each wave's first record
  uint32_t step_first, n_steps;    // word offset of the steps: {first quad, quads}
  int32_t lo, hi;                  // samples read relative to a tile's first: [lo, hi)
};

// Device data (32-bit words): [n_blk] QuadBlock, steps, records, operation blocks (the first
// idle), sums: [n_blk][wave][n_quads][rows / 16] uint16 LDS words of the outputs' windows.
struct QuadTables {
  bool use = false;
  int order = 0;              // TileOrder
  int rows = 0, n_blk = 0;    // outputs per block (32 or 64), blocks
  int n_quads = 0;            // padded to a multiple of 2
  uint32_t op_off = 0, sum_off = 0;  // word offsets of the operation blocks and the sums
  std::vector<uint32_t> data;
  double records = 0, max_records = 0;  // of the busiest SIMD, step by step: all blocks, the largest
};

// The plan's delays: output o sums row k at sign * shift[o * out_stride + k * row_stride].
struct QuadShifts {
  const int32_t *shift;
  int64_t out_stride, row_stride;
  int sign, n_out, n_rows;
  // Of rows k..k+3 (rows past the last: as the last).
  void quad(int o, int k, int32_t *s) const {
    const int32_t *p = shift + o * out_stride;
    for (int c = 0; c < 4; ++c) s[c] = sign * p[(k + c < n_rows ? k + c : n_rows - 1) * row_stride];
  }
};

// Modelled CU clocks of all blocks, per tile, for `rows` outputs per block, from two of the
// blocks' patterns; 1e300 where a quad's sums do not fit a set.
double guess_quad_cost(const QuadShifts &sh, int rows);
// false if a quad's sums do not fit a set, or on bad_alloc.
bool build_quad_tables(const QuadShifts &sh, int rows, QuadTables *t);

}  // namespace dd
