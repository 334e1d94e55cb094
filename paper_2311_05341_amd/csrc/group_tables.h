// Host tables of the group-sum forward kernel (fwd_group.hip): which partial
// sums over groups of neighbouring channels a block of DM rows shares, and the
// order in which they are built.  Plain C++, no device code.
//
// For a group of channels [c0, c0 + g) and a block of DM rows, the delays of
// row d relative to the group's first channel, r_c(d) = shift(c, d) -
// shift(c0, d), take few distinct values: neighbouring rows differ by much less
// than one sample of delay inside the group, so the rows of the block fall into
// a handful of patterns r.  The group's partial sum
//   P_r(k) = sum_{c in group} x(c, t0 + base + r_c + k),  base = shift(c0, first row),
// is built once per pattern and every row d adds P_{r(d)}(t - t0 + u_d),
// u_d = shift(c0, d) - base: one add per group instead of one per channel.
// The sums are integers, so the regrouping is exact.  Successive patterns are
// visited along a path on which one channel moves by one sample at a time:
// P += x(c, s + 1 + k) - x(c, s + k).
#pragma once

#include <stdint.h>

#include <vector>

namespace dd {

// Geometry shared by the host tables and the kernel.
constexpr int kGrpMaxRows = 64;
// DM rows per workgroup.  16-bit input, whose sums need one register per sample
// instead of one and a half, takes twice the rows per partial sum built.
constexpr int group_rows(int bits) { return bits == 16 ? 64 : 32; }
constexpr int kGrpWin = 512;        // LDS words of a row's window (one or two samples per word)
constexpr int kGrpWaves = 16;       // each builds its part of the next step's partial sums and adds up
constexpr int group_rows_per_wave(int bits) { return group_rows(bits) / kGrpWaves; }  // rows of the current step
constexpr int kGrpChunk = 252;      // words of a pattern row that one wave builds: 63 lanes x 4 (lane 63 only loads)
constexpr int kGrpMaxWords = 12 * kGrpChunk;  // longest pattern row
// LDS: two sets of partial sums (one step's each), a row of zeros, and a place that
// lanes without a word to store write to.
constexpr int kGrpZeroBytes = 4 * kGrpWin, kGrpTrashBytes = 1024;
constexpr int kGrpSetBytes = (160 * 1024 - 64 - kGrpZeroBytes - kGrpTrashBytes) / 2 / 64 * 64;
constexpr int kGrpStepPairs = 4;    // a step has at most this many pairs of groups
constexpr int kGrpOps = 8;                           // operations per block of them
constexpr int kGrpBlockWords = 12;                   // words of such a block
constexpr int kGrpRecWords = 4;
constexpr int64_t kGrpMaxOffset = (int64_t)0xFFFF0000;  // of an operation's window from its block's base

// A wave's work: a stream of records, each running one block of operations over
// the words [k0, k0 + kGrpChunk) of a pattern row.  Record word 0: the operation
// block, 1: flags, lanes that store in bits 8-15, k0 in bits 16-31, 2: the LDS
// address of the wave's words in the next pattern's row, 3: the rows' stride.
constexpr uint32_t kRecStart = 1u;  // the partial sums start from zero
constexpr uint32_t kRecLast = 2u;   // the wave's last record of the step
// An operation block: words 0-1 the byte offset (64 bits, signed) that its windows
// are relative to; 2-3 the operations' kinds, a byte each; 4-11 the byte offset of
// each operation's window (of its first load: rounded down to 4 bytes, 2 for 4-bit
// samples).  A kind is the window's first sample in that load (bits 0-1) and
constexpr uint32_t kOpMove = 4u;    // P += x(s + 1) - x(s)
constexpr uint32_t kOpDown = 8u;    // a move with the opposite sign
constexpr uint32_t kOpAdd = 16u;    // S += x(s); S are the sums of one window phase
constexpr uint32_t kOpFold = 32u;   // the last add of its phase: P += S, S = 0
constexpr uint32_t kOpWrite = 64u;  // P is a finished pattern, in the row at hand: go to the next row

// Sum entries of a (step, wave): per pair of groups and row of the wave, the LDS byte
// offsets of the two windows to add (a missing group: the row of zeros), and on a
// pair's first entry
constexpr int group_sum_words(int bits) { return kGrpStepPairs * 2 * group_rows_per_wave(bits); }
constexpr uint32_t kSumLast = 1u << 31;   // last pair of the step
constexpr uint32_t kSumFlush = 1u << 30;  // add the 16-bit sums to the totals after this pair
constexpr uint32_t kSumOffset = (1u << 18) - 1;

// One DM block's place in the table (18 words).
struct GroupBlock {
  uint32_t rec_first[kGrpWaves];  // first record of each wave's stream
  uint32_t sum_first;             // word offset of its sum entries: [step][wave][group_sum_words]
  uint32_t n_steps;
};

// The head of the table (16 words), followed by the GroupBlocks.
struct GroupHead {
  int64_t rec_off, op_off, sum_off;  // word offsets of the records, operation blocks and sum entries
  int64_t lo, hi;                    // samples read relative to a tile's start: [lo, hi)
  int64_t spare[3];
};
constexpr int kGrpHeadWords = sizeof(GroupHead) / 4;

struct GroupTables {
  bool use = false;            // the plan runs the group-sum kernel
  int n_blk = 0;
  std::vector<uint32_t> data;  // GroupHead, [n_blk] GroupBlock, records, operation blocks, sum entries
  GroupHead head = {};
  int lds_bytes = 0;           // of both sets
  double cost = 0;             // modelled CU clocks for all blocks, per time tile, from the patterns alone
  double work = 0, max_work = 0;  // building instructions of the busiest SIMD, step by step: all blocks, the largest
};

// Tables for shift[n_dm][n_chan] (never decreasing with d) and samples of
// `bits` (4, 8: two packed 16-bit sums per word; 16: one 32-bit sum) in channel
// rows pitch_bytes apart.  false if some group cannot be held, if the modelled clocks
// exceed max_cost (> 0), if one block's instructions are far above max_work (> 0), or on bad_alloc.
bool build_group_tables(const int32_t *shift, int n_dm, int n_chan, int bits, int64_t pitch_bytes, GroupTables *t,
                        double max_cost = 0, double max_work = 0);

}  // namespace dd
