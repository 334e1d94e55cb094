// Host side of a plan: validation, the FP64 integer shift table, delay spans
// and the tile shape.  No device code here.
//
// The shift table follows Sec. 1, Eq. 1 (cold-plasma delay relative to the top
// of the band) with channel c at f_high - c*df as in Sec. 4.1, the constant
// 4.148808e3 s MHz^2 cm^3/pc, divided by the sampling time and rounded half up.
// It is evaluated in IEEE FP64 with no contraction, in one fixed order, so the
// table is bit-for-bit reproducible; the device only receives the integers.
#pragma clang fp contract(off)

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <climits>
#include <new>

#include "dd_internal.h"
#include "run_parts.h"

namespace dd {

static const double kDispersionConstant = 4.148808e3;  // s MHz^2 cm^3 / pc

static double channel_freq(const dd_plan &p, int c) {
  if (!p.freqs.empty()) return p.freqs[c];
  return p.desc.f_high_mhz - (double)c * p.desc.chan_bw_mhz;
}

dd_status build_shift_table(dd_plan &p) {
  const int nc = p.desc.n_chan, nd = p.desc.n_dm;
  const double fh = p.desc.f_high_mhz;
  std::vector<double> k;
  try {
    k.resize(nc);
    p.shift.assign((size_t)nd * nc, 0);
  } catch (const std::bad_alloc &) {
    return fail(DD_ERR_NOMEM, "shift table allocation failed");
  }
  for (int c = 0; c < nc; ++c) {
    double f = channel_freq(p, c);
    if (!(f > 0.0) || !(f <= fh) || !isfinite(f))
      return fail(DD_ERR_RANGE, "channel " + std::to_string(c) + " frequency " + std::to_string(f) +
                                    " MHz is not in (0, f_high]");
    k[c] = 1.0 / (f * f) - 1.0 / (fh * fh);
  }
  const double t = p.desc.t_samp_s, d0 = p.desc.dm_start, step = p.desc.dm_step;
  const size_t work = (size_t)nd * nc;
  const int nthr = work < (1u << 20) ? 1 : (int)std::min<unsigned>(kMaxParts, std::max(1u, std::thread::hardware_concurrency()));
  // The kernels rely on delays never decreasing with d (each DM block is
  // staged from its first row's delays); Eq. 1 with dm_step >= 0 and
  // f_c <= f_high guarantees it, and so does monotone FP64 rounding.  Check.
  struct Part {
    bool bad = false, falls = false;
    int32_t mx = 0;
  } parts[kMaxParts];
  run_parts(nthr, [&](int i) {
    Part &part = parts[i];
    const int lo = (int)((int64_t)nd * i / nthr), hi = (int)((int64_t)nd * (i + 1) / nthr);
    for (int d = lo; d < hi; ++d) {
      const double dm = d0 + (double)d * step;
      int32_t *row = p.shift.data() + (size_t)d * nc;
      const int32_t *prev = d > lo ? row - nc : row;
      for (int c = 0; c < nc; ++c) {
        const double v = ((dm * kDispersionConstant) * k[c]) / t;
        const double s = floor(v + 0.5);
        if (!(s >= 0.0 && s <= 2147483647.0)) {
          part.bad = true;
          return;
        }
        row[c] = (int32_t)s;
      }
      int32_t falls = 0, mx = 0;
      for (int c = 0; c < nc; ++c) {
        falls |= row[c] < prev[c];
        mx = std::max(mx, row[c]);
      }
      part.falls |= falls != 0;
      part.mx = std::max(part.mx, mx);
    }
  });
  bool falls = false;
  int32_t mx = 0;
  for (int i = 0; i < nthr; ++i) {
    if (parts[i].bad) return fail(DD_ERR_RANGE, "a shift does not fit in int32");
    falls |= parts[i].falls;
    mx = std::max(mx, parts[i].mx);
    const int lo = (int)((int64_t)nd * i / nthr);  // the parts' first rows against the rows before them
    if (lo > 0)
      for (int c = 0; c < nc; ++c) falls |= p.shift[(size_t)lo * nc + c] < p.shift[(size_t)(lo - 1) * nc + c];
  }
  if (falls) return fail(DD_ERR_RANGE, "shift table decreases with DM");
  p.max_shift = mx;
  p.n_out = p.desc.n_samp - (int64_t)mx;
  if (p.n_out <= 0)
    return fail(DD_ERR_TOO_SHORT, "n_samp " + std::to_string(p.desc.n_samp) + " <= largest shift " +
                                      std::to_string(mx));
  return DD_OK;
}

// Largest delay spread max_c(shift[d_hi][c] - shift[d_lo][c]) over the DM blocks
// [b*dm_block, b*dm_block + dm_block) (the last block clipped).  Shifts never
// decrease with d, so the spread inside a block is last row minus first row.
int32_t max_dm_block_span(const dd_plan &p, int dm_block) {
  const int nc = p.desc.n_chan, nd = p.desc.n_dm;
  int32_t span = 0;
  for (int lo = 0; lo < nd; lo += dm_block) {
    const int hi = std::min(lo + dm_block, nd) - 1;
    const int32_t *a = p.shift.data() + (size_t)lo * nc, *b = p.shift.data() + (size_t)hi * nc;
    for (int c = 0; c < nc; ++c) span = std::max(span, b[c] - a[c]);
  }
  return span;
}

static const int kLdsLimit = 160 * 1024;

static int round_up(int64_t v, int a) { return (int)((v + a - 1) / a * a); }

// Tables of the integer forward kernel for tile shape (ns, dm_per_wave, waves).
// For DM block b, channel c: sbase = shift(c, first DM of b) rounded down to
// the staging unit (the samples in 16 bytes: 16 for u8, 32 for u4, 8 for u16);
// for each DM d of the block, with v = shift(c, d) - sbase the window's offset
// in the staged row, the entry is the LDS byte offset of its first word inside
// the channel's shifted copies (each row_bytes long): for 8- and 4-bit samples
// (one byte each once staged) four copies, (v % 4) * row_bytes + (v - v % 4);
// for 16-bit samples (byte offset 2v) two copies,
// (v % 2) * row_bytes + 2 * (v - v % 2).  Phase-load shapes (segs > 0) add
// the channel's place in the staging slot; for packed 4-bit samples the copies
// are the eight nibble phases of the packed row and the entry is
// (v % 8) * row_bytes + 4 * (v / 8).
// Fails with DD_ERR_RANGE if even one channel per LDS stage does not fit.
dd_status build_int_tables(const dd_plan &p, int ns, int dm_per_wave, int waves, int chan_block, int segs,
                           int lds_limit, IntTables *t, bool fill) {
  const int nc = p.desc.n_chan, nd = p.desc.n_dm;
  const int dblk = waves * dm_per_wave;
  const bool u16 = p.desc.dtype == DD_U16;
  const bool u4 = p.desc.dtype == DD_U4;
  const int unit = u4 ? 32 : u16 ? 8 : 16;
  const bool phase = segs > 0;  // phase-load staging (8-bit, packed 4-bit)
  if (phase && p.desc.dtype == DD_F32) return fail(DD_ERR_RANGE, "phase-load staging is for integer input");
  if (phase && u4 && (ns % 8 || chan_block > 16)) return fail(DD_ERR_RANGE, "shape not compiled for 4-bit phase loads");
  // copies of a staged row: byte phases (4, or 2 for 16-bit samples); packed
  // 4-bit phase loads keep the eight nibble phases of the packed row
  const int copies = phase && u4 ? 8 : u16 ? 2 : 4;
  const int span = max_dm_block_span(p, dblk);
  // samples of a staged row: the tile, the spread, the rounding of the stage base
  // (ring form: and the extra word the phase build reads past a chunk; packed
  // 4-bit phase loads: a spare word, which the odd nibble copies never fill)
  const int64_t rs = (int64_t)64 * ns + span + unit + (phase ? (u4 ? 8 : 0) : 16);
  if (rs > (1 << 23)) return fail(DD_ERR_RANGE, "delay spread too large");
  t->row_bytes = u16 ? round_up(2 * rs, 16) : phase && u4 ? round_up((rs + 1) / 2, 16) : round_up(rs, unit);
  int64_t lds;
  if (phase) {
    // LDS: kPhaseSlots slots of chan_block x copies, 1 KB load sink; a copy row
    // is loaded in at most `segs` 1 KB segments; entries are slot offsets
    lds = (int64_t)kPhaseSlots * chan_block * copies * t->row_bytes + 1024;
    if ((t->row_bytes + 1023) / 1024 > segs) return fail(DD_ERR_RANGE, "staged rows longer than the shape's loads");
    if ((int64_t)chan_block * copies * t->row_bytes > 65536)
      return fail(DD_ERR_RANGE, "staging slot too large for 16-bit LDS offsets");
  } else {
    // LDS: two buffers of the shifted copies, a ring of 3 raw slots (rows of raw
    // bytes + 16), 1 KB of scratch.  Loads per block: 1 KB segments of raw rows.
    const int raw = p.desc.dtype == DD_U4 ? t->row_bytes / 2 : t->row_bytes;
    lds = (int64_t)2 * chan_block * copies * t->row_bytes + (int64_t)3 * chan_block * (raw + 16) + 1024;
    if (chan_block * ((raw + 1023) / 1024) > 16) return fail(DD_ERR_RANGE, "too many staging segments");  // kStageSegs
    if ((int64_t)copies * t->row_bytes > 65536) return fail(DD_ERR_RANGE, "staged rows too long for 16-bit LDS offsets");
  }
  if (lds > lds_limit) return fail(DD_ERR_RANGE, "staged channel block exceeds LDS");
  t->chan_block = chan_block;
  t->segs = segs;
  t->lds_bytes = (int)lds;
  const int n_dblk = (nd + dblk - 1) / dblk;
  const int ew = int_entry_words(dm_per_wave, segs);  // 32-bit words per channel
  const int ncp = (nc + chan_block - 1) / chan_block * chan_block;  // channels rounded up to whole blocks
  t->offs_words = (size_t)n_dblk * waves * ncp * ew;
  t->sbase_words = (size_t)n_dblk * nc;
  if (!fill) return DD_OK;
  try {
    t->offs.assign(t->offs_words, 0);
    t->sbase.assign(t->sbase_words, 0);
  } catch (const std::bad_alloc &) {
    return fail(DD_ERR_NOMEM, "table allocation failed");
  }
  for (int b = 0; b < n_dblk; ++b) {
    const int32_t *s0 = p.shift.data() + (size_t)(b * dblk) * nc;
    int32_t *sb = t->sbase.data() + (size_t)b * nc;
    for (int c = 0; c < nc; ++c) sb[c] = s0[c] & ~(unit - 1);
    for (int w = 0; w < waves; ++w)
      for (int r = 0; r < dm_per_wave; ++r) {
        const int d = std::min(b * dblk + w * dm_per_wave + r, nd - 1);
        const int32_t *sd = p.shift.data() + (size_t)d * nc;
        uint32_t *o = t->offs.data() + (((size_t)b * waves + w) * ncp) * ew;
        for (int c = 0; c < ncp; ++c) {
          // window offset v (samples) inside the staged row -> byte offset of
          // its first word inside the channel's shifted copies; padding
          // channels (c >= nc, staged as zero rows) read their own row at 0
          const int32_t v = c < nc ? sd[c] - sb[c] : 0;
          const int32_t slot = phase ? (c % chan_block) * copies * t->row_bytes : 0;  // channel's copies in the slot
          const uint32_t e = u16             ? (uint32_t)(slot + (v & 1) * t->row_bytes + 2 * (v & ~1))
                             : phase && u4 ? (uint32_t)(slot + (v & 7) * t->row_bytes + 4 * (v >> 3))
                                           : (uint32_t)(slot + (v & 3) * t->row_bytes + (v & ~3));
          if (phase)
            o[(size_t)c * ew + r] = e;
          else
            o[(size_t)c * ew + (r >> 1)] |= e << (16 * (r & 1));
        }
      }
  }
  return DD_OK;
}

// Tables of the float kernel in direction `adjoint` for shape (ns, per_wave,
// waves, row_block); see FloatTables.
static dd_status build_float_tables(const dd_plan &p, bool adjoint, const int *shape, int lds_limit,
                                    FloatTables *t, bool fill) {
  const int nc = p.desc.n_chan, nd = p.desc.n_dm;
  const int ns = shape[0], per_wave = shape[1], waves = shape[2], rb = shape[3];
  const int n_rows = adjoint ? nd : nc, n_out = adjoint ? nc : nd;
  const int oblk = waves * per_wave;
  const int n_oblk = (n_out + oblk - 1) / oblk;
  auto sh = [&](int o, int k) -> int32_t {
    return adjoint ? -p.shift[(size_t)k * nc + o] : p.shift[(size_t)o * nc + k];
  };
  // staging bases and the largest spread
  std::vector<int32_t> sbase;
  try {
    sbase.assign((size_t)n_oblk * n_rows, 0);
  } catch (const std::bad_alloc &) {
    return fail(DD_ERR_NOMEM, "table allocation failed");
  }
  int64_t span = 0;
  for (int b = 0; b < n_oblk; ++b)
    for (int k = 0; k < n_rows; ++k) {
      int32_t mn = INT32_MAX, mx = INT32_MIN;
      for (int o = b * oblk; o < std::min(n_out, (b + 1) * oblk); ++o) {
        const int32_t v = sh(o, k);
        mn = std::min(mn, v);
        mx = std::max(mx, v);
      }
      sbase[(size_t)b * n_rows + k] = mn & ~3;  // rounds toward minus infinity
      span = std::max<int64_t>(span, (int64_t)mx - mn);
    }
  const int64_t floats = ((int64_t)64 * ns + span + 4 + 3) / 4 * 4;
  if (floats * 4 > (1 << 24)) return fail(DD_ERR_RANGE, "delay spread too large");
  t->row_bytes = (int)(floats * 4);
  const int64_t lds = (int64_t)3 * rb * t->row_bytes + 1024;  // ring of 3 slots and a 1 KiB load sink
  if (lds > lds_limit) return fail(DD_ERR_RANGE, "staged row block exceeds LDS");
  if (rb * ((t->row_bytes + 1023) / 1024) > std::min(64, 16 * waves))  // the kernel's load segments per block
    return fail(DD_ERR_RANGE, "too many staging segments");
  if (t->row_bytes > 65536) return fail(DD_ERR_RANGE, "staged rows too long for 16-bit LDS offsets");
  t->ns = ns;
  t->per_wave = per_wave;
  t->waves = waves;
  t->row_block = rb;
  t->lds_bytes = (int)lds;
  const int rp = per_wave < 2 ? 2 : per_wave;
  const int nrp = (n_rows + rb - 1) / rb * rb;
  t->offs_count = (size_t)n_oblk * waves * nrp * rp;
  t->sbase_count = sbase.size();
  if (!fill) return DD_OK;
  try {
    t->offs.assign(t->offs_count, 0);
  } catch (const std::bad_alloc &) {
    return fail(DD_ERR_NOMEM, "table allocation failed");
  }
  for (int b = 0; b < n_oblk; ++b)
    for (int w = 0; w < waves; ++w)
      for (int r = 0; r < per_wave; ++r) {
        const int o = std::min(b * oblk + w * per_wave + r, n_out - 1);
        uint16_t *dst = t->offs.data() + (((size_t)b * waves + w) * nrp) * rp + r;
        for (int k = 0; k < n_rows; ++k)
          dst[(size_t)k * rp] = (uint16_t)(4 * (sh(o, k) - sbase[(size_t)b * n_rows + k]));
      }
  t->sbase = std::move(sbase);
  return DD_OK;
}

int num_shapes(const dd_plan &p) {
  return p.desc.dtype == DD_F32 ? kNumF32Shapes : kNumIntShapes + kNumDirectShapes;
}

dd_status set_tiles(dd_plan &p, int direction, int shape, int order, bool fill) {
  if (direction != 0 && !(direction == 1 && p.desc.dtype == DD_F32))
    return fail(DD_ERR_ARG, "direction must be 0 (forward) or 1 (adjoint, float plans)");
  if (shape < 0 || shape >= num_shapes(p)) return fail(DD_ERR_ARG, "no such tile shape");
  if (order < 0 || order >= kNumOrders) return fail(DD_ERR_ARG, "no such workgroup order");
  TileCfg t;
  t.shape = shape;
  t.order = order;
  if (p.desc.dtype == DD_F32) {
    FloatTables ft;
    const dd_status st = build_float_tables(p, direction == 1, kF32Shapes[shape], kLdsLimit, &ft, fill);
    if (st != DD_OK) return st;
    ft.shape = shape;
    ft.order = order;
    p.qtab[direction].use = false;
    if (direction == 1) {
      p.ftab_adj = std::move(ft);
      return DD_OK;
    }
    t.ns = ft.ns;
    t.dm_per_wave = ft.per_wave;
    t.waves = ft.waves;
    t.chan_block = ft.row_block;
    t.row_bytes = ft.row_bytes;
    t.lds_bytes = ft.lds_bytes;
    p.ftab_fwd = std::move(ft);
    p.fwd = t;
    return DD_OK;
  }
  const int *k = int_shape(shape);
  IntTables tab;
  if (k[3] == 0) {  // direct-read kernel: no staging tables, any delay spread
    t.ns = k[0];
    t.dm_per_wave = k[1];
    t.waves = k[2];
    t.chan_block = 0;
    t.row_bytes = t.lds_bytes = 0;
    p.fwd = t;
    p.span_fwd = max_dm_block_span(p, t.waves * t.dm_per_wave);
    p.itab = IntTables();
    p.gtab.use = false;
    p.chosen = true;
    return DD_OK;
  }
  const dd_status st = build_int_tables(p, k[0], k[1], k[2], k[3], int_shape_segs(shape), kLdsLimit, &tab, fill);
  if (st != DD_OK) return st;
  t.ns = k[0];
  t.dm_per_wave = k[1];
  t.waves = k[2];
  t.chan_block = k[3];
  t.segs = tab.segs;
  t.row_bytes = tab.row_bytes;
  t.lds_bytes = tab.lds_bytes;
  p.fwd = t;
  p.span_fwd = max_dm_block_span(p, t.waves * t.dm_per_wave);
  p.itab = std::move(tab);
  p.gtab.use = false;
  p.chosen = true;
  return DD_OK;
}

// Default tiles: the first compiled shape (they are listed fastest first; for
// 8-bit plans the phase-load shapes before the others, an 8-wave one
// only where two of its workgroups fit in a CU's LDS) that holds the plan's
// delay spread, in the grouped workgroup order (as fast as time tiles fastest
// on the headline plan, with a third of its L2 fetch traffic).
// For an integer plan whose spread leaves only LDS shapes staging 1 or 2
// channels at a time, the direct-read kernel is faster (measured: 12.7 against
// 8.5-10 Tadds/s at 264-395 samples of delay per DM step) and is chosen.
// 4-bit plans read directly whatever their spread: 2 rows x 8 waves, each XCD
// taking whole time tiles.  Its packed 16-byte windows and in-place nibble adds
// beat staging even on narrow spreads (8192 ch x 2^20 x 4000 DMs at 1200-1500
// MHz: 50.1 against 44.1 Tadds/s for the best staged shape, the phase-load
// form; 4096 ch x 2^19 x 2048 DMs at 120-190 MHz: 50.0 against 25.3 for the
// best staged shape; grid order 1 there against 46.2 for the grouped order).
static dd_status choose_shapes(dd_plan &p) {
  if (p.desc.dtype == DD_U4) return set_tiles(p, 0, kNumIntShapes + 1, kOrderXcdTiles, false);
  const int dirs = p.desc.dtype == DD_F32 ? 2 : 1;
  for (int dir = 0; dir < dirs; ++dir) {
    dd_status last = DD_ERR_RANGE;
    for (int pass = 0; pass < 2 && last != DD_OK && last != DD_ERR_NOMEM; ++pass)
      for (int i = 0; i < num_shapes(p); ++i) {
        const bool phase = p.desc.dtype == DD_U8 && int_shape_segs(i) > 0;
        if (phase != (pass == 0)) continue;
        last = set_tiles(p, dir, i, kOrderDmGroups, false);
        // an 8-wave phase-load shape pays only when two of its workgroups share a CU
        if (last == DD_OK && phase && p.fwd.waves == 8 && 2 * p.fwd.lds_bytes > kLdsLimit) last = DD_ERR_RANGE;
        if (last == DD_OK || last == DD_ERR_NOMEM) break;
      }
    if (last == DD_ERR_NOMEM) return last;
    if (last != DD_OK) return fail(DD_ERR_RANGE, "delay spread exceeds every compiled staging shape");
  }
  // Direct shape for 8- and 16-bit samples: 4 rows x 4 waves (4096 ch x 2^20 at 120-190 MHz,
  // DM step 0.5: 30.0 against 25.9 Tadds/s for 2 x 8 with 8-bit samples, 11.7 against 8.2 with
  // 16-bit), each XCD taking whole time tiles (on 4096-channel plans at 120-190, 300-400 and
  // 1200-1500 MHz: 8-bit 33.0-34.3 against 30.5-31.2 Tadds/s for the grouped order, 16-bit
  // 17.0-17.8 against 16.1-16.7), except 8-bit plans too wide for 4-channel stages, which
  // keep the grouped order (4096 ch x 2^20 at 120-190 MHz, DM step 0.5: 30.0 against 29.3).
  // An 8-bit plan reads directly when its staged shape holds at most 4 channels per stage: on
  // those four plans (staged shapes 16, 17, 18 and 5) 33.0-34.3 against 15.0-24.4 Tadds/s.
  const int direct = kNumIntShapes;
  if (p.desc.dtype == DD_U8 && !is_direct(p.fwd) && p.fwd.chan_block <= 4)
    return set_tiles(p, 0, direct, p.fwd.chan_block <= 2 ? kOrderDmGroups : kOrderXcdTiles, false);
  // 16-bit plans: the 8-wave shape with 4 rows per wave and 4 channels per stage,
  // where two of its workgroups fit in a CU's LDS, so that one's barrier waits
  // overlap the other's adds: first in its phase-load form (the two copies loaded
  // straight into LDS: 1111.5 against 1326.9 ms on 8192 ch x 2^20 x 4000 DMs),
  // else in its raw-ring form (13-16% faster than the 16-wave default on 8192 x
  // 2^20 and on binned 4096-channel ranges; 11% slower on a plan with ~1000
  // samples of spread per 32 DMs, where only one fits).  Otherwise a plan left
  // with at most 4 channels per stage reads directly (4096-channel plans whose
  // staged shape was the 1-row, 16-wave raw ring: 17.0-17.8 against 14.6-15.1
  // Tadds/s), as does one with at most 2.
  if (p.desc.dtype == DD_U16 && !is_direct(p.fwd)) {
    if (p.fwd.chan_block <= 2) return set_tiles(p, 0, direct, kOrderXcdTiles, false);
    const int keep_shape = p.fwd.shape, keep_order = p.fwd.order;
    bool moved = false;
    for (int want_phase = 1; want_phase >= 0; --want_phase)
      for (int i = 0; i < kNumIntShapes; ++i) {
        const int *k = kIntShapes[i];
        if (k[0] != 16 || k[1] != 4 || k[2] != 8 || k[3] != 4 || (k[4] > 0) != (want_phase == 1)) continue;
        if (i == keep_shape) return moved ? set_tiles(p, 0, keep_shape, keep_order, false) : DD_OK;
        const dd_status st = set_tiles(p, 0, i, kOrderDmGroups, false);
        if (st == DD_ERR_NOMEM) return st;
        if (st == DD_OK && 2 * p.fwd.lds_bytes <= kLdsLimit) return DD_OK;
        moved = moved || st == DD_OK;
        break;
      }
    if (moved) {
      const dd_status st = set_tiles(p, 0, keep_shape, keep_order, false);
      if (st != DD_OK) return st;
    }
    if (p.fwd.chan_block <= 4) return set_tiles(p, 0, direct, kOrderXcdTiles, false);
  }
  return DD_OK;
}

static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// Modelled us of a launch: `longest` and `mean` of its workgroups, `rounds` of resident ones.
// Past the first round, workgroups in different phases overlap.
static double launch_us(double longest, double mean, double rounds, double overlap, double tail) {
  return rounds <= 1 ? longest : std::max(longest, overlap * mean * (rounds + tail));
}

// Whether an integer plan's forward runs by group sums (fwd_group.hip) instead of
// its shape's kernel.  Two models in turn:
//
// From the patterns alone (max_cost), before any tables are built: where group sums cannot
// come out a tenth ahead.  Both kernels run in rounds of resident workgroups (256 CUs): group
// sums one per CU, the other kernels two of 32 rows x 512 samples.  kModel: the group
// kernel's measured time against this model (8192 ch x 2^20 x 4000 DMs 8-bit: 353 ms
// against 513; 1024 ch x 101773 x 700: 1.09 against 1.48); rate: additions per CU clock of
// the other kernels (8-bit 40.8 Tadds/s on the 8-wave staged shape, 33-34 on the others;
// 4-bit 50; 16-bit 30 and 17).  This model is rough: it is up to 5 times off where a plan has few
// channels or workgroups, and refuses 128 ch x 32768 x 256 DMs of step 1 (42 us against 36)
// by far more than that.
//
// From the tables: a workgroup of group sums takes a start of 9 us (16-bit: 12) and about
// 9 clocks per building instruction of its busiest SIMD, step by step; one of the other
// kernels a start and a time per channel, less where a CU has only one of them; both less
// where few run.  Constants fitted to 1160 plans (32-4096 ch, 16-1500 DMs of step 0.02-2,
// 2000-300000 outputs at 1200-1550 MHz), timed both ways: group sums to 6-9%, the others to
// 5-8%.  Without this model 128 of 593 8-bit plans of that set ran by group sums that are up
// to 1.86 times as slow as their shape (200 ch x 82109 x 116 DMs: 98 against 78 us), 19 of 259
// 4-bit and 5 of 241 16-bit ones up to 1.31 and 1.39; with it 5, 1 and 1, at most 1.07, and
// 11 that would gain 2% or more (one 22%) run their shape.  Of 700 other plans 50 were slower
// by group sums without it; with it 7, at most 1.10, and 3 that would gain 2 to 4% run their shape.
// On the two plans above, 4-bit 8192 ch x 2^18 x 500 and 16-bit the same, group sums against
// the other kernels: 353 / 820, 1.09 / 1.78, 13.1 / 22.4 and 21.7 / 37.7 ms.
//
// A beam of a batch: the same two models without rounds, for many workgroups in flight, fitted
// to 330 plans (128-1024 ch, 64-512 DMs) in batches of themselves (group sums to 7%, the
// others to 2-4%).  There 8 of 157 4-bit beams were up to 1.26 times as slow by group sums; with
// the second model two (1.04 and 1.20).  Next to beams that gain by group sums, up to a tenth is
// given to them, since the two kernels fill each other's waits: eight 4-bit batches of 9-30
// beams took 1 to 5% longer with the line at equal times less 3%, and the same at equal
// times and at 5%, 10%, 20% and more above.
namespace {
struct GroupModel {
  // group sums: us of a workgroup and per instruction with all CUs busy, how much less with few;
  // several rounds
  double start, op, idle, overlap, tail;
  // the other kernel's workgroup, two of which share a CU; its us, and per channel
  int rows;
  double samples, own_start, own_chan;
  // shares of the time per channel: one on every CU, how much less with few; the start of a second one
  double alone, own_idle, second, own_overlap, own_tail;
  double margin;  // of the other kernel's time that group sums may take
  double batch_start, batch_op, batch_own_start, batch_own_chan;  // the same among many beams
};
constexpr GroupModel kGroup8 = {8.91, 0.00357, 0.119, 0.62, 1.13, 32, 512, 5.83, 0.2267, 0.715, 0.207, 1.02, 0.795, 0.724,
                                1.01, 4.43, 0.00256, 4.04, 0.1967};
constexpr GroupModel kGroup4 = {9.29, 0.00379, 0.140, 0.635, 1.30, 16, 1008, 9.71, 0.2482, 0.934, 0.418, 0.951, 0.663,
                                0.852, 0.97, 5.52, 0.00279, 5.45, 0.1676};
constexpr GroupModel kGroup16 = {11.96, 0.00413, 0.149, 0.796, 0.754, 32, 1024, 7.96, 0.6722, 0.668, 0.122, 0.947, 0.783,
                                 0.647, 1.0, 8.04, 0.0035, 6.28, 0.9156};
}  // namespace

SumsPay build_group_sums(const dd_plan &p, bool batch, GroupTables *t) {
  const double kModel = 0.74, kCus = 256;
  const int bits = p.desc.dtype == DD_U4 ? 4 : p.desc.dtype == DD_U16 ? 16 : 8;
  const bool best_staged = !is_direct(p.def_fwd) && p.def_fwd.waves == 8;
  const double rate = bits == 4 ? 80.0 : bits == 16 ? (best_staged ? 47.0 : 27.0) : best_staged ? 64.0 : 53.0;
  const int64_t tile = bits == 16 ? kGrpWin : 2 * kGrpWin;
  const int64_t n_blk = (p.desc.n_dm + group_rows(bits) - 1) / group_rows(bits), tiles = (p.n_out + tile - 1) / tile;
  const double groups = ceil((double)n_blk * (double)tiles / kCus);
  const double others = ceil((double)((p.desc.n_dm + 31) / 32) * (double)((p.n_out + 511) / 512) / (2 * kCus));
  // a beam of a batch: all its tiles against the plan's additions; a plan: the group kernel's rounds
  // at its mean cost per block against the others' rounds
  const double limit =
      batch ? 0.9 * (double)p.desc.n_dm * (double)p.n_out * p.desc.n_chan / rate / kModel / (double)tiles
            : 0.9 * others * (2.0 * 32 * 512) * p.desc.n_chan / rate / (groups * kModel) * (double)n_blk;
  const GroupModel m = bits == 8 ? kGroup8 : bits == 4 ? kGroup4 : kGroup16;
  const double slow = bits == 4 || best_staged ? 1.0 : bits == 8 ? 1.2 : 1.7;  // staged shapes of 16 waves, direct reads
  const double rounds = (double)n_blk * (double)tiles / kCus;
  const double own_wgs = ceil((double)p.desc.n_dm / m.rows) * ceil((double)p.n_out / m.samples);
  const double own_rounds = own_wgs / (2 * kCus), own_wg = m.own_start + m.own_chan * slow * p.desc.n_chan;
  // the most instructions per block that pay: of the largest block in a single round, else (and in
  // a batch) of all on average
  double max_work, near_work = 0;
  if (batch) {
    const double own = (m.batch_own_start + m.batch_own_chan * slow * p.desc.n_chan) * own_rounds;
    max_work = (own / rounds - m.batch_start) / m.batch_op;
    near_work = (1.1 * own / rounds - m.batch_start) / m.batch_op;
  } else {
    const double share = own_rounds <= 0.5 ? m.alone + m.own_idle * (own_rounds - 0.5)
                                           : m.second + (1.0 - m.second) * 2.0 * (std::min(own_rounds, 1.0) - 0.5);
    const double own = m.margin * (own_rounds <= 1 ? m.own_start + m.own_chan * slow * p.desc.n_chan * share
                                                   : launch_us(own_wg, own_wg, own_rounds, m.own_overlap, m.own_tail));
    const double op = m.op * (1.0 - m.idle * std::max(0.0, 1.0 - rounds));
    max_work = ((rounds <= 1 ? own : own / (m.overlap * (rounds + m.tail))) - m.start) / op;
  }
  near_work = std::max(near_work, max_work);
  if (near_work <= 0) return kSumsLose;
  const GroupTables *g = &p.gtab;
  if (p.gtab.data.empty()) {
    if (!build_group_tables(p.shift.data(), p.desc.n_dm, p.desc.n_chan, bits, p.in_pitch_bytes, t, limit, near_work) ||
        t->data.size() * 4 > p.def_table_bytes) {
      *t = GroupTables();
      return kSumsLose;
    }
    g = t;
  }
  const double work = rounds <= 1 && !batch ? g->max_work : g->work / (double)n_blk;
  if (g->cost <= limit && work < max_work) return kSumsPay;
  if (g->cost <= limit && work < near_work) return kSumsNear;
  *t = GroupTables();
  return kSumsLose;
}

// Whether a direction of a float plan runs by quad sums (quad_f32.hip) instead of its
// shape's kernel, and with how many outputs per block: where the modelled time, in rounds
// of one workgroup per CU, is below 0.62 of the other kernel's (kRate: additions per CU
// clock; 22.7 measured on 1024 ch x 131900 x 512 DMs).  At 1200-1500 MHz, quad sums against
// the other kernel by what the model says: 0.26-0.40 of it: 0.35-0.57 measured (that plan's
// forward: 1618 against 4919 us); 0.41-0.53: 0.41-0.73; 0.58-0.62: 0.77-0.93; 0.64 (512 ch x
// 35996 x 200 DMs of step 1, 256 ch x 16944 x 70): 1.14 and 1.26, since steps of one or two
// quads wait at their barriers.  Then, with the tables at hand, where it is also faster in a
// second model: a start per workgroup, a time per record of the busiest SIMD, step by step,
// and per quad, against the two-outputs-per-wave shapes' start and time per row.  Constants
// fitted to 658 plans and directions (32-1024 ch, 24-1024 DMs), both kernels to 7%.  Without it 7 of the 633
// taken were slower by shared sums, up to 1.26 times (adjoint of 200 ch x 66828 x 126 DMs of
// step 0.5: 198 against 157 us), with it 2 (that one and 1.07), and one that would gain 23% of
// 33 us runs its shape.
static void choose_quads(dd_plan &p, int dir) {
  const FloatTables &t = dir ? p.ftab_adj : p.ftab_fwd;
  const double kRate = 23.0, kCus = 256;
  const int nd = p.desc.n_dm, nc = p.desc.n_chan;
  const QuadShifts sh = {p.shift.data(), dir ? 1 : (int64_t)nc, dir ? (int64_t)nc : 1, dir ? -1 : 1, dir ? nc : nd,
                         dir ? nd : nc};
  const int64_t out_len = dir ? p.desc.n_samp : p.n_out, tiles = (out_len + kQuadWin - 1) / kQuadWin;
  const int64_t oblk = t.waves * t.per_wave, n_oblk = (sh.n_out + oblk - 1) / oblk;
  const int64_t others_tiles = (out_len + 64 * t.ns - 1) / (64 * t.ns);
  double best = 0.62 * ceil((double)(n_oblk * others_tiles) / kCus) * (double)(oblk * 64 * t.ns) * sh.n_rows / kRate;
  int rows = 0;
  for (int r : {64, 32}) {
    const int64_t n_blk = (sh.n_out + r - 1) / r;
    const double v = ceil((double)(n_blk * tiles) / kCus) * guess_quad_cost(sh, r) / (double)n_blk;
    if (v < best) best = v, rows = r;
  }
  QuadTables q;
  if (!rows || !build_quad_tables(sh, rows, &q) ||
      q.data.size() * 4 > up256(t.offs_count * 2) + up256(t.sbase_count * 4))  // (they take those tables' place)
    return;
  if (t.per_wave == 2) {
    const double start = rows == 64 ? 8.30 : 6.78, rec = rows == 64 ? 0.307 : 0.42, quad = rows == 64 ? 0.255 : 0.071;
    const double fixed = start + quad * ((sh.n_rows + 3) / 4);
    const double sums = launch_us(fixed + rec * q.max_records, fixed + rec * q.records / q.n_blk,
                                  (double)(q.n_blk * tiles) / kCus, 0.9, 0.86);
    const double own_wg = t.row_block == 8 ? 10.4 + 0.533 * sh.n_rows : 9.0 + 0.61 * sh.n_rows;
    if (sums > launch_us(own_wg, own_wg, (double)(n_oblk * others_tiles) / kCus, 0.925, 0.82)) return;
  }
  // Orders, measured on 1024 ch x 135212 x 512 DMs of step 0.5, the same of step 0.1 and 512
  // ch x 33576 x 200 (two rounds of workgroups).  Forward, by tiles per XCD / groups of
  // blocks / runs of tiles / tiles first: 2157 / 2258 / 2397 / 2417, 1607 / 1707 / 1796 /
  // 1822 and 177 / 174 / 179 / 174 us.  Adjoint: 2218 / 2245 / 2177 / 2171, 1633 / 1706 /
  // 1706 / 1715 and 164 / 173 / 154 / 152 us; 1024 ch x 2^17 x 1024: 4885 / 4817 / 4743 / 4751.
  q.order = dir ? kOrderXcdRuns : q.n_blk * tiles > 2 * (int64_t)kCus ? kOrderXcdTiles : kOrderDmGroups;
  q.use = true;
  p.qtab[dir] = std::move(q);
}

dd_status choose_forward_tiles(dd_plan &p) {
  dd_status st = choose_shapes(p);
  if (st != DD_OK) return st;
  p.def_fwd = p.fwd;
  p.def_table_bytes = table_bytes(p);
  p.def_shape[0] = p.fwd.shape;
  p.def_order[0] = p.fwd.order;
  p.def_shape[1] = p.ftab_adj.shape;
  p.def_order[1] = p.ftab_adj.order;
  // the tables of shared sums, or those of the shapes that they do not replace
  if (p.desc.dtype == DD_F32) {
    for (int dir = 0; dir < 2 && st == DD_OK; ++dir) {
      choose_quads(p, dir);
      const FloatTables &t = dir ? p.ftab_adj : p.ftab_fwd;
      if (!p.qtab[dir].use) st = set_tiles(p, dir, t.shape, t.order);
    }
  } else {
    GroupTables t;
    if (build_group_sums(p, false, &t) == kSumsPay) {
      p.gtab = std::move(t);
      p.gtab.use = true;
    } else {
      st = set_tiles(p, 0, p.fwd.shape, p.fwd.order);
    }
  }
  p.chosen = false;
  return st;
}

// Device workspace layout.  Integer plans: [offs words][sbase int32].
// Float plans: [forward offs][forward sbase][adjoint offs][adjoint sbase].
TableLayout table_layout(const dd_plan &p) {
  TableLayout L;
  if (p.desc.dtype != DD_F32) {
    if (!is_direct(p.fwd)) L.int_sbase = up256(p.itab.offs_words * sizeof(uint32_t));
    return L;
  }
  size_t off = 0;
  const FloatTables *tabs[2] = {&p.ftab_fwd, &p.ftab_adj};
  for (int k = 0; k < 2; ++k) {
    L.f_offs[k] = off;
    off += up256(tabs[k]->offs_count * 2);
    L.f_sbase[k] = off;
    off += up256(tabs[k]->sbase_count * 4);
  }
  return L;
}

size_t table_bytes(const dd_plan &p) {
  if (p.desc.dtype != DD_F32 && is_direct(p.fwd)) return up256(p.shift.size() * sizeof(int32_t));
  if (p.desc.dtype != DD_F32)
    return up256(p.itab.offs_words * sizeof(uint32_t)) + up256(p.itab.sbase_words * sizeof(int32_t));
  return up256(p.ftab_fwd.offs_count * 2) + up256(p.ftab_fwd.sbase_count * 4) + up256(p.ftab_adj.offs_count * 2) +
         up256(p.ftab_adj.sbase_count * 4);
}

// Table sizes follow the layouts of build_int_tables / build_float_tables
// (offs: per output block, wave and padded row, `entry_bytes` bytes of
// entries; sbase: per output block and row, one int32).
static size_t shape_table_bytes(int64_t n_out, int64_t n_rows, const int *k, int64_t entry_bytes) {
  const int64_t per_wave = k[1], waves = k[2], rb = k[3];
  const int64_t n_oblk = (n_out + waves * per_wave - 1) / (waves * per_wave);
  const int64_t rows_pad = (n_rows + rb - 1) / rb * rb;
  return up256((size_t)(n_oblk * waves * rows_pad * entry_bytes)) + up256((size_t)(n_oblk * n_rows * 4));
}

size_t tune_table_bytes(const dd_plan &p) {
  const int64_t nc = p.desc.n_chan, nd = p.desc.n_dm;
  size_t fwd = 0, adj = 0;
  if (p.desc.dtype != DD_F32) {
    for (int i = 0; i < kNumIntShapes; ++i)
      fwd = std::max(fwd, shape_table_bytes(nd, nc, kIntShapes[i], 4 * int_entry_words(kIntShapes[i][1], kIntShapes[i][4])));
    return std::max(fwd, up256((size_t)nd * (size_t)nc * sizeof(int32_t)));  // direct shapes: the shift table
  }
  for (int i = 0; i < kNumF32Shapes; ++i) {
    const int64_t eb = 2 * std::max(kF32Shapes[i][1], 2);  // max(per_wave, 2) uint16 entries
    fwd = std::max(fwd, shape_table_bytes(nd, nc, kF32Shapes[i], eb));
    adj = std::max(adj, shape_table_bytes(nc, nd, kF32Shapes[i], eb));
  }
  return fwd + adj;
}

}  // namespace dd
