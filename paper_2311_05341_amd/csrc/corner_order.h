// Which order the workgroups of the corner turn (corner.hip) take.  Plain C++, no device code.
#pragma once

#include <stdint.h>

namespace dd {

// Whether each XCD takes a run of time tiles (corner.hip), or all of them walk the channel
// tiles of one time tile after another.  Runs finish a line of the output, or a line of the
// input that two channel tiles share, in one XCD's L2; in order, spectra are read as they lie.
// bits: of a sample; tile_chan: channels of a tile; out_or: output address | its row pitch.
//
// Runs against the order by time tiles, us:
// * Float rows of whole lines are read a little faster in order (1024 ch x 100000: 166 / 158).
// * A multiple of 8 channel tiles (but for just 8 of samples wider than 4 bits): the order by
//   time tiles, too, keeps a channel tile on its XCD, and runs pay only for turns far larger
//   than the caches (8-bit 4096 ch x 436460: 739 / 1041, 8192 x 40002: 151 / 173); below, 8
//   XCDs each with a time tile of their own cost up to 15% (float 16384 x 5000: 155 / 138,
//   16-bit 16384 x 5000: 72 / 65, 4-bit 16384 x 8300: 40 / 35, 8-bit 32768 x 1994: 28 / 25).
//   The line is at 1.7e8 samples for all types, over rows of whole lines of 8 or 16 bits at
//   1.4 GB read and written (8-bit 4096 ch x 136192: 1.07 times, x 253562: 0.92; 4-bit 2048 x
//   166912: 0.91).  Spectra that do not end on a line pay in any case.
// * One channel tile over rows of whole lines: only its spectra can share lines (4-bit 257 ch x
//   231424: 23 / 31, 16-bit 128 x 200000: 16 / 14, 8-bit 64 x 2152448: 63 / 55); large ones of
//   at least half a tile gain a little (8-bit 256 x 2294784: 225 / 240).  Short 4-bit ones do
//   not gain over other rows either (256 x 271658: 27 / 24).
// * All others gain, up to half (8-bit 1024 x 2318480: 977 / 2006, float 3000 x 70002: 360 / 608).
// Of 1010 turns timed both ways, 84 were 2.5 to 21% slower by runs; 16 of them still take runs
// (4-bit 512 x 103042 11%, the others at most 8%), and 15 that would gain 2.5 to 7% do not.
inline bool corner_runs(int bits, int n_chan, int64_t n_samp, int64_t in_pitch, uint64_t out_or, int tile_chan) {
  const int n_ctiles = (n_chan + tile_chan - 1) / tile_chan;
  const double samples = (double)n_chan * (double)n_samp;
  const bool whole = out_or % 128 == 0, big = samples >= 1.7e8;
  if (bits == 32 && whole) return false;
  if (n_ctiles % 8 == 0 && (n_ctiles > 8 || bits == 4))
    return (whole && bits > 4 ? samples * bits / 4 >= 1.4e9 : big) || in_pitch % 128 != 0;
  if (n_ctiles > 1) return true;
  if (whole) return (big && 2 * n_chan >= tile_chan) || (in_pitch > 128 && in_pitch % 128 != 0);
  return !(bits == 4 && !big && in_pitch % 128 == 0);
}

}  // namespace dd
