// Forward transform for integer input by shared group sums (tables:
// group_tables.h).
//
// A workgroup owns 32 (16-bit input: 64) DM rows x one time tile and runs through groups of
// neighbouring channels.  Per group, its waves compute the partial sums of the group's few
// delay patterns over the tile's window into LDS, and each adds to its own DM rows the window
// of the pattern a row follows, at the row's own offset: one LDS read and one add per row,
// word and group, where a kernel that sums channel by channel does one per channel.
//
// LDS words: 8- and 4-bit input packs two 16-bit partial sums per word, the
// samples k and k + kGrpWin of the tile, so that a window at any offset starts
// on a word and lane i owns words i, i + 64, ...: no byte phases, no bank
// conflicts.  16-bit input keeps one 32-bit sum per word.
//
// Steps: the LDS holds the partial sums of two steps (a few groups each).  Between
// two barriers every wave builds its part of the next step's partial sums and adds
// up its rows of the current step's; half of the waves of each SIMD start with the
// one, half with the other, so vector work and LDS reads overlap.  A building wave
// streams records, each a block of 8 operations (add a channel's window, or move a
// channel by one sample), loading the channel rows straight from global memory 8
// operations ahead of their use: lane i takes the words 4i..4i+3 of its 252-word
// chunk of a pattern row, later samples come from lane i + 1 (DPP; lane 63 only
// loads).
//
// Bound by instruction issue: on 8192 ch x 2^20 x 4000 DMs (8-bit) the vector units
// are 67% busy, LDS 58%, and waves wait 39% of their time.
// Measured (8-bit 8192 ch x 2^20 x 4000 DMs): 353 ms, 94 Tadds/s, against 820 ms for
// the staged kernel.  What mattered, on the way there: branches (a branch-free move
// and one load site per operation: 464 -> 400 ms; waves specialised into builders and
// summers, 2 and 2 per SIMD, left the builders' serial instruction stream exposed:
// 699), loads aligned to 4 bytes (a wave's unaligned dword load takes 17 clocks, an
// aligned one 5.4), exact load counts in every wait (a conditional load turns them
// into full waits), groups small enough that a step has a part for almost every wave.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dd_internal.h"
#include "group_tables.h"
#include "tile_order.h"

namespace dd {
namespace {

struct GroupArgs {
  const uint8_t *x;      // channel rows
  const uint32_t *tab;   // GroupTables::data
  float *out;            // [n_dm][out_pitch]
  int64_t n_out, out_pitch;
  int32_t n_dm;
  int64_t row_bytes;     // readable bytes of a row (a multiple of 16)
  int64_t total;         // readable bytes of the input
  int32_t out_mode;      // an OutMode; other than kOutFloat for 16-bit input only
};

template <typename T>
__device__ __forceinline__ T scalar_load(const T *p, int64_t i) {
  return ((const __attribute__((address_space(4))) T *)p)[i];
}

// LDS-only barrier: the loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Lane i's value of v from lane i + 1 (lane 63: zero).
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);  // wave_shl:1
}

typedef __attribute__((address_space(3))) uint32_t lds_word;
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

struct Rec {
  uint32_t h[kGrpRecWords];
  uint32_t base[2], kinds[2];
  uint32_t off[kGrpOps];
};

// One operation's window as loaded: lane i's samples 4i..4i+3 (8-bit input: w[1]
// the same kGrpWin later; 4-bit: 16 bits each).
struct Raw {
  uint32_t w[2];
};

// Byte offset of word k (0, 1) of a lane's window.
template <int BITS>
__device__ __forceinline__ int lane_byte(int lane, int k) {
  return BITS == 4 ? 2 * lane + k * (kGrpWin / 2) : BITS == 8 ? 4 * lane + k * kGrpWin : 8 * lane + 4 * k;
}

// Loads of a record's windows, whose offsets count from byte `org` of the input.
// Loads are aligned.  EDGE: the tile may reach past the input's ends; loads are
// then moved inside it (a load lies wholly inside or outside, and no output uses
// what lies outside).
template <int BITS, bool EDGE>
struct Windows {
  __amdgpu_buffer_rsrc_t rs;
  int64_t org, total;
  const uint8_t *x;

  __device__ __forceinline__ Windows(const GroupArgs &a, int64_t org_) : org(org_), total(a.total), x(a.x) {
    if constexpr (!EDGE) {
      uint64_t b = (uint64_t)a.x + (uint64_t)org;
      asm("" : "+s"(b));  // a descriptor in scalar registers
      rs = __builtin_amdgcn_make_buffer_rsrc((void *)b, 0, -1, 0x00020000);
    }
  }
  __device__ __forceinline__ void load(Raw &w, uint32_t off, int lane) const {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int l = lane_byte<BITS>(lane, k);
      if constexpr (EDGE) {
        using T = typename std::conditional<BITS == 4, uint16_t, uint32_t>::type;
        w.w[k] = *(const T *)(x + max(min(org + off + l, total - (int)sizeof(T)), (int64_t)0));
      } else if constexpr (BITS == 4) {
        w.w[k] = __builtin_amdgcn_raw_buffer_load_b16(rs, l, (int)off, 0);
      } else {
        w.w[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, l, (int)off, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // loads stay in the order of their use
  }
};

// The lane's four sample words, in the order loaded.
template <int BITS>
__device__ __forceinline__ void unpack(const Raw &w, uint32_t (&x)[4]) {
  if constexpr (BITS == 8) {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = __builtin_amdgcn_perm(w.w[1], w.w[0], 0x0C040C00u + 0x00010001u * j);
  } else if constexpr (BITS == 4) {
    const uint32_t v = __builtin_amdgcn_perm(w.w[1], w.w[0], 0x05040100u);
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = (v >> (4 * j)) & 0x000F000Fu;
  } else {
    x[0] = w.w[0] & 0xFFFFu;
    x[1] = w.w[0] >> 16;
    x[2] = w.w[1] & 0xFFFFu;
    x[3] = w.w[1] >> 16;
  }
}

// P += the sums S of windows of phase m (bits 8q and 8q + 1 of kinds): sample j of
// a window is word j + m, from the next lane past word 3; S = 0.  In asm (three
// scalar branches; left to itself the compiler selects among copies).  The scalar
// instructions before the first DPP read of S cover its two wait states.
template <int Q>
__device__ __forceinline__ void fold(uint32_t (&P)[4], uint32_t (&S)[4], uint32_t kinds) {
#define DD_NEXT " wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
  asm("s_bitcmp1_b32 %8, %9\n\t"
      "s_cbranch_scc1 .Lf2%=\n\t"
      "s_bitcmp1_b32 %8, %10\n\t"
      "s_cbranch_scc1 .Lf1%=\n\t"
      "v_add_u32 %0, %4, %0\n\tv_add_u32 %1, %5, %1\n\tv_add_u32 %2, %6, %2\n\tv_add_u32 %3, %7, %3\n\t"
      "s_branch .Lfd%=\n"
      ".Lf1%=:\n\t"
      "v_add_u32 %0, %5, %0\n\tv_add_u32 %1, %6, %1\n\tv_add_u32 %2, %7, %2\n\t"
      "v_add_u32_dpp %3, %4, %3" DD_NEXT
      "s_branch .Lfd%=\n"
      ".Lf2%=:\n\t"
      "s_bitcmp1_b32 %8, %10\n\t"
      "s_cbranch_scc1 .Lf3%=\n\t"
      "v_add_u32 %0, %6, %0\n\tv_add_u32 %1, %7, %1\n\t"
      "v_add_u32_dpp %2, %4, %2" DD_NEXT
      "v_add_u32_dpp %3, %5, %3" DD_NEXT
      "s_branch .Lfd%=\n"
      ".Lf3%=:\n\t"
      "v_add_u32 %0, %7, %0\n\t"
      "v_add_u32_dpp %1, %4, %1" DD_NEXT
      "v_add_u32_dpp %2, %5, %2" DD_NEXT
      "v_add_u32_dpp %3, %6, %3" DD_NEXT
      ".Lfd%=:\n\t"
      "v_mov_b32 %4, 0\n\tv_mov_b32 %5, 0\n\tv_mov_b32 %6, 0\n\tv_mov_b32 %7, 0"
      : "+v"(P[0]), "+v"(P[1]), "+v"(P[2]), "+v"(P[3]), "+v"(S[0]), "+v"(S[1]), "+v"(S[2]), "+v"(S[3])
      : "s"(kinds), "i"(8 * Q + 1), "i"(8 * Q)
      : "scc");
#undef DD_NEXT
}

// The window's sample words 0..4 of a window of phase m.
template <int BITS>
__device__ __forceinline__ void window(const Raw &w, uint32_t m, uint32_t (&x)[5]) {
  uint32_t v[4];
  if constexpr (BITS == 8) {
    Raw s;
#pragma unroll
    for (int k = 0; k < 2; ++k) s.w[k] = __builtin_amdgcn_alignbyte(next_lane(w.w[k]), w.w[k], m);
    unpack<BITS>(s, v);
  } else if constexpr (BITS == 4) {
    Raw s;
    const uint32_t sh = 4 * (m & 3);
#pragma unroll
    for (int k = 0; k < 2; ++k) s.w[k] = (w.w[k] | next_lane(w.w[k]) << 16) >> sh;
    unpack<BITS>(s, v);
  } else {
    Raw s;
    const uint32_t sh = 16 * (m & 1);
    s.w[0] = __builtin_amdgcn_alignbit(w.w[1], w.w[0], sh);
    s.w[1] = __builtin_amdgcn_alignbit(next_lane(w.w[0]), w.w[1], sh);
    unpack<BITS>(s, v);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = v[j];
  x[4] = next_lane(v[0]);
}

// Operation Q of a record (its kind in byte Q of kinds).  A move is P += d or P -= d
// with d(j) = x(j + 1) - x(j), without a branch: with b = 1 for down and m = -b,
// P + ((d - b) xor m) is either (asm: the compiler knows no subtraction with a
// scalar borrow); P goes into the row at hand in any case, and a finished row is
// left behind.
template <int BITS, int Q>
__device__ __forceinline__ void run_op(uint32_t (&P)[4], uint32_t (&S)[4], const Raw &w, uint32_t kinds, uint32_t &dst,
                                       uint32_t step) {
  constexpr int B = 8 * Q;
  if (kinds & (kOpMove << B)) {
    uint32_t x[5], d[4];
    window<BITS>(w, kinds >> B, x);
    static_assert(kOpDown == 8 && kOpWrite == 64, "bits 3 and 6");
    const uint32_t m = (uint32_t)((int32_t)(kinds << (28 - B)) >> 31);
    const uint64_t borrow = (uint64_t)m << 32 | m;
    uint64_t unused;
    asm("v_subb_co_u32 %0, %4, %6, %5, %10\n\t"
        "v_subb_co_u32 %1, %4, %7, %6, %10\n\t"
        "v_subb_co_u32 %2, %4, %8, %7, %10\n\t"
        "v_subb_co_u32 %3, %4, %9, %8, %10"
        : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]), "=&s"(unused)
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "s"(borrow));
#pragma unroll
    for (int j = 0; j < 4; ++j) P[j] += d[j] ^ m;
    *(__attribute__((address_space(3))) v4u *)(uintptr_t)dst = v4u{P[0], P[1], P[2], P[3]};
    dst += step & (uint32_t)((int32_t)(kinds << (25 - B)) >> 31);
  }
  if (kinds & (kOpAdd << B)) {
    uint32_t x[4];
    unpack<BITS>(w, x);
#pragma unroll
    for (int j = 0; j < 4; ++j) S[j] += x[j];
    if (kinds & (kOpFold << B)) {
      fold<Q>(P, S, kinds);
      if (kinds & (kOpWrite << B)) {
        *(__attribute__((address_space(3))) v4u *)(uintptr_t)dst = v4u{P[0], P[1], P[2], P[3]};
        dst += step;
      }
    }
  }
}

// Output of one exact total by OutMode: float32, the raw 32-bit total, or low
// (read back) + 2^16 * this total converted once.
__device__ __forceinline__ void store_total(float *o, uint32_t v, int mode) {
  if (mode == kOutRawTotals)
    *(uint32_t *)o = v;
  else if (mode == kOutCombineHigh)
    *o = (float)((double)*(const uint32_t *)o + 65536.0 * (double)v);
  else
    *o = (float)v;
}

constexpr int kGrpThreads = 64 * kGrpWaves;
constexpr int kGrpLdsBytes = 2 * kGrpSetBytes + kGrpZeroBytes + kGrpTrashBytes;

template <int BITS>
constexpr int tile_samples() { return BITS == 16 ? kGrpWin : 2 * kGrpWin; }

template <int BITS, bool EDGE>
__device__ __forceinline__ void group_tile(uint8_t *lds, const GroupArgs &a, const GroupBlock *gb, int blk, int64_t t0,
                                           int wave, int lane) {
  constexpr int R = group_rows_per_wave(BITS);
  constexpr int kSumWords = group_sum_words(BITS);
  constexpr int NW = kGrpWin / 64;  // words per lane and row
  constexpr bool PACKED = BITS != 16;

  const GroupHead *th = (const GroupHead *)a.tab;

  // ---- building: this wave's record stream
  const uint32_t *rp = a.tab + scalar_load(&th->rec_off, 0) + (uint64_t)scalar_load(&gb->rec_first[wave], 0) * kGrpRecWords;
  const uint32_t *const ops = a.tab + scalar_load(&th->op_off, 0);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
  const uint32_t trash = lds0 + 2 * kGrpSetBytes + kGrpZeroBytes + 16u * lane;
  uint32_t P[4] = {0, 0, 0, 0}, S[4] = {0, 0, 0, 0};
  Rec cur, next;                 // the record in hand, its windows loaded or on the way, and the one after it
  uint32_t head[kGrpRecWords];   // the head of the record after those
  Raw win[kGrpOps];
  auto load_head = [&]() {
#pragma unroll
    for (int i = 0; i < kGrpRecWords; ++i) head[i] = scalar_load(rp, i);
    rp += kGrpRecWords;
  };
  // Record `head` into r, and the next head (the table holds records past the last stream).
  auto load_rec = [&](Rec &r) {
    const uint32_t *o = ops + (uint64_t)head[0] * kGrpBlockWords;
#pragma unroll
    for (int i = 0; i < kGrpRecWords; ++i) r.h[i] = head[i];
    r.base[0] = scalar_load(o, 0);
    r.base[1] = scalar_load(o, 1);
    r.kinds[0] = scalar_load(o, 2);
    r.kinds[1] = scalar_load(o, 3);
#pragma unroll
    for (int q = 0; q < kGrpOps; ++q) r.off[q] = scalar_load(o, 4 + q);
    load_head();
  };
  auto windows = [&](const Rec &r) {
    const int64_t base = (int64_t)((uint64_t)r.base[1] << 32 | r.base[0]);
    return Windows<BITS, EDGE>(a, (t0 + (r.h[1] >> 16)) * BITS / 8 + base);  // (t0, chunks: even)
  };
  // Run a step's records, loading the windows of the next record as those of the
  // record in hand are used, and the record after that one meanwhile.
  auto build_step = [&]() {
    for (bool last = false; !last;) {
      Rec after;
      load_rec(after);
      const Windows<BITS, EDGE> ahead = windows(next);
      const uint32_t flags = cur.h[1];
      last = (flags & kRecLast) != 0;
      // lane 63 and lanes past the row write to a spare place that does not move
      const bool lane_ok = lane < (int)((flags >> 8) & 255);
      uint32_t dst = lane_ok ? lds0 + cur.h[2] + 16 * lane : trash;
      const uint32_t step = lane_ok ? cur.h[3] : 0;
      if (flags & kRecStart) {
#pragma unroll
        for (int j = 0; j < 4; ++j) P[j] = S[j] = 0;
      }
#define DD_OP(Q)                                                         \
  run_op<BITS, (Q) % 4>(P, S, win[Q], cur.kinds[(Q) / 4], dst, step); \
  ahead.load(win[Q], next.off[Q], lane);
      DD_OP(0) DD_OP(1) DD_OP(2) DD_OP(3) DD_OP(4) DD_OP(5) DD_OP(6) DD_OP(7)
#undef DD_OP
      cur = next;
      next = after;
    }
  };

  // ---- adding up: this wave's rows of the current step
  const uint32_t *ep = a.tab + scalar_load(&th->sum_off, 0) + scalar_load(&gb->sum_first, 0) + wave * kSumWords + lane;
  uint32_t acc[R][NW], lo[PACKED ? R : 1][PACKED ? NW : 1], hi[PACKED ? R : 1][PACKED ? NW : 1];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      acc[r][j] = 0;
      if constexpr (PACKED) lo[r][j] = hi[r][j] = 0;
    }
  const uint32_t base = lds0 + 4u * lane;
  auto sum_step = [&](uint32_t ev) {  // ev: the step's entries, one per lane
#pragma unroll
    for (int p = 0; p < kGrpStepPairs; ++p) {
      const uint32_t marks = (uint32_t)__builtin_amdgcn_readlane((int)ev, p * 2 * R);
#pragma unroll
      for (int r0 = 0; r0 < R; r0 += 2) {  // two rows' windows at a time
        uint32_t w[2][2][NW];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)ev, (p * 2 + h) * R + r0 + r);
            const lds_word *q = (const lds_word *)(uintptr_t)(base + (h == 0 && r0 + r == 0 ? e & kSumOffset : e));
#pragma unroll
            for (int j = 0; j < NW; ++j) w[h][r][j] = q[64 * j];
          }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int j = 0; j < NW; ++j) acc[r0 + r][j] += w[0][r][j] + w[1][r][j];
        if (r0 + 2 < R) __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PACKED) {
        if (marks & kSumFlush) {
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int j = 0; j < NW; ++j) {
              lo[r][j] += acc[r][j] & 0xFFFFu;
              hi[r][j] += acc[r][j] >> 16;
              acc[r][j] = 0;
            }
        }
      }
      if (marks & kSumLast) break;
    }
  };

  // ---- one step's partial sums ahead
  if (threadIdx.x < kGrpWin / 4) *(__attribute__((address_space(3))) v4u *)(uintptr_t)(lds0 + 2 * kGrpSetBytes + 16 * threadIdx.x) = v4u{0, 0, 0, 0};
  load_head();
  load_rec(cur);
  load_rec(next);
  {
    const Windows<BITS, EDGE> w = windows(cur);
#pragma unroll
    for (int q = 0; q < kGrpOps; ++q) w.load(win[q], cur.off[q], lane);
  }
  const int n_steps = (int)scalar_load(&gb->n_steps, 0);
  // Between two barriers the first kind of wave adds up step i and then builds step
  // i + 1, the other builds first (the streams end with a step of idle records).
  const bool sum_first = (wave >> 2) & 1;
#pragma unroll 1
  for (int i = 0; i <= n_steps; ++i) {
    const int s = sum_first ? i : i - 1;
    const uint32_t ev = ep[(int64_t)max(min(s, n_steps - 1), 0) * (kGrpWaves * kSumWords)];
    build_step();
    if (sum_first) lds_barrier();
    if (s >= 0 && s < n_steps) sum_step(ev);
    if (!sum_first) lds_barrier();
  }

  // Word j of lane i is sample t0 + i + 64j (packed: and kGrpWin later).
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int d = blk * group_rows(BITS) + wave * R + r;
    if (d >= a.n_dm) break;
    float *o = a.out + (int64_t)d * a.out_pitch;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const int64_t t = t0 + lane + 64 * j;
      if constexpr (PACKED) {
        if (t < a.n_out) o[t] = (float)lo[r][j];
        if (t + kGrpWin < a.n_out) o[t + kGrpWin] = (float)hi[r][j];
      } else {
        if (t < a.n_out) store_total(o + t, acc[r][j], a.out_mode);
      }
    }
  }
}

template <int BITS>
__device__ __forceinline__ void run_tile(uint8_t *lds, const GroupArgs &a, int blk, int tblk) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t0 = (int64_t)tblk * tile_samples<BITS>();
  const GroupHead *head = (const GroupHead *)a.tab;
  const GroupBlock *gb = (const GroupBlock *)(a.tab + kGrpHeadWords) + blk;
  const int64_t end = (t0 + scalar_load(&head->hi, 0) + (BITS == 16 ? 0 : kGrpWin)) * BITS / 8 + 8;
  if (t0 + scalar_load(&head->lo, 0) < 0 || end > a.row_bytes)
    group_tile<BITS, true>(lds, a, gb, blk, t0, wave, lane);
  else
    group_tile<BITS, false>(lds, a, gb, blk, t0, wave, lane);
}

template <int BITS>
__global__ __launch_bounds__(kGrpThreads) void fwd_group_kernel(GroupArgs a, int n_blk, int n_tiles, int order) {
  extern __shared__ __align__(16) uint8_t lds[];
  int blk, tblk;
  tile_of(blockIdx.x, n_blk, n_tiles, order, blk, tblk);
  run_tile<BITS>(lds, a, blk, tblk);
}

// One counter per XCD (the counter slot of a group has 256 bytes).
__global__ void reset_group_counter_kernel(unsigned long long *counter) {
  for (int x = 0; x < kXcds; ++x) counter[x] = 0ull;
}

// Readable bytes of an input row: its samples rounded up to 16 bytes, inside the pitch.
__host__ __device__ inline int64_t readable_row_bytes(int64_t n_samp, int bits) {
  return (n_samp * bits / 8 + 15) / 16 * 16;
}

// Persistent batched form, the counterpart of those in fwd_int.hip and
// fwd_direct.hip.  A beam's table is its plan's group-sum table (BeamDesc.offs).
// Work items are (beam, time tile, DM block), beams in decreasing cost order, DM
// block fastest; list x holds the time tiles x, x + 8, ... of every beam, and a
// workgroup claims from its own XCD's list (workgroup w runs on XCD w % 8), so that
// the DM blocks of a tile share its input in one L2, then from the other lists in
// turn (64 beams of 256-1024 ch: 6.6 against 10.5 ms for one list in DM-block order).  The
// claim of the next item is issued when an item starts and read when it
// ends; a tile ends with a barrier after its last LDS read.  A workgroup returns
// when all lists are exhausted: every wave reaches the exit.
template <int BITS>
__global__ __launch_bounds__(kGrpThreads) void fwd_group_batched_kernel(const BeamDesc *__restrict__ beams, int n_beams,
                                                                        long long n_items,
                                                                        unsigned long long *__restrict__ counter) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ int claimed;
  int list = (int)(blockIdx.x % kXcds), tries = 0;
  int lo = 0, begin = 0;  // the beam of the last claim, and its first item in the list
  if (threadIdx.x == 0) claimed = (int)atomicAdd(counter + list, 1ull);
  for (;;) {
    lds_barrier();  // publishes the claim
    const int item = __builtin_amdgcn_readfirstlane(claimed);
    lds_barrier();  // every wave has read it before thread 0 writes the next one
    int n = 0;
    while (lo < n_beams) {
      n = (scalar_load(&beams[lo].tiles_t, 0) - list + kXcds - 1) / kXcds * scalar_load(&beams[lo].tiles_d, 0);
      if (item < begin + n) break;
      begin += n;
      ++lo;
    }
    if (lo == n_beams) {  // the list is exhausted: go on with the next one
      if (++tries == kXcds) return;
      list = (list + 1) % kXcds;
      lo = begin = 0;
      if (threadIdx.x == 0) claimed = (int)atomicAdd(counter + list, 1ull);
      continue;
    }
    int next = 0;
    if (threadIdx.x == 0) next = (int)atomicAdd(counter + list, 1ull);  // the following claim, read after this tile
    const BeamDesc *b = beams + __builtin_amdgcn_readfirstlane(lo);
    const int k = item - begin, tiles_d = scalar_load(&b->tiles_d, 0);
    const int kt = __builtin_amdgcn_readfirstlane(k / tiles_d);
    const int tblk = list + kXcds * kt, blk = k - kt * tiles_d;
    GroupArgs a;
    a.x = scalar_load(&b->x, 0);
    a.tab = scalar_load(&b->offs, 0);
    a.out = scalar_load(&b->out, 0);
    a.n_out = scalar_load(&b->n_out, 0);
    a.out_pitch = scalar_load(&b->out_pitch, 0);
    a.n_dm = scalar_load(&b->n_dm, 0);
    a.row_bytes = readable_row_bytes(scalar_load(&b->n_samp, 0), BITS);
    a.total = (scalar_load(&b->n_chan, 0) - 1) * scalar_load(&b->pitch, 0) + a.row_bytes;
    a.out_mode = kOutFloat;
    run_tile<BITS>(lds, a, __builtin_amdgcn_readfirstlane(blk), __builtin_amdgcn_readfirstlane(tblk));
    if (threadIdx.x == 0) claimed = next;
  }
}

template <int BITS>
int launch_group_bits(const GroupArgs &a, int n_blk, int lds_bytes, int order, hipStream_t st) {
  const int64_t tiles = (a.n_out + tile_samples<BITS>() - 1) / tile_samples<BITS>();
  if (tiles * n_blk >= ((int64_t)1 << 31)) return (int)hipErrorInvalidConfiguration;
  const void *fn = (const void *)fwd_group_kernel<BITS>;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL((fwd_group_kernel<BITS>), dim3((unsigned)(tiles * n_blk)), dim3(kGrpThreads), lds_bytes, st, a,
                     n_blk, (int)tiles, order);
  return (int)hipGetLastError();
}

}  // namespace

int launch_forward_group(const dd_plan &p, const void *tables, const void *d_in, float *d_out, int64_t out_pitch,
                         void *stream, int64_t out_limit, int out_mode) {
  const GroupTables &t = p.gtab;
  const int bits = p.desc.dtype == DD_U4 ? 4 : p.desc.dtype == DD_U16 ? 16 : 8;
  GroupArgs a;
  a.x = (const uint8_t *)d_in;
  a.tab = (const uint32_t *)tables;
  a.out = d_out;
  a.n_out = out_limit > 0 && out_limit < p.n_out ? out_limit : p.n_out;
  a.out_pitch = out_pitch;
  a.n_dm = p.desc.n_dm;
  a.row_bytes = ((p.desc.n_samp * bits / 8 + 15) / 16 * 16);  // inside the pitch, a multiple of 16
  a.total = (p.desc.n_chan - 1) * p.in_pitch_bytes + a.row_bytes;
  a.out_mode = out_mode;
  const hipStream_t st = (hipStream_t)stream;
  if (bits == 4) return launch_group_bits<4>(a, t.n_blk, kGrpLdsBytes, p.fwd.order, st);
  if (bits == 16) return launch_group_bits<16>(a, t.n_blk, kGrpLdsBytes, p.fwd.order, st);
  return launch_group_bits<8>(a, t.n_blk, kGrpLdsBytes, p.fwd.order, st);
}

int group_tile_samples(int dtype) { return dtype == DD_U16 ? tile_samples<16>() : tile_samples<8>(); }

int batch_group_kernels(int dtype, BatchLaunch *out) {
  const void *fn = dtype == DD_U4    ? (const void *)fwd_group_batched_kernel<4>
                   : dtype == DD_U16 ? (const void *)fwd_group_batched_kernel<16>
                                     : (const void *)fwd_group_batched_kernel<8>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kGrpLdsBytes);
  int dev = 0, n_cu = 0;
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return (int)e;
  out->reset_fn = (const void *)reset_group_counter_kernel;
  out->main_fn = fn;
  out->grid = n_cu;  // one workgroup takes a CU's LDS
  out->block = kGrpThreads;
  out->lds_bytes = kGrpLdsBytes;
  return 0;
}

}  // namespace dd
