// Float forward and adjoint by shared sums of four rows (tables and the order of the
// sums: quad_tables.h; the same sums row by row: kernels_f32.hip).
//
// A workgroup owns 16 * R outputs x one tile of kQuadWin samples.  The LDS holds the
// quad sums of two steps (a few quads each): between two barriers every wave builds its
// part of the next step's sums and adds up its outputs of the current step's, half of the
// waves of each SIMD starting with the one, half with the other.  A building wave streams
// records of 4 operations, loading the rows straight from memory a record ahead.  Lane i
// owns words i, i + 64, ... in both: loads, stores and LDS reads of a wave are contiguous
// and free of bank conflicts.
//
// The floor is LDS: one word read per four rows, output and sample, where the kernels that
// stage rows read one per row (they run at 80% of it).  Bound by instruction issue and the
// barriers: on 1024 ch x 2^17 x 1024 DMs (6.2 patterns of 770 words per quad on average, 3.6
// quads a step, whose busiest wave has 1.4 times the mean of records) LDS is 47% busy,
// vector units 45% (adjoint: both 43%).  Forward and adjoint of that plan: 17.0 ms by
// staged rows, 8.8 by quad sums; 1024 ch x 131900 x 512 DMs of step 0.1: 9.6 and 3.3.  On the
// way there: windows loaded when a pattern needs them, one pattern after another: 10.9; a
// stream loaded ahead with a bounded descriptor per operation: 13.4, without where the
// block's windows lie inside their rows: 10.8; rows taken over by one asm branch instead of
// the compiler's copies: 9.5; 256 words of a pattern per record instead of 192: 9.0.  8 waves
// of 128 outputs' registers each (384 or 576 words per record): 12.8 and 13.4; 32 outputs:
// 11.2.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dd_internal.h"
#include "quad_tables.h"
#include "tile_order.h"

namespace dd {
namespace {

struct QuadArgs {
  const float *x;       // rows
  const uint32_t *tab;  // QuadTables::data
  float *out;
  int64_t row_pitch, out_pitch;
  int32_t n_rows, row_len, n_outputs, out_len;
  int32_t n_blk, n_quads;
  uint32_t pitch_bytes;  // of the rows (three of them within 32 bits, or every tile is an edge)
  uint32_t op_off, sum_off;
};

template <typename T>
__device__ __forceinline__ T scalar_load(const T *p, int64_t i) {
  return ((const __attribute__((address_space(4))) T *)p)[i];
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef __attribute__((address_space(3))) float lds_float;

struct QuadRec {
  uint32_t head[kQuadRecWords], op[kQuadOpWords];
};

// Words 2p and 2p + 1 of a window.
typedef float v2f __attribute__((ext_vector_type(2)));

// x[c] = w, c in bits 4Q and 4Q + 1 of kinds.  (In asm: left to itself the compiler copies
// every row in every branch.)
template <int Q, int NP>
__device__ __forceinline__ void take_row(v2f (&x)[4][NP], const v2f (&w)[NP], uint32_t kinds) {
#define DD_BRANCHES(M0, M1, M2, M3)                                                             \
  "s_bitcmp1_b32 %[k], %[b0]\n\ts_cbranch_scc1 .Lo%=\n\ts_bitcmp1_b32 %[k], %[b1]\n\t"           \
  "s_cbranch_scc1 .L2%=\n\t" M0 "s_branch .Le%=\n.L2%=:\n\t" M2 "s_branch .Le%=\n.Lo%=:\n\t"      \
  "s_bitcmp1_b32 %[k], %[b1]\n\ts_cbranch_scc1 .L3%=\n\t" M1 "s_branch .Le%=\n.L3%=:\n\t" M3 ".Le%=:"
  static_assert(NP == 2 || NP == 3, "pairs of words");
  if constexpr (NP == 3) {
    asm(DD_BRANCHES("v_mov_b64 %0, %12\n\tv_mov_b64 %1, %13\n\tv_mov_b64 %2, %14\n\t",
                    "v_mov_b64 %3, %12\n\tv_mov_b64 %4, %13\n\tv_mov_b64 %5, %14\n\t",
                    "v_mov_b64 %6, %12\n\tv_mov_b64 %7, %13\n\tv_mov_b64 %8, %14\n\t",
                    "v_mov_b64 %9, %12\n\tv_mov_b64 %10, %13\n\tv_mov_b64 %11, %14\n\t")
        : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[0][2]), "+v"(x[1][0]), "+v"(x[1][1]), "+v"(x[1][2]), "+v"(x[2][0]),
          "+v"(x[2][1]), "+v"(x[2][2]), "+v"(x[3][0]), "+v"(x[3][1]), "+v"(x[3][2])
        : "v"(w[0]), "v"(w[1]), "v"(w[2]), [k] "s"(kinds), [b0] "i"(4 * Q), [b1] "i"(4 * Q + 1)
        : "scc");
  } else {
    asm(DD_BRANCHES("v_mov_b64 %0, %8\n\tv_mov_b64 %1, %9\n\t", "v_mov_b64 %2, %8\n\tv_mov_b64 %3, %9\n\t",
                    "v_mov_b64 %4, %8\n\tv_mov_b64 %5, %9\n\t", "v_mov_b64 %6, %8\n\tv_mov_b64 %7, %9\n\t")
        : "+v"(x[0][0]), "+v"(x[0][1]), "+v"(x[1][0]), "+v"(x[1][1]), "+v"(x[2][0]), "+v"(x[2][1]), "+v"(x[3][0]),
          "+v"(x[3][1])
        : "v"(w[0]), "v"(w[1]), [k] "s"(kinds), [b0] "i"(4 * Q), [b1] "i"(4 * Q + 1)
        : "scc");
  }
#undef DD_BRANCHES
}

// EDGE: some of the block's windows may reach outside their rows.
template <int R, bool EDGE>
__device__ __forceinline__ void quad_tile(uint8_t *lds, const QuadArgs &a, const QuadBlock *qb, int blk, int t0, int wave,
                                          int lane) {
  constexpr int NW = kQuadWin / 64;
  constexpr int W = quad_lane_words(kQuadWaves * R);
  lds_float *const base = (lds_float *)(__attribute__((address_space(3))) void *)lds + lane;
  uint32_t lane_byte[EDGE ? W : 1];
#pragma unroll
  for (int j = 0; j < (EDGE ? W : 1); ++j) {
    lane_byte[j] = 4u * (uint32_t)(lane + 64 * j);
    asm("" : "+v"(lane_byte[j]));
  }
  const int n_steps = (int)scalar_load(&qb->n_steps, 0);
  const uint32_t *const steps = a.tab + scalar_load(&qb->step_first, 0);

  // ---- building: this wave's record stream
  const uint32_t *rp = a.tab + (uint64_t)scalar_load(&qb->rec_first[wave], 0) * kQuadRecWords;
  const uint32_t *const ops = a.tab + a.op_off;
  QuadRec cur, next;             // the record in hand, its windows loaded or on the way, and the one after it
  uint32_t head[kQuadRecWords];  // the head of the record after those
  v2f x[4][W / 2], win[kQuadOps][W / 2];
  auto load_head = [&]() {
#pragma unroll
    for (int i = 0; i < kQuadRecWords; ++i) head[i] = scalar_load(rp, i);
    rp += kQuadRecWords;
  };
  // Record `head` into r, and the next head (the table holds records past the last stream).
  auto load_rec = [&](QuadRec &r) {
    const uint32_t *o = ops + (uint64_t)(head[0] & ~kQuadLast) * kQuadOpWords;
#pragma unroll
    for (int i = 0; i < kQuadRecWords; ++i) r.head[i] = head[i];
#pragma unroll
    for (int i = 0; i < kQuadOpWords; ++i) r.op[i] = scalar_load(o, i);
    load_head();
  };
  // The words start + lane + 64j of operation Q's row.  EDGE: zeros outside the row: a
  // negative start wraps past the row's end.  (Whole offsets in registers: an instruction's
  // own offset would be added to a wrapped one.)
  auto record_base = [&](const QuadRec &r) -> uint64_t {  // the quad's first row at the least of the starts
    if constexpr (EDGE) return 0;
    const int64_t s = (int64_t)t0 + (int32_t)r.op[2] + 64 * W * (int)(r.head[1] & 0xFFFFu);
    uint64_t p = (uint64_t)(a.x + (int64_t)(r.op[0] >> 15) * 4 * a.row_pitch + s);
    asm("" : "+s"(p));  // a descriptor in scalar registers
    return p;
  };
  auto load_window = [&](const QuadRec &r, uint64_t rec_base, auto qc) {
    constexpr int Q = decltype(qc)::value;
    const uint32_t kind = r.op[1] >> (4 * Q), rel = r.op[3 + Q / 2] >> (16 * (Q & 1)) & 0xFFFFu;
    const bool none = (kind & kQuadNone) != 0;
    if constexpr (EDGE) {
      const int row = none ? 0 : 4 * (int)(r.op[0] >> 15) + (int)(kind & 3u);
      uint64_t p = (uint64_t)(a.x + (int64_t)row * a.row_pitch);
      asm("" : "+s"(p));
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, none ? 0 : 4 * a.row_len, 0x00020000);
      const uint32_t s = 4u * ((uint32_t)t0 + r.op[2] + rel + 64 * W * (r.head[1] & 0xFFFFu));
#pragma unroll
      for (int j = 0; j < W; ++j) {
        uint32_t v = s + lane_byte[j];
        asm("" : "+v"(v));
        win[Q][j / 2][j % 2] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)v, 0, 0));
      }
    } else {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)rec_base, 0, none ? 0 : -1, 0x00020000);
      const uint32_t off = (kind & 3u) * a.pitch_bytes + 4u * rel;
#pragma unroll
      for (int j = 0; j < W; ++j)
        win[Q][j / 2][j % 2] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(lane_byte[0] + 256u * j), (int)off, 0));
    }
    __builtin_amdgcn_sched_barrier(0);  // loads stay in the order of their use
  };
  auto run_op = [&](const QuadRec &r, auto qc, lds_float *&dst, int words) {
    constexpr int Q = decltype(qc)::value;
    const uint32_t kind = r.op[1] >> (4 * Q);
    take_row<Q, W / 2>(x, win[Q], r.op[1]);
    if (kind & kQuadWrite) {
      float v[W];
#pragma unroll
      for (int j = 0; j < W; ++j)
        v[j] = ((x[0][j / 2][j % 2] + x[1][j / 2][j % 2]) + x[2][j / 2][j % 2]) + x[3][j / 2][j % 2];
      if (words >= 64 * W) {
#pragma unroll
        for (int j = 0; j < W; ++j) dst[64 * j] = v[j];
      } else {
#pragma unroll
        for (int j = 0; j < W - 1; ++j)
          if (j == 0 || words > 64 * j) dst[64 * j] = v[j];
        asm volatile("; part of a chunk");  // (keeps the branches apart)
      }
      dst += r.op[0] & 0x7FFFu;
    }
  };
  // Run a step's records, loading the windows of the next record as those of the record in
  // hand are used.
  auto build_step = [&]() {
    for (bool last = false; !last;) {
      QuadRec after;
      load_rec(after);
      last = (cur.head[0] & kQuadLast) != 0;
      lds_float *dst = base + (cur.head[1] >> 16);
      const uint64_t rec_base = record_base(next);
      const int words = (int)(cur.op[0] & 0x7FFFu) - 64 * W * (int)(cur.head[1] & 0xFFFFu);
#define DD_OP(Q)                                                  \
  run_op(cur, std::integral_constant<int, Q>(), dst, words); \
  load_window(next, rec_base, std::integral_constant<int, Q>());
      DD_OP(0) DD_OP(1) DD_OP(2) DD_OP(3)
#undef DD_OP
      cur = next;
      next = after;
    }
  };

  float tot[R][NW], part[R][NW];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < NW; ++j) tot[r][j] = part[r][j] = 0.0f;
  const uint32_t *const sums = a.tab + a.sum_off + ((int64_t)blk * kQuadWaves + wave) * a.n_quads * (R / 2) + lane;
  const int last_quad = (a.n_rows + 3) / 4 - 1;
  auto sum_step = [&](int q0, int n, uint32_t ev) {  // ev: the windows' places, a word per lane
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
#pragma unroll
      for (int r0 = 0; r0 < R; r0 += 2) {  // two outputs' windows at a time
        const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)ev, i * (R / 2) + r0 / 2);
        float w[2][NW];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const lds_float *q = (const lds_float *)base + (r ? e >> 16 : e & 0xFFFFu);
#pragma unroll
          for (int j = 0; j < NW; ++j) w[r][j] = q[64 * j];
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int j = 0; j < NW; ++j) part[r0 + r][j] += w[r][j];
      }
      if ((q0 + i) % 8 == 7 || q0 + i == last_quad) {  // the end of 32 rows
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NW; ++j) {
            tot[r][j] += part[r][j];
            part[r][j] = 0.0f;
          }
      }
    }
  };

  // Between two barriers the first kind of wave adds up step i and then builds step i + 1,
  // the other builds first (waves w, w + 4, ... share a SIMD; the streams end with a
  // record for a step that is none).
  const bool sum_first = (wave >> 2) & 1;
#pragma unroll
  for (int j = 0; j < W / 2; ++j) x[0][j] = x[1][j] = x[2][j] = x[3][j] = 0.0f;
  load_head();
  load_rec(cur);
  load_rec(next);
  const uint64_t first_base = record_base(cur);
  load_window(cur, first_base, std::integral_constant<int, 0>());
  load_window(cur, first_base, std::integral_constant<int, 1>());
  load_window(cur, first_base, std::integral_constant<int, 2>());
  load_window(cur, first_base, std::integral_constant<int, 3>());
#pragma unroll 1
  for (int i = 0; i <= n_steps; ++i) {
    const int s = sum_first ? i : i - 1;
    const int sq = max(min(s, n_steps - 1), 0) * kQuadStepWords;
    const int q0 = (int)scalar_load(steps, sq), n = s < 0 || s >= n_steps ? 0 : (int)scalar_load(steps, sq + 1);
    const uint32_t ev = sums[q0 * (R / 2)];
    build_step();
    if (sum_first) lds_barrier();
    sum_step(q0, n, ev);
    if (!sum_first) lds_barrier();
  }

#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int o = (blk * kQuadWaves + wave) * R + r;
    if (o >= a.n_outputs) break;
    float *orow = a.out + (int64_t)o * a.out_pitch;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const int64_t t = (int64_t)t0 + lane + 64 * j;
      if (t < a.out_len) orow[t] = tot[r][j];
    }
  }
}

template <int R>
__global__ __launch_bounds__(64 * kQuadWaves) void quad_kernel(QuadArgs a, int n_tiles, int order) {
  extern __shared__ __align__(16) uint8_t lds[];
  int blk, tile;
  tile_of(blockIdx.x, a.n_blk, n_tiles, order, blk, tile);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t0 = tile * kQuadWin;
  const QuadBlock *qb = (const QuadBlock *)a.tab + blk;
  if (a.pitch_bytes == 0 || (int64_t)t0 + scalar_load(&qb->lo, 0) < 0 || (int64_t)t0 + scalar_load(&qb->hi, 0) > a.row_len)
    quad_tile<R, true>(lds, a, qb, blk, t0, wave, lane);
  else
    quad_tile<R, false>(lds, a, qb, blk, t0, wave, lane);
}

}  // namespace

int launch_quad(const QuadTables &q, const void *tables, const float *x, int64_t row_pitch, int n_rows, int64_t row_len,
                float *out, int64_t out_pitch, int n_outputs, int64_t out_len, void *stream) {
  QuadArgs a;
  a.x = x;
  a.tab = (const uint32_t *)tables;
  a.out = out;
  a.row_pitch = row_pitch;
  a.out_pitch = out_pitch;
  a.n_rows = n_rows;
  a.row_len = (int32_t)row_len;
  a.n_outputs = n_outputs;
  a.out_len = (int32_t)out_len;
  a.n_blk = q.n_blk;
  a.n_quads = q.n_quads;
  a.op_off = q.op_off;
  a.sum_off = q.sum_off;
  a.pitch_bytes = row_pitch < (1 << 28) ? 4 * (uint32_t)row_pitch : 0;
  const int64_t tiles = (out_len + kQuadWin - 1) / kQuadWin;
  if (tiles * q.n_blk >= ((int64_t)1 << 31)) return (int)hipErrorInvalidConfiguration;
  const int lds = 2 * kQuadSetBytes;
  const void *fn = q.rows == 64 ? (const void *)quad_kernel<64 / kQuadWaves> : (const void *)quad_kernel<32 / kQuadWaves>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return (int)e;
  const dim3 grid((unsigned)(tiles * q.n_blk)), block(64 * kQuadWaves);
  if (q.rows == 64)
    hipLaunchKernelGGL(quad_kernel<64 / kQuadWaves>, grid, block, lds, (hipStream_t)stream, a, (int)tiles, q.order);
  else
    hipLaunchKernelGGL(quad_kernel<32 / kQuadWaves>, grid, block, lds, (hipStream_t)stream, a, (int)tiles, q.order);
  return (int)hipGetLastError();
}

}  // namespace dd
