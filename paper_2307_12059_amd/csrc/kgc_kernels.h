// Kernels of the TransE completion join for gfx950 (CDNA4, wave64).
//
//   stage_operands   kernel 1: norms of the connector outputs (Section 4.3: a = h + r, b = t) with the zero
//                    vector as pivot (Section 4.5), and the bf16 operands of the contraction
//   join_l2          kernel 2: ||a - b||^2 for a tile of heads x tails by bf16 MFMA, filter, exact re-score
//   join_l1          kernel 3: sum |a - b| for a tile by float32 vector arithmetic, filter, exact re-score
// Both join kernels end in recheck_and_emit / wave_append (kgc_device.h).
#pragma once
#include "kgc_device.h"

namespace kgc {

// Number of extra contraction columns that carry the norms (three bf16 pieces of each float32 norm).
constexpr int kNormCols = 6;
// Operands are stored K-slice-major: X[ks][slot][32] bf16, so one tile's slice is contiguous.
constexpr int kSliceK = 32;
// Row stride (elements) of a slice in LDS: 32 + 8 padding = 80 bytes, which spreads eight consecutive
// rows' 16-byte fragments over all banks.
constexpr int kLdsRow = 40;
// Swizzle of the streaming kernel's LDS slices: rows are 64 bytes (four 16-byte chunks) without padding, and
// chunk c of row r is stored at position c ^ lds_swizzle(r).  With r = ...b3 b2 b1 b0 the swizzle is
// (b2 << 1) | (b1 ^ b3): eight or sixteen consecutive rows reading the same logical chunk, and four
// consecutive rows writing all their chunks, then fall on distinct banks whether the LDS serves 128 or
// 256 bytes per cycle.
__device__ __forceinline__ int lds_swizzle(int row) { return (((row >> 2) & 1) << 1) | (((row >> 1) ^ (row >> 3)) & 1); }
// Running maxima are kept in this many slots so that the atomics of kernel 1 do not pile on one address.
constexpr int kMaxSlots = 1024;

// device-side scalars of one join
struct JoinParams {
  float thr;            // filter threshold: on the squared distance (L2) or on the float32 sum (L1)
  float base;           // L1: what the rounding of coordinates h + r can add to a sum (L2: 0, unused)
  float pad[2];
};

struct DevCounters {
  unsigned long long hits;        // true number of qualifying triples
  unsigned long long candidates;  // triples re-scored in double
  unsigned long long tile_cursor; // next free entry of the surviving-tile list (per relation batch)
  unsigned int n_active;          // rows (relation, head tile) of the batch that still have tail tiles
  unsigned int exact_need;        // most accumulator blocks any one batch wanted to list (see list_block)
  unsigned long long tiles;       // surviving tiles over all batches
  unsigned long long exact_total; // accumulator blocks scored by the block form of the exact stage (L1: blocks summed by k_l1_blocks), over all batches
  unsigned int fact_need, pad;    // most pairs any one batch of the relation-factorised kernel wanted to list
  unsigned int max_a[1024];       // running maxima of ||bf16(h + r)||^2 (L2) or ||e||_1 (L1), float bits, spread over slots
  unsigned int max_b[1024];       // running maxima of ||bf16(t)||^2 (L2) or ||r||_1 (L1)
  unsigned int sample[256];       // triples within delta by workgroup of k_sample_close
  unsigned int n_exact;           // accumulator blocks listed for the exact stage by the pruned L2 join kernels (per batch)
  unsigned int pair_mode;         // pruned L2 batch: 1 = its rows keep so few tiles that they are taken tile by tile
  unsigned long long n_fact;      // pairs listed by the relation-factorised kernel (per batch)
  unsigned long long l1_sample;   // sampled tiles << 32 | their blocks (k_l1_micro_pairs, per batch)
};

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// relation numbers of a batch's records become numbers of the whole join (kgc_join_se)
__global__ void k_shift_relation(kgc_triple* rec, uint64_t n, int32_t r0) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) rec[i].r += r0;
}

// dense join over a window of head tiles: the (relation, 256-row tile) rows that the operand staging has to fill
__global__ void k_window_rows(uint32_t* rows, unsigned int* n_rows, int RB, int n_tiles, int w0, int w1) {
  const int per_rel = w1 - w0;
  const int64_t total = (int64_t)RB * per_rel;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    rows[i] = (uint32_t)((i / per_rel) * n_tiles + w0 + i % per_rel);
  if (blockIdx.x == 0 && threadIdx.x == 0) *n_rows = (unsigned int)total;
}

// Around the tile lists of a pruned batch: the running total of surviving tiles, and which L2 join kernel takes the
// batch (when the host allows the choice): tile by tile when its rows keep few tiles.
//   phase 0, after k_rows_from_bitmap: at most kPairModeTilesPerRow tiles per active row on average.
//   phase 1, after a bound test that listed the new tiles itself (BoundL2Args::list_*) and before k_rows_from_bitmap:
//            the flat list is the batch's list when it is short against the number of rows (and fits); the rows then
//            count once per tile.  Otherwise the cursors start over and k_rows_from_bitmap builds the lists per row.
constexpr unsigned long long kPairModeTilesPerRow = 3;
__global__ void k_batch_tiles(DevCounters* c, int allow_pairs, int phase, unsigned long long n_rows, unsigned long long list_cap) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    if (phase == 0) {
      c->tiles += c->tile_cursor;
      c->pair_mode = (allow_pairs && c->tile_cursor <= kPairModeTilesPerRow * c->n_active && c->tile_cursor < 0xffffffffull) ? 1u : 0u;
    } else {
      const unsigned long long n = c->tile_cursor;
      const unsigned long long few = n_rows / 8 > 4096 ? n_rows / 8 : 4096;
      if (allow_pairs && n <= few && n <= list_cap && n < 0xffffffffull) {
        c->tiles += n; c->n_active = (unsigned int)n; c->pair_mode = 1u;
      } else {
        c->tile_cursor = 0; c->n_active = 0; c->pair_mode = 0u;
      }
    }
  }
}

// slot -> entity for the dense order: identity, -1 on the padding rows
__global__ void k_identity_slots(int32_t* slot_ent, int64_t N, int64_t Nslots) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < Nslots) slot_ent[i] = i < N ? (int32_t)i : -1;
}

// ---------------------------------------------------------------------------------------------
// Kernel 1.  One block stages kStageRows consecutive slots of one relation (IS_A: the row is
// a = h + r; otherwise the row is b = t and there is a single "relation").  The rows are rounded to bf16
// into an LDS tile, their squared norms ||.||^2 are summed in float32 from the rounded values, and the staged rows
//     A:  [ a~ (d) | nA_hi nA_mid nA_lo | 1 1 1 | 0 ... ]
//     B:  [ -2 b~ (d) | 1 1 1 | nB_hi nB_mid nB_lo | 0 ... ]
// are written slice by slice, 16 bytes per thread, so that the dot product of an A row and a B row is
// nA + nB - 2 a~.b~ = ||a~ - b~||^2.  The three pieces are the float32 norm cut into 8-bit mantissa
// chunks, exact in bf16.  Padding rows get a norm of 1e30 so they never pass the filter.  The squared
// norms are also written out plainly; with the zero pivot they are distA^2 and distB^2 of Section 4.5.
//
// Filter slack (slack_delta >= 0, the joins).  Rounding to bf16 moves a row x by e = ||x - x~||, which this
// kernel MEASURES per row (it holds x and x~) instead of bounding it by 2^-8 ||x||.  By the triangle
// inequality (the argument of Lemma 1, Section 4.4) a true hit ||a - b|| <= delta has
//     ||a~ - b~||^2 <= (delta + e_a + e_b)^2 <= delta^2 + (2 delta e_a + 2 e_a^2) + (2 delta e_b + 2 e_b^2),
// so each row's own term 2 delta e + 2 e^2 is taken off its norm column and the join compares against
// delta^2 (plus the float32 accumulation bound): rows that round well pay nothing for those that do not.
// e is widened by 0.1 % and by 2^-23 ||x|| (the float32 addition h + r and its own summation).
//
// Work split: a block of four waves stages kStageRows = 64 consecutive slots, 16 per wave, and nothing is shared
// between the waves (no block barrier).  A wave reads two rows per load instruction, 32 lanes x 4 consecutive
// dimensions each (one 16-byte or 8-byte load per lane where base and row length allow), keeps the per-row sums of
// squares in registers (8 row pairs), writes the rounded values to its own LDS tile, reduces the sums across lanes
// with a halving exchange (9 shuffles for 16 rows), adds the norm columns, and copies the tile out slice by slice,
// 1 KiB per store instruction.
constexpr int kStageRows = 64;
constexpr int kStageWaveRows = 16;

// four consecutive elements of a row from column c on (n = d - c of them exist); vec: 16-byte (f32) / 8-byte (bf16) loads allowed
__device__ __forceinline__ void stage_ld4(const void* base, int64_t off, int n, int dtype, bool vec, float v[4]) {
  v[0] = v[1] = v[2] = v[3] = 0.f;
  if (n <= 0) return;
  if (vec && n >= 4) {
    if (dtype == KGC_BF16) {
      const uint2 t = *(const uint2*)((const uint16_t*)base + off);
      v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
      v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
    } else {
      const float4 t = *(const float4*)((const float*)base + off);
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (k < n) v[k] = ld_elem(base, off + k, dtype);
}

// sums of 8 per-lane values over the 32 lanes of each half wave: afterwards lane l holds the total of value
// ((l >> 4) & 1) * 4 + ((l >> 3) & 1) * 2 + ((l >> 2) & 1)
__device__ __forceinline__ float stage_reduce8(const float v[8], int lane) {
  float a[4], b[2], c;
  const bool b4 = lane & 16, b3 = lane & 8, b2 = lane & 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float send = b4 ? v[i] : v[i + 4], keep = b4 ? v[i + 4] : v[i];
    a[i] = keep + __shfl_xor(send, 16, 64);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float send = b3 ? a[i] : a[i + 2], keep = b3 ? a[i + 2] : a[i];
    b[i] = keep + __shfl_xor(send, 8, 64);
  }
  {
    const float send = b2 ? b[0] : b[1], keep = b2 ? b[1] : b[0];
    c = keep + __shfl_xor(send, 4, 64);
  }
  c += __shfl_xor(c, 2, 64);
  c += __shfl_xor(c, 1, 64);
  return c;
}

// DROP (the relation-factorised join): a row with an element that is no finite number is staged as a padding slot, and ent_out
// (may be NULL) gets the slots' entities without such rows.  No pair with one can be a hit, but its G and u are no numbers, and the
// factorised kernel lets those keep every set open that they are in (rows whose norms leave float32's range need that): one
// row cost 2 N R listed pairs (N = 15,000, R = 1,345, d = 100: 23.2 ms a call against 0.49).  The sum of the squared rounding errors tells:
// v - bf16(v) is a NaN for an infinite or NaN v, and never for a finite one (whose error may overflow to infinity).
template <bool IS_A, bool DROP = false>
__device__ __forceinline__ void stage_operands(const void* __restrict__ E, const void* __restrict__ Rv,
                                               int dtype, int d, int r0, int RB,
                                               const int32_t* __restrict__ slot_ent, int64_t Nslots, int KS,
                                               uint16_t* __restrict__ out, float* __restrict__ norms,
                                               unsigned int* __restrict__ max_slots,
                                               const uint32_t* __restrict__ active_rows,
                                               const unsigned int* __restrict__ n_active, int nH, int bm,
                                               int64_t rel_stride, const int32_t* __restrict__ n_rows_dev,
                                               float slack_delta, int64_t n_identity, int32_t* __restrict__ ent_out = nullptr) {
  extern __shared__ __attribute__((aligned(16))) uint16_t tile_all[];   // [4 waves][16 rows][KS * 32 + 8]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int W = KS * kSliceK + 8;
  uint16_t* tile = tile_all + wave * kStageWaveRows * W;
  const int esz = dtype == KGC_BF16 ? 2 : 4;
  // vector loads: every row of E (and of Rv) starts on a 4-element boundary of an aligned array
  const bool vec = (d % 4 == 0) && ((uintptr_t)E % (4 * esz) == 0) && (!(IS_A && Rv) || (uintptr_t)Rv % (4 * esz) == 0);
  const bool slack = slack_delta >= 0.f && slack_delta <= 3e38f;       // (an infinite threshold passes everything anyway)
  // dense joins stage every row group of every relation of the batch; pruned joins only the head tiles
  // (rows of the active list) that still have tail tiles to meet
  const int64_t groups_per_rel = Nslots / kStageRows;
  const int groups_per_tile = bm / kStageRows;
  const int64_t ngroups = active_rows ? (int64_t)*n_active * groups_per_tile : groups_per_rel * RB;
  float vmax = 0.f;
  for (int64_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
    int rl;
    int64_t slot0;
    if (active_rows) {
      const int64_t row = (int64_t)active_rows[g / groups_per_tile];
      rl = (int)(row / nH);
      slot0 = (row - (int64_t)rl * nH) * bm + (g % groups_per_tile) * kStageRows;
    } else {
      rl = (int)(g / groups_per_rel);
      slot0 = (g - (int64_t)rl * groups_per_rel) * kStageRows;
    }
    // n_rows_dev: only the first *n_rows_dev slots (rounded up to a 256-row tile) hold rows this time
    if (n_rows_dev && slot0 >= ((int64_t)*n_rows_dev + 255) / 256 * 256) continue;
    slot0 += wave * kStageWaveRows;
    const int ent_l = lane >= kStageWaveRows ? -1 : slot_ent ? slot_ent[slot0 + lane] : (slot0 + lane < n_identity ? (int)(slot0 + lane) : -1);
    const int64_t ro = (int64_t)(r0 + rl) * d;
    const int64_t eo = (int64_t)(r0 + rl) * rel_stride;       // per-relation source rows (0: one array for all)
    float sq[8], er[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sq[i] = er[i] = 0.f;
    for (int c0 = 0; c0 < KS * kSliceK; c0 += 128) {
      const int c = c0 + 4 * l32;
      float rv[4] = {0.f, 0.f, 0.f, 0.f};
      if (IS_A && Rv) stage_ld4(Rv, ro + c, d - c, dtype, vec, rv);     // Rv == nullptr: the plain row (a = h)
      float x[8][4];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int ent = __shfl(ent_l, 2 * i + half, 64);
        stage_ld4(E, eo + (int64_t)(ent < 0 ? 0 : ent) * d + c, ent < 0 ? 0 : d - c, dtype, vec, x[i]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint16_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float v = x[i][k] + rv[k];                     // (columns past d and padding rows: 0 + 0)
          o[k] = f32_to_bf16_rne(v);
          const float f = bf16_to_f32(o[k]);
          sq[i] += f * f;
          er[i] += (v - f) * (v - f);
          if (!IS_A) o[k] = f32_to_bf16_rne(-2.f * f);        // B rows carry -2 b~ (exact: a sign flip and an exponent step)
        }
        if (c < KS * kSliceK)
          *(uint2*)(&tile[(2 * i + half) * W + c]) = make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
      }
    }
    // per-row totals: lane l now speaks for row 2 * i + half with i from bits 4, 3, 2 of l (four lanes hold the same)
    const float sqr = stage_reduce8(sq, lane), err = stage_reduce8(er, lane);
    {
      const int i = (((lane >> 4) & 1) << 2) | (((lane >> 3) & 1) << 1) | ((lane >> 2) & 1);
      const int row = 2 * i + half;
      int ent_r = __shfl(ent_l, row, 64);
      if constexpr (DROP) {
        if (!(err == err)) ent_r = -1;
        unsigned long long gone = __builtin_amdgcn_ballot_w64(!(err == err) && (lane & 3) == 0);
        while (gone) {                                         // (the same for the whole wave)
          const int r = __shfl(row, (int)__builtin_ctzll(gone), 64);
          for (int c = lane; c < d; c += 64) tile[r * W + c] = 0;
          gone &= gone - 1ull;
        }
        if (ent_out && (lane & 3) == 0) ent_out[slot0 + row] = ent_r;
      }
      float nrm = ent_r >= 0 ? sqr : 1e30f;
      const float plain = nrm;                                 // the maxima behind the accumulation bound stay plain
      if (slack && ent_r >= 0) {
        const float e = sqrtf(err) * 1.001f + 1.2e-7f * sqrtf(sqr);
        nrm = sqr - (2.f * slack_delta * e + 2.f * e * e) * 1.0001f;
      }
      if ((lane & 3) == 0) {
        uint16_t piece[3];
        float rem = nrm;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          piece[q] = f32_to_bf16_trunc(rem);
          rem -= bf16_to_f32(piece[q]);
        }
        const uint16_t one = 0x3F80u;
#pragma unroll
        for (int q = 0; q < kNormCols; ++q)
          tile[row * W + d + q] = (q < 3) == IS_A ? piece[q % 3] : one;
        if (norms) norms[(int64_t)rl * Nslots + slot0 + row] = plain;
        if (ent_r >= 0) vmax = fmaxf(vmax, plain);
      }
    }
    // the tile is this wave's own: its LDS operations complete in order, the fence keeps the compiler from moving them
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    {   // write out: slice ks of these 16 rows is 16 * 64 contiguous bytes
      const int row = lane >> 2, part = lane & 3;
      uint16_t* obase = out + ((int64_t)rl * KS * Nslots + slot0) * kSliceK + lane * 8;
      for (int ks = 0; ks < KS; ++ks) {
        const uint4 v = *(const uint4*)(&tile[row * W + ks * kSliceK + part * 8]);
        *(uint4*)(obase + (int64_t)ks * Nslots * kSliceK) = v;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  }
  if (max_slots) {   // one atomic per wave, spread over kMaxSlots addresses
    for (int off = 32; off > 0; off >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, off, 64));
    if (lane == 0) atomicMax(&max_slots[(blockIdx.x * 4 + wave) % kMaxSlots], __float_as_uint(vmax));   // non-negative floats order like their bits
  }
}

template <bool IS_A>
__global__ __launch_bounds__(256, 4) void k_stage_operands(const void* __restrict__ E, const void* __restrict__ Rv,
                                                        int dtype, int d, int r0, int RB,
                                                        const int32_t* __restrict__ slot_ent, int64_t Nslots, int KS,
                                                        uint16_t* __restrict__ out, float* __restrict__ norms,
                                                        unsigned int* __restrict__ max_slots,
                                                        const uint32_t* __restrict__ active_rows,
                                                        const unsigned int* __restrict__ n_active, int nH, int bm,
                                                        int64_t rel_stride = 0, const int32_t* __restrict__ n_rows_dev = nullptr,
                                                        float slack_delta = -1.f,
                                                        int64_t n_identity = 0) {      // slot_ent == NULL: slot s holds entity s, s < n_identity
  stage_operands<IS_A>(E, Rv, dtype, d, r0, RB, slot_ent, Nslots, KS, out, norms, max_slots, active_rows, n_active, nH, bm, rel_stride,
                       n_rows_dev, slack_delta, n_identity);
}
// Both sides of the relation-factorised join, which are the same plain rows in the two operand forms, in one launch:
// blockIdx.y = 0 stages the head side, 1 the tail side.  ent_out: the slots' entities, -1 for rows that are left out (DROP).
__global__ __launch_bounds__(256, 4) void k_stage_pair(const void* __restrict__ E, int dtype, int d, const int32_t* __restrict__ slot_ent,
                                                       int64_t Nslots, int KS, uint16_t* __restrict__ out_a, uint16_t* __restrict__ out_b,
                                                       unsigned int* __restrict__ max_a, unsigned int* __restrict__ max_b, float delta,
                                                       int32_t* __restrict__ ent_out) {
  if (blockIdx.y == 0)
    stage_operands<true, true>(E, nullptr, dtype, d, 0, 1, slot_ent, Nslots, KS, out_a, nullptr, max_a, nullptr, nullptr, 0, kStageRows, 0,
                               nullptr, delta, 0, ent_out);
  else
    stage_operands<false, true>(E, nullptr, dtype, d, 0, 1, slot_ent, Nslots, KS, out_b, nullptr, max_b, nullptr, nullptr, 0, kStageRows, 0,
                                nullptr, delta, 0);
}

// squared norms scattered back to entity order (kgc_norms)
__global__ void k_scatter_norms(const float* __restrict__ norms, const int32_t* __restrict__ slot_ent, int64_t Nslots,
                                int64_t N, int RB, float* __restrict__ outp) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)RB * Nslots) return;
  const int rl = (int)(i / Nslots);
  const int ent = slot_ent[i - (int64_t)rl * Nslots];
  if (ent >= 0) outp[(int64_t)rl * N + ent] = norms[i];
}

// max over rows of the L1 norm (used for the float32 error bound of the L1 filter); a half-wave takes four rows at a
// time, their loads in flight together
__global__ __launch_bounds__(256) void k_row_l1_max(const void* __restrict__ X, int64_t rows, int d, int dtype,
                                                    unsigned int* __restrict__ max_bits) {
  const int j = threadIdx.x & 31;
  const int64_t hw = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 5;
  const int64_t nhw = ((int64_t)gridDim.x * blockDim.x) >> 5;
  float vmax = 0.f;
  for (int64_t row = hw; row < rows; row += 4 * nhw) {
    float s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = 0.f;
    for (int c = j; c < d; c += 32) {
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = ld_elem(X, (row + q * nhw < rows ? row + q * nhw : row) * d + c, dtype);      // (past the end: this row again)
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] += fabsf(v[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s[q] += __shfl_xor(s[q], 16, 32);
      s[q] += __shfl_xor(s[q], 8, 32);
      s[q] += __shfl_xor(s[q], 4, 32);
      s[q] += __shfl_xor(s[q], 2, 32);
      s[q] += __shfl_xor(s[q], 1, 32);
      vmax = fmaxf(vmax, s[q]);
    }
  }
  if (j == 0) atomicMax(&max_bits[blockIdx.x % kMaxSlots], __float_as_uint(vmax));
}

// Filter thresholds, computed on the device so that no host round trip sits between kernel 1 and the join.
//
// L2.  The staged norm columns already carry every row's own rounding slack (see k_stage_operands), so that a
// true hit has D' = ||a~ - b~||^2 - slack_a - slack_b <= delta^2.  The contraction returns D' with an accumulated
// float32 error of at most e_acc, so the filter keeps D' <= delta^2 + e_acc and loses no hit.
// L1.  The float32 sum of |fl(fl(h + r) - t)| differs from the exact sum by at most
// 2^-23 (max||h||_1 + max||r||_1) + (d + 2) 2^-23 (delta + that); the filter keeps sums below delta + margin.
__global__ __launch_bounds__(64) void k_join_params(DevCounters* cnt, JoinParams* prm, float delta, int p, int dtype,
                                                    int d, int kp) {
  float ma = 0.f, mb = 0.f;
  for (int i = threadIdx.x; i < 1024; i += 64) {
    ma = fmaxf(ma, __uint_as_float(cnt->max_a[i]));
    mb = fmaxf(mb, __uint_as_float(cnt->max_b[i]));
  }
  for (int off = 32; off > 0; off >>= 1) {
    ma = fmaxf(ma, __shfl_xor(ma, off, 64));
    mb = fmaxf(mb, __shfl_xor(mb, off, 64));
  }
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  float thr, base = 0.f;
  if (p == 1) base = 1.2e-7f * (ma + mb);
  if (delta < 0.f) {
    thr = -1.f;                                   // squared distances and sums are >= 0: nothing passes
  } else if (p == 2) {
    const float eacc = (float)(kp + 16) * 1.2e-7f * 2.f * (ma + mb);
    thr = (delta * delta + eacc) * (1.f + 1e-6f);
  } else {
    thr = (delta + base + (float)(d + 2) * 1.2e-7f * (delta + base)) * (1.f + 1e-6f);
  }
  prm->thr = thr;
  prm->base = base;
}

// ---------------------------------------------------------------------------------------------
struct JoinArgs {
  const uint16_t* A;        // staged A operands of this relation batch: [RB][KS][Nslots][32]   (L2)
  const uint16_t* B;        // staged B operands: [KS][Nslots][32]                              (L2)
  const JoinParams* prm;
  int64_t Nslots;
  int KS;                   // 32-wide slices
  int k16;                  // 16-wide MFMA steps that hold data (the last slice may be half empty)
  int nH, nT;               // tiles along heads / tails
  int r0, RB;               // first relation and number of relations of this batch
  RecheckCtx cx;
};

// Kernel 2.  One block scores one (relation, head tile, tail tile): D = A_tile * B_tile^T over the
// augmented K (Section 4.3's dist for p = 2, squared, on bf16-rounded operands), with bf16 MFMA
// 32x32x16 and float32 accumulation.  K slices go global -> registers -> LDS, double buffered.
// WGM x WGN waves; each wave owns a (BM/WGM) x (BN/WGN) sub-tile as TM x TN MFMA tiles.
template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(WGM* WGN * 64) void k_join_l2(const JoinArgs a) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int LA = (BM * 4) / NT, LB = (BN * 4) / NT;   // 16-byte chunks per thread per slice
  static_assert(LA * NT == BM * 4 && LB * NT == BN * 4, "tile rows must divide over the threads");
  static_assert(TM >= 1 && TN >= 1, "wave tile too small");

  __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * kLdsRow];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BN * kLdsRow];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;

  const int tT = (int)blockIdx.x, tH = (int)blockIdx.y, rl = (int)blockIdx.z;

  const int64_t slice_elems = a.Nslots * kSliceK;
  const uint16_t* Ab = a.A + (int64_t)rl * a.KS * slice_elems + (int64_t)tH * BM * kSliceK;
  const uint16_t* Bb = a.B + (int64_t)tT * BN * kSliceK;

  uint4 ra[LA], rb[LB];
  auto gload = [&](int ks) {
    const uint4* ga = (const uint4*)(Ab + (int64_t)ks * slice_elems);
    const uint4* gb = (const uint4*)(Bb + (int64_t)ks * slice_elems);
#pragma unroll
    for (int i = 0; i < LA; ++i) ra[i] = ga[tid + i * NT];
#pragma unroll
    for (int i = 0; i < LB; ++i) rb[i] = gb[tid + i * NT];
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int c = tid + i * NT;
      *(uint4*)(&As[buf][(c >> 2) * kLdsRow + (c & 3) * 8]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int c = tid + i * NT;
      *(uint4*)(&Bs[buf][(c >> 2) * kLdsRow + (c & 3) * 8]) = rb[i];
    }
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  gload(0);
  sstore(0);
  __syncthreads();

  const int arow = wm * WTM + (lane & 31);
  const int brow = wn * WTN + (lane & 31);
  const int koff = (lane >> 5) * 8;

  for (int ks = 0; ks < a.KS; ++ks) {
    const int buf = ks & 1;
    if (ks + 1 < a.KS) gload(ks + 1);
    const int steps = (a.k16 - ks * 2) >= 2 ? 2 : 1;
    for (int s = 0; s < steps; ++s) {
      bf16x8_t fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[i] = *(const bf16x8_t*)(&As[buf][(arow + i * 32) * kLdsRow + s * 16 + koff]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[j] = *(const bf16x8_t*)(&Bs[buf][(brow + j * 32) * kLdsRow + s * 16 + koff]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (ks + 1 < a.KS) sstore(buf ^ 1);
    __syncthreads();
  }

  // ---- epilogue: filter on the squared distance, then the rare exact path ----
  const float thr = a.prm->thr;
  float mn = acc[0][0][0];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) mn = fminf(mn, acc[i][j][v]);
  if (__builtin_amdgcn_ballot_w64(mn <= thr) == 0ull) return;

  // MFMA 32x32 accumulator layout: register v of lane l holds row 8*(v/4) + 4*(l/32) + (v%4), column l%32.
  const int64_t hbase = (int64_t)tH * BM + wm * WTM;
  const int64_t tbase = (int64_t)tT * BN + wn * WTN;
  constexpr int NW = (TM * TN + 3) / 4;      // 64-element words of the candidate mask
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    unsigned long long cm = 0ull;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int tile = w * 4 + q;
      if (tile < TM * TN) {
        const int i = tile / TN, j = tile % TN;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (acc[i][j][v] <= thr) cm |= 1ull << (q * 16 + v);
      }
    }
    if (__builtin_amdgcn_ballot_w64(cm != 0ull) == 0ull) continue;
    recheck_and_emit(cm, a.r0 + rl, a.cx, [&](int e, int src, int64_t& hslot, int64_t& tslot) {
      const int tile = w * 4 + (e >> 4), v = e & 15;
      const int i = tile / TN, j = tile % TN;
      hslot = hbase + i * 32 + 8 * (v >> 2) + 4 * (src >> 5) + (v & 3);
      tslot = tbase + j * 32 + (src & 31);
    });
  }
}

// ---------------------------------------------------------------------------------------------
// Kernel 2, streaming form.  One block owns one (relation, head tile) and walks over a range of tail
// tiles; the K slices of all those tiles form one continuous stream that is prefetched two slices
// ahead through registers into a double-buffered LDS stage, so the global-memory latency of a slice
// is covered by the MFMA work of the two slices before it, also across tile boundaries.
// Tail-tile range: dense mode splits [0, nT) evenly over gridDim.z, the slowest grid dimension (x = head tile,
// y = relation), so that one range of tail rows stays in the L2 caches while every head tile of every
// relation passes over it; pruned mode reads the row's list of surviving tail tiles.
struct JoinStreamArgs {
  const uint16_t* A;
  const uint16_t* B;
  const JoinParams* prm;
  int64_t Nslots;
  int KS, k16;
  int nH, nT;
  int r0, RB;
  const uint32_t* row_start; // NULL: dense.  Else row = r_local * nH + head tile owns cols[row_start[row] .. + row_count[row])
  const uint32_t* row_count;
  const uint32_t* cols;      // surviving tail tile numbers, ascending within a row
  const uint32_t* active_rows;   // pruned mode: the rows with row_count > 0 ...
  const unsigned int* n_active;  // ... and how many there are; the grid strides over them
  RecheckCtx cx;
  ExactEntry* xlist;                  // where the kernel lists the accumulator blocks that hold candidates (k_exact_blocks
  unsigned int* xcount;               // scores them), how many it has listed, and how many the list holds; a block that
  unsigned int xcap;                  // finds the list full is counted, not stored (the host enlarges the list and reruns)
  const uint32_t* tile_rows;          // pruned mode, tile-at-a-time kernel: the row of every entry of cols ...
  const unsigned long long* tile_total;   // ... how many entries there are ...
  const unsigned int* pair_mode;      // ... and whether that kernel (1) or the row-walking one (0) takes this batch
  int cols_lds;                       // head-resident listed kernel: entries of LDS reserved for a row's tile list
  int b_per_rel;                      // 1: the tail operands are staged per relation, [RB][KS][Nslots][32] like A
  // Group assignment (k_join_l2_direct<.., kEpiAssignMin>): heads are all entities in identity order, tails
  // the pivots of a covering round, staged in an array of their own with tail_slots rows.
  int64_t tail_slots;                 // rows per K slice of B when it differs from Nslots (0: the same)
  const int32_t* tail_rows_dev;       // device count of valid tail rows (tail tiles past it are skipped); may be NULL
  float thr_value;                    // filter threshold on the squared distance when prm == NULL
  unsigned long long* best;           // kEpiAssignMin: per entity, min over the pivots within reach of (pivot position << 32);
                                      // kEpiMinDist: one word, min over all scored pairs of the float bits of the squared distance
  const int32_t* group_of;            // entities that already belong to a group (>= 0) are left alone
  int32_t* near_all; int32_t* near_first;   // kEpiNear: per entity, min over all pivots / those of the first tile of (distance bits, position)
  int64_t n_heads;                    // entities (head slots past it are padding)
  // k_join_l2_direct over tile lists, optional: candidates leave to a list that k_exact_pairs scores (NULL: the owning wave scores them)
  ExactEntry* plist; unsigned long long* pcount; unsigned int pcap;
};
enum { kEpiJoin = 0, kEpiAssignMin = 1, kEpiMinDist = 2, kEpiNear = 3 };
constexpr int kNearBits = 12;              // kEpiNear: low bits of a key that hold the pivot's position (kOrderPivots of them at most)

// A 32 x 32 accumulator block with candidates, at the end of a tile: listed for k_exact_blocks.  A full list drops
// the entry but still counts it: the host then sees how long the list has to be and runs the join again.
__device__ __forceinline__ void list_block(const JoinStreamArgs& a, int32_t r, int64_t hs0, int64_t ts0) {
  if (lane_id() == 0) {
    const unsigned int idx = atomicAdd(a.xcount, 1u);
    if (idx < a.xcap) a.xlist[idx] = ExactEntry{r, (int32_t)hs0, (int32_t)ts0, 0};
  }
}

// The exact stage of the L2 joins that list blocks: one wave per listed block (exact_block_l2), the grid strides over
// the list.  Workgroups of kExactWaves waves: the waves of a workgroup score their blocks side by side and reserve
// their output records with ONE atomic on the hit counter between them (two barriers per round; the sums of a round
// sit in the LDS buffer of the round's parity, so a wave that is already in the next round does not overwrite what a
// slower one still reads).  One atomic per block was measured at 18 of the kernel's 46 microseconds on a list of
// 2,400 blocks: atomics on one address are served one after the other, 8 ns each.
constexpr int kExactWaves = 16;
template <bool BF16, bool VEC>
__global__ __launch_bounds__(kExactWaves * 64, 1) void k_exact_blocks(const ExactEntry* __restrict__ list, const unsigned int* __restrict__ count,
                                                      unsigned int cap, unsigned long long* __restrict__ total,
                                                      unsigned int* __restrict__ need, const RecheckCtx cx) {
  __shared__ unsigned int wave_hits[2][kExactWaves];
  __shared__ unsigned long long wave_base[2][kExactWaves];
  const unsigned int n = *count < cap ? *count : cap;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *total += n;
    if (*count > *need) *need = *count;
  }
  // entry e goes to wave e / gridDim.x of workgroup e % gridDim.x: a short list is spread over all workgroups (and with
  // them over all compute units), not over the waves of the first few
  const unsigned int wv = (unsigned int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), per_round = gridDim.x * kExactWaves;
  int round = 0;
  for (unsigned int e0 = 0; e0 < n; e0 += per_round, ++round) {          // the same number of rounds for the whole workgroup
    const int par = round & 1;
    auto reserve = [&](int hits) -> unsigned long long {
      if ((threadIdx.x & 63) == 0) wave_hits[par][wv] = (unsigned int)hits;
      __syncthreads();
      if (threadIdx.x == 0) {
        unsigned int sum = 0u;
        for (int w = 0; w < kExactWaves; ++w) sum += wave_hits[par][w];
        unsigned long long base = sum ? atomicAdd(cx.hit_counter, (unsigned long long)sum) : 0ull;
        for (int w = 0; w < kExactWaves; ++w) { wave_base[par][w] = base; base += wave_hits[par][w]; }
      }
      __syncthreads();
      return wave_base[par][wv];
    };
    const unsigned int e = e0 + blockIdx.x + gridDim.x * wv;
    if (e < n) {                                                         // (the same for the whole wave)
      const ExactEntry x = list[e];
      exact_block_l2<BF16, VEC>(x.r, cx, (int64_t)x.hs0, (int64_t)x.ts0, reserve);
    } else {
      (void)reserve(0);
    }
  }
}

// LISTED: the block walks tile lists (pruned mode); otherwise the grid enumerates the dense problem and the
// kernel holds no load of the list in its inner loop (such a load would make every tile end wait for all
// outstanding prefetches).
template <int BM, int BN, int WGM, int WGN, int MINB, bool LISTED>
__global__ __launch_bounds__(WGM* WGN * 64, MINB) void k_join_l2_stream(const JoinStreamArgs a) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int LA = (BM * 4) / NT, LB = (BN * 4) / NT;
  constexpr int ASZ = BM * kSliceK, BSZ = BN * kSliceK;      // elements per LDS buffer (64-byte rows, swizzled)
  static_assert(LA * NT == BM * 4 && LB * NT == BN * 4, "tile rows must divide over the threads");

  __shared__ __attribute__((aligned(16))) uint16_t As[2 * ASZ];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2 * BSZ];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  int ncand_lane = 0;                                        // candidates this lane sent to the exact stage

  // pruned mode: the grid strides over the rows (relation, head tile) that still have tail tiles
  for (unsigned int row_i = blockIdx.x;; row_i += gridDim.x) {
  int tH, rl, t_begin, t_end;
  const uint32_t* cols = nullptr;
  if constexpr (LISTED) {
    if (row_i >= *a.n_active) break;
    const int64_t row = (int64_t)a.active_rows[row_i];
    rl = (int)(row / a.nH); tH = (int)(row - (int64_t)rl * a.nH);
    t_begin = (int)a.row_start[row]; t_end = t_begin + (int)a.row_count[row];
    cols = a.cols;
    __syncthreads();                    // the previous row is done with the LDS buffers
  } else {
    // grid = (head tiles, tail-tile ranges, relations): blocks that run together share a tail-tile range
    tH = (int)blockIdx.x; rl = (int)blockIdx.y;
    t_begin = (int)(((int64_t)a.nT * blockIdx.z) / gridDim.z);
    t_end = (int)(((int64_t)a.nT * (blockIdx.z + 1)) / gridDim.z);
  }
  const int ntiles = t_end - t_begin;
  if (ntiles <= 0) break;
  const int KS = a.KS;
  const int64_t slice_bytes = a.Nslots * kSliceK * 2;

  // per-thread byte offset inside a tile slice; uniform bases are kept apart so they can live in SGPRs
  const uint32_t voff = (uint32_t)tid * 16u;
  const char* Abase = (const char*)a.A + ((int64_t)rl * KS * a.Nslots + (int64_t)tH * BM) * (kSliceK * 2);
  const char* Bbase = (const char*)a.B + (a.b_per_rel ? (int64_t)rl * KS * a.Nslots * (kSliceK * 2) : 0);
  int tcol = cols ? (int)cols[t_begin] : t_begin;
  const char* pA = Abase;                                            // slice being prefetched
  const char* pB = Bbase + (int64_t)tcol * BN * (kSliceK * 2);

  // LDS addresses (elements): where this thread stores its chunks (chunk i sits NT / 4 rows below chunk 0),
  // and where it reads its fragments
  const int st0 = (tid >> 2) * kSliceK + (((tid & 3) ^ lds_swizzle(tid >> 2)) * 8);
  constexpr int st_step = (NT / 4) * kSliceK;      // NT / 4 is a multiple of 16 rows, so the swizzle repeats
  // fragment of MFMA step s: logical 16-byte chunk 2 s + lane / 32 of row lane % 32; rows 32 apart share the swizzle
  const int rsw = lds_swizzle(lane & 31);
  const int rd_a = (wm * WTM + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_b = (wn * WTN + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_step = (((lane >> 5) ^ rsw) & 2) ? -16 : 16;   // chunk ^ 2: the second step's fragment

  // staging registers as vectors (not arrays), so they are plain SSA values for the compiler
  typedef uint32_t rega_t __attribute__((ext_vector_type(4 * LA)));
  typedef uint32_t regb_t __attribute__((ext_vector_type(4 * LB)));
  rega_t ra;
  regb_t rb;

#define KGC_GLOAD()                                                                               \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < LA; ++i) {                                              \
      const uint4 t = *(const uint4*)(pA + voff + (uint32_t)(i * NT * 16));                       \
      ra[4 * i] = t.x; ra[4 * i + 1] = t.y; ra[4 * i + 2] = t.z; ra[4 * i + 3] = t.w;             \
    }                                                                                             \
    _Pragma("unroll") for (int i = 0; i < LB; ++i) {                                              \
      const uint4 t = *(const uint4*)(pB + voff + (uint32_t)(i * NT * 16));                       \
      rb[4 * i] = t.x; rb[4 * i + 1] = t.y; rb[4 * i + 2] = t.z; rb[4 * i + 3] = t.w;             \
    }                                                                                             \
  } while (0)
#define KGC_SSTORE(AW, BW)                                                                        \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < LA; ++i)                                                \
      *(uint4*)(&(AW)[st0 + i * st_step]) = make_uint4(ra[4 * i], ra[4 * i + 1], ra[4 * i + 2], ra[4 * i + 3]); \
    _Pragma("unroll") for (int i = 0; i < LB; ++i)                                                \
      *(uint4*)(&(BW)[st0 + i * st_step]) = make_uint4(rb[4 * i], rb[4 * i + 1], rb[4 * i + 2], rb[4 * i + 3]); \
  } while (0)
#define KGC_MFMA_STEP(FA, FB)                                                                     \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                \
      _Pragma("unroll") for (int j = 0; j < TN; ++j)                                              \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(FA[i], FB[j], acc[i][j], 0, 0, 0);    \
  } while (0)

  // prologue: first slice -> registers -> LDS buffer 0
  KGC_GLOAD();
  KGC_SSTORE(As, Bs);
  __syncthreads();

  const float thr = a.prm->thr;
  const int last_two = (a.k16 - (KS - 1) * 2) >= 2;   // does the last slice of a tile hold two MFMA steps of data?
  int buf = 0;

  for (int ti = 0; ti < ntiles; ++ti) {
    f32x16_t acc[TM][TN];          // first written by the ks == 0 step, whose MFMAs take a zero C operand
    const int tcol_cur = tcol;

    for (int ks = 0; ks < KS; ++ks) {
      // ---- issue the loads of the next slice of the stream (next K slice, or slice 0 of the next tile) ----
      const bool last_slice = (ks == KS - 1);
      const bool has_next = !(last_slice && ti == ntiles - 1);
      if (has_next) {
        if (last_slice) {
          tcol = cols ? (int)cols[t_begin + ti + 1] : t_begin + ti + 1;
          pA = Abase;
          pB = Bbase + (int64_t)tcol * BN * (kSliceK * 2);
        } else {
          pA += slice_bytes;
          pB += slice_bytes;
        }
        KGC_GLOAD();
      }
      // ---- MFMA on the current slice ----
      const uint16_t* Ac = As + buf * ASZ + rd_a;
      const uint16_t* Bc = Bs + buf * BSZ + rd_b;
      {
        // all fragments of both MFMA steps are requested first, so the second step's LDS latency hides
        // behind the first step's MFMAs (the last slice of a tile may hold one step only)
        const bool two = !last_slice || last_two;
        bf16x8_t fa[TM], fb[TN], ga[TM], gb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j] = *(const bf16x8_t*)(Bc + j * 32 * kSliceK);
        if (two) {
#pragma unroll
          for (int i = 0; i < TM; ++i) ga[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK + rd_step);
#pragma unroll
          for (int j = 0; j < TN; ++j) gb[j] = *(const bf16x8_t*)(Bc + j * 32 * kSliceK + rd_step);
        }
        if (ks == 0) {
          const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], zero16, 0, 0, 0);
        } else {
          KGC_MFMA_STEP(fa, fb);
        }
        if (two) KGC_MFMA_STEP(ga, gb);
      }
      // ---- stage the prefetched slice into the other buffer ----
      if (has_next) KGC_SSTORE(As + (buf ^ 1) * ASZ, Bs + (buf ^ 1) * BSZ);
      __syncthreads();
      buf ^= 1;
    }

    // ---- end of a tile: filter on the squared distance, then the rare exact path ----
    float mn = acc[0][0][0];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) mn = fminf(mn, acc[i][j][v]);
    const bool has = __builtin_amdgcn_ballot_w64(mn <= thr) != 0ull;
    // MFMA 32x32 accumulator layout: register v of lane l holds row 8*(v/4) + 4*(l/32) + (v%4), column l%32.
    const int64_t hbase = (int64_t)tH * BM + wm * WTM;
    const int64_t tbase = (int64_t)tcol_cur * BN + wn * WTN;
    // Surviving tiles hold their candidates in patches: each accumulator block that has some is re-scored as a
    // whole in double precision by a kernel of its own: here it is only listed (list_block).
    if (has) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          int n = 0;
#pragma unroll
          for (int v = 0; v < 16; ++v) n += (acc[i][j][v] <= thr) ? 1 : 0;
          if (__builtin_amdgcn_ballot_w64(n != 0) != 0ull) {
            ncand_lane += n;
            list_block(a, a.r0 + rl, hbase + i * 32, tbase + j * 32);
          }
        }
    }
  }
#undef KGC_GLOAD
#undef KGC_SSTORE
#undef KGC_MFMA_STEP
  if (!LISTED) break;
  }   // rows
  for (int off = 32; off > 0; off >>= 1) ncand_lane += __shfl_xor(ncand_lane, off, 64);
  if (lane == 0 && ncand_lane) atomicAdd(a.cx.cand_counter, (unsigned long long)ncand_lane);
}

// ---------------------------------------------------------------------------------------------
// Kernel 2, head-resident form.  As the streaming form, but the block first copies ALL K slices of its
// head tile (the staged a = h + r rows, BM x KS x 64 bytes) into LDS and keeps them there, so only the
// tail rows are streamed: half the global -> LDS traffic per tile, and the L2 only has to hold the tail
// range.  Tail slices are prefetched two slices ahead through two register sets.  Needs
// (KS * BM + 2 * BN) * 64 bytes of LDS: KS <= 8 (d <= 250) with one 256 x 256 block per CU, or with two 128 x 128 blocks per CU whose barriers and
// tile ends then fall at different times, so that one block's MFMAs fill the other's bubbles.
template <int BM, int BN, int WGM, int WGN, int MINB, int QCAP, bool LISTED>
__global__ __launch_bounds__(WGM* WGN * 64, MINB) void k_join_l2_ares(const JoinStreamArgs a) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int LA = (BM * 4) / NT, LB = (BN * 4) / NT;
  constexpr int ASZ = BM * kSliceK, BSZ = BN * kSliceK;
  static_assert(LA * NT == BM * 4 && LB * NT == BN * 4, "tile rows must divide over the threads");

  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // [KS][BM][32] head slices, then [2][BN][32] tail slices
  const int KS = a.KS;
  uint16_t* Ares = lds;
  uint16_t* Bs = lds + KS * ASZ;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  int ncand_lane = 0;                                        // candidates this lane sent to the exact stage
  if (LISTED && a.pair_mode && *a.pair_mode) return;         // this batch goes tile by tile (k_join_l2_pairs)

  for (unsigned int row_i = blockIdx.x;; row_i += gridDim.x) {
  int tH, rl, t_begin, t_end;
  const uint32_t* cols = nullptr;
  const uint32_t* lcols = nullptr;      // the row's tile list in LDS, when it fits (see below)
  if constexpr (LISTED) {
    if (row_i >= *a.n_active) break;
    const int64_t row = (int64_t)a.active_rows[row_i];
    rl = (int)(row / a.nH); tH = (int)(row - (int64_t)rl * a.nH);
    t_begin = (int)a.row_start[row]; t_end = t_begin + (int)a.row_count[row];
    cols = a.cols;
    __syncthreads();                    // the previous row is done with the LDS buffers
  } else {
    tH = (int)blockIdx.x; rl = (int)blockIdx.y;
    t_begin = (int)(((int64_t)a.nT * blockIdx.z) / gridDim.z);
    t_end = (int)(((int64_t)a.nT * (blockIdx.z + 1)) / gridDim.z);
  }
  const int ntiles = t_end - t_begin;
  if (ntiles <= 0) break;
  const int64_t slice_bytes = a.Nslots * kSliceK * 2;
  const uint32_t voff = (uint32_t)tid * 16u;
  const char* Abase = (const char*)a.A + ((int64_t)rl * KS * a.Nslots + (int64_t)tH * BM) * (kSliceK * 2);
  const char* Bbase = (const char*)a.B + (a.b_per_rel ? (int64_t)rl * KS * a.Nslots * (kSliceK * 2) : 0);
  int tcol = cols ? (int)cols[t_begin] : t_begin;
  const char* pB = Bbase + (int64_t)tcol * BN * (kSliceK * 2);

  const int st0 = (tid >> 2) * kSliceK + (((tid & 3) ^ lds_swizzle(tid >> 2)) * 8);
  constexpr int st_step = (NT / 4) * kSliceK;
  const int rsw = lds_swizzle(lane & 31);
  const int rd_a = (wm * WTM + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_b = (wn * WTN + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_step = (((lane >> 5) ^ rsw) & 2) ? -16 : 16;

  // ---- head tile: all K slices into LDS, once; four slices' loads in flight together (a row with one or two
  // ---- tiles is mostly memory round trips); past the last slice the loads repeat it and nothing is stored
  for (int ks0 = 0; ks0 < KS; ks0 += 4) {
    uint4 t[4][LA];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ks = ks0 + j < KS ? ks0 + j : KS - 1;
#pragma unroll
      for (int i = 0; i < LA; ++i) t[j][i] = *(const uint4*)(Abase + (int64_t)ks * slice_bytes + voff + (uint32_t)(i * NT * 16));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (ks0 + j < KS) {
#pragma unroll
        for (int i = 0; i < LA; ++i) *(uint4*)(&Ares[(ks0 + j) * ASZ + st0 + i * st_step]) = t[j][i];
      }
  }

  // The tile list of the row goes to LDS behind the tail buffers when there is room (a.cols_lds entries): the
  // loop then holds no global load besides the prefetches, whose outstanding count the compiler can follow
  // exactly; a list read from global memory makes every tile change wait for all of them.
  if (LISTED && ntiles <= a.cols_lds) {
    uint32_t* l = (uint32_t*)(Bs + 2 * BSZ);
    for (int t = tid; t < ntiles; t += NT) l[t] = cols[t_begin + t];
    lcols = l;
  }
  // the list must be complete before the first prefetches: with one or two K slices per tile they already move
  // on to the second tile (the barrier also publishes the head tile; all threads of a block take the same path)
  if (LISTED) __syncthreads();
  typedef uint32_t regb_t __attribute__((ext_vector_type(4 * LB)));
  regb_t rb0, rb1;
  int pf_k = 0, pf_t = 0, pf_i = 0;
#define KGC_GLOAD(RB)                                                                             \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < LB; ++i) {                                              \
      const uint4 t = *(const uint4*)(pB + voff + (uint32_t)(i * NT * 16));                       \
      RB[4 * i] = t.x; RB[4 * i + 1] = t.y; RB[4 * i + 2] = t.z; RB[4 * i + 3] = t.w;             \
    }                                                                                             \
    /* advance the cursor; past the end of the stream it stays on the last slice, so that the loads can be   */ \
    /* issued unconditionally (straight-line code lets the compiler count outstanding loads exactly)        */ \
    if (++pf_i < total) {                                                                         \
      if (++pf_k == KS) {                                                                         \
        pf_k = 0;                                                                                 \
        ++pf_t;                                                                                   \
        tcol = lcols ? (int)lcols[pf_t] : cols ? (int)cols[t_begin + pf_t] : t_begin + pf_t;          \
        pB = Bbase + (int64_t)tcol * BN * (kSliceK * 2);                                          \
      } else {                                                                                    \
        pB += slice_bytes;                                                                        \
      }                                                                                           \
    }                                                                                             \
  } while (0)
#define KGC_SSTORE(BUF, RB)                                                                       \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < LB; ++i)                                                \
      *(uint4*)(&Bs[(BUF) * BSZ + st0 + i * st_step]) =                                           \
          make_uint4(RB[4 * i], RB[4 * i + 1], RB[4 * i + 2], RB[4 * i + 3]);                     \
  } while (0)
#define KGC_MFMA_STEP(FA, FB)                                                                     \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                \
      _Pragma("unroll") for (int j = 0; j < TN; ++j)                                              \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(FA[i], FB[j], acc[i][j], 0, 0, 0);    \
  } while (0)

  const float thr = a.prm->thr;
  const int last_two = (a.k16 - (KS - 1) * 2) >= 2;
  const int total = ntiles * KS;
  int ck = 0, ct = 0;
  int tcol_cur = tcol;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // MFMA on tail slice in buffer BUF against head slice ck; at the end of a tile the filter on the squared
  // distance, the rare exact path, and the move to the next tile.  MFMA 32x32 accumulator layout: register v
  // of lane l holds row 8*(v/4) + 4*(l/32) + (v%4), column l%32.
#define KGC_COMPUTE(BUF)                                                                          \
  do {                                                                                            \
    const uint16_t* Ac = Ares + ck * ASZ + rd_a;                                                  \
    const uint16_t* Bc = Bs + (BUF) * BSZ + rd_b;                                                 \
    const bool last_slice = (ck == KS - 1);                                                       \
    const bool two = !last_slice || last_two;                                                     \
    bf16x8_t fa[TM], fb[TN];                                                                      \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK); \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) fb[j] = *(const bf16x8_t*)(Bc + j * 32 * kSliceK); \
    if (ck == 0) {                                                                                \
      const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], zero16, 0, 0, 0);     \
    } else {                                                                                      \
      KGC_MFMA_STEP(fa, fb);                                                                      \
    }                                                                                             \
    if (two) {                                                                                    \
      _Pragma("unroll") for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK + rd_step); \
      _Pragma("unroll") for (int j = 0; j < TN; ++j) fb[j] = *(const bf16x8_t*)(Bc + j * 32 * kSliceK + rd_step); \
      KGC_MFMA_STEP(fa, fb);                                                                      \
    }                                                                                             \
    if (last_slice) {                                                                             \
      /* End of a tile: does any element pass the filter?  Candidates come in patches, so every accumulator    */ \
      /* block that holds some is listed for the exact kernel (list_block): no queue, no extra barrier.         */ \
      /* MFMA 32x32 accumulator layout: register v of lane l holds row 8*(v/4) + 4*(l/32) + (v%4), column l%32. */ \
      float mn = acc[0][0][0];                                                                    \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
          _Pragma("unroll") for (int v = 0; v < 16; ++v) mn = fminf(mn, acc[i][j][v]);            \
      if (__builtin_amdgcn_ballot_w64(mn <= thr) != 0ull) {                                       \
        const int64_t hbase = (int64_t)tH * BM + wm * WTM;                                        \
        const int64_t tbase = (int64_t)tcol_cur * BN + wn * WTN;                                  \
        _Pragma("unroll") for (int i = 0; i < TM; ++i)                                            \
          _Pragma("unroll") for (int j = 0; j < TN; ++j) {                                        \
            int n = 0;                                                                            \
            _Pragma("unroll") for (int v = 0; v < 16; ++v) n += (acc[i][j][v] <= thr) ? 1 : 0;    \
            if (__builtin_amdgcn_ballot_w64(n != 0) != 0ull) {                                    \
              ncand_lane += n;                                                                    \
              list_block(a, a.r0 + rl, hbase + i * 32, tbase + j * 32);                           \
            }                                                                                     \
          }                                                                                       \
      }                                                                                           \
      ck = 0;                                                                                     \
      if (++ct < ntiles) tcol_cur = lcols ? (int)lcols[ct] : cols ? (int)cols[t_begin + ct] : t_begin + ct; \
    } else {                                                                                      \
      ++ck;                                                                                       \
    }                                                                                             \
  } while (0)

  // prologue: tail slices 0 and 1 in flight, slice 0 staged (the barrier also publishes the head tile)
  KGC_GLOAD(rb0);
  KGC_GLOAD(rb1);
  KGC_SSTORE(0, rb0);
  __syncthreads();

  // Both steps run to their end in every iteration (an odd number of slices only skips the second step's
  // arithmetic): with no way out of the middle of the body, every path reaches the top of the loop with
  // the same loads outstanding, so the compiler needs no wait there.
  for (int i = 0; i < total; i += 2) {
    // even step: slice i is in buffer 0; set 0 is free for slice i + 2; set 1 holds slice i + 1
    KGC_GLOAD(rb0);
    KGC_COMPUTE(0);
    KGC_SSTORE(1, rb1);
    __syncthreads();
    // odd step: slice i + 1 is in buffer 1; set 1 is free for slice i + 3; set 0 holds slice i + 2
    KGC_GLOAD(rb1);
    if (i + 1 < total) KGC_COMPUTE(1);
    KGC_SSTORE(0, rb0);
    __syncthreads();
  }
#undef KGC_GLOAD
#undef KGC_SSTORE
#undef KGC_MFMA_STEP
#undef KGC_COMPUTE
  if (!LISTED) break;
  }   // rows
  for (int off = 32; off > 0; off >>= 1) ncand_lane += __shfl_xor(ncand_lane, off, 64);
  if (lane == 0 && ncand_lane) atomicAdd(a.cx.cand_counter, (unsigned long long)ncand_lane);
}

// ---------------------------------------------------------------------------------------------
// Kernel 2, one surviving tile at a time (pruned joins whose rows keep only a tile or two each).  Walking such a
// row costs the row-walking kernels a chain of some ten memory round trips (row record, tile list, head tile,
// the tail slices one behind the other) for a microsecond of arithmetic.  Here a block takes one (row, tail tile)
// entry of the list, reads ALL K slices of both 128-row tiles with every load in flight at once, and multiplies out
// of LDS: three round trips per tile.  The host launches both kernels; a device flag set from the batch's tile and
// row counts (k_batch_tiles) says which of them works.  LDS: 2 * KS * 8 KiB.
__global__ __launch_bounds__(256, 2) void k_join_l2_pairs(const JoinStreamArgs a) {
  constexpr int BM = 128, BN = 128, NT = 256, WGN = 2, WTM = 64, WTN = 64, TM = 2, TN = 2;
  constexpr int LA = (BM * 4) / NT;
  constexpr int ASZ = BM * kSliceK;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // [KS][128][32] head slices, then the same for the tail tile
  if (!*a.pair_mode) return;
  const int KS = a.KS;
  uint16_t* As = lds;
  uint16_t* Bs = lds + KS * ASZ;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const unsigned int total = (unsigned int)*a.tile_total;
  const int64_t slice_bytes = a.Nslots * kSliceK * 2;
  const uint32_t voff = (uint32_t)tid * 16u;
  const int st0 = (tid >> 2) * kSliceK + (((tid & 3) ^ lds_swizzle(tid >> 2)) * 8);
  constexpr int st_step = (NT / 4) * kSliceK;
  const int rsw = lds_swizzle(lane & 31);
  const int rd_a = (wm * WTM + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_b = (wn * WTN + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_step = (((lane >> 5) ^ rsw) & 2) ? -16 : 16;
  const float thr = a.prm->thr;
  const bool last_two = (a.k16 - (KS - 1) * 2) >= 2;
  int ncand_lane = 0;
  // A block walks its tiles (entries blockIdx.x, + gridDim.x, ... of the list) in batches of up to kPairsBatch: the
  // batch's list entries are read into the LDS first, so that no load of the list sits among the tile loads (loads
  // return in order: waiting for a list entry would wait for every tile load asked for before it).  The first four K
  // slices of the NEXT tile are asked for as soon as the current tile is in the LDS, so that their memory round trip
  // runs beside the current tile's arithmetic.  Which of a tile's 32 x 32 blocks hold candidates is noted per wave,
  // and the batch's blocks are listed for the exact kernel at its end with ONE atomic on the list's length for the
  // whole workgroup (atomics on one address are served one after the other, and their round trip would sit in
  // every tile's path).
  constexpr int kPairsBatch = 32;
  __shared__ uint32_t my_row[kPairsBatch], my_col[kPairsBatch];
  __shared__ uint8_t my_has[kPairsBatch][4];
  __shared__ unsigned int list_n[4];
  __shared__ unsigned int list_base;
  typedef uint32_t regt_t __attribute__((ext_vector_type(16 * LA)));   // 4 slices x LA chunks x 4 registers: vectors, so
  regt_t ta, tb;                                                       // that they are plain SSA values for the compiler
#define KGC_PAIRS_ASK(ROW, TCOL)                                                                              \
  do {                                                                                                       \
    const int rl_ = (int)((ROW) / (uint32_t)a.nH), tH_ = (int)((ROW) - (uint32_t)rl_ * (uint32_t)a.nH);      \
    const char* Ab_ = (const char*)a.A + ((int64_t)rl_ * KS * a.Nslots + (int64_t)tH_ * BM) * (kSliceK * 2); \
    const char* Bb_ = (const char*)a.B + (a.b_per_rel ? (int64_t)rl_ * KS * a.Nslots * (kSliceK * 2) : 0) +  \
                      (int64_t)(TCOL) * BN * (kSliceK * 2);                                                  \
    _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                          \
      const int ks = j < KS ? j : KS - 1; /* past the last slice the loads repeat it and nothing is stored */ \
      _Pragma("unroll") for (int i = 0; i < LA; ++i) {                                                       \
        const uint4 x_ = *(const uint4*)(Ab_ + (int64_t)ks * slice_bytes + voff + (uint32_t)(i * NT * 16));  \
        const uint4 y_ = *(const uint4*)(Bb_ + (int64_t)ks * slice_bytes + voff + (uint32_t)(i * NT * 16));  \
        ta[4 * (j * LA + i)] = x_.x; ta[4 * (j * LA + i) + 1] = x_.y; ta[4 * (j * LA + i) + 2] = x_.z; ta[4 * (j * LA + i) + 3] = x_.w; \
        tb[4 * (j * LA + i)] = y_.x; tb[4 * (j * LA + i) + 1] = y_.y; tb[4 * (j * LA + i) + 2] = y_.z; tb[4 * (j * LA + i) + 3] = y_.w; \
      }                                                                                                      \
    }                                                                                                        \
  } while (0)
  for (unsigned int e0 = blockIdx.x; e0 < total; e0 += kPairsBatch * gridDim.x) {      // (the same for the whole block)
    // the batch's entries e0, e0 + gridDim.x, ...
    const unsigned int left = (total - e0 + gridDim.x - 1) / gridDim.x;
    const int nb = left < (unsigned int)kPairsBatch ? (int)left : kPairsBatch;
    __syncthreads();                                         // the previous batch is listed
    if (tid < nb) { my_row[tid] = a.tile_rows[e0 + (unsigned int)tid * gridDim.x]; my_col[tid] = a.cols[e0 + (unsigned int)tid * gridDim.x]; }
    __syncthreads();
    KGC_PAIRS_ASK(my_row[0], my_col[0]);
    for (int it = 0; it < nb; ++it) {
    const uint32_t row = my_row[it], tcol_now = my_col[it];
    const int rl = (int)(row / (uint32_t)a.nH), tH = (int)(row - (uint32_t)rl * (uint32_t)a.nH);
    __syncthreads();                                         // the previous tile is done with the LDS
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < KS) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
          *(uint4*)(&As[j * ASZ + st0 + i * st_step]) = make_uint4(ta[4 * (j * LA + i)], ta[4 * (j * LA + i) + 1], ta[4 * (j * LA + i) + 2], ta[4 * (j * LA + i) + 3]);
          *(uint4*)(&Bs[j * ASZ + st0 + i * st_step]) = make_uint4(tb[4 * (j * LA + i)], tb[4 * (j * LA + i) + 1], tb[4 * (j * LA + i) + 2], tb[4 * (j * LA + i) + 3]);
        }
      }
    if (KS > 4) {                                            // the slices after the fourth: loaded now (d > 122)
      const char* Abase = (const char*)a.A + ((int64_t)rl * KS * a.Nslots + (int64_t)tH * BM) * (kSliceK * 2);
      const char* Bbase = (const char*)a.B + (a.b_per_rel ? (int64_t)rl * KS * a.Nslots * (kSliceK * 2) : 0) +
                          (int64_t)tcol_now * BN * (kSliceK * 2);
      for (int ks0 = 4; ks0 < KS; ks0 += 4) {
        uint4 ua[4][LA], ub[4][LA];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int ks = ks0 + j < KS ? ks0 + j : KS - 1;
#pragma unroll
          for (int i = 0; i < LA; ++i) {
            ua[j][i] = *(const uint4*)(Abase + (int64_t)ks * slice_bytes + voff + (uint32_t)(i * NT * 16));
            ub[j][i] = *(const uint4*)(Bbase + (int64_t)ks * slice_bytes + voff + (uint32_t)(i * NT * 16));
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (ks0 + j < KS) {
#pragma unroll
            for (int i = 0; i < LA; ++i) {
              *(uint4*)(&As[(ks0 + j) * ASZ + st0 + i * st_step]) = ua[j][i];
              *(uint4*)(&Bs[(ks0 + j) * ASZ + st0 + i * st_step]) = ub[j][i];
            }
          }
      }
    }
    __syncthreads();
    if (it + 1 < nb) KGC_PAIRS_ASK(my_row[it + 1], my_col[it + 1]);      // the next tile's loads
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    for (int ks = 0; ks < KS; ++ks) {
      const uint16_t* Ac = As + ks * ASZ + rd_a;
      const uint16_t* Bc = Bs + ks * ASZ + rd_b;
      const int nstep = (ks < KS - 1 || last_two) ? 2 : 1;
      for (int step = 0; step < nstep; ++step) {
        bf16x8_t fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK + step * rd_step);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j] = *(const bf16x8_t*)(Bc + j * 32 * kSliceK + step * rd_step);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
      }
    }
    // the filter on the squared distance: which of the wave's blocks hold candidates
    unsigned int has = 0u;                                   // bit i * TN + j: block (i, j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        int n = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) n += (acc[i][j][v] <= thr) ? 1 : 0;
        ncand_lane += n;
        if (__builtin_amdgcn_ballot_w64(n != 0) != 0ull) has |= 1u << (i * TN + j);
      }
    if (lane == 0) my_has[it][wave] = (uint8_t)has;
    }   // tiles of the batch
    // the batch's blocks with candidates onto the list: wave w takes the notes of all four waves for tiles w, w + 4, ...
    __syncthreads();
    unsigned int mine = 0u;
    for (int it = wave; it < nb; it += 4)
      mine += (unsigned int)__builtin_popcount((unsigned int)my_has[it][0] | ((unsigned int)my_has[it][1] << 8) |
                                               ((unsigned int)my_has[it][2] << 16) | ((unsigned int)my_has[it][3] << 24));
    if (lane == 0) list_n[wave] = mine;
    __syncthreads();
    if (tid == 0) {
      const unsigned int sum = list_n[0] + list_n[1] + list_n[2] + list_n[3];
      list_base = sum ? atomicAdd(a.xcount, sum) : 0u;
    }
    __syncthreads();
    if (lane == 0 && mine) {
      unsigned int idx = list_base;
      for (int w = 0; w < wave; ++w) idx += list_n[w];
      for (int it = wave; it < nb; it += 4) {
        const uint32_t row = my_row[it];
        const int rl = (int)(row / (uint32_t)a.nH), tH = (int)(row - (uint32_t)rl * (uint32_t)a.nH);
        for (int w = 0; w < 4; ++w) {
          const unsigned int has = my_has[it][w];
          const int64_t hbase = (int64_t)tH * BM + (w / WGN) * WTM;
          const int64_t tbase = (int64_t)my_col[it] * BN + (w % WGN) * WTN;
          for (int b = 0; b < TM * TN; ++b)
            if ((has >> b) & 1u) {
              if (idx < a.xcap) a.xlist[idx] = ExactEntry{a.r0 + rl, (int32_t)(hbase + (b / TN) * 32), (int32_t)(tbase + (b % TN) * 32), 0};
              ++idx;
            }
        }
      }
    }
  }   // batches
#undef KGC_PAIRS_ASK
  for (int off = 32; off > 0; off >>= 1) ncand_lane += __shfl_xor(ncand_lane, off, 64);
  if (lane == 0 && ncand_lane) atomicAdd(a.cx.cand_counter, (unsigned long long)ncand_lane);
}

// ---------------------------------------------------------------------------------------------
// Kernel 2, barrier-free form (dense mode only).  The head tile is resident in LDS as above, but the tail
// rows never pass through LDS: every wave reads the MFMA fragments of ITS OWN WTN tail columns straight from
// the staged operand array into registers (lane l takes row l % 32 of a 32-row group, 16 bytes at offset
// 16 * (l / 32) for the first K step of a slice and 32 bytes further for the second: the layout the MFMA
// wants), two slices ahead of their use through three register sets.  Nothing in the loop is shared between
// waves, so it holds no barrier and no LDS store: the LDS only serves the head fragments, and the waves of
// a block drift apart, so that one wave's MFMAs cover the other's waits.  The waves that share tail columns
// (same wn) read the same lines, mostly one after the other out of the CU's vector cache.
// LDS: KS * BM * 64 bytes: BM = 256 up to KS = 9 (d <= 282), BM = 128 up to KS = 19 (d <= 602).  In the join
// form (EPI = kEpiJoin) candidates are re-scored by the owning wave; kEpiAssignMin is the epilogue of the
// group assignment (see JoinStreamArgs).
// LISTED (pruned joins over many entities, kEpiJoin): the grid strides over the active rows, and a row's tile list
// sits in the LDS behind the head slices (a.cols_lds entries), so that the tile loop holds no load of the list among
// its prefetches.
constexpr int kListPart = 16, kListParts = 8;      // LISTED: tiles of a part of a row, and parts of a row, at least and at most
template <int BM, int WGM, int WGN, int EPI, bool LISTED = false>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void k_join_l2_direct(const JoinStreamArgs a) {
  constexpr int BN = 256;
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int LA = (BM * 4) / NT;
  constexpr int ASZ = BM * kSliceK;
  constexpr int ROWB = kSliceK * 2;                       // bytes of one staged row slice
  static_assert(LA * NT == BM * 4, "tile rows must divide over the threads");

  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // [KS][BM][32] head slices
  const int KS = a.KS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;

  for (unsigned int blk_i = blockIdx.x;; blk_i += gridDim.x) {
  unsigned int row_i = blk_i;
  int tH, rl, t_begin, ntiles;
  const uint32_t* tlist = nullptr;                         // LISTED: the row's tile list in the LDS
  if constexpr (LISTED) {
    // Workgroups go to the eight XCDs in turn, and neighbouring active rows (one relation, neighbouring head tiles)
    // meet the same tail tiles: within every 256 consecutive workgroups, those of one XCD take 32 neighbouring rows,
    // so that a tail tile is fetched into one L2, not into all eight.
    const unsigned int n_act = *a.n_active;
    if ((blk_i & ~255u) >= n_act) break;                   // (the same for the whole block)
    row_i = (blk_i & ~255u) + (blk_i & 7u) * 32u + ((blk_i >> 3) & 31u);
    if (row_i >= n_act) continue;                          // (a hole of the last, partial set of 256)
    // (the same for the whole block: kept in scalar registers)
    const int64_t row = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a.active_rows[row_i]);
    rl = (int)(row / a.nH); tH = (int)(row - (int64_t)rl * a.nH);
    t_begin = __builtin_amdgcn_readfirstlane((int)a.row_start[row]); ntiles = __builtin_amdgcn_readfirstlane((int)a.row_count[row]);
    // A long row is cut into as many parts as have kListPart tiles, at most gridDim.y: where a few rows hold most of a
    // batch's tiles (a group against all rows without one), one workgroup each would leave the chip idle.
    const int parts = ntiles / kListPart < (int)gridDim.y ? (ntiles / kListPart > 1 ? ntiles / kListPart : 1) : (int)gridDim.y;
    const int part = (int)blockIdx.y;
    if (part >= parts) continue;                           // (the same for the whole block)
    const int p0 = (int)((int64_t)ntiles * part / parts), p1 = (int)((int64_t)ntiles * (part + 1) / parts);
    t_begin += p0;
    ntiles = p1 - p0;
    __syncthreads();                                       // the previous row is done with the LDS
  } else {
    tH = (int)blockIdx.x; rl = (int)blockIdx.y;
    int nT = a.nT;
    if (EPI == kEpiAssignMin && a.tail_rows_dev) {        // only the tail tiles that hold pivots of this round
      const int used = (*a.tail_rows_dev + BN - 1) / BN;
      nT = used < nT ? used : nT;
    }
    t_begin = (int)(((int64_t)nT * blockIdx.z) / gridDim.z);
    ntiles = (int)(((int64_t)nT * (blockIdx.z + 1)) / gridDim.z) - t_begin;
  }
  if (ntiles <= 0) break;                                  // (an active row has tiles; the same for the whole block)
  const int64_t slice_bytes_a = a.Nslots * ROWB;
  const int64_t slice_bytes = (a.tail_slots ? a.tail_slots : a.Nslots) * ROWB;

  // ---- head tile: all K slices into LDS, once (swizzled as in the other forms) ----
  {
    const char* Abase = (const char*)a.A + ((int64_t)rl * KS * a.Nslots + (int64_t)tH * BM) * ROWB;
    const uint32_t voff = (uint32_t)tid * 16u;
    const int st0 = (tid >> 2) * kSliceK + (((tid & 3) ^ lds_swizzle(tid >> 2)) * 8);
    constexpr int st_step = (NT / 4) * kSliceK;
    for (int ks = 0; ks < KS; ++ks) {
      uint4 t[LA];
#pragma unroll
      for (int i = 0; i < LA; ++i) t[i] = *(const uint4*)(Abase + (int64_t)ks * slice_bytes_a + voff + (uint32_t)(i * NT * 16));
#pragma unroll
      for (int i = 0; i < LA; ++i) *(uint4*)(&lds[ks * ASZ + st0 + i * st_step]) = t[i];
    }
  }
  // LISTED: the row's tiles in segments of what the LDS holds of the list (a.cols_lds entries; nearly always one segment)
  const int row_tiles = ntiles;
  for (int seg0 = 0; seg0 < (LISTED ? row_tiles : 1); seg0 += (LISTED ? a.cols_lds : 1)) {
  if constexpr (LISTED) {
    if (seg0 > 0) __syncthreads();                         // the previous segment's list is no longer read
    ntiles = row_tiles - seg0 < a.cols_lds ? row_tiles - seg0 : a.cols_lds;
    uint32_t* l = (uint32_t*)(lds + KS * ASZ);
    for (int t = tid; t < ntiles; t += NT) l[t] = a.cols[t_begin + seg0 + t];
    tlist = l;
  }
  __syncthreads();          // the head tile (and the tile list) is complete: no barrier in the tile loop

  const int rsw = lds_swizzle(lane & 31);
  const int rd_a = (wm * WTM + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_step = (((lane >> 5) ^ rsw) & 2) ? -16 : 16;

  // tail fragments of this lane: row (lane % 32) of each 32-row group of the wave's columns
  // (LISTED: the tile part of the address is the same for the whole wave and stays in scalar registers, the lane's
  // part is a 32-bit offset: the kernel has no register to spare)
  const uint32_t boff = (uint32_t)((wn * WTN + (lane & 31)) * ROWB + (lane >> 5) * 16);
  const char* Bw = (const char*)a.B + (a.b_per_rel ? (int64_t)rl * KS * a.Nslots * ROWB : 0) + (LISTED ? 0u : boff);
  const char* pB = Bw + (int64_t)(LISTED ? __builtin_amdgcn_readfirstlane((int)tlist[0]) : t_begin) * BN * ROWB;
  const int total = ntiles * KS;
  int pf_k = 0, pf_t = 0, pf_i = 0;

  typedef uint32_t regq_t __attribute__((ext_vector_type(8 * TN)));   // TN column groups x 2 K steps x 4 registers
  regq_t q0, q1, q2;
#define KGC_GLOAD(Q)                                                                              \
  do {                                                                                            \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) {                                              \
      const uint4 t0 = *(const uint4*)(pB + ((LISTED ? boff : 0u) + (uint32_t)(j * 32 * ROWB)));  \
      const uint4 t1 = *(const uint4*)(pB + ((LISTED ? boff : 0u) + (uint32_t)(j * 32 * ROWB + 32))); \
      Q[8 * j] = t0.x; Q[8 * j + 1] = t0.y; Q[8 * j + 2] = t0.z; Q[8 * j + 3] = t0.w;             \
      Q[8 * j + 4] = t1.x; Q[8 * j + 5] = t1.y; Q[8 * j + 6] = t1.z; Q[8 * j + 7] = t1.w;         \
    }                                                                                             \
    /* the cursor stops on the last slice, so the loads are unconditional (and the compiler can count them) */ \
    if (++pf_i < total) {                                                                         \
      if (++pf_k == KS) {                                                                         \
        pf_k = 0;                                                                                 \
        ++pf_t;                                                                                   \
        pB = Bw + (int64_t)(LISTED ? __builtin_amdgcn_readfirstlane((int)tlist[pf_t]) : t_begin + pf_t) * BN * ROWB; \
      } else {                                                                                    \
        pB += slice_bytes;                                                                        \
      }                                                                                           \
    }                                                                                             \
  } while (0)
#define KGC_FRAG(Q, J, STEP)                                                                      \
  __builtin_bit_cast(bf16x8_t, u32x4_t{Q[8 * (J) + 4 * (STEP)], Q[8 * (J) + 4 * (STEP) + 1],      \
                                       Q[8 * (J) + 4 * (STEP) + 2], Q[8 * (J) + 4 * (STEP) + 3]})

  // kEpiNear takes the transpose: a lane then holds one head row (column of the accumulator) and many pivots, whose
  // minimum needs no exchange between lanes
#define KGC_MFMA(FA, FB, C)                                                                       \
  (EPI == kEpiNear ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(FB, FA, C, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(FA, FB, C, 0, 0, 0))
  const float thr = a.prm ? a.prm->thr : a.thr_value;
  float run_min = 3e38f;                                   // kEpiMinDist
  int near[EPI == kEpiNear ? TM : 1];                      // kEpiNear: smallest key of this lane's head row in each block of 32
  if constexpr (EPI == kEpiNear)
#pragma unroll
    for (int i = 0; i < TM; ++i) near[i] = 0x7fffffff;
  const int last_two = (a.k16 - (KS - 1) * 2) >= 2;
  int ck = 0, ct = 0;
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // kEpiNear: the keys so far to memory (the two halves of the wave hold pivots of the same head rows)
#define KGC_NEAR_OUT(OUT)                                                                         \
  do {                                                                                            \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) {                                              \
      const int key = min(near[i], __shfl_xor(near[i], 32, 64));                                  \
      const int64_t e = (int64_t)tH * BM + wm * WTM + i * 32 + (lane & 31);                       \
      if (lane < 32 && e < a.n_heads) atomicMin(&(OUT)[e], key);                                  \
    }                                                                                             \
  } while (0)
  // One slice: head fragments from LDS, tail fragments from register set Q; at the end of a tile the filter
  // on the squared distance and the rare exact path.  MFMA 32x32 accumulator layout: register v of lane l
  // holds row 8*(v/4) + 4*(l/32) + (v%4), column l%32.
#define KGC_COMPUTE(Q)                                                                            \
  do {                                                                                            \
    const uint16_t* Ac = lds + ck * ASZ + rd_a;                                                   \
    const bool last_slice = (ck == KS - 1);                                                       \
    const bool two = !last_slice || last_two;                                                     \
    bf16x8_t fa[TM];                                                                              \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK); \
    if (ck == 0) {                                                                                \
      const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
          acc[i][j] = KGC_MFMA(fa[i], KGC_FRAG(Q, j, 0), zero16); \
    } else {                                                                                      \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
          acc[i][j] = KGC_MFMA(fa[i], KGC_FRAG(Q, j, 0), acc[i][j]); \
    }                                                                                             \
    if (two) {                                                                                    \
      _Pragma("unroll") for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(Ac + i * 32 * kSliceK + rd_step); \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
          acc[i][j] = KGC_MFMA(fa[i], KGC_FRAG(Q, j, 1), acc[i][j]); \
    }                                                                                             \
    if (last_slice) {                                                                             \
      if constexpr (EPI == kEpiNear) {                                                            \
        const int where = (t_begin + ct) * BN + wn * WTN + 4 * (lane >> 5);                       \
        _Pragma("unroll") for (int i = 0; i < TM; ++i) {                                          \
          int key = 0x7fffffff;                                                                   \
          _Pragma("unroll") for (int j = 0; j < TN; ++j)                                          \
            _Pragma("unroll") for (int v = 0; v < 16; ++v)                                        \
              key = min(key, (__float_as_int(acc[i][j][v]) & ~((1 << kNearBits) - 1)) | (j * 32 + 8 * (v >> 2) + (v & 3))); \
          near[i] = min(near[i], key | where);                                                    \
        }                                                                                         \
        if (t_begin + ct == 0) KGC_NEAR_OUT(a.near_first);                                        \
      }                                                                                           \
      float mn = acc[0][0][0];                                                                    \
      _Pragma("unroll") for (int i = 0; i < TM; ++i)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                            \
          _Pragma("unroll") for (int v = 0; v < 16; ++v) mn = fminf(mn, acc[i][j][v]);            \
      if (EPI == kEpiNear) {                                                                      \
      } else if (EPI == kEpiMinDist) {                                                            \
        run_min = fminf(run_min, mn);        /* only the smallest squared distance is wanted */    \
      } else if (__builtin_amdgcn_ballot_w64(mn <= thr) != 0ull) {                                \
        const int64_t hbase = (int64_t)tH * BM + wm * WTM;                                        \
        const int64_t tbase = (int64_t)(LISTED ? __builtin_amdgcn_readfirstlane((int)tlist[ct]) : t_begin + ct) * BN + wn * WTN; \
        constexpr int NW = (TM * TN + 3) / 4;                                                     \
        _Pragma("unroll") for (int w = 0; w < NW; ++w) {                                          \
          unsigned long long cm = 0ull;                                                           \
          _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                         \
            const int tile = w * 4 + q;                                                           \
            if (tile < TM * TN) {                                                                 \
              const int i = tile / TN, j = tile % TN;                                             \
              _Pragma("unroll") for (int v = 0; v < 16; ++v)                                      \
                if (acc[i][j][v] <= thr) cm |= 1ull << (q * 16 + v);                              \
            }                                                                                     \
          }                                                                                       \
          if (__builtin_amdgcn_ballot_w64(cm != 0ull) == 0ull) continue;                          \
          auto map = [=](int e, int src, int64_t& hslot, int64_t& tslot) {                        \
            const int tile = w * 4 + (e >> 4), v = e & 15;                                        \
            const int i = tile / TN, j = tile % TN;                                               \
            hslot = hbase + i * 32 + 8 * (v >> 2) + 4 * (src >> 5) + (v & 3);                     \
            tslot = tbase + j * 32 + (src & 31);                                                  \
          };                                                                                      \
          if (EPI == kEpiJoin) {                                                                  \
            if (LISTED && a.plist) list_pairs(cm, a.r0 + rl, a.plist, a.pcount, a.pcap, map);     \
            else recheck_and_emit(cm, a.r0 + rl, a.cx, map);                                      \
          } else {                                                                                \
            /* only the lowest pivot position within reach matters to the round (the low word, a distance in the */ \
            /* float32 form, stays 0).  At most a quarter of the pairs within reach: every lane files its own     */ \
            if (__builtin_amdgcn_ballot_w64(__builtin_popcountll(cm) > 16) == 0ull) {              \
              while (cm) {                                                                        \
                const int e = (int)__builtin_ctzll(cm);                                           \
                cm &= cm - 1ull;                                                                  \
                int64_t hslot, tslot;                                                             \
                map(e, lane, hslot, tslot);                                                       \
                if (hslot < a.n_heads && a.group_of[hslot] < 0)                                   \
                  atomicMin(&a.best[hslot], (unsigned long long)(uint32_t)tslot << 32);           \
              }                                                                                   \
              continue;                                                                           \
            }                                                                                     \
            /* many (a radius that spans the rows): per element one lane of each half, whose 32 lanes hold one  */ \
            /* head row and pivots in ascending order, files it, and only if nothing lower is there yet (N =    */ \
            /* 20,000, d = 512, one group: 5.9 -> 0.36 ms for the rounds, which atomics on one row bounded)     */ \
            _Pragma("unroll 1") for (int e = 0; e < 64; ++e) {                                    \
              const bool in = (cm >> e) & 1ull;                                                   \
              const unsigned long long b = __builtin_amdgcn_ballot_w64(in);                       \
              if (b == 0ull) continue;                                                            \
              const uint32_t half = (uint32_t)(lane < 32 ? b : b >> 32);                          \
              if (in && (lane & 31) == __builtin_ctz(half)) {                                     \
                int64_t hslot, tslot;                                                             \
                map(e, lane, hslot, tslot);                                                       \
                const unsigned long long v64 = (unsigned long long)(uint32_t)tslot << 32;         \
                if (hslot < a.n_heads && a.group_of[hslot] < 0 &&                                 \
                    __hip_atomic_load(&a.best[hslot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > v64) \
                  atomicMin(&a.best[hslot], v64);                                                 \
              }                                                                                   \
            }                                                                                     \
          }                                                                                       \
        }                                                                                         \
      }                                                                                           \
      ck = 0;                                                                                     \
      ++ct;                                                                                       \
    } else {                                                                                      \
      ++ck;                                                                                       \
    }                                                                                             \
  } while (0)

  // slices i, i + 1 in flight; every step first asks for slice i + 2 (into the set slice i - 1 has left)
  KGC_GLOAD(q0);
  KGC_GLOAD(q1);
  for (int i = 0; i < total; i += 3) {
    KGC_GLOAD(q2);
    KGC_COMPUTE(q0);
    KGC_GLOAD(q0);
    if (i + 1 < total) KGC_COMPUTE(q1);
    KGC_GLOAD(q1);
    if (i + 2 < total) KGC_COMPUTE(q2);
  }
  if constexpr (EPI == kEpiNear) KGC_NEAR_OUT(a.near_all);
#undef KGC_GLOAD
#undef KGC_FRAG
#undef KGC_MFMA
#undef KGC_NEAR_OUT
#undef KGC_COMPUTE
  if (!LISTED && EPI == kEpiMinDist) {                     // (not listed: a single pass)
    for (int off = 32; off > 0; off >>= 1) run_min = fminf(run_min, __shfl_xor(run_min, off, 64));
    if (lane == 0) atomicMin(a.best, (unsigned long long)__float_as_uint(fmaxf(run_min, 0.f)));   // non-negative floats order like their bits
  }
  }   // segments of the row's tile list
  if (!LISTED) break;
  }   // rows
}

// ---------------------------------------------------------------------------------------------
// Relation-factorised L2 join.  For the TransE distance of Section 4.3,
//     ||h + r - t||^2 = ||h - t||^2 + 2 r.h - 2 r.t + ||r||^2,
// and the only part that needs a d-long contraction per (h, t) pair, ||h - t||^2, does not depend on the
// relation (the observation Section 5.2 makes for the tail side, taken one step further).  One block keeps
// a head tile in LDS, forms the tile G = ||h~ - t~||^2 ONCE with the matrix pipes (plain entity rows on both
// sides, same augmented-K operands as the other forms) and keeps it in registers while it walks the relations.
// The filter asks of a pair whether G + 2 r.h <= lim_r + 2 r.t (lim_r: fact_params).  Asked pair by pair that is an
// addition and half a minimum each, and the vector pipes bound the kernel (19.6 ms of the dense N = 15,000, R = 1,345
// join at 88 % of the plain vector rate).  Rounding is monotonic, so a set of pairs of one relation is decided at once:
//     min G + min 2 r.h  >  lim_r + max 2 r.t   over the set   =>   none of its pairs passes.
// (r.h and r.t are those of the bf16-rounded rows, and G is less the rows' rounding slacks.)
// A wave asks this at three levels, each over what the level before left open:
//   1. its whole TM * 32 x 64 pairs, one RELATION per lane (minima and maxima of r.e over 64 rows: k_fact_dot);
//   2. eight head rows x one tail column, one COLUMN per lane: one coalesced load of r.t, TM * 4 additions and half as
//      many minima per relation; the row minima of 2 r.h are wave-uniform and come through the scalar cache;
//   3. the pairs themselves, with the accumulators in registers, for the (relation, eight rows) still open.
// On embeddings in clusters level 1 leaves a relation open where its source cluster has a member among the head rows or
// its target cluster among the tail columns, level 2 where eight rows hold both a member of the source cluster and a
// neighbour of the tail.  The candidates are those of the pair-wise filter.
// Measured (dense joins, rows in order, kernel alone): N = 15,000, R = 1,345, d = 100: 257 us; N = 100,000, R = 200, d = 200: 3.6 ms,
// 1.15 PFLOP/s over its contraction.  What bounds it there is issue: matrix pipes 50 % and vector pipes 39 % busy (358 us and
// 4.24 ms) before the accumulators were no longer cleared (a zero operand), minima lost their canonicalising v_max, exchanges
// between lanes left the LDS, and level 1 kept what a block's tiles share in registers and the rest in flight under the
// contraction, as are the next tile's first rows; 59 % and 32 % now.  L1, 40,000, 18, 100: 611 -> 414 us; 20,011, 37, 512: 574 ->
// 374 us.
// (With one level of 32 rows in place of levels 1 and 2, in the caller's order, half of all (relation, wave) pairs on 500 clusters
// went to level 3.)
// Candidates leave through a queue per wave (in LDS, no atomics; one atomic a flush, and those on one word are served one after
// the other, about 8 ns each: up to 512 entries where the LDS has room) to a list in memory that
// k_exact_pairs scores: a wave that scored its own would wait three memory round trips for one or two pairs.
// A list that was too short is made longer by the host, which then runs the call again.
struct JoinFactArgs {
  const uint16_t* A;         // staged head operands of the plain entity rows: [KS][Nslots][32]
  const uint16_t* B;         // staged tail operands: [KS][Nslots][32]
  const float* u;            // [RBp][Nslots] r . e~ (float32, e~: the bf16-rounded row), zero rows from RB on
  const float* limr;         // [RBp] threshold on G + 2 r.h - 2 r.t, i.e. thr_r - ||r||^2
  const float* umin8;        // [Nslots / 64][RBp][8] min of 2 r.e over 8 rows
  const float* umin64;       // [Nslots / 64][RBp] min of 2 r.e over 64 rows ...
  const float* umax64;       // ... and max
  int64_t Nslots;
  int KS, k16;
  int nT;
  int r0, RB, RBp;           // RBp: rows of the per-relation tables (RB rounded up to kFactChunk)
  int zrel;                  // relations per block along grid z
  ExactEntry* list;          // candidates for k_exact_pairs
  unsigned long long* list_count;  // (may run past list_cap)
  unsigned int list_cap;
  unsigned long long give_up;      // with so many pairs listed the host takes another form: the waves end
  int queue;                 // candidates a wave holds back, kFactQueue at least
};
constexpr int kFactQueue = 64;         // candidates a wave holds back, at least: as many as the LDS has room for (JoinFactArgs::queue)
constexpr int kFactBatch = 4;          // relations whose r.t and r.h a lane has in flight together
constexpr int kFactChunks = 3;         // chunks of 64 relations whose level-1 loads are in flight together
constexpr int kFactIds = 64 + 64 * kFactChunks;      // relations that level 1 has left open and level 2 has not taken yet
inline __host__ __device__ size_t fact_wave_lds(int queue) { return (size_t)queue * 8 + kFactIds * 2; }      // (with kFactQueue, eight times this beside 19 slices of 128 rows fill the LDS)

// Per-relation filter thresholds of the factorised join: limr[rl] = thr_r - ||r||^2.  A hit x = h + r - t, ||x|| <= delta,
// has on the bf16-rounded rows x~ = h~ + r - t~ with ||x~|| <= delta + e_h + e_t (e = the distance that the rounding moves a
// row), and with products of the ROUNDED rows the expansion of ||x~||^2 is exact, so that, as in k_stage_operands,
//     (||h~ - t~||^2 - slack_h - slack_t) + 2 r.h~ - 2 r.t~ + ||r||^2 <= delta^2.
// The staged norms carry the slacks: every row pays for its own rounding, and the length of r does not enter.  (Products of
// the caller's rows left a term 2 (delta + ||r||) m, m from the largest norms: N = 1,000, R = 16, d = 32, relations 16 times
// as long as delta: 37,789 candidates where the per-relation kernel has 76, 190 us a call against 100.)
// thr_r = delta^2 + e_acc + e_u: e_acc bounds the float32 accumulation of the contraction as in k_join_params; e_u bounds the
// float32 errors of the two products, (d + 12) 2^-24 ||r|| ||e~|| each and doubled (taken twice), of ||r||^2 and of the
// final sums.
// One wave, kFactChunk relations from rl0 on: the maxima of the staged norms, ||r||^2 in float32, the thresholds.
constexpr int kFactChunk = 8;          // rows of the per-relation tables are rounded up to this
__device__ __forceinline__ void fact_params(const DevCounters* __restrict__ cnt, const void* __restrict__ Rv, int dtype, int r0, int rl0, int RB,
                                            int RBp, float delta, int d, int kp, float* __restrict__ limr) {
  if (rl0 >= RBp) return;                                              // (RBp is a multiple of kFactChunk)
  const int lane = threadIdx.x & 63;
  float ma = 0.f, mb = 0.f, rn[kFactChunk];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    ma = fmaxf(ma, __uint_as_float(cnt->max_a[i * 64 + lane]));
    mb = fmaxf(mb, __uint_as_float(cnt->max_b[i * 64 + lane]));
  }
#pragma unroll
  for (int i = 0; i < kFactChunk; ++i) rn[i] = 0.f;
  for (int k = lane; k < d; k += 64)
#pragma unroll
    for (int i = 0; i < kFactChunk; ++i) {
      const float x = ld_elem(Rv, (int64_t)(r0 + (rl0 + i < RB ? rl0 + i : RB - 1)) * d + k, dtype);
      rn[i] += x * x;
    }
  for (int off = 32; off > 0; off >>= 1) {
    ma = fmaxf(ma, __shfl_xor(ma, off, 64));
    mb = fmaxf(mb, __shfl_xor(mb, off, 64));
#pragma unroll
    for (int i = 0; i < kFactChunk; ++i) rn[i] += __shfl_xor(rn[i], off, 64);
  }
  const float na = sqrtf(ma) * 1.01f, nb = sqrtf(mb) * 1.01f;
  const float eacc = (float)(kp + 16) * 1.2e-7f * 2.f * (ma + mb);
#pragma unroll
  for (int i = 0; i < kFactChunk; ++i) {
    const float rnorm = sqrtf(rn[i]) * 1.0001f;
    const float eu = 4.f * (float)(d + 12) * 6e-8f * rnorm * (na + nb) + 2e-6f * (rn[i] + ma + mb);
    const float thr = (delta * delta + eacc + eu) * (1.f + 1e-6f);
    // nothing passes a negative threshold (nor a relation that is not there: those are not walked either); norms that leave
    // float32's range decide nothing, every pair of the relation goes to the exact stage
    float lim = thr < 1e37f && rn[i] < 1e37f ? thr - rn[i] : __builtin_inff();
    if (rl0 + i >= RB || delta < 0.f) lim = -__builtin_inff();
    if (lane == 0) limr[rl0 + i] = lim;
  }
}

// The smaller of two floats in one instruction, as the median of them and -infinity: fminf puts a canonicalising v_max before
// every operand the compiler has not seen computed, which doubles the minima over accumulators (and it turns a median with a
// constant infinity back into fminf: the empty asm hides the value).  A median with a NaN is the smallest of its numbers: a NaN
// gives -infinity here, and a set that holds one stays open; the maximum below passes over it.  That loses nothing: rows that hold
// no numbers are left out (stage_operands), so that a product r.t is a NaN only where ||r||^2 or a row's ||t||^2 is beyond
// float32 (|r.t| <= ||r|| ||t||), and then the relation's threshold, or every one, is infinite or a NaN and keeps the set open.
__device__ __forceinline__ float vmin2(float a, float b) {
  float lowest = -__builtin_inff();
  asm("" : "+s"(lowest));
  return __builtin_amdgcn_fmed3f(a, b, lowest);
}
__device__ __forceinline__ float vmax2(float a, float b) {
  float highest = __builtin_inff();
  asm("" : "+s"(highest));
  return __builtin_amdgcn_fmed3f(a, b, highest);
}
// lane l < 32: the smaller of a in lanes l and l + 32; lane l >= 32: the smaller of b in lanes l - 32 and l
__device__ __forceinline__ float min_halves(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return vmin2(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
template <int CTRL>
__device__ __forceinline__ float dpp_min(float x) {
  return vmin2(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)));
}
template <int CTRL>
__device__ __forceinline__ float dpp_max(float x) {
  return vmax2(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)));
}
// the minimum over the wave, in every lane: exchanges inside 16 lanes (quad permutes, mirrors), then between them
__device__ __forceinline__ float wave_min(float x) {
  x = dpp_min<0xB1>(x);                                    // quad_perm [1, 0, 3, 2]
  x = dpp_min<0x4E>(x);                                    // quad_perm [2, 3, 0, 1]
  x = dpp_min<0x141>(x);                                   // row_half_mirror
  x = dpp_min<0x140>(x);                                   // row_mirror
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = vmin2(__uint_as_float(s[0]), __uint_as_float(s[1]));
  return min_halves(x, x);
}

// u[rl][slot] = r . e~ for the relations of a batch and the bf16-rounded row of every slot's entity (why rounded:
// fact_params; 0 for padding slots and for rows from RB on), and the extremes of 2 r.e~ over 8 and over 64 consecutive
// slots (padding does not count), on the float32 matrix pipes: a wave takes 32 relations x 64 slots, operands straight into
// registers in the permuted order of dimensions that k_small_dot explains, every load of 64 dimensions issued before the
// first is used.  The 128 x 128 vector tile kernel that did the products before left most of the chip idle on a thin product
// (R = 2, d = 200: 60 us of latency) and needed a pass that cleared u and one that took the extremes: 204 us for the three,
// now 82 us (N = 15,000, R = 1,345, d = 100, float32 rows; 4.0 GFLOP, 81 MB written; 89 with the extremes taken through the
// LDS), N = 100,000, R = 200, d = 200: 284 -> 136 us.  One more workgroup per 32 relations makes their thresholds.
template <bool BF16, bool VEC>
__global__ __launch_bounds__(256) void k_fact_dot(const void* __restrict__ Rv, const void* __restrict__ E,
                                                  const int32_t* __restrict__ slot_ent, int64_t Nslots, int r0, int RB, int RBp,
                                                  int d, float* __restrict__ u, float* __restrict__ umin8,
                                                  float* __restrict__ umin64, float* __restrict__ umax64,
                                                  const DevCounters* __restrict__ cnt, float delta, int kp, float* __restrict__ limr) {
  if (blockIdx.x == gridDim.x - 1) {
    fact_params(cnt, Rv, BF16 ? KGC_BF16 : KGC_F32, r0, (int)blockIdx.y * 32 + (int)(threadIdx.x >> 6) * kFactChunk, RB, RBp, delta, d, kp, limr);
    return;
  }
  const int lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);         // this wave's 64 slots (Nslots is a multiple of 256)
  const int rl0 = (int)blockIdx.y * 32;
  const int64_t xo = (int64_t)(r0 + (rl0 + row < RB ? rl0 + row : RB - 1)) * d;      // (past the end: a valid row, dropped)
  int ent[2];
  int64_t yo[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    ent[j] = slot_ent[g * 64 + 32 * j + row];
    yo[j] = (int64_t)(ent[j] < 0 ? 0 : ent[j]) * d;
  }
  f32x16_t acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) acc[j] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int kG = 8;                                                   // groups of 8 dimensions per chunk
  for (int k0 = 0; k0 < d; k0 += 8 * kG) {
    f32x4_t xv[kG], yv[2][kG];
#pragma unroll
    for (int q = 0; q < kG; ++q) {
      const int k = k0 + 8 * q + 4 * half;
      xv[q] = exact_ld4<BF16, VEC>(Rv, xo, k, d);
#pragma unroll
      for (int j = 0; j < 2; ++j) yv[j][q] = exact_ld4<BF16, VEC>(E, yo[j], k, d);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < kG; ++q) {
      if (k0 + 8 * q >= d) break;                                         // the same for the whole wave
      if (!BF16) {                                                        // (as k_stage_operands rounds them)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) yv[j][q][e] = bf16_to_f32(f32_to_bf16_rne(yv[j][q][e]));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[q][e], yv[j][q][e], acc[j], 0, 0, 0);
    }
  }
  // register v of lane l holds relation 8 (v / 4) + 4 (l / 32) + v % 4, slot l % 32
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int rl = rl0 + 8 * (v >> 2) + 4 * half + (v & 3);
    float lo[2], hi[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float x = ent[j] >= 0 && rl < RB ? acc[j][v] : 0.f;
      if (rl < RBp) u[(int64_t)rl * Nslots + g * 64 + 32 * j + row] = x;
      lo[j] = ent[j] >= 0 ? 2.f * x : 3e38f;
      hi[j] = ent[j] >= 0 ? 2.f * x : -3e38f;
      lo[j] = dpp_min<0x141>(dpp_min<0x4E>(dpp_min<0xB1>(lo[j])));         // eight slots: two exchanges in a quad, one of its neighbour
      hi[j] = dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(hi[j])));
      if (rl < RBp && (lane & 7) == 0) umin8[(g * RBp + rl) * 8 + 4 * j + (row >> 3)] = lo[j];
    }
    float l = dpp_min<0x140>(vmin2(lo[0], lo[1])), h = dpp_max<0x140>(vmax2(hi[0], hi[1]));
    {   // the two sixteens of a half wave
      const auto sl = __builtin_amdgcn_permlane16_swap(__float_as_uint(l), __float_as_uint(l), false, false);
      const auto sh = __builtin_amdgcn_permlane16_swap(__float_as_uint(h), __float_as_uint(h), false, false);
      l = vmin2(__uint_as_float(sl[0]), __uint_as_float(sl[1]));
      h = vmax2(__uint_as_float(sh[0]), __uint_as_float(sh[1]));
    }
    if (rl < RBp && row == 0) { umin64[g * RBp + rl] = l; umax64[g * RBp + rl] = h; }
  }
}

// A wave-uniform read-only array of an earlier launch, read through the scalar cache whatever else the kernel stores.
typedef const __attribute__((address_space(4))) float* scalar_f32_t;
__device__ __forceinline__ scalar_f32_t scalar_f32(const float* p) { return (scalar_f32_t)(uintptr_t)p; }

// Two shapes, both with wave tiles of 128 x 64 (two LDS reads and one read through the vector cache per four MFMAs): 256 x 256
// up to KS = 9, 128 x 512 beyond, where every tail row is read by one wave.  (128 x 256 with wave tiles of 64 x 64 asked the
// vector cache for 64 bytes a cycle.)
template <int WGM, int WGN>
__global__ __launch_bounds__(WGM* WGN * 64, 1) void k_join_l2_fact(const JoinFactArgs a) {
  constexpr int TM = 4, TN = 2;                            // a wave holds 64 tail columns: one per lane in the bound
  constexpr int NT = WGM * WGN * 64;
  constexpr int WTM = TM * 32, WTN = TN * 32;
  constexpr int BM = WGM * WTM, BN = WGN * WTN;
  constexpr int LA = (BM * 4) / NT;
  constexpr int ASZ = BM * kSliceK;
  constexpr int ROWB = kSliceK * 2;
  static_assert(LA * NT == BM * 4, "tile rows must divide over the threads");
  constexpr int NG = TM * 4;                               // groups of eight head rows
  static_assert(TM % 2 == 0, "a wave's rows are whole groups of 64 slots");

  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // [KS][BM][32] head slices, then the waves' queues
  const int KS = a.KS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  constexpr int NC = kFactChunks;
  char* wlds = (char*)(lds + (size_t)KS * ASZ) + wave * fact_wave_lds(a.queue);
  uint16_t* ids = (uint16_t*)wlds;  // relations of the batch (fewer than 65,536) that level 1 left open
  uint2* q = (uint2*)(wlds + kFactIds * 2);                // candidates: relation << 16 | head row of the wave, tail slot
  int qn = 0;                                              // entries in the queue (the same in all lanes)

  const int tH = (int)blockIdx.x;
  const int t_begin = (int)(((int64_t)a.nT * blockIdx.y) / gridDim.y);
  int t_end = (int)(((int64_t)a.nT * (blockIdx.y + 1)) / gridDim.y);
  const int rl_begin = (int)blockIdx.z * a.zrel;
  // The tables' padding rows are not walked: a NaN keeps a pair open whatever the threshold (rows whose norms leave
  // float32's range), and the exact stage would read past the last relation.
  const int rl_end = rl_begin + a.zrel < a.RB ? rl_begin + a.zrel : a.RB;
  if (t_end <= t_begin || rl_end <= rl_begin) return;
  const int64_t slice_bytes = a.Nslots * ROWB;

  // ---- head tile: all K slices into LDS, once ----
  {
    const char* Abase = (const char*)a.A + (int64_t)tH * BM * ROWB;
    const uint32_t voff = (uint32_t)tid * 16u;
    const int st0 = (tid >> 2) * kSliceK + (((tid & 3) ^ lds_swizzle(tid >> 2)) * 8);
    constexpr int st_step = (NT / 4) * kSliceK;
    for (int ks = 0; ks < KS; ++ks) {
      uint4 t[LA];
#pragma unroll
      for (int i = 0; i < LA; ++i) t[i] = *(const uint4*)(Abase + (int64_t)ks * slice_bytes + voff + (uint32_t)(i * NT * 16));
#pragma unroll
      for (int i = 0; i < LA; ++i) *(uint4*)(&lds[ks * ASZ + st0 + i * st_step]) = t[i];
    }
  }
  __syncthreads();                                         // the only barrier: from here on the waves run on their own
  if (((int64_t)(t_end - 1) * BN + wn * WTN) >= a.Nslots) --t_end;      // (BN = 512: half of the last tile may not be there)
  if (t_end <= t_begin) return;

  const int rsw = lds_swizzle(lane & 31);
  const int rd_a = (wm * WTM + (lane & 31)) * kSliceK + (((lane >> 5) ^ rsw) * 8);
  const int rd_step = (((lane >> 5) ^ rsw) & 2) ? -16 : 16;
  const uint32_t boff = (uint32_t)((wn * WTN + (lane & 31)) * ROWB + (lane >> 5) * 16);
  const int last_two = (a.k16 - (KS - 1) * 2) >= 2;
  const int hrow0 = tH * BM + wm * WTM;                    // this wave's first head row
  const scalar_f32_t um8 = scalar_f32(a.umin8 + (int64_t)(hrow0 >> 6) * a.RBp * 8);
  const float* um64 = a.umin64 + (int64_t)(hrow0 >> 6) * a.RBp;
  const scalar_f32_t limr = scalar_f32(a.limr);

  // the queue's entries to the list, with one atomic; entries past its end are counted only
#define KGC_FLUSH()                                                                               \
  do {                                                                                            \
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");                                        \
    __builtin_amdgcn_wave_barrier();                                                              \
    const int fl = lane_id_here();                                                                \
    unsigned long long base = 0ull;                                                               \
    if (fl == 0) base = atomicAdd(a.list_count, (unsigned long long)qn);                          \
    base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32) | \
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);                         \
    for (int k = fl; k < qn && base + (unsigned)k < a.list_cap; k += 64) {                        \
      ExactEntry e;                                                                               \
      e.r = a.r0 + (int32_t)(q[k].x >> 16); e.hs0 = hrow0 + (int32_t)(q[k].x & 0xffffu); e.ts0 = (int32_t)q[k].y; e.pad = 0; \
      a.list[base + (unsigned)k] = e;                                                             \
    }                                                                                             \
    if (base > a.give_up) return;                                                                 \
    qn = 0;                                                                                       \
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");                                        \
    __builtin_amdgcn_wave_barrier();                                                              \
  } while (0)

  const char* pB = (const char*)a.B + (int64_t)t_begin * BN * ROWB + boff;
  bf16x8_t nb0[TN], nb1[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    nb0[j] = *(const bf16x8_t*)(pB + j * 32 * ROWB);
    nb1[j] = *(const bf16x8_t*)(pB + j * 32 * ROWB + 32);
  }
  bf16x8_t fa[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[i] = *(const bf16x8_t*)(lds + rd_a + i * 32 * kSliceK);
  // level 1's first chunks: what does not change from tile to tile
  float um_first[NC], lim_first[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int rl = rl_begin + 64 * c + lane < rl_end ? rl_begin + 64 * c + lane : rl_end - 1;
    um_first[c] = um64[rl];
    lim_first[c] = a.limr[rl];
#pragma unroll
    for (int h = 1; h < TM / 2; ++h) um_first[c] = fminf(um_first[c], um64[(int64_t)h * a.RBp + rl]);
  }
  for (int tT = t_begin; tT < t_end; ++tT) {
    // ---- G = ||h~ - t~||^2: tail fragments straight from the staged array, the next slice's in flight ----
    f32x16_t acc[TM][TN];
    const int tcol = tT * BN + wn * WTN;                                  // this wave's first tail column
    const float* ux64 = a.umax64 + (int64_t)(tcol >> 6) * a.RBp;
    float ux_first[NC];                                    // ... and what does, in flight under the contraction
#pragma unroll
    for (int c = 0; c < NC; ++c) ux_first[c] = ux64[rl_begin + 64 * c + lane < rl_end ? rl_begin + 64 * c + lane : rl_end - 1];
    // Order inside a slice, pinned by scheduling barriers: the next slice's loads first (left to itself the compiler issues
    // them behind six MFMAs), then per block row its MFMAs followed by the LDS read of that row's fragment of the next step.
    for (int ks = 0; ks < KS; ++ks) {
      const bool wrap = ks + 1 == KS, two = !wrap || last_two;
      bf16x8_t fb0[TN], fb1[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) { fb0[j] = nb0[j]; fb1[j] = nb1[j]; }
      // (the last slice asks for the next tile's first, which the bounds below then hide; the last tile's for its own)
      if (!wrap) pB += slice_bytes;
      else pB = (const char*)a.B + (int64_t)(tT + 1 < t_end ? tT + 1 : tT) * BN * ROWB + boff;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        nb0[j] = *(const bf16x8_t*)(pB + j * 32 * ROWB);
        nb1[j] = *(const bf16x8_t*)(pB + j * 32 * ROWB + 32);
      }
      __builtin_amdgcn_sched_barrier(0);
      const uint16_t* An = lds + (wrap ? 0 : (ks + 1) * ASZ) + rd_a;      // the next slice's first step (the first of all behind the last)
      const uint16_t* A1 = two ? lds + ks * ASZ + rd_a + rd_step : An;
      if (ks == 0) {                                       // (a zero operand: no register is cleared)
        const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb0[j], zero16, 0, 0, 0);
          fa[i] = *(const bf16x8_t*)(A1 + i * 32 * kSliceK);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb0[j], acc[i][j], 0, 0, 0);
          fa[i] = *(const bf16x8_t*)(A1 + i * 32 * kSliceK);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (two) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb1[j], acc[i][j], 0, 0, 0);
          fa[i] = *(const bf16x8_t*)(An + i * 32 * kSliceK);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }

    // ---- column minima of eight rows: lane l ends up with column l of the wave's 64.  MFMA 32x32 accumulator layout:
    // register v of lane l holds row 8*(v/4) + 4*(l/32) + (v%4), column l%32. ----
    float gm[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int i = g >> 2, v = (g & 3) * 4;
      float m[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) m[j] = vmin2(vmin2(acc[i][j][v], acc[i][j][v + 1]), vmin2(acc[i][j][v + 2], acc[i][j][v + 3]));
      gm[g] = min_halves(m[0], m[1]);
    }
    float gt = gm[0];
#pragma unroll
    for (int g = 1; g < NG; ++g) gt = vmin2(gt, gm[g]);
    gt = wave_min(gt);

    const float* ut0 = a.u + tcol + lane;
    const float* uh0 = a.u + hrow0 + lane;
    int cnt = 0, rb = rl_begin;
    for (;;) {
      // ---- level 1: one relation per lane, NC chunks of 64 with their loads in flight together ----
      while (rb < rl_end && cnt <= kFactIds - 64 * NC) {
        float um[NC], lm[NC], ux[NC];
        if (rb == rl_begin) {
#pragma unroll
          for (int c = 0; c < NC; ++c) { um[c] = um_first[c]; lm[c] = lim_first[c]; ux[c] = ux_first[c]; }
        } else {
          float uh[NC][TM / 2];
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int rl = rb + 64 * c + lane < rl_end ? rb + 64 * c + lane : rl_end - 1;
            ux[c] = ux64[rl];
            lm[c] = a.limr[rl];
#pragma unroll
            for (int h = 0; h < TM / 2; ++h) uh[c][h] = um64[(int64_t)h * a.RBp + rl];
          }
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            um[c] = uh[c][0];
#pragma unroll
            for (int h = 1; h < TM / 2; ++h) um[c] = fminf(um[c], uh[c][h]);
          }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (rb + 64 * c >= rl_end) break;                               // (the same for the whole wave)
          const int rl = rb + 64 * c + lane;
          const bool open = rl < rl_end && !(gt + um[c] > lm[c] + ux[c]);
          const unsigned long long b = __builtin_amdgcn_ballot_w64(open);
          if (open) ids[cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = (uint16_t)rl;
          cnt += __builtin_popcountll(b);
        }
        rb += 64 * NC;
      }
      const bool last = rb >= rl_end;
      const int take = last ? cnt : cnt / kFactBatch * kFactBatch;        // (not the last: more than a quarter full)
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
      // ---- level 2: the open relations, kFactBatch at a time, the next batch's r.t and r.h in flight ----
      int nr[kFactBatch];
      float nt[kFactBatch], nh[kFactBatch][TM / 2];
#define KGC_FACT_LOAD(e0)                                                                         \
  _Pragma("unroll") for (int k = 0; k < kFactBatch; ++k) {                                        \
    const int e = (e0) + k < take ? (e0) + k : take - 1;                                          \
    nr[k] = __builtin_amdgcn_readfirstlane((int)ids[e]);                                          \
    const int64_t uo = (int64_t)nr[k] * a.Nslots;                                                 \
    nt[k] = ut0[uo];                                                                              \
    _Pragma("unroll") for (int h = 0; h < TM / 2; ++h) nh[k][h] = uh0[uo + 64 * h];               \
  }
      if (take > 0) KGC_FACT_LOAD(0);
      for (int e0 = 0; e0 < take; e0 += kFactBatch) {
        int rk[kFactBatch];
        float ut[kFactBatch], uh[kFactBatch][TM / 2];
#pragma unroll
        for (int k = 0; k < kFactBatch; ++k) {
          rk[k] = nr[k]; ut[k] = nt[k];
#pragma unroll
          for (int h = 0; h < TM / 2; ++h) uh[k][h] = nh[k][h];
        }
        if (e0 + kFactBatch < take) KGC_FACT_LOAD(e0 + kFactBatch);
        unsigned int todo = 0u;                            // relations of the batch that level 2 leaves open
#pragma unroll
        for (int k = 0; k < kFactBatch; ++k) {
          const scalar_f32_t ug = um8 + (int64_t)rk[k] * 8;
          float m = gm[0] + ug[0];
#pragma unroll
          for (int g = 1; g < NG; ++g) m = fminf(m, gm[g] + ug[(int64_t)(g >> 3) * a.RBp * 8 + (g & 7)]);
          if (__builtin_amdgcn_ballot_w64(!(m > limr[rk[k]] + 2.f * ut[k])) != 0ull && e0 + k < take) todo |= 1u << k;
        }
        while (todo) {                                     // one body for the batch's relations: it is long
          const int k = __builtin_ctz(todo);
          todo &= todo - 1u;
          int rel = rk[0];
          float utk = ut[0], uhk[TM / 2];
#pragma unroll
          for (int h = 0; h < TM / 2; ++h) uhk[h] = uh[0][h];
#pragma unroll
          for (int kk = 1; kk < kFactBatch; ++kk)
            if (k == kk) {
              rel = rk[kk]; utk = ut[kk];
#pragma unroll
              for (int h = 0; h < TM / 2; ++h) uhk[h] = uh[kk][h];
            }
          const float lim = limr[rel] + 2.f * utk;
          float ug[NG];
#pragma unroll
          for (int g = 0; g < NG; ++g) ug[g] = um8[((int64_t)(g >> 3) * a.RBp + rel) * 8 + (g & 7)];
          // ---- level 3: the pairs of the open eights ----
          const int lq = lane_id_here();
          float limj[TN];
#pragma unroll
          for (int j = 0; j < TN; ++j) limj[j] = __shfl(lim, 32 * j + (lq & 31), 64);
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            if (__builtin_amdgcn_ballot_w64(!(gm[g] + ug[g] > lim)) == 0ull) continue;
            uint32_t cm = 0u;
#pragma unroll
            for (int v = 0; v < 4; ++v) {                  // rows 8 g + 4 (lane / 32) + v of the wave
              const float x = 2.f * __shfl(uhk[g >> 3], 8 * (g & 7) + 4 * (lq >> 5) + v, 64);
#pragma unroll
              for (int j = 0; j < TN; ++j)
                if (!(acc[g >> 2][j][4 * (g & 3) + v] + x > limj[j])) cm |= 1u << (j * 4 + v);
            }
            for (;;) {                                     // one pair per lane and round into the queue
              const unsigned long long b = __builtin_amdgcn_ballot_w64(cm != 0u);
              if (b == 0ull) break;
              const int n = __builtin_popcountll(b);
              if (qn + n > a.queue) KGC_FLUSH();
              if (cm != 0u) {
                const int e = __builtin_ctz(cm);
                const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                q[pos] = make_uint2((uint32_t)rel << 16 | (uint32_t)(8 * g + 4 * (lq >> 5) + (e & 3)), (uint32_t)(tcol + (e >> 2) * 32 + (lq & 31)));
                cm &= cm - 1u;
              }
              qn += n;
            }
          }
        }
      }
#undef KGC_FACT_LOAD
      // what did not fill a batch goes to the front
      const uint16_t rest = ids[take + lane < cnt ? take + lane : 0];
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
      if (take + lane < cnt) ids[lane] = rest;
      cnt -= take;
      if (last) break;
    }
  }
  if (qn > 0) KGC_FLUSH();
#undef KGC_FLUSH
}

// Exact scores of the pairs listed by k_join_l2_fact.  A wave takes up to 64 consecutive entries, four at a time (one per
// 16-lane group: the loads of a row are coalesced), gathers the results so that lane l speaks for entry l, and the
// workgroup's waves reserve their output records with one atomic between them per round.  Four entries are a chain of
// memory round trips, so a short list is spread over waves (64 each: N = 1,000, R = 16, 115 pairs 13 us, and
// 82 us for 1,034 pairs of 282 dimensions); more than 256 workgroups would wait on the atomics instead.
constexpr unsigned int kExactPairWaves = 1024;
__global__ __launch_bounds__(256) void k_exact_pairs(const ExactEntry* __restrict__ list, const unsigned long long* __restrict__ count,
                                                     unsigned int cap, unsigned int* __restrict__ need, const RecheckCtx cx) {
  __shared__ unsigned int wave_hits[4];
  __shared__ unsigned long long base_s;
  const unsigned int n = *count <= cap ? (unsigned int)*count : 0u;      // (a list that did not fit: the host runs the call again)
  const int lane = lane_id(), wave = (int)(threadIdx.x >> 6), grp = lane >> 4, sub = lane & 15;
  // entries a wave takes at a time: a short list is dealt to 1,024 waves, four to 64 each
  const unsigned int share = (n + kExactPairWaves * 4u - 1u) / (kExactPairWaves * 4u) * 4u;
  const unsigned int per = share < 4u ? 4u : share < 64u ? share : 64u;
  for (unsigned int e0 = blockIdx.x * 4u * per; e0 < n; e0 += gridDim.x * 4u * per) {       // the same for the whole block
    const unsigned int first = e0 + (unsigned)wave * per;
    int32_t r = 0, h = -1, t = -1;
    if ((unsigned)lane < per && first + (unsigned)lane < n) {
      const ExactEntry en = list[first + (unsigned)lane];
      r = en.r; h = cx.slot_ent[en.hs0]; t = cx.slot_ent_t[en.ts0];
      if (h < 0 || t < 0 || (cx.no_self && h == t)) h = -1;
    }
    double sum = 0.0;                                      // of entry `lane` (one root for 64 entries, not one for four)
    for (int s = 0; s < (int)(per >> 2); ++s) {
      if (first + (unsigned)s * 4u >= n) break;            // the same for the whole wave
      const int src = 4 * s + grp;
      const int32_t hs = __shfl(h, src, 64), rs = __shfl(r, src, 64), ts = __shfl(t, src, 64);
      const double g = hs >= 0 ? group16_exact_sum(cx, hs, rs, ts, sub) : 0.0;
      const double gl = __shfl(g, 16 * (lane & 3), 64);
      if ((lane >> 2) == s) sum = gl;
    }
    const double dist = cx.p == 2 ? sqrt(sum) : sum;
    const bool hit = h >= 0 && dist <= cx.delta;
    const float distf = (float)dist;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(hit);
    if (lane == 0) wave_hits[wave] = (unsigned int)__builtin_popcountll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
      const unsigned int total = wave_hits[0] + wave_hits[1] + wave_hits[2] + wave_hits[3];
      base_s = total ? atomicAdd(cx.hit_counter, (unsigned long long)total) : 0ull;
    }
    __syncthreads();
    unsigned long long pos = base_s;
    for (int w = 0; w < wave; ++w) pos += wave_hits[w];
    pos += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (hit && pos < cx.cap) {
      kgc_triple rec;
      rec.h = h; rec.r = r; rec.t = t; rec.dist = distf;
      cx.out[pos] = rec;
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && *count) {
    atomicAdd(cx.cand_counter, (unsigned long long)n);
    atomicMax(need, *count < 0xffffffffull ? (unsigned int)*count : 0xffffffffu);
  }
}

// ---------------------------------------------------------------------------------------------
// Top-1 search (the smallest triple distance, Section 3.3).  Three small kernels around the join:
//   k_top1_sample  exact distances of `n` pseudo-random triples (one per 16-lane group), minimum by atomicMin
//                  on the bits of the non-negative double: an upper bound of the top-1 distance to start from;
//   k_top1_min     over the records a join returned: pass 0 the minimum of (distance bits << 32 | r), pass 1,
//                  among the records that attain it, the minimum of (h << 32 | t);
//   k_top1_exact   the double-precision distance of the chosen triple.
struct Top1State {
  unsigned long long sample_min;   // bits of a double
  unsigned long long key_dr;       // (float distance bits << 32) | r
  unsigned long long key_ht;       // (h << 32) | t
  double dist;                     // exact distance of (key_ht, r of key_dr)
  unsigned long long sub_min;      // float bits of the smallest squared distance the sub-sampled dense pass saw
  double sub_bound;                // the distance bound that follows from it
};

__device__ __forceinline__ uint32_t top1_hash(uint32_t x) {
  x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
  return x;
}

// The minimum is taken per wave first: with one atomic per sample the 65,536 on one word were the kernel's time (190 us).
__global__ __launch_bounds__(256) void k_top1_sample(RecheckCtx cx, int64_t N, int r_begin, int R, int n, int no_self,
                                                     Top1State* st, double* all = nullptr) {
  const int sub = threadIdx.x & 15;
  unsigned long long best = ~0ull;                        // bits of non-negative doubles order like the numbers
  for (int64_t g = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4; g < n; g += ((int64_t)gridDim.x * blockDim.x) >> 4) {
    const uint32_t a = top1_hash((uint32_t)g * 3u + 1u), b = top1_hash((uint32_t)g * 3u + 2u), c = top1_hash((uint32_t)g * 3u + 3u);
    const int32_t h = (int32_t)(((uint64_t)a * (uint64_t)N) >> 32);
    int32_t t = (int32_t)(((uint64_t)b * (uint64_t)N) >> 32);
    const int32_t r = r_begin + (int32_t)(((uint64_t)c * (uint64_t)R) >> 32);      // R relations from r_begin on
    if (no_self && t == h) t = (t + 1 == N) ? 0 : t + 1;  // N >= 2 is checked on the host
    const double dist = group16_exact_dist(cx, h, r, t, sub);      // (all 16 lanes of a group run the same rounds)
    const unsigned long long bits = (unsigned long long)__double_as_longlong(dist);
    best = bits < best ? bits : best;
    if (all && sub == 0) all[g] = dist;                   // top-k: the sample stays on the device until it is asked for
  }
  for (int off = 16; off < 64; off <<= 1) {
    const unsigned long long o = (unsigned long long)__shfl_xor((long long)best, off, 64);
    best = o < best ? o : best;
  }
  if ((threadIdx.x & 63) == 0 && best != ~0ull) atomicMin(&st->sample_min, best);
}

// How many of kSampleTriples random triples lie within cx.delta, counted by workgroup: one triple per 16-lane group and step.
static_assert(sizeof(DevCounters::sample) == 256 * 4, "a word per workgroup");
constexpr int kSampleBlocks = 256, kSampleSteps = 4, kSampleTriples = kSampleBlocks * 16 * kSampleSteps;      // (a step is two memory round trips)
__global__ __launch_bounds__(256) void k_sample_close(RecheckCtx cx, int64_t N, int r_begin, int R, unsigned int* __restrict__ counts) {
  __shared__ unsigned int n_s;
  if (threadIdx.x == 0) n_s = 0;
  __syncthreads();
  const int sub = threadIdx.x & 15, grp = threadIdx.x >> 4;
  unsigned int n = 0;
  for (int i = 0; i < kSampleSteps; ++i) {
    const uint32_t k = ((uint32_t)blockIdx.x * kSampleSteps + (uint32_t)i) * 16u + (uint32_t)grp;
    const int32_t h = (int32_t)(((uint64_t)top1_hash(k * 3u + 1u) * (uint64_t)N) >> 32);
    const int32_t t = (int32_t)(((uint64_t)top1_hash(k * 3u + 2u) * (uint64_t)N) >> 32);
    const int32_t r = r_begin + (int32_t)(((uint64_t)top1_hash(k * 3u + 3u) * (uint64_t)R) >> 32);
    if (group16_exact_dist(cx, h, r, t, sub) <= cx.delta) ++n;
  }
  if (sub == 0 && n) atomicAdd(&n_s, n);
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = n_s;
}

__global__ __launch_bounds__(256) void k_top1_min(const kgc_triple* __restrict__ rec, const unsigned long long* __restrict__ count,
                                                  unsigned long long cap, int pass, Top1State* st) {
  const unsigned long long n = *count < cap ? *count : cap;
  unsigned long long best = ~0ull;
  const unsigned long long want = st->key_dr;           // pass 1: written by pass 0, an earlier launch
  for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (unsigned long long)gridDim.x * blockDim.x) {
    const kgc_triple x = rec[i];
    const unsigned long long kdr = ((unsigned long long)__float_as_uint(x.dist) << 32) | (uint32_t)x.r;
    if (pass == 0) best = kdr < best ? kdr : best;
    else if (kdr == want) {
      const unsigned long long kht = ((unsigned long long)(uint32_t)x.h << 32) | (uint32_t)x.t;
      best = kht < best ? kht : best;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)(best & 0xffffffffull), off, 64);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(best >> 32), off, 64);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    best = o < best ? o : best;
  }
  if ((threadIdx.x & 63) == 0 && best != ~0ull) atomicMin(pass == 0 ? &st->key_dr : &st->key_ht, best);
}

// Disjoint head and tail samples for the sub-sampled dense pass: 2 m entities evenly spread over [0, N),
// even positions to the heads, odd positions to the tails (so the pass scores no self pair); N >= 2 m.
__global__ void k_top1_pick(int64_t N, int m, int32_t* heads, int32_t* tails) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= m) return;
  heads[i] = (int32_t)(((int64_t)(2 * i) * N) / (2 * (int64_t)m));
  tails[i] = (int32_t)(((int64_t)(2 * i + 1) * N) / (2 * (int64_t)m));
}

// The smallest squared distance of the sub-sampled pass is taken on bf16-rounded rows with float32
// accumulation; the true distance of that pair is at most sqrt(D + e_acc) + m (same m and e_acc as the join's
// filter threshold, see k_join_params), which bounds the top-1 distance from above.
__global__ __launch_bounds__(64) void k_top1_bound(const DevCounters* cnt, int dtype, int kp, Top1State* st) {
  float ma = 0.f, mb = 0.f;
  for (int i = threadIdx.x; i < 1024; i += 64) {
    ma = fmaxf(ma, __uint_as_float(cnt->max_a[i]));
    mb = fmaxf(mb, __uint_as_float(cnt->max_b[i]));
  }
  for (int off = 32; off > 0; off >>= 1) {
    ma = fmaxf(ma, __shfl_xor(ma, off, 64));
    mb = fmaxf(mb, __shfl_xor(mb, off, 64));
  }
  if (threadIdx.x != 0) return;
  const float D = __uint_as_float((uint32_t)st->sub_min);
  const float u = 1.01f / 256.f;
  const float m = u * (sqrtf(ma) * 1.01f + (dtype == KGC_BF16 ? 0.f : sqrtf(mb) * 1.01f));
  const float eacc = (float)(kp + 16) * 1.2e-7f * 2.f * (ma + mb);
  st->sub_bound = ((double)sqrtf(D + eacc) + (double)m) * (1.0 + 1e-5);
}

// ---- top-k: the k smallest of the n records a join returned, by radix select on the float bits of the
// distance (non-negative floats order like their bits), 8 bits per pass from the top.  State on the device:
//   prefix / mask  the bits fixed so far;  need  how many records are still wanted among those that match.
struct TopkState {
  unsigned int hist[256];
  unsigned int prefix, mask;
  unsigned long long need;        // records still to take among the keys that match the prefix
  unsigned long long taken_less;  // emit: records with a smaller key written so far
  unsigned long long taken_eq;    // emit: records with the k-th key written so far
};

__global__ void k_topk_init(TopkState* ts, unsigned long long k) {
  const int i = threadIdx.x;
  if (i < 256) ts->hist[i] = 0u;
  if (i == 0) { ts->prefix = 0u; ts->mask = 0u; ts->need = k; ts->taken_less = 0ull; ts->taken_eq = 0ull; }
}

__global__ __launch_bounds__(256) void k_topk_hist(const kgc_triple* __restrict__ rec, const unsigned long long* __restrict__ count,
                                                   unsigned long long cap, int shift, TopkState* ts) {
  __shared__ unsigned int h[256];
  h[threadIdx.x] = 0u;
  __syncthreads();
  const unsigned long long n = *count < cap ? *count : cap;
  const unsigned int prefix = ts->prefix, mask = ts->mask;
  for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (unsigned long long)gridDim.x * blockDim.x) {
    const unsigned int key = __float_as_uint(rec[i].dist);
    if ((key & mask) == prefix) atomicAdd(&h[(key >> shift) & 255u], 1u);
  }
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&ts->hist[threadIdx.x], h[threadIdx.x]);
}

// which digit holds the need-th record among the matching keys (one workgroup, one digit per thread: a prefix sum);
// fix it and clear the histogram
__global__ __launch_bounds__(256) void k_topk_digit(int shift, TopkState* ts) {
  __shared__ unsigned int incl[256];
  const int b = threadIdx.x;
  const unsigned int c = ts->hist[b];
  const unsigned long long need = ts->need;
  incl[b] = c;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const unsigned int v = b >= off ? incl[b - off] : 0u;
    __syncthreads();
    incl[b] += v;
    __syncthreads();
  }
  const unsigned long long hi = incl[b], lo = hi - c;
  const bool none = b == 255 && hi < need;                // fewer records than asked for: the last digit, all of them counted
  if ((lo < need && hi >= need) || none) {                // one thread (need > 0)
    ts->need = need - (none ? hi : lo);                   // still wanted inside the chosen digit
    ts->prefix |= (unsigned int)b << shift;
    ts->mask |= 255u << shift;
  }
  ts->hist[b] = 0u;
}

// after four passes prefix is the k-th smallest key T and need the number of records with key == T to take:
// every record below T goes out, and the first `need` of those at T that get there
__global__ __launch_bounds__(256) void k_topk_emit(const kgc_triple* __restrict__ rec, const unsigned long long* __restrict__ count,
                                                   unsigned long long cap, unsigned long long k, TopkState* ts,
                                                   kgc_triple* __restrict__ out) {
  const unsigned long long n = *count < cap ? *count : cap;
  const unsigned int T = ts->prefix;
  const unsigned long long need_eq = ts->need;
  const unsigned long long n_less = (n < k ? n : k) - (need_eq < (n < k ? n : k) ? need_eq : (n < k ? n : k));
  for (unsigned long long i = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (unsigned long long)gridDim.x * blockDim.x) {
    const kgc_triple x = rec[i];
    const unsigned int key = __float_as_uint(x.dist);
    if (n <= k) { out[i] = x; continue; }                 // fewer records than asked for: all of them
    if (key < T) out[atomicAdd(&ts->taken_less, 1ull)] = x;
    else if (key == T) {
      const unsigned long long j = atomicAdd(&ts->taken_eq, 1ull);
      if (j < need_eq) out[n_less + j] = x;
    }
  }
}

__global__ __launch_bounds__(64) void k_top1_exact(RecheckCtx cx, Top1State* st) {
  const int sub = threadIdx.x & 15;
  const int32_t r = (int32_t)(uint32_t)(st->key_dr & 0xffffffffull);
  const int32_t h = (int32_t)(uint32_t)(st->key_ht >> 32), t = (int32_t)(uint32_t)(st->key_ht & 0xffffffffull);
  const double dist = group16_exact_dist(cx, h, r, t, sub);
  if (threadIdx.x == 0) st->dist = dist;
}

// ---------------------------------------------------------------------------------------------
struct JoinL1Args {
  const JoinParams* prm;
  int64_t Nslots;
  int nH, nT;
  int r0, RB;
  const uint32_t* row_start;   // NULL: dense (one block per tile, grid = (nT, nH, RB)); else see JoinStreamArgs
  const uint32_t* row_count;
  const uint32_t* cols;
  const uint32_t* active_rows;
  const unsigned int* n_active;
  const unsigned int* block_count; const unsigned long long* tile_total; unsigned int block_most;      // not NULL: a batch that l1_by_blocks sends to k_l1_blocks is left alone
  RecheckCtx cx;
};
// A pruned batch goes by 32 x 32 blocks where the bound leaves at most six of a tile's sixteen (a block of its own costs twice
// its share of a tile: four times the rows to load for a pair), or where there are so few that whole tiles would leave the chip
// idle, and never where there are more than their list may hold (`most`).
constexpr unsigned int kL1FewBlocks = 16384;
__device__ __forceinline__ unsigned int l1_block_line(const unsigned long long* tiles, unsigned int most) {
  const unsigned long long line = 6ull * *tiles > kL1FewBlocks ? 6ull * *tiles : kL1FewBlocks;
  return line < most ? (unsigned int)line : most;
}
__device__ __forceinline__ bool l1_by_blocks(const unsigned int* blocks, const unsigned long long* tiles, unsigned int most) {
  return *blocks <= l1_block_line(tiles, most);
}

// Kernel 3.  One block of 256 threads scores 128 x 128 tiles of (heads, tails) for one relation in
// float32 vector arithmetic only: acc += |(h_k + r_k) - t_k| (Section 4.3's dist for p = 1).  A tile is
// staged through LDS in 16-dimension slices, dimension-major, a = h + r formed while staging; each
// thread keeps an 8 x 8 block of sums in registers (two 4-row groups x two 4-column groups).  In pruned
// mode the block walks the surviving tail tiles of its (relation, head tile) row.
// The kernel is bound by the vector units (two operations per pair and dimension), so dimensions are left out where they
// decide nothing (padding rows stand far from all others: as copies of row 0 they were 23 of 24 M candidates of a
// structured-embedding join, all of them re-scored for nothing): terms are >= 0 and rounding is monotonic, a sum that has passed the threshold stays above it.  After
// every slice a wave takes the minimum of each lane's 64 sums (32 operations against the slice's 2,048); once at most
// kL1Early pairs of its 4,096 are still at or below the threshold, they are its candidates -- a superset of those that
// the full sum would leave, decided in double -- and the wave only helps to stage.  A tile ends with its last wave.
// N = 20,000, R = 18, d = 100, every pair: 8.4 ms (clusters of spread 0.1) and 20 ms (0.7), where all sums to the end are
// 37 ms at the plain vector rate; structured embedding, N = 15,000, R = 64, pruned: 4.35 -> 1.95 ms (mostly the padding).
constexpr int kL1Tile = 128;
constexpr int kL1K = 16;
constexpr int kL1Early = 8;        // open pairs of a wave that go to the exact stage before the last dimension
template <bool BF16, bool VEC>
__global__ __launch_bounds__(256, 3) void k_join_l1(const JoinL1Args a) {
  constexpr int BM = kL1Tile, BN = kL1Tile, BK = kL1K;
  __shared__ __attribute__((aligned(16))) float As[BK][BM];
  __shared__ __attribute__((aligned(16))) float Bs[BK][BN];
  __shared__ int32_t hent[BM], tent[BN];
  __shared__ BlockQueue queue;
  __shared__ uint32_t decided[2][4];      // per slice (alternating) and wave: the wave's candidates are known
  if (a.block_count && l1_by_blocks(a.block_count, a.tile_total, a.block_most)) return;

  const int tid = threadIdx.x, wave = tid >> 6;
  if (tid == 0) { queue.count = 0u; queue.pending = 0u; queue.flag = 0u; queue.nhits = 0u; }   // published by the first barrier
  for (unsigned int row_i = blockIdx.x;; row_i += gridDim.x) {
  int tH, rl, t_begin, t_end;
  const uint32_t* cols = nullptr;
  if (a.row_start) {
    if (row_i >= *a.n_active) break;
    const int64_t row = (int64_t)a.active_rows[row_i];
    rl = (int)(row / a.nH); tH = (int)(row - (int64_t)rl * a.nH);
    t_begin = (int)a.row_start[row]; t_end = t_begin + (int)a.row_count[row];
    cols = a.cols;
    __syncthreads();                      // the previous row is done with hent
  } else {
    t_begin = (int)blockIdx.x; t_end = t_begin + 1; tH = (int)blockIdx.y; rl = (int)blockIdx.z;
  }
  if (t_end <= t_begin) break;
  const int r = a.r0 + rl;
  const int d = a.cx.d;
  const float thr = a.prm->thr;
  const int tx = tid & 15, ty = tid >> 4;
  // staging assignment: thread -> (row = tid / 2, eight dimensions starting at (tid % 2) * 8)
  const int srow = tid >> 1, sk0 = (tid & 1) * 8;
  const int64_t ro = (int64_t)r * a.cx.rstride;
  if (tid < BM) hent[tid] = a.cx.slot_ent[(int64_t)tH * BM + tid];

#pragma unroll 1
  for (int ti = t_begin; ti < t_end; ++ti) {
    const int tT = cols ? (int)cols[ti] : ti;
    __syncthreads();                        // previous tile done with tent / As / Bs
    if (tid >= BM) tent[tid - BM] = a.cx.slot_ent_t[(int64_t)tT * BN + (tid - BM)];
    __syncthreads();
    float acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
    const int he = hent[srow], te = tent[srow];
    const int64_t ho = (int64_t)r * a.cx.hstride + (int64_t)(he < 0 ? 0 : he) * d,
                  to = (int64_t)r * a.cx.tstride + (int64_t)(te < 0 ? 0 : te) * d;

    unsigned long long cm[1] = {0ull};
    bool done = false;                      // the same for the whole wave
    int par = 0;
    f32x4_t xh[2], xr[2], xt[2];            // a slice's elements of this thread: head, relation, tail
#define KGC_L1_LOAD(k0)                                                     \
  _Pragma("unroll") for (int q = 0; q < 2; ++q) {                           \
    const int k = (k0) + sk0 + 4 * q;                                       \
    xh[q] = exact_ld4<BF16, VEC>(a.cx.E, ho, k, d);                         \
    xr[q] = exact_ld4<BF16, VEC>(a.cx.Rv, ro, k, d);                        \
    xt[q] = exact_ld4<BF16, VEC>(a.cx.Et, to, k, d);                        \
  }
    KGC_L1_LOAD(0);
#pragma unroll 1
    for (int k0 = 0; k0 < d; k0 += BK, par ^= 1) {
      __syncthreads();                      // previous slice fully consumed
      if (k0 > 0 && (decided[par ^ 1][0] & decided[par ^ 1][1] & decided[par ^ 1][2] & decided[par ^ 1][3])) break;   // (the same for the whole block)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        As[sk0 + q][srow] = he < 0 ? 1e38f : xh[q >> 2][q & 3] + xr[q >> 2][q & 3];
        Bs[sk0 + q][srow] = te < 0 ? -1e38f : xt[q >> 2][q & 3];
      }
      __syncthreads();
      if (k0 + BK < d) { KGC_L1_LOAD(k0 + BK); }      // the next slice, in flight while this one is summed
      if (!done) {
#pragma unroll
        for (int k = 0; k < BK; ++k) {
          const float4 a0 = *(const float4*)(&As[k][ty * 4]);
          const float4 a1 = *(const float4*)(&As[k][64 + ty * 4]);
          const float4 b0 = *(const float4*)(&Bs[k][tx * 4]);
          const float4 b1 = *(const float4*)(&Bs[k][64 + tx * 4]);
          const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
          const float bv[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] += fabsf(av[i] - bv[j]);
        }
        // (the minimum passes over a NaN, whose pair is no candidate either)
        float m = acc[0][0];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 8; ++j) m = fminf(m, acc[i][j]);
        const unsigned long long open = __builtin_amdgcn_ballot_w64(m <= thr);
        const bool last = k0 + BK >= d;
        done = open == 0ull || last;
        if (open != 0ull && (last || __builtin_popcountll(open) <= kL1Early)) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (acc[i][j] <= thr) cm[0] |= 1ull << (i * 8 + j);
          if (!last) {                      // several pairs of one lane count one by one
            int n = __builtin_popcountll(cm[0]);
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) n += __shfl_xor(n, off, 64);
            done = n <= kL1Early;
            if (!done) cm[0] = 0ull;
          }
        }
      }
      if ((tid & 63) == 0) decided[par][wave] = done ? 1u : 0u;
    }
#undef KGC_L1_LOAD

    // the exact path is entered by the whole block or not at all
    if (__builtin_amdgcn_ballot_w64(cm[0] != 0ull) != 0ull && (tid & 63) == 0) queue.flag = 1u;
    __syncthreads();
    if (queue.flag) {
      const int64_t hbase = (int64_t)tH * BM, tbase = (int64_t)tT * BN;
      block_recheck<4, 1, 1>(cm, r, a.cx, &queue, [=](int e, int src, int64_t& hslot, int64_t& tslot) {
        const int stid = wave * 64 + src;
        const int sx = stid & 15, sy = stid >> 4;
        const int i = e >> 3, j = e & 7;
        hslot = hbase + (i >> 2) * 64 + sy * 4 + (i & 3);
        tslot = tbase + (j >> 2) * 64 + sx * 4 + (j & 3);
      });
    }
  }
  if (!a.row_start) break;
  }   // rows
}

// ---------------------------------------------------------------------------------------------
// Pruned L1 joins by pairs of micro-tiles.  A surviving 128 x 128 tile of small groups holds a few 32 x 32 blocks that the
// bound lets through among sixteen, and k_join_l1 sums all of it, one workgroup per row of tiles: the structured-embedding
// join of N = 15,000, R = 64 spent 1.9 ms there, N = 40,000, R = 18, whose 105 tiles are fewer than compute units, 200 us.
// Here the bound is asked again for the sixteen pairs of every surviving tile (k_l1_micro_pairs), the blocks it leaves are
// listed and dealt to waves (k_l1_blocks), and the pairs within the filter's threshold go to k_exact_pairs: 46 + 392 + 189 us and 8 + 27 + 13 us.
// One wave per listed 32 x 32 block: rows staged 16 dimensions at a time into the wave's own LDS, 4 x 4 sums per lane; a block
// ends when every sum has passed the threshold (terms are >= 0).  Bound by the vector units, two operations per pair and
// dimension.  Candidates leave through a queue per wave.
constexpr int kL1PairQueue = 256;
constexpr int kL1BlockStride = 36;     // floats per dimension in LDS: 16-byte rows, and the two halves of a row's dimensions on different banks
template <bool BF16, bool VEC>
__global__ __launch_bounds__(256) void k_l1_blocks(const ExactEntry* __restrict__ list, const unsigned int* __restrict__ count, unsigned int cap,
                                                   const unsigned long long* __restrict__ tiles, unsigned int most, unsigned int* __restrict__ need,
                                                   unsigned long long* __restrict__ total, const JoinParams* __restrict__ prm, const RecheckCtx cx,
                                                   ExactEntry* __restrict__ pairs, unsigned long long* __restrict__ pair_count,
                                                   unsigned int pair_cap) {
  __shared__ __attribute__((aligned(16))) float stage[4][2][kL1K * kL1BlockStride];
  __shared__ int32_t queue[4][3][kL1PairQueue];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  float* const As = stage[wave][0];
  float* const Bs = stage[wave][1];
  int32_t (&q)[3][kL1PairQueue] = queue[wave];
  int qn = 0;
  auto flush = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    unsigned long long base = 0ull;
    if (lane == 0) base = atomicAdd(pair_count, (unsigned long long)qn);
    base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);
    for (int k = lane; k < qn && base + (unsigned)k < pair_cap; k += 64) pairs[base + (unsigned)k] = ExactEntry{q[0][k], q[1][k], q[2][k], 0};
    qn = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  };
  if (!l1_by_blocks(count, tiles, most)) return;
  const unsigned int n = *count <= cap ? *count : 0u;      // (a list that did not fit: the host makes it longer and runs the call again)
  if (blockIdx.x == 0 && threadIdx.x == 0 && *count) { atomicMax(need, *count); *total += n; }
  const float thr = prm->thr;
  const int d = cx.d;
  const int row = lane >> 1, sk0 = (lane & 1) * 8, ly = lane >> 3, lx = lane & 7;
  for (unsigned int e = blockIdx.x * 4u + (unsigned)wave; e < n; e += gridDim.x * 4u) {
    const ExactEntry en = list[e];
    const int r = __builtin_amdgcn_readfirstlane(en.r), hs0 = __builtin_amdgcn_readfirstlane(en.hs0), ts0 = __builtin_amdgcn_readfirstlane(en.ts0);
    const int he = cx.slot_ent[hs0 + row], te = cx.slot_ent_t[ts0 + row];
    const int64_t ho = (int64_t)r * cx.hstride + (int64_t)(he < 0 ? 0 : he) * d, to = (int64_t)r * cx.tstride + (int64_t)(te < 0 ? 0 : te) * d,
                  ro = (int64_t)r * cx.rstride;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
    f32x4_t xh[2], xr[2], xt[2];
#define KGC_L1_LOAD(k0)                                                     \
  _Pragma("unroll") for (int g = 0; g < 2; ++g) {                           \
    const int k = (k0) + sk0 + 4 * g;                                       \
    xh[g] = exact_ld4<BF16, VEC>(cx.E, ho, k, d);                           \
    xr[g] = exact_ld4<BF16, VEC>(cx.Rv, ro, k, d);                          \
    xt[g] = exact_ld4<BF16, VEC>(cx.Et, to, k, d);                          \
  }
    KGC_L1_LOAD(0);
    bool open = true;                  // the same for the whole wave
    for (int k0 = 0; k0 < d && open; k0 += kL1K) {
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");       // the previous slice is consumed (a wave's LDS operations complete in order)
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        As[(sk0 + g) * kL1BlockStride + row] = he < 0 ? 1e38f : xh[g >> 2][g & 3] + xr[g >> 2][g & 3];
        Bs[(sk0 + g) * kL1BlockStride + row] = te < 0 ? -1e38f : xt[g >> 2][g & 3];
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
      if (k0 + kL1K < d) { KGC_L1_LOAD(k0 + kL1K); }
#pragma unroll
      for (int k = 0; k < kL1K; ++k) {
        const float4 av = *(const float4*)(As + k * kL1BlockStride + ly * 4);
        const float4 bv = *(const float4*)(Bs + k * kL1BlockStride + lx * 4);
        const float x[4] = {av.x, av.y, av.z, av.w}, y[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] += fabsf(x[i] - y[j]);
      }
      float m = acc[0][0];             // (passes over a NaN, whose pair is no candidate either)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) m = fminf(m, acc[i][j]);
      open = __builtin_amdgcn_ballot_w64(m <= thr) != 0ull;
    }
#undef KGC_L1_LOAD
    if (!open) continue;
    uint32_t cm = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (acc[i][j] <= thr) cm |= 1u << (i * 4 + j);
    for (;;) {                         // one pair per lane and round into the queue
      const unsigned long long b = __builtin_amdgcn_ballot_w64(cm != 0u);
      if (b == 0ull) break;
      const int m = __builtin_popcountll(b);
      if (qn + m > kL1PairQueue) flush();
      if (cm != 0u) {
        const int c = __builtin_ctz(cm);
        const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
        q[0][pos] = r; q[1][pos] = hs0 + ly * 4 + (c >> 2); q[2][pos] = ts0 + lx * 4 + (c & 3);
        cm &= cm - 1u;
      }
      qn += m;
    }
  }
  if (qn > 0) flush();
}

}  // namespace kgc
