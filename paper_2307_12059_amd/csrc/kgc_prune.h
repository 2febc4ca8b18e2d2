// Block-level pruning for the TransE completion join (gfx950).
//
// The paper filters pairs with one pivot p: dist(a, b) >= |dist(p, a) - dist(p, b)| (Lemma 1, Section 4.4)
// and turns that into index ranges over pivot-sorted lists (Lemma 2).  On embeddings whose norms
// concentrate, the single zero pivot of Section 4.5 separates little, so this build applies the same
// triangle-inequality argument with LOCAL pivots: entities are grouped around pivot entities, stored
// group by group, and every 32-row micro-tile m gets a centre c_m and a radius rho_m >= dist(e, c_m)
// for its rows.  For a = h + r with h in micro-tile H and b = t in micro-tile T,
//     dist(a, b) >= dist(c_H + r, c_T) - rho_H - rho_T          (triangle inequality, twice)
// so the pair of micro-tiles is skipped when that bound exceeds delta.  A join tile is evaluated iff one
// of its micro-tile pairs survives.  All of it is done in the metric of the join (L1 or L2); bounds are
// computed in float32 and widened by a relative slack so that rounding can only keep more, never drop.
#pragma once
#include "kgc_device.h"

namespace kgc {

constexpr int kMicro = 32;                 // rows per micro-tile (the MFMA tile height)
constexpr int kGroupRounds = 6;            // covering rounds
constexpr int kPivotsPerRound = 4096;      // pivots drawn from the uncovered entities per round
constexpr int kMaxGroups = kGroupRounds * kPivotsPerRound;
constexpr int kSmallGroup = 16;            // smaller groups are packed, unpadded, into the tail region
constexpr float kBoundSlack = 2e-4f;       // relative widening of float32 distance sums (d <= 960 terms)

struct GroupState {
  int32_t n_unc;        // uncovered entities in the current list
  int32_t n_unc_next[2]; // ... appended to the next list, by the round's parity (a round's start reads the count the
                        // round before left and clears its own)
  int32_t n_piv;        // pivots of the current round
  int32_t n_groups;     // groups formed so far
  int32_t n_slots;      // rows after layout, multiple of the slot alignment
  int32_t tail_base;    // first slot of the unpadded tail region
  int32_t tail_fill;    // running count of rows placed in the tail region
  int32_t n_big;        // groups of at least kSmallGroup rows: each is one unit of the two-level bound test
  int32_t max_unit;     // micro-tiles of the largest of them
};

// Start of a round: pivots are an even-stride sample (one in 2^shift, at most kPivotsPerRound) of the
// uncovered list; nearest-pivot records are reset.
// `best` is indexed by the position in the uncovered list, or (by_entity) by the entity itself; the pivot
// list is padded with -1 up to kPivotsPerRound (the grid covers max(N, kPivotsPerRound) threads).
// The first round (init_N > 0) also sets up the state: every entity uncovered and in no group.  A later round first
// closes the one before it (its pivots become groups, the entities it left uncovered are this round's list): what
// the threads read of the state is not what thread 0 writes.
__global__ void k_round_begin(GroupState* gs, int32_t* unc, int32_t* piv_ent, unsigned long long* best,
                              int shift, int by_entity, int64_t init_N, int32_t* group_of, int round) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool first = init_N > 0;
  const int n_unc = first ? (int)init_N : gs->n_unc_next[(round & 1) ^ 1];
  int n_piv = n_unc >> shift;
  n_piv = n_piv < 1 ? (n_unc > 0 ? 1 : 0) : n_piv;
  n_piv = n_piv < kPivotsPerRound ? n_piv : kPivotsPerRound;
  if (first && i < n_unc) { unc[i] = (int32_t)i; group_of[i] = -1; }
  if (i < kPivotsPerRound) {
    const int64_t pos = i < n_piv ? (int64_t)i * n_unc / n_piv : -1;   // n_piv > 0 where read
    piv_ent[i] = pos < 0 ? -1 : (first ? (int32_t)pos : unc[pos]);
  }
  if (i < n_unc) best[by_entity ? (first ? (int32_t)i : unc[i]) : i] = ~0ull;
  if (i == 0) {
    if (first) { gs->n_groups = 0; gs->n_slots = 0; gs->tail_base = 0; gs->tail_fill = 0; gs->n_big = 0; }
    else gs->n_groups += gs->n_piv;                        // the round before
    gs->n_unc = n_unc; gs->n_piv = n_piv; gs->n_unc_next[round & 1] = 0;
  }
}

// End of a round: an uncovered entity joins the group of the pivot the assignment found within tau, if any.
__global__ void k_round_commit(GroupState* gs, const int32_t* unc, const unsigned long long* best,
                               int32_t* group_of, int32_t* unc_next, int by_entity, int round) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= gs->n_unc) return;
  const int ent = unc[i];
  const unsigned long long b = best[by_entity ? ent : i];
  if (b != ~0ull) group_of[ent] = gs->n_groups + (int)(uint32_t)(b >> 32);
  else unc_next[atomicAdd(&gs->n_unc_next[round & 1], 1)] = ent;
}

// before the layout: group sizes and fill counts to zero, every slot to "padding"; the last round (number last_round)
// is closed
__global__ void k_group_clear(int32_t* gsize, int32_t* gfill, int n_groups_max, int32_t* slot_ent, int64_t n_slots,
                              GroupState* gs, int last_round) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    gs->n_groups += gs->n_piv;
    gs->n_unc = gs->n_unc_next[last_round & 1];
    gs->n_piv = 0;
  }
  if (i < n_groups_max) { gsize[i] = 0; gfill[i] = 0; }
  if (i < n_slots) slot_ent[i] = -1;
}

// counter[g] += 1 for every lane that asks, and the old value plus the lane's rank among those of the same g.  Lanes that
// share the group of the first lane still waiting go together, with one atomic, kSameGroupRounds times; the rest one by one:
// where one group holds much of the rows (N = 1,000,000, Zipf sizes, the largest 15 %) the atomics on its counter are
// served one after the other.  Two rounds take part of that away: 2.0 -> 1.6 ms each for k_group_hist and k_scatter_slots
// there, 22 -> 15 us for the latter with N = 100,000 in 2,000 groups.
constexpr int kSameGroupRounds = 2;
__device__ __forceinline__ int group_add(int32_t* counter, int g, bool want) {
  const int lane = lane_id();
  int pos = 0;
#pragma unroll 1
  for (int k = 0; k < kSameGroupRounds; ++k) {
    const unsigned long long w = __builtin_amdgcn_ballot_w64(want);
    if (w == 0ull) return pos;
    const int first = (int)__builtin_ctzll(w);
    const int gf = __shfl(g, first, 64);
    const unsigned long long m = __builtin_amdgcn_ballot_w64(want && g == gf);
    int base = 0;
    if (lane == first) base = atomicAdd(&counter[gf], (int)__builtin_popcountll(m));
    base = __shfl(base, first, 64);
    if (want && g == gf) {
      pos = base + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull));
      want = false;
    }
  }
  if (want) pos = atomicAdd(&counter[g], 1);
  return pos;
}

__global__ void k_group_hist(const int32_t* group_of, int64_t N, int32_t* gsize) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int g = i < N ? group_of[i] : -1;
  (void)group_add(gsize, g < 0 ? 0 : g, g >= 0);
}

constexpr int kTailAligned = 1024;
// Slot layout: groups of at least kSmallGroup rows start on a micro-tile boundary and are padded to one;
// all other rows follow, packed.  One block of 1024 threads: each thread owns a contiguous run of groups,
// an exclusive scan over the threads' padded sizes gives the run offsets.
// The padded groups are also numbered 0 .. n_big - 1 in slot order and their micro-tile ranges written to
// unit_first / unit_n: they are the units of the two-level bound test.
__global__ __launch_bounds__(1024) void k_group_layout(GroupState* gs, const int32_t* gsize, int32_t* goff, int64_t N,
                                                       int slot_align, int32_t* unit_first, int32_t* unit_n) {
  __shared__ int part[1024];
  __shared__ int placed_part[1024];
  __shared__ int big_part[1024];
  const int tid = threadIdx.x;
  const int G = gs->n_groups;
  const int per = (G + 1023) / 1024;
  const int g0 = tid * per, g1 = (g0 + per < G) ? g0 + per : G;
  __shared__ int largest;
  if (tid == 0) largest = 0;
  int sum = 0, placed = 0, nbig = 0, most = 0;
  for (int g = g0; g < g1; ++g) {
    const int sz = gsize[g];
    if (sz >= kSmallGroup) { sum += (sz + kMicro - 1) / kMicro * kMicro; placed += sz; ++nbig; most = sz > most ? sz : most; }
  }
  part[tid] = sum;
  placed_part[tid] = placed;
  big_part[tid] = nbig;
  __syncthreads();
  for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, 64));
  if ((tid & 63) == 0) atomicMax(&largest, most);      // (one per wave: 1,024 on one word took 3 us; read after the scan's barriers)
  for (int off = 1; off < 1024; off <<= 1) {          // inclusive scan, Hillis-Steele
    const int v = tid >= off ? part[tid - off] : 0;
    const int w = tid >= off ? placed_part[tid - off] : 0;
    const int x = tid >= off ? big_part[tid - off] : 0;
    __syncthreads();
    part[tid] += v;
    placed_part[tid] += w;
    big_part[tid] += x;
    __syncthreads();
  }
  int cur = part[tid] - sum;                           // exclusive prefix of this thread's run
  int ui = big_part[tid] - nbig;
  for (int g = g0; g < g1; ++g) {
    const int sz = gsize[g];
    if (sz >= kSmallGroup) {
      const int padded = (sz + kMicro - 1) / kMicro * kMicro;
      goff[g] = cur;
      unit_first[ui] = cur / kMicro;
      unit_n[ui] = padded / kMicro;
      ++ui;
      cur += padded;
    } else {
      goff[g] = -1;
    }
  }
  if (tid == 1023) {
    // many rows without a group: they start on a whole tile of every shape, so that the kernel that takes the pairs among
    // them (see part_pays) leaves no tile of theirs to the lists
    int total_padded = part[1023];
    if (N - placed_part[1023] >= kTailAligned) total_padded = (total_padded + slot_align - 1) / slot_align * slot_align;
    gs->n_big = big_part[1023];
    gs->max_unit = (largest + kMicro - 1) / kMicro;
    gs->tail_base = total_padded;
    gs->tail_fill = 0;
    const int64_t total = (int64_t)total_padded + (N - placed_part[1023]);
    gs->n_slots = (int32_t)((total + slot_align - 1) / slot_align * slot_align);
  }
}

__global__ void k_scatter_slots(GroupState* gs, const int32_t* group_of, const int32_t* goff, int32_t* gfill,
                                int64_t N, int32_t* slot_ent) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int g = i < N ? group_of[i] : -1;
  const int off = g >= 0 ? goff[g] : -1;
  const int in_group = group_add(gfill, off >= 0 ? g : 0, off >= 0);
  const int in_tail = group_add(&gs->tail_fill, 0, i < N && off < 0);
  if (i < N) slot_ent[off >= 0 ? off + in_group : gs->tail_base + in_tail] = (int32_t)i;
}

// ---------------------------------------------------------------------------------------------
// Row order of the relation-factorised join: rows that lie close together become neighbours, so that the sets of pairs its
// bounds are taken over (a wave's 128 x 64 pairs, eight rows x a column) hold few clusters.  Every row goes to the nearest of
// P evenly spread rows ("pivots", an eighth of the rows, 256 to 4,096), and the pivots' runs lie side by side where the
// pivots share the nearest of the first 256 pivots, which are evenly spread too: a cluster that several pivots cut into
// runs stays together.  One contraction of all rows with the pivots (k_join_l2_direct<.., kEpiNear>) finds both; nothing is
// read back and no slot is padding, so the order costs four launches.  Any order is a valid one: which pivot a row ends
// up with does not touch the result.  Measured at N = 15,000, d = 100 (1,792 pivots): begin 3, operands 6, contraction 16, sort 17 us,
// and the join kernel 4,670 -> 358 us with R = 1,345 (two thirds of its relations had been open to level 2); N = 100,000, d = 200:
// 318 us in all, join kernel 9,010 -> 4,240 us.
constexpr int kOrderPivots = 4096;
static_assert(kOrderPivots <= 1 << kNearBits, "a pivot's position must fit the low bits of a key");
// Position i of the pivot list: tile i / 256 takes every m-th of the P evenly spread rows (m tiles).
__global__ void k_order_begin(int64_t N, int P, int32_t* __restrict__ piv_ent, int32_t* __restrict__ near_all, int32_t* __restrict__ near_first) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P) {
    const int m = P / 256;
    piv_ent[i] = (int32_t)((int64_t)((i % 256) * m + i / 256) * N / P);
  }
  if (i < N) near_all[i] = near_first[i] = 0x7fffffff;
}
// the operands of that contraction in one launch: blockIdx.y = 0 all rows in the caller's order, 1 the pivots
__global__ __launch_bounds__(256, 4) void k_order_stage(const void* __restrict__ E, int dtype, int d, int64_t N, int64_t Npad, int KS,
                                                        const int32_t* __restrict__ piv_ent, int P, uint16_t* __restrict__ rows,
                                                        uint16_t* __restrict__ pivots) {
  if (blockIdx.y == 0)
    stage_operands<true, true>(E, nullptr, dtype, d, 0, 1, nullptr, Npad, KS, rows, nullptr, nullptr, nullptr, nullptr, 0, kStageRows, 0, nullptr,
                               -1.f, N);
  else      // (a pivot that is no number would be the nearest of all rows, or of none)
    stage_operands<false, true>(E, nullptr, dtype, d, 0, 1, piv_ent, P, KS, pivots, nullptr, nullptr, nullptr, nullptr, 0, kStageRows, 0, nullptr,
                                -1.f, 0);
}
// Counting sort of the rows by pivot, one workgroup: sizes of the runs, offsets (the pivots of one of the first 256 side by
// side), places.
__global__ __launch_bounds__(1024) void k_order_sort(const int32_t* __restrict__ near_all, const int32_t* __restrict__ near_first,
                                                     const int32_t* __restrict__ piv_ent, int64_t N, int64_t Nslots, int P,
                                                     int32_t* __restrict__ slot_ent) {
  __shared__ int run[kOrderPivots];
  __shared__ int area[256], wave_sum[4];
  const int tid = threadIdx.x;
  for (int p = tid; p < P; p += 1024) run[p] = 0;
  if (tid < 256) area[tid] = 0;
  __syncthreads();
  constexpr int kU = 8;                                    // rows a thread has in flight
  for (int64_t e0 = tid; e0 < N; e0 += 1024 * kU) {
    int p[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) p[q] = e0 + 1024 * q < N ? near_all[e0 + 1024 * q] & ((1 << kNearBits) - 1) : -1;
#pragma unroll
    for (int q = 0; q < kU; ++q)
      if (p[q] >= 0) atomicAdd(&run[p[q]], 1);
  }
  __syncthreads();
  int of[kOrderPivots / 1024], size[kOrderPivots / 1024], before[kOrderPivots / 1024];
#pragma unroll
  for (int q = 0; q < kOrderPivots / 1024; ++q) {
    const int p = tid + 1024 * q;
    of[q] = p < P ? near_first[piv_ent[p]] & 255 : 0;
    size[q] = p < P ? run[p] : 0;
  }
#pragma unroll
  for (int q = 0; q < kOrderPivots / 1024; ++q) before[q] = size[q] ? atomicAdd(&area[of[q]], size[q]) : 0;
  __syncthreads();
  // exclusive scan of the 256 areas by the first four waves
  int mine = 0, sum = 0;
  if (tid < 256) {
    mine = sum = area[tid];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(sum, off, 64);
      if ((tid & 63) >= off) sum += v;
    }
    if ((tid & 63) == 63) wave_sum[tid >> 6] = sum;
  }
  __syncthreads();
  if (tid < 256) {
    for (int w = 0; w < (tid >> 6); ++w) sum += wave_sum[w];
    area[tid] = sum - mine;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kOrderPivots / 1024; ++q)
    if (tid + 1024 * q < P) run[tid + 1024 * q] = area[of[q]] + before[q];
  __syncthreads();
  for (int64_t e0 = tid; e0 < N; e0 += 1024 * kU) {
    int p[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) p[q] = e0 + 1024 * q < N ? near_all[e0 + 1024 * q] & ((1 << kNearBits) - 1) : -1;
#pragma unroll
    for (int q = 0; q < kU; ++q)
      if (p[q] >= 0) slot_ent[atomicAdd(&run[p[q]], 1)] = (int32_t)(e0 + 1024 * q);
  }
  for (int64_t s = N + tid; s < Nslots; s += 1024) slot_ent[s] = -1;
}

// One wave per micro-tile: centre = mean of its rows, radius = max distance of a row to the centre (in
// the join's metric), widened for float32 rounding.  An empty micro-tile gets radius -1.
// The rows are read once, 64 dimensions at a time with the lanes on consecutive dimensions: the 32 loads of a chunk
// are independent of each other (one memory round trip), the chunk's centre values come from their sum, and each
// row's distance to the centre grows by its part of the chunk; the 32 row sums are then added across the lanes by a
// halving exchange (32 shuffles).
// With MAXL1 the largest L1 norm of a row, which the L1 filter's error bound asks for, is taken on the way (max_l1; the float32 sums
// run in another order than k_row_l1_max's: the bound they enter is widened by far more): two summaries and two passes of
// k_row_l1_max over 384 MB of connector rows each took 201 + 147 us, now 240.
__device__ __forceinline__ float micro_row_totals(const float (&rs)[kMicro], int lane) {
  // after the five halving steps lane l holds the sum of row 16 b5 + 8 b4 + 4 b3 + 2 b2 + b1 (bits of l)
  float a16[16], a8[8], a4[4], a2[2], a1;
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
#pragma unroll
  for (int i = 0; i < 16; ++i) a16[i] = (b5 ? rs[i + 16] : rs[i]) + __shfl_xor(b5 ? rs[i] : rs[i + 16], 32, 64);
#pragma unroll
  for (int i = 0; i < 8; ++i) a8[i] = (b4 ? a16[i + 8] : a16[i]) + __shfl_xor(b4 ? a16[i] : a16[i + 8], 16, 64);
#pragma unroll
  for (int i = 0; i < 4; ++i) a4[i] = (b3 ? a8[i + 4] : a8[i]) + __shfl_xor(b3 ? a8[i] : a8[i + 4], 8, 64);
#pragma unroll
  for (int i = 0; i < 2; ++i) a2[i] = (b2 ? a4[i + 2] : a4[i]) + __shfl_xor(b2 ? a4[i] : a4[i + 2], 4, 64);
  a1 = (b1 ? a2[1] : a2[0]) + __shfl_xor(b1 ? a2[0] : a2[1], 2, 64);
  return a1 + __shfl_xor(a1, 1, 64);
}
template <int P, bool MAXL1 = false>
__global__ __launch_bounds__(64) void k_micro_summary(const void* __restrict__ E, int dtype, int d,
                                                      const int32_t* __restrict__ slot_ent, int64_t n_micro,
                                                      float* __restrict__ cent, float* __restrict__ rad,
                                                      float* __restrict__ cnorm, int r0 = 0, int64_t rel_stride = 0,
                                                      unsigned int* __restrict__ max_l1 = nullptr) {
  // blockIdx.y: relation of a batch, for per-relation rows E[(r0 + y) * rel_stride + ...] (summaries then lie
  // relation after relation); one relation and rel_stride 0 for the TransE join
  static_assert(kMicro == 32, "the row sums below are laid out for 32 rows");
  const int64_t m = blockIdx.x;
  if (m >= n_micro) return;
  const int lane = threadIdx.x;
  E = (const char*)E + (int64_t)(r0 + (int)blockIdx.y) * rel_stride * (dtype == KGC_BF16 ? 2 : 4);
  cent += (int64_t)blockIdx.y * n_micro * d; rad += (int64_t)blockIdx.y * n_micro; cnorm += (int64_t)blockIdx.y * n_micro;
  const int32_t ent_l = lane < kMicro ? slot_ent[m * kMicro + lane] : -1;
  const int cnt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(ent_l >= 0));
  float* c = cent + m * d;
  if (cnt == 0) {
    for (int k = lane; k < d; k += 64) c[k] = 0.f;
    if (lane == 0) { rad[m] = -1.f; cnorm[m] = 0.f; }
    return;
  }
  const float inv = 1.f / (float)cnt;
  float c2 = 0.f;
  float rs[kMicro];                                   // this lane's part of every row's distance to the centre
#pragma unroll
  for (int q = 0; q < kMicro; ++q) rs[q] = 0.f;
  float l1[MAXL1 ? kMicro : 1];                       // ... and of its L1 norm
#pragma unroll
  for (int q = 0; q < (MAXL1 ? kMicro : 1); ++q) l1[q] = 0.f;
  for (int k0 = 0; k0 < d; k0 += 64) {
    const int k = k0 + lane;
    float v[kMicro];
#pragma unroll
    for (int q = 0; q < kMicro; ++q) v[q] = 0.f;
    if (k < d) {
#pragma unroll
      for (int q = 0; q < kMicro; ++q) {
        const int32_t ent = __builtin_amdgcn_readlane(ent_l, q);
        if (ent >= 0) v[q] = ld_elem(E, (int64_t)ent * d + k, dtype);
      }
      if constexpr (MAXL1) {
#pragma unroll
        for (int q = 0; q < kMicro; ++q) l1[q] += fabsf(v[q]);
      }
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < kMicro; ++q) sum += v[q];
      const float ck = sum * inv;
      c[k] = ck;
      c2 += ck * ck;
#pragma unroll
      for (int q = 0; q < kMicro; ++q) {
        const float x = v[q] - ck;
        if (__builtin_amdgcn_readlane(ent_l, q) >= 0) rs[q] += (P == 2) ? x * x : fabsf(x);
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) c2 += __shfl_xor(c2, off, 64);
  if (lane == 0) cnorm[m] = sqrtf(c2) * (1.f + kBoundSlack);
  const float a1 = micro_row_totals(rs, lane);
  float rmax = (P == 2) ? sqrtf(a1) : a1;             // (a missing row has sum 0)
  for (int off = 32; off > 0; off >>= 1) rmax = fmaxf(rmax, __shfl_xor(rmax, off, 64));
  if (lane == 0) rad[m] = rmax * (1.f + kBoundSlack) + 1e-30f;
  if constexpr (MAXL1) {
    float n = micro_row_totals(l1, lane);             // (a missing row has sum 0)
    for (int off = 32; off > 0; off >>= 1) n = fmaxf(n, __shfl_xor(n, off, 64));
    if (lane == 0) atomicMax(&max_l1[(blockIdx.x + blockIdx.y * gridDim.x) % kMaxSlots], __float_as_uint(n));      // non-negative floats order like their bits
  }
}

// ---------------------------------------------------------------------------------------------
// Generic 128 x 128 distance tile in float32 vector arithmetic (no MFMA): rows x_i (+ shift), columns y_j,
// dist_p(x_i + shift, y_j) for p = 1 or 2 (p = 0: the dot product x_i . y_j, MATRIX epilogue only), K staged through LDS in 16-dimension slices, 8 x 8 results
// per thread.  Two epilogues:
//   ASSIGN  first column within delta (= the group radius tau) of every row -> atomicMin on a packed
//           (column position, distance bits) word
//   MATRIX  the p-th power of every distance is written to a row-major n_rows x n_cols matrix
//   BOUND   rows and columns are micro-tile centres; a micro-tile pair survives when
//           dist - rho_row - rho_col <= delta (with slack), and then sets the bit of its join tile
enum { kEpiAssign = 0, kEpiBound = 1, kEpiMatrix = 2, kEpiBoundUnits = 3 };

// Units of the two-level bound test (see k_bound_l2_units further down): a padded group's run of micro-tiles, or a
// single micro-tile of the packed tail region.
struct UnitTable {
  const int32_t* first;   // big units: first micro-tile ...
  const int32_t* n;       // ... and number of micro-tiles
  int n_big;              // units 0 .. n_big - 1 are padded groups
  int tail_first;         // unit n_big + i is micro-tile tail_first + i
  int n_units;
};
__device__ __forceinline__ void unit_range(const UnitTable& ut, int u, int& first, int& n) {
  if (u < ut.n_big) { first = ut.first[u]; n = ut.n[u]; }
  else { first = ut.tail_first + (u - ut.n_big); n = 1; }
}

constexpr int kInlineMicroPairs = 8;   // unit pairs with at most this many micro-tile pairs are refined where they are found
struct BoundPairs {
  unsigned long long* list;     // (rl << 48) | (unit of heads << 24) | unit of tails
  unsigned long long* count;    // entries asked for (may exceed cap)
  unsigned long long cap;
};


struct TileDistArgs {
  const void* X; int dtypeX; const int32_t* row_ids; const int32_t* n_rows_dev; int64_t n_rows;
  const void* Y; int dtypeY; const int32_t* col_ids; const int32_t* n_cols_dev; int64_t n_cols;
  const void* shift; int dtype_shift; int r0;     // optional vector added to every row: shift[(r0 + blockIdx.z) * d ...]
  int d;
  unsigned long long* best;                        // ASSIGN
  float* matrix;                                   // MATRIX
  int64_t matrix_rel_stride;                       // MATRIX: relation blockIdx.z writes its n_rows x n_cols block this many floats further on
  int symmetric;                                   // MATRIX with X == Y and no shift: only the blocks on and above the diagonal work, and write both halves
  const float* rad; float delta; uint32_t* bitmap; // BOUND
  int nH, words_per_row, micro_per_bm, micro_per_bn;
  // BOUND with per-relation summaries (the general form): relation blockIdx.z reads rows z * x_rel_rows + i of X and
  // z * y_rel_rows + j of Y (0: one set for all relations); rad_rows: radii of the rows when they differ from the columns'
  int64_t x_rel_rows, y_rel_rows; const float* rad_rows;
  // BOUND on units (L1): rows / columns are unit centres, rad their radii; survivors are refined on the
  // micro-tile summaries below (small pairs on the spot, the others through the list)
  UnitTable ut; BoundPairs bp;
  const float* fine_cent; const float* fine_rad; int64_t n_micro;
  const JoinParams* prm;                           // L1 BOUND with a shift: see l1_reach
};

// What the float32 sum of |fl(c_H + r) - c_T| less the radii may come to for a pair that the exact bound keeps.  kBoundSlack pays
// for roundings in proportion to the distance; that of the coordinates c_H + r goes with their size instead, 2^-24 (||c_H||_1 +
// ||r||_1) at most, and JoinParams::base is twice that for the largest rows there are (the spare factor covers the roundings of
// the centres' own means).  Rows at 12,288 under a relation of 5e-4 per dimension, half a unit in their last place: sum 0.0625
// for a distance of 0.032.  Without a shift (connector rows, prm NULL) there is no such rounding.
__device__ __forceinline__ float l1_reach(float delta, const JoinParams* prm) { return delta * (1.f + kBoundSlack) + (prm ? prm->base : 0.f); }

// L1 bound of one unit pair on its micro-tile pairs: dist_1(c_H + r, c_T) - rho_H - rho_T <= delta, centre
// distances summed over d by the calling lane; `lane_count` lanes starting at `lane0` share the pairs.
__device__ __forceinline__ void refine_unit_pair_l1(const TileDistArgs& a, int rl, int uH, int uT, int lane0, int lane_count) {
  int fH, nHm, fT, nTm;
  unit_range(a.ut, uH, fH, nHm);
  unit_range(a.ut, uT, fT, nTm);
  const int64_t so = (int64_t)(a.r0 + rl) * a.d;
  const int64_t total = (int64_t)nHm * nTm;
  const float reach = l1_reach(a.delta, a.prm);
  for (int64_t i = lane0; i < total; i += lane_count) {
    const int64_t mH = fH + i / nTm, mT = fT + i % nTm;
    const float rH = a.fine_rad[mH], rT = a.fine_rad[mT];
    if (rH < 0.f || rT < 0.f) continue;
    const float* cH = a.fine_cent + mH * a.d;
    const float* cT = a.fine_cent + mT * a.d;
    float s = 0.f;
    for (int k = 0; k < a.d; ++k) s += fabsf(cH[k] + ld_elem(a.shift, so + k, a.dtype_shift) - cT[k]);
    if (s * (1.f - kBoundSlack) - rH - rT <= reach) {
      const int tH = (int)(mH / a.micro_per_bm), tT = (int)(mT / a.micro_per_bn);
      uint32_t* w = &a.bitmap[((int64_t)rl * a.nH + tH) * a.words_per_row + (tT >> 5)];
      if (!(*w & (1u << (tT & 31)))) atomicOr(w, 1u << (tT & 31));
    }
  }
}

template <int P, int EPI>
__global__ __launch_bounds__(256) void k_tile_dist(const TileDistArgs a) {
  constexpr int BM = 128, BN = 128, BK = 16;
  __shared__ __attribute__((aligned(16))) float As[BK][BM];
  __shared__ __attribute__((aligned(16))) float Bs[BK][BN];
  __shared__ int32_t rid[BM], cid[BN];
  const int tid = threadIdx.x;
  const int64_t n_rows = a.n_rows_dev ? (int64_t)*a.n_rows_dev : a.n_rows;
  const int64_t n_cols = a.n_cols_dev ? (int64_t)*a.n_cols_dev : a.n_cols;
  const int64_t row0 = (int64_t)blockIdx.y * BM, col0 = (int64_t)blockIdx.x * BN;
  if (row0 >= n_rows || col0 >= n_cols) return;
  if (EPI == kEpiMatrix && a.symmetric && blockIdx.y > blockIdx.x) return;      // the mirror block writes this one
  if (tid < BM) {
    const int64_t r = row0 + tid;
    rid[tid] = r < n_rows ? (a.row_ids ? a.row_ids[r] : (int32_t)r) : -1;
  } else {
    const int64_t c = col0 + (tid - BM);
    cid[tid - BM] = c < n_cols ? (a.col_ids ? a.col_ids[c] : (int32_t)c) : -1;
  }
  __syncthreads();
  const int d = a.d;
  const int tx = tid & 15, ty = tid >> 4;
  float acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
  const int srow = tid >> 1, sk0 = (tid & 1) * 8;
  // L1 bounds: terms are >= 0 and rounding is monotonic, so a wave none of whose sums is at or below what its pairs'
  // radii allow (the largest of a thread's rows and of its columns, widened for the roundings of the comparison at the
  // end) has ruled all of them out, and a tile of four such waves ends there.
  constexpr bool kEarly = P == 1 && (EPI == kEpiBound || EPI == kEpiBoundUnits);
  __shared__ uint32_t decided[2][4];                           // per slice (alternating) and wave
  float open_to = 0.f;
  const float reach = P == 1 ? l1_reach(a.delta, a.prm) : a.delta * (1.f + kBoundSlack);      // (L2: without a shift only)
  int par = 0;
  if constexpr (kEarly) {
    const float* rad_r = (a.rad_rows ? a.rad_rows : a.rad) + (int64_t)blockIdx.z * a.x_rel_rows;
    const float* rad_c = a.rad + (int64_t)blockIdx.z * a.y_rel_rows;
    float mr = -1.f, mc = -1.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lr = (i >> 2) * 64 + ty * 4 + (i & 3), lc = (i >> 2) * 64 + tx * 4 + (i & 3);
      const float vr = rid[lr] >= 0 ? rad_r[row0 + lr] : -1.f, vc = cid[lc] >= 0 ? rad_c[col0 + lc] : -1.f;
      mr = vr > mr || vr != vr ? vr : mr;      // (a NaN stays)
      mc = vc > mc || vc != vc ? vc : mc;
    }
    // (-1: all of the thread's rows, or columns, are empty; NaN: every pair stays open)
    open_to = mr < 0.f || mc < 0.f ? -1.f : (reach + mr + mc) / (1.f - kBoundSlack) * (1.f + 1e-5f);
  }
  const int re = rid[srow], ce = cid[srow];
  const int64_t xo = ((int64_t)blockIdx.z * a.x_rel_rows + (re < 0 ? 0 : re)) * d,
                yo = ((int64_t)blockIdx.z * a.y_rel_rows + (ce < 0 ? 0 : ce)) * d;
  const int64_t so = (int64_t)(a.r0 + (int)blockIdx.z) * d;
  for (int k0 = 0; k0 < d; k0 += BK, par ^= 1) {
    float va[8], vb[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int k = k0 + sk0 + q;
      const bool in = k < d;
      float x = in ? ld_elem(a.X, xo + k, a.dtypeX) : 0.f;
      if (in && a.shift) x += ld_elem(a.shift, so + k, a.dtype_shift);
      va[q] = x;
      vb[q] = in ? ld_elem(a.Y, yo + k, a.dtypeY) : 0.f;
    }
    __syncthreads();
    if (kEarly && k0 > 0 && (decided[par ^ 1][0] & decided[par ^ 1][1] & decided[par ^ 1][2] & decided[par ^ 1][3])) return;      // (the whole block)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      As[sk0 + q][srow] = va[q];
      Bs[sk0 + q][srow] = vb[q];
    }
    __syncthreads();
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
        for (int j = 0; j < 8; ++j) {
          if (P == 0) {
            acc[i][j] += av[i] * bv[j];
          } else {
            const float x = av[i] - bv[j];
            acc[i][j] += (P == 2) ? x * x : fabsf(x);
          }
        }
    }
    if constexpr (kEarly) {
      bool open = false;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) open |= !(acc[i][j] > open_to);
      const unsigned long long b = __builtin_amdgcn_ballot_w64(open);
      if ((tid & 63) == 0) decided[par][tid >> 6] = b == 0ull ? 1u : 0u;
    }
  }
  // rows of this thread: (i >> 2) * 64 + ty * 4 + (i & 3); columns: (j >> 2) * 64 + tx * 4 + (j & 3)
  if (EPI == kEpiAssign) {
    // Among the columns (pivots) within tau of the row, the one with the LOWEST position wins, not the
    // nearest: when a natural cluster received several pivots, all its rows then agree on one of them
    // instead of splitting the cluster between them.
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lr = (i >> 2) * 64 + ty * 4 + (i & 3);
      unsigned long long bestv = ~0ull;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int lc = (j >> 2) * 64 + tx * 4 + (j & 3);
        const float dist = (P == 2) ? sqrtf(acc[i][j]) : acc[i][j];
        if (cid[lc] >= 0 && dist <= a.delta) {
          const unsigned long long v =
              ((unsigned long long)(uint32_t)(col0 + lc) << 32) | (unsigned long long)__float_as_uint(dist);
          bestv = v < bestv ? v : bestv;
        }
      }
      // the 16 threads that share a row are 16 consecutive lanes
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)(bestv & 0xffffffffull), off, 16);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(bestv >> 32), off, 16);
        const unsigned long long o = ((unsigned long long)hi << 32) | lo;
        bestv = o < bestv ? o : bestv;
      }
      if (tx == 0 && rid[lr] >= 0 && bestv != ~0ull) atomicMin(&a.best[row0 + lr], bestv);
    }
  } else if (EPI == kEpiMatrix) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lr = (i >> 2) * 64 + ty * 4 + (i & 3);
      if (rid[lr] < 0) continue;
#pragma unroll
      for (int jg = 0; jg < 2; ++jg) {
        const int lc = jg * 64 + tx * 4;
        float* o = a.matrix + (int64_t)blockIdx.z * a.matrix_rel_stride + (row0 + lr) * n_cols + col0 + lc;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (cid[lc + j] >= 0) o[j] = acc[i][jg * 4 + j];
        if (a.symmetric && blockIdx.y != blockIdx.x) {       // sum of (x_i - x_j)^2 = sum of (x_j - x_i)^2, term by term
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (cid[lc + j] >= 0) a.matrix[(int64_t)blockIdx.z * a.matrix_rel_stride + (col0 + lc + j) * n_cols + row0 + lr] = acc[i][jg * 4 + j];
        }
      }
    }
  } else if (EPI == kEpiBoundUnits) {
    const int rl = (int)blockIdx.z;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lr = (i >> 2) * 64 + ty * 4 + (i & 3);
      if (rid[lr] < 0) continue;
      const float rr = a.rad[row0 + lr];
      if (rr < 0.f) continue;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int lc = (j >> 2) * 64 + tx * 4 + (j & 3);
        if (cid[lc] < 0) continue;
        const float rc = a.rad[col0 + lc];
        if (rc < 0.f) continue;
        const float dist = (P == 2) ? sqrtf(acc[i][j]) : acc[i][j];
        if (dist * (1.f - kBoundSlack) - rr - rc > reach) continue;
        const int uH = (int)(row0 + lr), uT = (int)(col0 + lc);
        int fH, nHm, fT, nTm;
        unit_range(a.ut, uH, fH, nHm);
        unit_range(a.ut, uT, fT, nTm);
        unsigned long long pos = a.bp.cap;
        if ((int64_t)nHm * nTm > kInlineMicroPairs) pos = atomicAdd(a.bp.count, 1ull);
        if (pos < a.bp.cap)
          a.bp.list[pos] = ((unsigned long long)(uint32_t)rl << 48) | ((unsigned long long)(uint32_t)uH << 24) |
                           (unsigned long long)(uint32_t)uT;
        else
          refine_unit_pair_l1(a, rl, uH, uT, 0, 1);
      }
    }
  } else {
    const int rl = (int)blockIdx.z;
    const float* rad_r = (a.rad_rows ? a.rad_rows : a.rad) + (int64_t)rl * a.x_rel_rows;
    const float* rad_c = a.rad + (int64_t)rl * a.y_rel_rows;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lr = (i >> 2) * 64 + ty * 4 + (i & 3);
      if (rid[lr] < 0) continue;
      const float rr = rad_r[row0 + lr];
      if (rr < 0.f) continue;                                  // empty micro-tile
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int lc = (j >> 2) * 64 + tx * 4 + (j & 3);
        if (cid[lc] < 0) continue;
        const float rc = rad_c[col0 + lc];
        if (rc < 0.f) continue;
        const float dist = (P == 2) ? sqrtf(acc[i][j]) : acc[i][j];
        const float lb = dist * (1.f - kBoundSlack) - rr - rc;  // radii already carry their slack
        if (lb <= reach) {
          const int tH = (int)((row0 + lr) / a.micro_per_bm), tT = (int)((col0 + lc) / a.micro_per_bn);
          atomicOr(&a.bitmap[((int64_t)rl * a.nH + tH) * a.words_per_row + (tT >> 5)], 1u << (tT & 31));
        }
      }
    }
  }
}

// The same MATRIX results for small operands (a few hundred to a few thousand rows and columns: micro-tile centres,
// relation vectors), where the 128 x 128 tiles above leave most of the chip idle: 32 x 32 results per block of 256
// threads, K through LDS 128 dimensions at a time, four rows x one column per thread.  out[i][j] = ||x_i - y_j||^2
// (P = 2) or x_i . y_j (P = 0), row-major n_rows x n_cols; X rows of the given type, Y rows float32.
// With `rad` set (P = 2, X = Y = the micro-tile centres) the result is not the squared centre distance D itself but
// the part of the flat bound test that depends on the pair alone, reach^2 (1 + slack) + D (d + 8) 2^-24 - D with
// reach = delta (1 + slack) + rad_i + rad_j (see k_bound_l2), so that the test does not form it again for every
// group of relations; a pair with an empty micro-tile (rad < 0) gets -3e38 and never passes.
template <int P>
__global__ __launch_bounds__(256) void k_small_matrix(const void* __restrict__ X, int dtypeX, int64_t n_rows,
                                                      const float* __restrict__ Y, int64_t n_cols, int d,
                                                      float* __restrict__ out, const float* __restrict__ rad = nullptr,
                                                      float delta = 0.f, int symmetric = 0) {      // symmetric (X == Y): blocks above the diagonal write both halves
  constexpr int KC = 128;                                 // dimensions per pass through LDS (d <= 128: one pass, two barriers)
  __shared__ float xs[32][KC + 1], ys[32][KC + 1];
  const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
  const int64_t row0 = (int64_t)blockIdx.y * 32, col0 = (int64_t)blockIdx.x * 32;
  if (symmetric && blockIdx.y > blockIdx.x) return;        // the mirror block writes this one
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < d; k0 += KC) {
    const int kn = d - k0 < KC ? d - k0 : KC;
    __syncthreads();
    // 32 rows x kn dimensions of each operand, consecutive threads on consecutive dimensions of a row
    for (int e = tid; e < 32 * KC; e += 256) {
      const int rw = e / KC, k = e - rw * KC;
      const bool in = k < kn;
      xs[rw][k] = (in && row0 + rw < n_rows) ? ld_elem(X, (row0 + rw) * d + k0 + k, dtypeX) : 0.f;
      ys[rw][k] = (in && col0 + rw < n_cols) ? Y[(col0 + rw) * d + k0 + k] : 0.f;
    }
    __syncthreads();
    for (int k = 0; k < kn; ++k) {
      const float b = ys[tx][k];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = xs[ty + 8 * q][k];
        if (P == 0) acc[q] += a * b;
        else { const float x = a - b; acc[q] += x * x; }
      }
    }
  }
  if (col0 + tx < n_cols) {
    const float rT = rad ? rad[col0 + tx] : 0.f;
    const float dsl = delta * (1.f + kBoundSlack), dk = (float)(d + 8) * 6e-8f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (row0 + ty + 8 * q < n_rows) {
        float v = acc[q];
        if (rad) {
          const float rH = rad[row0 + ty + 8 * q];
          const float reach = dsl + (rH + rT);                 // (the same for both orders of the pair)
          v = (rH < 0.f || rT < 0.f) ? -3e38f : reach * reach * (1.f + kBoundSlack) + v * dk - v;
        }
        out[(row0 + ty + 8 * q) * n_cols + col0 + tx] = v;
        if (symmetric && blockIdx.y != blockIdx.x) out[(col0 + tx) * n_cols + row0 + ty + 8 * q] = v;   // (sum of (x_i - x_j)^2 = sum of (x_j - x_i)^2 term by term, and the pair term is symmetric too)
      }
  }
}

// out[i][j] = x_i . y_j for small operands, on the float32 matrix pipes: one wave per 32 x 32 results, no LDS and no
// barrier.  v_mfma_f32_32x32x2_f32 takes A[i][k] from lane 32 k + i and B[k][j] from lane 32 k + j (k = 0, 1); a dot
// product does not care in which order its dimensions are taken as long as both operands agree, so lane (row, half)
// reads the four consecutive elements 8 g + 4 half .. + 3 of its row in one load and feeds them to four successive
// steps.  All loads of up to 128 dimensions are issued before the first is used: a chunk costs one memory round trip.
// Products and sums are float32 (the bound test charges (d + 8) 2^-24 ||x|| ||y|| for them, which holds for any order
// of a float32 sum of d products).  X rows of the given storage type, Y rows float32; VEC: rows may be read four
// elements at a time (both bases on 16-byte boundaries -- 8 for bf16 rows -- and d a multiple of four).
template <bool BF16, bool VEC>
__global__ __launch_bounds__(64) void k_small_dot(const void* __restrict__ X, int64_t n_rows, const float* __restrict__ Y,
                                                  int64_t n_cols, int d, float* __restrict__ out) {
  const int lane = threadIdx.x, row = lane & 31, half = lane >> 5;
  const int64_t row0 = (int64_t)blockIdx.y * 32, col0 = (int64_t)blockIdx.x * 32;
  const int64_t xr = row0 + row < n_rows ? row0 + row : n_rows - 1;      // (past the end: a valid row, the results are dropped)
  const int64_t yc = col0 + row < n_cols ? col0 + row : n_cols - 1;
  const int64_t xo = xr * d, yo = yc * d;
  f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  constexpr int kG = 16;                                                  // groups of 8 dimensions per chunk (d <= 128: one chunk)
  for (int k0 = 0; k0 < d; k0 += 8 * kG) {
    f32x4_t xv[kG], yv[kG];
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      const int k = k0 + 8 * g + 4 * half;
      xv[g] = exact_ld4<BF16, VEC>(X, xo, k, d);
      yv[g] = exact_ld4<false, VEC>(Y, yo, k, d);
    }
    __builtin_amdgcn_sched_barrier(0);                                    // (the loads stay together, ahead of the arithmetic)
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      if (k0 + 8 * g >= d) break;                                         // the same for the whole wave
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[g][e], yv[g][e], acc, 0, 0, 0);
    }
  }
  // register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
  if (col0 + row < n_cols) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t i = row0 + 8 * (v >> 2) + 4 * half + (v & 3);
      if (i < n_rows) out[i * n_cols + col0 + row] = acc[v];
    }
  }
}

// Connector rows of the structured-embedding model, out[r][i][c] = sum_k W[r][c][k] e_i[k], on the float32 matrix pipes
// (operands as in k_small_dot; products and sums are float32 as in a vector kernel).  A wave takes 32 entities x 128
// outputs, so that an entity's fragment meets four of the map's, and the four waves of a workgroup share the map's rows
// in the vector cache; bound by the matrix pipes (64 cycles per step and SIMD).
// N = 15,000, R = 64, d = 100, one side: 515 -> 406 us against the 128 x 128 vector tiles.  Rows must start on a boundary of
// four elements (element by element its loads are slower than those tiles, which other sizes take).
template <bool BF16>
__global__ __launch_bounds__(256) void k_connect(const void* __restrict__ E, int64_t N, const void* __restrict__ W, int d,
                                                 float* __restrict__ out) {
  const int lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32;
  const int col0 = (int)blockIdx.y * 128;
  if (row0 >= N) return;                                                  // (no barrier follows)
  const int64_t xr = row0 + row < N ? row0 + row : N - 1;                 // (past the end: a valid row, the results are dropped)
  const int64_t xo = xr * d, wo = (int64_t)blockIdx.z * d * d;
  const int nb = (d - col0 + 31) / 32 < 4 ? (d - col0 + 31) / 32 : 4;     // blocks of 32 outputs that exist
  int64_t yo[4];
  f32x16_t acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = col0 + 32 * j + row;
    yo[j] = wo + (int64_t)(c < d ? c : d - 1) * d;
    acc[j] = f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  }
  // Dimensions in ascending order, two per step (lanes 0 - 31 hold the even one, 32 - 63 the odd one): the sums are those
  // of a chain of fused multiply-adds, bit for bit.  So both halves read the eight elements of a group.
  constexpr int kG = 2;                                                   // groups of 8 dimensions per chunk
  for (int k0 = 0; k0 < d; k0 += 8 * kG) {
    f32x4_t xv[kG][2], yv[4][kG][2];
#pragma unroll
    for (int g = 0; g < kG; ++g)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int k = k0 + 8 * g + 4 * q;
        xv[g][q] = exact_ld4<BF16, true>(E, xo, k, d);
#pragma unroll
        for (int j = 0; j < 4; ++j) yv[j][g][q] = exact_ld4<BF16, true>(W, yo[j], k, d);
      }
    __builtin_amdgcn_sched_barrier(0);                                    // (the loads stay together, ahead of the arithmetic)
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      if (k0 + 8 * g >= d) break;                                         // the same for the whole wave
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int q = e >> 1, i = 2 * (e & 1);
        const float x = half ? xv[g][q][i + 1] : xv[g][q][i];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, half ? yv[j][g][q][i + 1] : yv[j][g][q][i], acc[j], 0, 0, 0);
      }
    }
  }
  float* o = out + (int64_t)blockIdx.z * N * d;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = col0 + 32 * j + row;
    if (j >= nb || c >= d) continue;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t i = row0 + 8 * (v >> 2) + 4 * half + (v & 3);
      if (i < N) o[i * d + c] = acc[j][v];
    }
  }
}

// L2 only.  u[rl][m] = r . c_m and rn[rl] = ||r||^2 for the relations of a batch: one wave per (rl, m).
__global__ __launch_bounds__(256) void k_rel_centre_dot(const void* __restrict__ Rv, int dtype, int d, int r0, int RB,
                                                        const float* __restrict__ cent, int64_t n_micro,
                                                        float* __restrict__ u, float* __restrict__ rn) {
  const int lane = threadIdx.x & 63;
  const int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t per_rel = n_micro + 1;                       // the extra item computes ||r||^2
  if (w >= per_rel * RB) return;
  const int rl = (int)(w / per_rel);
  const int64_t m = w - (int64_t)rl * per_rel;
  const int64_t ro = (int64_t)(r0 + rl) * d;
  float s = 0.f;
  if (m == n_micro) {
    for (int k = lane; k < d; k += 64) { const float x = ld_elem(Rv, ro + k, dtype); s += x * x; }
  } else {
    const float* c = cent + m * d;
    for (int k = lane; k < d; k += 64) s += ld_elem(Rv, ro + k, dtype) * c[k];
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) {
    if (m == n_micro) rn[rl] = s; else u[(int64_t)rl * n_micro + m] = s;
  }
}

// L2 only.  The squared centre distance of a micro-tile pair under relation r expands into parts that do
// not need a d-dimensional loop per (r, H, T):
//     ||c_H + r - c_T||^2 = ||c_H - c_T||^2 + 2 (r.c_H - r.c_T) + ||r||^2 = D[H][T] + 2 (u[r][H] - u[r][T]) + rn[r]
// (the same observation that makes distB independent of r in Section 5.2, applied to the bound).  The float32 cancellation error of the sum is bounded by
// err = 2 (d + 8) 2^-24 ||r|| (||c_H|| + ||c_T||) + (d + 8) 2^-24 D and added on the keeping side: D itself is a float32
// sum of d squared differences (relative error at most (d + 4) 2^-24 in the worst case), and for TransE data it is far
// larger than reach^2 (r cancels c_H - c_T), so its error is charged in full, not absorbed in the slack of reach^2.
constexpr int kRelChunk = 16;
struct BoundL2Args {
  const float* D; const float* u; const float* rn; const float* rad; const float* cnorm;
  int64_t n_micro; int RB; int d; float delta;
  uint32_t* bitmap; int nH, words_per_row, micro_per_bm, micro_per_bn;
  // micro-tile level of the two-level test without the D and u matrices (D == NULL): centre distances are then
  // summed directly from the centres and the relation vector
  const float* cent; const void* Rv; int dtype; int r0;
  int64_t both_from;      // pairs whose head and tail number both reach this are left out: another kernel takes their rows
  // k_bound_l2 only, optional (NULL: off): every tile whose bit is set for the first time is also appended to a flat
  // list -- its tail tile to list_cols, its row (relation, head tile) to list_rows and to list_active -- so that a
  // batch with few surviving tiles needs no pass over the bitmap (see k_batch_tiles)
  uint32_t* list_cols; uint32_t* list_rows; uint32_t* list_active; unsigned long long* list_count; unsigned long long list_cap;
};
constexpr int kHeadChunk = 16;
constexpr int kHeadsFlat = 64;       // head micro-tiles per block of the flat test (four groups of kHeadChunk)
// PAIR_READY: a.D holds the pair's part of the right side, ready made (k_small_matrix with radii), not the plain
// squared centre distance: a test then costs one load, one addition and one comparison.
// UNITS: the unit level of the two-level test (see below): `a` describes UNITS, and a surviving (relation, unit pair)
// is appended to the list `bp` -- or refined on the spot on the micro-tile arrays `fine` when the pair is small or
// the list is full -- instead of setting bits.
template <bool LIST>
__device__ __forceinline__ void refine_unit_pair(const BoundL2Args& a, const UnitTable& ut, int rl, int uH, int uT, int lane0,
                                                 int lane_count);
// The surviving (relation rl0 + q, unit pair) of a wave: bit q of `keep` per lane (head unit mH the same for the wave,
// tail unit mT the lane's).  A pair of small units (in the packed tail region both are single micro-tiles) is
// finished on the spot; pairs with many micro-tile pairs go through the list, whose length is advanced ONCE per
// relation for all lanes of the wave that append (atomics on one address are served one after the other: with one
// per entry the unit level of a join with many survivors spent most of its time there).  Called by all active lanes.
template <bool LIST>
__device__ __forceinline__ void unit_pairs_out(uint32_t keep, int rl0, int mH, int mT, const BoundL2Args& fine,
                                               const UnitTable& ut, const BoundPairs& bp) {
  if (__builtin_amdgcn_ballot_w64(keep != 0u) == 0ull) return;
  int fH, nHm, fT, nTm;
  unit_range(ut, mH, fH, nHm);
  unit_range(ut, mT, fT, nTm);
  // (without the matrices a micro-tile pair costs a loop over d: then every pair but a single one is listed)
  const bool big = (int64_t)nHm * nTm > (fine.D ? kInlineMicroPairs : 1);
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll 1
  for (int q = 0; q < kRelChunk; ++q) {
    const bool k = (keep >> q) & 1u;
    if (__builtin_amdgcn_ballot_w64(k) == 0ull) continue;
    const unsigned long long ml = __builtin_amdgcn_ballot_w64(k && big);
    unsigned long long pos = bp.cap;
    if (ml) {
      const int leader = (int)__builtin_ctzll(ml);
      unsigned long long base = 0ull;
      if (lane == leader) base = atomicAdd(bp.count, (unsigned long long)__builtin_popcountll(ml));
      const uint32_t blo = (uint32_t)__shfl((int)(uint32_t)(base & 0xffffffffull), leader, 64);
      const uint32_t bhi = (uint32_t)__shfl((int)(uint32_t)(base >> 32), leader, 64);
      if (k && big) pos = (((unsigned long long)bhi << 32) | blo) + (unsigned long long)__builtin_popcountll(ml & ((1ull << lane) - 1ull));
    }
    if (k) {
      if (pos < bp.cap)
        bp.list[pos] = ((unsigned long long)(uint32_t)(rl0 + q) << 48) | ((unsigned long long)(uint32_t)mH << 24) |
                       (unsigned long long)(uint32_t)mT;
      else
        refine_unit_pair<LIST>(fine, ut, rl0 + q, mH, mT, 0, 1);
    }
  }
}
// LIST (UNITS only): the micro-tile level also lists the tiles it keeps (see keep_tile)
template <bool PAIR_READY, bool UNITS, bool LIST = false>
__global__ __launch_bounds__(256) void k_bound_l2(const BoundL2Args a, const BoundL2Args fine, const UnitTable ut,
                                                  const BoundPairs bp) {
  // block = 256 tail micro-tiles x kHeadsFlat head micro-tiles x kRelChunk relations; the per-(head, relation)
  // terms sit in LDS, the thread's own per-relation terms in registers, so one test costs one (shared) D load per
  // kRelChunk relations, one addition and one comparison -- and most chunks of relations end at one comparison
  __shared__ __attribute__((aligned(16))) float aH[kHeadsFlat][kRelChunk];   // 2 r.c_H + ||r||^2 - kk ||c_H|| ||r|| per (head micro-tile, relation)
  __shared__ float srnS[kRelChunk];
  __shared__ float radH[kHeadsFlat], aHmin[kHeadsFlat];
  const int tid = threadIdx.x;
  const int64_t mT = (int64_t)blockIdx.x * blockDim.x + tid;
  const int64_t mH0 = (int64_t)blockIdx.y * kHeadsFlat;
  const int rl0 = (int)blockIdx.z * kRelChunk;
  const float kk = 2.f * (float)(a.d + 12) * 6e-8f;
  {
    // 256 threads = kRelChunk relations x 16 neighbouring heads per pass: a row of u is read 64 bytes at a time (one
    // thread per relation and sixteenth of the heads would pull a whole cache line per value: 64 lines per load
    // instruction, 0.4 GB through the vector caches per launch for a matrix of 4 MB)
    const int q = tid >> 4, j = tid & 15;
    const int rl = rl0 + q;
    const float rnq = rl < a.RB ? a.rn[rl] : 0.f;
    const float srn = sqrtf(rnq);
#pragma unroll
    for (int pass = 0; pass < kHeadsFlat / 16; ++pass) {
      const int hq = pass * 16 + j;
      const int64_t mH = mH0 + hq;
      const bool in = rl < a.RB && mH < a.n_micro;
      const float ah = in ? 2.f * a.u[(int64_t)rl * a.n_micro + mH] + rnq * (1.f - 2.4e-7f) : 0.f;
      aH[hq][q] = in ? ah - (kk * a.cnorm[mH]) * srn : 0.f;
    }
    if (tid < kRelChunk) srnS[tid] = sqrtf(rl0 + tid < a.RB ? a.rn[rl0 + tid] : 0.f);
    if (tid < kHeadsFlat) {
      const int64_t m = mH0 + tid;
      radH[tid] = m < a.n_micro ? a.rad[m] : -1.f;
    }
  }
  __syncthreads();
  {
    // the smallest left side of every head micro-tile over the chunk's relations: four threads per head
    const int hq = tid >> 2, part = tid & 3;
    float mn = 3e38f;
    if (mH0 + hq < a.n_micro) {
#pragma unroll
      for (int i = 0; i < 4; ++i) mn = rl0 + part * 4 + i < a.RB ? fminf(mn, aH[hq][part * 4 + i]) : mn;
    }
    mn = fminf(mn, __shfl_xor(mn, 1, 64));
    mn = fminf(mn, __shfl_xor(mn, 2, 64));
    if (part == 0) aHmin[hq] = mn;
  }
  __syncthreads();
  if (mT >= a.n_micro) return;
  const float rT = a.rad[mT];
  if (rT < 0.f || (mT >= a.both_from && mH0 >= a.both_from)) return;      // empty micro-tile, or pairs left out
  const float cT = a.cnorm[mT];
  const int heads_here = a.n_micro - mH0 < kHeadsFlat ? (int)(a.n_micro - mH0) : kHeadsFlat;
  // dist^2 <= lim + ek sqrt(rn), ek = kk (||c_H|| + ||c_T||)
  //   <=>   (2 u_H + rn) - kk ||c_H|| sqrt(rn)  <=  (lim - D) + (2 u_T + kk ||c_T|| sqrt(rn)):
  // the left side is formed once per (head micro-tile, relation) and block, the last term once per (thread, relation),
  // lim - D once per micro-tile pair, which leaves one addition and one comparison per test.  The extra roundings of
  // this order (two each at most 2^-24 of |2 u_H + rn| and of |2 u_T|, three of D) are paid for on the keeping side:
  // 4 more units in the (d + 8) factor of ek, 2.4e-7 of rn and of D.
  float bT[kRelChunk];
  const int nrel = a.RB - rl0 < kRelChunk ? a.RB - rl0 : kRelChunk;
#pragma unroll
  for (int q = 0; q < kRelChunk; ++q)
    bT[q] = q < nrel ? 2.f * a.u[(int64_t)(rl0 + q) * a.n_micro + mT] + (kk * cT) * srnS[q] : -3e38f;   // past the batch: never passes
  // One comparison first for the whole chunk: no relation can pass when even the smallest left side exceeds the right
  // side with the largest per-relation term (float addition is monotonic, so this is the 16 tests' own arithmetic:
  // nothing is widened).  For TransE data the two sides are 6 sigma apart, so almost every chunk ends here.
  float bmax = bT[0];
#pragma unroll
  for (int q = 1; q < kRelChunk; ++q) bmax = fmaxf(bmax, bT[q]);
  const int tT = UNITS ? 0 : (int)(mT / a.micro_per_bn);
  const float dsl = a.delta * (1.f + kBoundSlack);
  const float dk = (float)(a.d + 8) * 6e-8f;
  for (int hg = 0; hg < kHeadsFlat; hg += kHeadChunk) {
  if (mH0 + hg >= a.n_micro) break;                              // the same for the block
  // the centre distances of a group of heads, all loads in flight together (a head past the end reads the group's first row; it is skipped below)
  float Dv[kHeadChunk];
  {
    const float* Dp = a.D + (mH0 + hg) * a.n_micro + mT;
    const int nvalid = a.n_micro - (mH0 + hg) < kHeadChunk ? (int)(a.n_micro - (mH0 + hg)) : kHeadChunk;
#pragma unroll
    for (int hq = 0; hq < kHeadChunk; ++hq) Dv[hq] = Dp[hq < nvalid ? (int64_t)hq * a.n_micro : 0];
  }
#pragma unroll
  for (int hl = 0; hl < kHeadChunk; ++hl) {
    const int hq = hg + hl;
    float rhs;
    if (PAIR_READY) {
      if (hq >= heads_here) break;                               // past the end (the same for the block)
      rhs = Dv[hl];                                              // (-3e38 for an empty micro-tile)
    } else {
      const float rH = radH[hq];
      if (rH < 0.f) continue;                                    // empty or past the end
      const float D = Dv[hl];
      const float reach = dsl + rH + rT;
      rhs = reach * reach * (1.f + kBoundSlack) + D * dk - D;
    }
    const int64_t mH = mH0 + hq;
    if (__builtin_amdgcn_ballot_w64(aHmin[hq] <= rhs + bmax) == 0ull) continue;
    bool any = false;
#pragma unroll
    for (int q = 0; q < kRelChunk; ++q) any |= aH[hq][q] <= rhs + bT[q];
    if (__builtin_amdgcn_ballot_w64(any) == 0ull) continue;      // almost always: nothing survives
    uint32_t keep = 0u;
#pragma unroll
    for (int q = 0; q < kRelChunk; ++q) keep |= (aH[hq][q] <= rhs + bT[q]) ? (1u << q) : 0u;
    if constexpr (UNITS) {
      unit_pairs_out<LIST>(keep, rl0, (int)mH, (int)mT, fine, ut, bp);
      continue;
    }
    const int tH = (int)(mH / a.micro_per_bm);
    while (keep) {
      const int q = __builtin_ctz(keep);
      keep &= keep - 1u;
      const int64_t row = (int64_t)(rl0 + q) * a.nH + tH;
      const uint32_t bit = 1u << (tT & 31);
      const uint32_t old = atomicOr(&a.bitmap[row * a.words_per_row + (tT >> 5)], bit);
      if (a.list_count && !(old & bit)) {                        // the tile is new: also onto the flat list
        const unsigned long long idx = atomicAdd(a.list_count, 1ull);
        if (idx < a.list_cap) { a.list_cols[idx] = (uint32_t)tT; a.list_rows[idx] = (uint32_t)row; a.list_active[idx] = (uint32_t)row; }
      }
    }
  }
  }   // groups of heads
}

// ---------------------------------------------------------------------------------------------
// Two-level bound test (L2).  When groups span several micro-tiles, the flat test over micro-tile pairs does
// the same work many times: all micro-tiles of a group sit within the group's radius of one another.  A
// UNIT is a padded group (its run of micro-tiles) or, in the packed tail region, a single micro-tile.  The
// same bound is first taken on unit pairs -- centre = mean of the micro-tile centres, radius = max over
// the micro-tiles of (distance of its centre to the unit centre + its radius), so every row of the unit is
// inside -- and only the micro-tile pairs of surviving unit pairs are tested.  Survivors go through a list;
// a lane that finds the list full tests its pair's micro-tiles on the spot.
// One workgroup of sixteen waves per unit, the micro-tiles dealt over the waves; P: the join's metric (radii in that
// metric).  (One wave per unit walked the largest group alone, three times: 6.9 ms of the N = 1,000,000 workload with
// 4,700 micro-tiles in one group.)
constexpr int kUnitWaves = 16;
template <int P>
__global__ __launch_bounds__(kUnitWaves * 64) void k_unit_summary(const float* __restrict__ cent, const float* __restrict__ rad, int d,
                                                                  UnitTable ut, float* __restrict__ centU, float* __restrict__ radU,
                                                                  float* __restrict__ cnormU) {
  __shared__ float part[kUnitWaves][64];
  __shared__ int part_n[kUnitWaves];
  __shared__ float part_r[kUnitWaves];
  const int u = (int)blockIdx.x;
  if (u >= ut.n_units) return;
  const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6);
  int first, n;
  unit_range(ut, u, first, n);
  float* c = centU + (int64_t)u * d;
  // the centre: its chunk of 64 dimensions is written by wave 0 and read by all after the barrier
  float c2 = 0.f;
  int cntm = 0;
  for (int k0 = 0; k0 < d; k0 += 64) {
    const int k = k0 + lane;
    float s = 0.f;
    int cn = 0;
    for (int m = first + wave; m < first + n; m += kUnitWaves) {
      if (rad[m] < 0.f) continue;                       // the same for the whole wave
      ++cn;
      if (k < d) s += cent[(int64_t)m * d + k];
    }
    part[wave][lane] = s;
    if (lane == 0) part_n[wave] = cn;
    __syncthreads();
    if (wave == 0) {
      float t = 0.f;
      cntm = 0;
#pragma unroll
      for (int w = 0; w < kUnitWaves; ++w) { t += part[w][lane]; cntm += part_n[w]; }
      const float ck = cntm > 0 ? t * (1.f / (float)cntm) : 0.f;
      if (k < d) { c[k] = ck; c2 += ck * ck; }
    }
    __syncthreads();
  }
  float rmax = 0.f;
  for (int m = first + wave; m < first + n; m += kUnitWaves) {
    const float rm = rad[m];
    if (rm < 0.f) continue;
    float s = 0.f;
    for (int k = lane; k < d; k += 64) { const float x = cent[(int64_t)m * d + k] - c[k]; s += (P == 2) ? x * x : fabsf(x); }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    rmax = fmaxf(rmax, ((P == 2) ? sqrtf(s) : s) * (1.f + kBoundSlack) + rm);
  }
  if (lane == 0) part_r[wave] = rmax;
  __syncthreads();
  if (wave == 0) {
    for (int off = 32; off > 0; off >>= 1) c2 += __shfl_xor(c2, off, 64);
    rmax = lane < kUnitWaves ? part_r[lane] : 0.f;
    for (int off = 32; off > 0; off >>= 1) rmax = fmaxf(rmax, __shfl_xor(rmax, off, 64));
    if (lane == 0) {
      radU[u] = cntm > 0 ? rmax * (1.f + kBoundSlack) + 1e-30f : -1.f;
      cnormU[u] = cntm > 0 ? sqrtf(c2) * (1.f + kBoundSlack) : 0.f;
    }
  }
}

// The same where no unit has more than kSmallUnit micro-tiles: a wave per unit, whose micro-tiles' centres are read once, side
// by side (the chunk's centre comes from their sum, and each one's distance grows by its part of the chunk).  N = 100,000,
// d = 200, units of one to three: 5.3 us, where the workgroups of sixteen waves take 24 for the launch of 1,024 threads and
// two barriers per 64 dimensions.
constexpr int kSmallUnit = 4;
template <int P>
__global__ __launch_bounds__(64) void k_unit_summary_small(const float* __restrict__ cent, const float* __restrict__ rad, int d,
                                                           UnitTable ut, float* __restrict__ centU, float* __restrict__ radU,
                                                           float* __restrict__ cnormU) {
  const int u = (int)blockIdx.x;
  if (u >= ut.n_units) return;
  const int lane = threadIdx.x;
  int first, n;
  unit_range(ut, u, first, n);
  float rm[kSmallUnit], dist[kSmallUnit];
  int cntm = 0;
#pragma unroll
  for (int i = 0; i < kSmallUnit; ++i) {
    rm[i] = i < n ? rad[first + i] : -1.f;                // (-1: an empty micro-tile, or none; the same for the whole wave)
    cntm += !(rm[i] < 0.f);
    dist[i] = 0.f;
  }
  const float inv = cntm > 0 ? 1.f / (float)cntm : 0.f;
  float c2 = 0.f;
  for (int k = lane; k < d; k += 64) {
    float v[kSmallUnit], s = 0.f;
#pragma unroll
    for (int i = 0; i < kSmallUnit; ++i) v[i] = cent[(int64_t)(first + (i < n ? i : 0)) * d + k];
#pragma unroll
    for (int i = 0; i < kSmallUnit; ++i)
      if (!(rm[i] < 0.f)) s += v[i];
    const float ck = s * inv;
    centU[(int64_t)u * d + k] = ck;
    c2 += ck * ck;
#pragma unroll
    for (int i = 0; i < kSmallUnit; ++i) { const float x = v[i] - ck; dist[i] += (P == 2) ? x * x : fabsf(x); }
  }
  for (int off = 32; off > 0; off >>= 1) {
    c2 += __shfl_xor(c2, off, 64);
#pragma unroll
    for (int i = 0; i < kSmallUnit; ++i) dist[i] += __shfl_xor(dist[i], off, 64);
  }
  float rmax = 0.f;
#pragma unroll
  for (int i = 0; i < kSmallUnit; ++i)
    if (!(rm[i] < 0.f)) rmax = fmaxf(rmax, ((P == 2) ? sqrtf(dist[i]) : dist[i]) * (1.f + kBoundSlack) + rm[i]);
  if (lane == 0) {
    radU[u] = cntm > 0 ? rmax * (1.f + kBoundSlack) + 1e-30f : -1.f;
    cnormU[u] = cntm > 0 ? sqrtf(c2) * (1.f + kBoundSlack) : 0.f;
  }
}

// the micro-tile level of the test for one surviving unit pair and relation; `lane_count` lanes starting at
// `lane0` share the micro-tile pairs (1 lane = on the spot in the unit-level kernel, a block in k_bound_refine)
// a surviving join tile: its bit in the bitmap, and -- LIST: the first time -- its entry on the flat list (see
// k_batch_tiles).  A template parameter and not a test of a.list_count: with both forms in one kernel the atomic of the
// plain form became a returning one too, and a join with many surviving tiles (N = 1,000,000) lost a third of its
// bound test's speed.
template <bool LIST>
__device__ __forceinline__ void keep_tile(const BoundL2Args& a, int rl, int tH, int tT) {
  const int64_t row = (int64_t)rl * a.nH + tH;
  uint32_t* w = &a.bitmap[row * a.words_per_row + (tT >> 5)];
  const uint32_t bit = 1u << (tT & 31);
  if (*w & bit) return;                                          // (most micro-tile pairs of a tile find it set)
  if constexpr (!LIST) {
    atomicOr(w, bit);
  } else {
    const uint32_t old = atomicOr(w, bit);
    if (!(old & bit)) {
      const unsigned long long idx = atomicAdd(a.list_count, 1ull);
      if (idx < a.list_cap) { a.list_cols[idx] = (uint32_t)tT; a.list_rows[idx] = (uint32_t)row; a.list_active[idx] = (uint32_t)row; }
    }
  }
}
template <bool LIST>
__device__ __forceinline__ void refine_unit_pair(const BoundL2Args& a, const UnitTable& ut, int rl, int uH, int uT, int lane0,
                                                 int lane_count) {
  int fH, nHm, fT, nTm;
  unit_range(ut, uH, fH, nHm);
  unit_range(ut, uT, fT, nTm);
  const float rnq = a.rn[rl], srn = sqrtf(rnq);
  const float dsl = a.delta * (1.f + kBoundSlack);
  const float kk = 2.f * (float)(a.d + 12) * 6e-8f;
  const int64_t total = (int64_t)nHm * nTm;
  for (int64_t i = lane0; i < total; i += lane_count) {
    const int64_t mH = fH + i / nTm, mT = fT + i % nTm;
    const float rH = a.rad[mH], rT = a.rad[mT];
    if (rH < 0.f || rT < 0.f) continue;
    if (!a.D) {           // small problems: no matrices, the distance of c_H + r and c_T summed over d
      // (the coordinates c_H + r are rounded: 2^-24 (||c_H|| + ||r||) of distance, taken twice; see l1_reach)
      const float* cH = a.cent + mH * a.d;
      const float* cT = a.cent + mT * a.d;
      const int64_t so = (int64_t)(a.r0 + rl) * a.d;
      float sq = 0.f;
      for (int k = 0; k < a.d; ++k) {
        const float x = cH[k] + ld_elem(a.Rv, so + k, a.dtype) - cT[k];
        sq += x * x;
      }
      if (sqrtf(sq) * (1.f - kBoundSlack) - 1.2e-7f * (a.cnorm[mH] + srn) - rH - rT <= dsl) keep_tile<LIST>(a, rl, (int)(mH / a.micro_per_bm), (int)(mT / a.micro_per_bn));
      continue;
    }
    const float D = a.D[mH * a.n_micro + mT];
    const float reach = dsl + rH + rT;
    const float rhs = reach * reach * (1.f + kBoundSlack) + D * ((float)(a.d + 8) * 6e-8f) - D;
    const float ek = kk * (a.cnorm[mH] + a.cnorm[mT]);
    const float lhs = (2.f * a.u[(int64_t)rl * a.n_micro + mH] + rnq * (1.f - 2.4e-7f)) - 2.f * a.u[(int64_t)rl * a.n_micro + mT] -
                      ek * srn;
    if (lhs <= rhs) keep_tile<LIST>(a, rl, (int)(mH / a.micro_per_bm), (int)(mT / a.micro_per_bn));
  }
}

// Unit level: the flat kernel's arithmetic on unit summaries (a.D, a.u, a.rad, a.cnorm and a.n_micro then
// describe UNITS); survivors are appended to the list, or refined on the spot when the list is full.
// `fine` holds the micro-tile level arrays for that case.
template <bool LIST>
__global__ __launch_bounds__(256) void k_bound_l2_units(const BoundL2Args a, const BoundL2Args fine, const UnitTable ut,
                                                        const BoundPairs bp) {
  __shared__ float aH[kHeadChunk][kRelChunk];
  __shared__ float srnS[kRelChunk];
  __shared__ float radH[kHeadChunk], cnH[kHeadChunk];
  const int tid = threadIdx.x;
  const int64_t mT = (int64_t)blockIdx.x * blockDim.x + tid;
  const int64_t mH0 = (int64_t)blockIdx.y * kHeadChunk;
  const int rl0 = (int)blockIdx.z * kRelChunk;
  {
    const int q = tid / kHeadChunk, hq = tid % kHeadChunk;      // neighbouring threads on neighbouring heads: 64 bytes of a row of u
    const int rl = rl0 + q;
    const int64_t mH = mH0 + hq;
    const float rnq = rl < a.RB ? a.rn[rl] : 0.f;
    aH[hq][q] = (rl < a.RB && mH < a.n_micro) ? 2.f * a.u[(int64_t)rl * a.n_micro + mH] + rnq * (1.f - 2.4e-7f) : 0.f;
    if (tid < kRelChunk) srnS[tid] = sqrtf((rl0 + tid < a.RB) ? a.rn[rl0 + tid] : 0.f);
    if (tid < kHeadChunk) {
      const int64_t m = mH0 + tid;
      radH[tid] = m < a.n_micro ? a.rad[m] : -1.f;
      cnH[tid] = m < a.n_micro ? a.cnorm[m] : 0.f;
    }
  }
  __syncthreads();
  if (mT >= a.n_micro) return;
  const float rT = a.rad[mT];
  if (rT < 0.f || (mT >= a.both_from && mH0 >= a.both_from)) return;
  const float cT = a.cnorm[mT];
  float bT[kRelChunk];
  const int nrel = a.RB - rl0 < kRelChunk ? a.RB - rl0 : kRelChunk;
#pragma unroll
  for (int q = 0; q < kRelChunk; ++q) bT[q] = q < nrel ? 2.f * a.u[(int64_t)(rl0 + q) * a.n_micro + mT] : -3e38f;
  const float dsl = a.delta * (1.f + kBoundSlack);
  const float kk = 2.f * (float)(a.d + 12) * 6e-8f;
  // the centre distances of the block's heads, all loads in flight together (a head past the end reads the first row; it is skipped below)
  float Dv[kHeadChunk];
  {
    const float* Dp = a.D + mH0 * a.n_micro + mT;
    const int nvalid = a.n_micro - mH0 < kHeadChunk ? (int)(a.n_micro - mH0) : kHeadChunk;
#pragma unroll
    for (int hq = 0; hq < kHeadChunk; ++hq) Dv[hq] = Dp[hq < nvalid ? (int64_t)hq * a.n_micro : 0];
  }
#pragma unroll
  for (int hq = 0; hq < kHeadChunk; ++hq) {
    const float rH = radH[hq];
    if (rH < 0.f) continue;
    const int64_t mH = mH0 + hq;
    const float D = Dv[hq];
    const float reach = dsl + rH + rT;
    const float rhs = reach * reach * (1.f + kBoundSlack) + D * ((float)(a.d + 8) * 6e-8f) - D;
    const float ek = kk * (cnH[hq] + cT);
    uint32_t keep = 0u;
#pragma unroll
    for (int q = 0; q < kRelChunk; ++q) keep |= (aH[hq][q] - bT[q] - ek * srnS[q] <= rhs) ? (1u << q) : 0u;
    unit_pairs_out<LIST>(keep, rl0, (int)mH, (int)mT, fine, ut, bp);
  }
}

// L1 form of k_bound_refine (below): the listed unit pairs on their micro-tile summaries.
__global__ __launch_bounds__(256) void k_bound_refine_l1(const TileDistArgs a) {
  const unsigned long long n = *a.bp.count < a.bp.cap ? *a.bp.count : a.bp.cap;
  for (unsigned long long e = blockIdx.x; e < n; e += gridDim.x) {
    const unsigned long long v = a.bp.list[e];
    refine_unit_pair_l1(a, (int)(v >> 48), (int)((v >> 24) & 0xffffffull), (int)(v & 0xffffffull),
                        (int)(blockIdx.y * blockDim.x + threadIdx.x), (int)(gridDim.y * blockDim.x));
  }
}

// Micro-tile level for the listed unit pairs.  The grid strides over the list in x; the gridDim.y blocks of
// one x share the micro-tile pairs of an entry, so that a pair of large groups (millions of micro-tile pairs
// in one entry) does not hang on a single block.
template <bool LIST>
__global__ __launch_bounds__(256) void k_bound_refine(const BoundL2Args fine, const UnitTable ut, const BoundPairs bp) {
  const unsigned long long n = *bp.count < bp.cap ? *bp.count : bp.cap;
  for (unsigned long long e = blockIdx.x; e < n; e += gridDim.x) {
    const unsigned long long v = bp.list[e];
    refine_unit_pair<LIST>(fine, ut, (int)(v >> 48), (int)((v >> 24) & 0xffffffull), (int)(v & 0xffffffull),
                     (int)(blockIdx.y * blockDim.x + threadIdx.x), (int)(gridDim.y * blockDim.x));
  }
}

// Tile lists from the bitmap.  A wave takes kBitmapRowsPerLane x 64 (relation, head tile) rows: every lane counts
// the surviving tail tiles of its rows (almost all rows are empty); the wave reserves its part of the column list and
// of the active-row list with ONE atomic each (thousands of atomics on the same two counters cost more than the
// whole scan), and the rows that have tiles are then written out by the whole wave, one row after the other, tile
// numbers ascending.
constexpr int kBitmapRowsPerLane = 8;
constexpr int kBitmapShortWords = 64;
// (few rows: one per lane, so that more waves write out the lists, a chain per row; 7,500 rows that all have tiles: 284 -> 43 us)
constexpr int64_t kBitmapFewRows = 1 << 15;
__host__ __device__ inline int bitmap_rows_per_lane(int words_per_row, int64_t n_rows) {
  return words_per_row <= kBitmapShortWords && n_rows > kBitmapFewRows ? kBitmapRowsPerLane : 1;
}
__global__ __launch_bounds__(256) void k_rows_from_bitmap(const uint32_t* __restrict__ bitmap, int words_per_row,
                                                         int64_t n_rows, uint32_t* __restrict__ row_start,
                                                         uint32_t* __restrict__ row_count, uint32_t* __restrict__ cols,
                                                         unsigned long long* __restrict__ total,
                                                         uint32_t* __restrict__ active_rows,
                                                         unsigned int* __restrict__ n_active,
                                                         uint32_t* __restrict__ tile_rows,        // may be NULL: the row of every entry of cols
                                                         int nH = 1, int h0 = 0, int h1 = 0x7fffffff,     // window: only head tiles [h0, h1)
                                                         int t0 = 0, int t1 = 0x7fffffff,                 // ... and tail tiles [t0, t1) count
                                                         const unsigned int* skip = nullptr,              // non-zero: the lists exist already, nothing to do
                                                         unsigned long long* tiles_total = nullptr,       // running total of listed tiles (with skip)
                                                         int xh = 0x7fffffff, int xt = 0x7fffffff) {      // tiles with head >= xh and tail >= xt do not count
  if (skip && *skip) return;
  // word i of a row holds tail tiles 32 i .. 32 i + 31: the bits of those inside [t0, t1)
  auto col_mask = [=](int i, int64_t row) -> uint32_t {
    const int end = xt < t1 && (int)(row % nH) >= xh ? xt : t1;
    const int lo = t0 - 32 * i, hi = end - 32 * i;
    if (hi <= 0 || lo >= 32) return 0u;
    const uint32_t mlo = lo <= 0 ? 0xffffffffu : 0xffffffffu << lo;
    const uint32_t mhi = hi >= 32 ? 0xffffffffu : (1u << hi) - 1u;
    return mlo & mhi;
  };
  auto row_in = [=](int64_t row) -> bool { const int tH = (int)(row % nH); return tH >= h0 && tH < h1; };
  const int lane = threadIdx.x & 63;
  // rows of up to kBitmapShortWords words are counted one per lane, kBitmapRowsPerLane of them; longer rows by the
  // whole wave, one after the other, 64 per wave
  const int rpl = bitmap_rows_per_lane(words_per_row, n_rows);
  const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * (64 * rpl);
  if (row0 >= n_rows) return;                                  // whole waves leave together
  uint32_t cnt[kBitmapRowsPerLane];
#pragma unroll
  for (int k = 0; k < kBitmapRowsPerLane; ++k) {
    const int64_t base_row = row0 + k * 64;
    cnt[k] = 0;
    if (k >= rpl) continue;
    if (words_per_row <= kBitmapShortWords) {   // short rows: every lane counts its own
      if (base_row + lane < n_rows && row_in(base_row + lane)) {
        const uint32_t* w = bitmap + (base_row + lane) * words_per_row;
        for (int i = 0; i < words_per_row; ++i) cnt[k] += __builtin_popcount(w[i] & col_mask(i, base_row + lane));
      }
    } else {                                 // long rows: the wave counts them one after the other, words over lanes
      // eight rows at a time, their words in flight together (one row after the other was a chain of memory round trips:
      // 0.40 ms per batch of 200,000 rows of 500 bytes on the N = 1,000,000 workload)
      for (int rr = 0; rr < 64 && base_row + rr < n_rows; rr += 8) {
        uint32_t c[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) c[j] = 0u;
        for (int i = lane; i < words_per_row; i += 64) {
          uint32_t v[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int64_t row = base_row + rr + j < n_rows ? base_row + rr + j : base_row + rr;      // (past the end: a valid row, dropped)
            v[j] = bitmap[row * words_per_row + i];
          }
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (v[j]) c[j] += __builtin_popcount(v[j] & col_mask(i, base_row + rr + j));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (__builtin_amdgcn_ballot_w64(c[j] != 0u) == 0ull) continue;      // (most rows)
          for (int off = 32; off > 0; off >>= 1) c[j] += __shfl_xor(c[j], off, 64);
          if (lane == rr + j && base_row + rr + j < n_rows && row_in(base_row + rr + j)) cnt[k] = c[j];
        }
      }
    }
  }
  // this lane's tiles and rows, their exclusive prefix over the wave, one reservation per wave
  uint32_t ltiles = 0, lrows = 0;
#pragma unroll
  for (int k = 0; k < kBitmapRowsPerLane; ++k) { ltiles += cnt[k]; lrows += cnt[k] ? 1u : 0u; }
  uint32_t ptiles = ltiles, prows = lrows;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t ot = __shfl_up(ptiles, off, 64), orw = __shfl_up(prows, off, 64);
    if (lane >= off) { ptiles += ot; prows += orw; }
  }
  const uint32_t wtiles = __shfl(ptiles, 63, 64), wrows = __shfl(prows, 63, 64);
  unsigned long long wbase = 0;
  unsigned int abase = 0;
  if (lane == 0 && wrows) {
    wbase = atomicAdd(total, (unsigned long long)wtiles);
    abase = atomicAdd(n_active, wrows);
    if (tiles_total) atomicAdd(tiles_total, (unsigned long long)wtiles);
  }
  wbase = ((unsigned long long)(uint32_t)__shfl((int)(uint32_t)(wbase >> 32), 0, 64) << 32) |
          (uint32_t)__shfl((int)(uint32_t)(wbase & 0xffffffffull), 0, 64);
  abase = (unsigned int)__shfl((int)abase, 0, 64);
  unsigned long long my_base = wbase + (ptiles - ltiles);
  unsigned int my_act = abase + (prows - lrows);
  unsigned long long bases[kBitmapRowsPerLane];
#pragma unroll
  for (int k = 0; k < kBitmapRowsPerLane; ++k) {
    const int64_t my_row = row0 + k * 64 + lane;
    bases[k] = cnt[k] ? my_base : 0ull;
    if (k < rpl && my_row < n_rows) {
      row_start[my_row] = (uint32_t)bases[k];
      row_count[my_row] = cnt[k];
      if (cnt[k]) active_rows[my_act++] = (uint32_t)my_row;   // rows that still have work, in any order
    }
    my_base += cnt[k];
  }
  if (!wrows) return;
#pragma unroll 1
  for (int k = 0; k < rpl; ++k) {
    uint32_t c = 0;
    unsigned long long bk = 0;
#pragma unroll
    for (int q = 0; q < kBitmapRowsPerLane; ++q) { c = (q == k) ? cnt[q] : c; bk = (q == k) ? bases[q] : bk; }
    unsigned long long live = __builtin_amdgcn_ballot_w64(c != 0u);
    while (live) {
      const int src = (int)__builtin_ctzll(live);
      live &= live - 1ull;
      const unsigned long long base = ((unsigned long long)(uint32_t)__shfl((int)(uint32_t)(bk >> 32), src, 64) << 32) |
                                      (uint32_t)__shfl((int)(uint32_t)(bk & 0xffffffffull), src, 64);
      const uint32_t* w = bitmap + (row0 + k * 64 + src) * words_per_row;
      // ascending order: words in chunks of 64, prefix of popcounts across lanes
      uint32_t run = 0;
      for (int i0 = 0; i0 < words_per_row; i0 += 64) {
        const int i = i0 + lane;
        uint32_t word = i < words_per_row ? (w[i] & col_mask(i, row0 + k * 64 + src)) : 0u;
        const uint32_t pc = __builtin_popcount(word);
        uint32_t pre = pc;
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t o = __shfl_up(pre, off, 64);
          if (lane >= off) pre += o;
        }
        uint32_t pos = run + pre - pc;
        while (word) {
          const int bit = __builtin_ctz(word);
          word &= word - 1;
          if (tile_rows) tile_rows[base + pos] = (uint32_t)(row0 + k * 64 + src);
          cols[base + pos++] = (uint32_t)(i * 32 + bit);
        }
        run += __shfl(pre, 63, 64);
      }
    }
  }
}

// The bound once more for the sixteen micro-tile pairs of every surviving 128 x 128 tile of a pruned L1 join (k_l1_blocks): a wave
// takes tiles of one row, a lane per dimension.  A tile is a few memory round trips, so a batch of few rows, whose tiles a wave each
// would walk alone, deals every row's tiles to as many waves as there are for it.  The waves end once more blocks are listed than
// l1_by_blocks accepts (*count only grows, and keeps within 256 a wave of that line): the batch then goes by whole tiles.  That is
// mostly known far earlier: every eighth wave reports its first tile, one anywhere in its row, and the first report after which
// those hold clearly more blocks than the line (eight a tile, six are allowed) puts *count past it: N = 16,000, R = 40, 625,000
// tiles with all blocks within reach: 697 us with the line alone, 16 with the reports, beside 26.6 ms for the whole tiles.
// Atomics on one word are served one after the other, 8 ns each, so a workgroup asks for the last entries of its waves' queues
// at once, and only its first wave flushes early, to see the count for all four (4,959, 7, 39: 28 us with 64 entries a wave, 17
// so; N = 15,000, R = 64, by blocks: 44 and 30).  (More waves, or a look at the reports at every flush, cost more than they saved.)
struct L1MicroArgs {
  const uint32_t* row_start; const uint32_t* row_count; const uint32_t* cols; const uint32_t* active_rows;      // see JoinStreamArgs
  const unsigned int* n_active;
  int nH, r0;
  const float* cent_h; const float* rad_h; const float* cent_t; const float* rad_t;      // micro-tile summaries of heads and tails ...
  int64_t h_rel, t_rel;                // ... and how many of them per relation (0: the same for all)
  const void* shift; int dtype, d;     // added to the heads' centres: shift[(r0 + relation) * d ...] (NULL: nothing)
  float delta; const JoinParams* prm;  // (see l1_reach)
  ExactEntry* list; unsigned int* count; unsigned int cap;      // surviving blocks: relation, first head slot, first tail slot
  const unsigned long long* tiles; unsigned int most;           // see l1_by_blocks
  unsigned long long* sample;                                   // sampled tiles << 32 | their blocks
};
constexpr unsigned int kL1SampleTiles = 64, kL1SampleBlocks = 8;      // tiles a decision takes at least, and blocks a tile it takes more than
constexpr unsigned int kL1Whole = 0x80000000u;                  // *count of a batch that was sent to whole tiles early (more than may be listed)
constexpr int kL1MicroQueue = 256, kL1MicroEarly = 64;      // blocks a wave holds back, and the first of a workgroup
__global__ __launch_bounds__(256) void k_l1_micro_pairs(const L1MicroArgs a) {
  static_assert(kL1Tile == 4 * 32, "four micro-tiles a side");
  __shared__ int32_t queue[4][3][kL1MicroQueue];
  __shared__ int stop_s, qn_s[4];
  __shared__ unsigned int base_s;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int32_t (&q)[3][kL1MicroQueue] = queue[wave];
  const int room = wave == 0 ? kL1MicroEarly : kL1MicroQueue;
  int qn = 0;
  if (threadIdx.x == 0) stop_s = 0;
  __syncthreads();
  const unsigned int line = l1_block_line(a.tiles, a.most);
  const bool early = *a.tiles * kL1SampleBlocks > line;
  bool report = ((blockIdx.x * 4u + (unsigned)wave) & 7u) == 0u && early;
  bool over = false;                   // more blocks than the line, as of a flush of this workgroup (or *count put past it)
  auto flush = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    unsigned int base = 0u;
    if (lane == 0) base = atomicAdd(a.count, (unsigned int)qn);
    base = (unsigned int)__builtin_amdgcn_readfirstlane((int)base);
    for (int k = lane; k < qn && base + (unsigned)k < a.cap; k += 64) a.list[base + (unsigned)k] = ExactEntry{q[0][k], q[1][k], q[2][k], 0};
    if (base + (unsigned)qn > line) {
      over = true;
      __hip_atomic_store(&stop_s, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    qn = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
  };
  const unsigned int n_rows = *a.n_active;
  const float reach = l1_reach(a.delta, a.prm);
  const unsigned int waves = gridDim.x * 4u, me = blockIdx.x * 4u + (unsigned)wave;
  const unsigned int parts = n_rows >= waves ? 1u : waves / (n_rows ? n_rows : 1u);      // of a row (a part past its tiles is empty)
  for (unsigned int item = me; item < n_rows * parts && !over; item += waves) {
    const unsigned int i = item % n_rows, part = item / n_rows;
    const int64_t row = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a.active_rows[i]);
    const int rl = (int)(row / a.nH), tH = (int)(row - (int64_t)rl * a.nH);
    const int64_t mh = rl * a.h_rel + tH * 4;
    const int t0 = __builtin_amdgcn_readfirstlane((int)a.row_start[row]), nt = __builtin_amdgcn_readfirstlane((int)a.row_count[row]);
    const unsigned int mine = (unsigned)nt > part ? ((unsigned)nt - part + parts - 1u) / parts : 0u;
    unsigned int turn = mine ? ((me * 0x9E3779B1u) >> 8) % mine : 0u;      // (a sample of first tiles alone would be one of the rows' largest groups)
    const int p = lane >> 2;           // the pair that this lane will hold the total of: head micro-tile p / 4, tail micro-tile p % 4
    const float rh = a.rad_h[mh + (p >> 2)];
    int tT_next = mine ? (int)a.cols[t0 + (int)(part + turn * parts)] : 0;
    for (unsigned int left = mine; left; --left) {
      over = over || __builtin_amdgcn_readfirstlane(__hip_atomic_load(&stop_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != 0;
      if (over) break;
      const int tT = __builtin_amdgcn_readfirstlane(tT_next);
      const int64_t mt = rl * a.t_rel + (int64_t)tT * 4;
      const float rt = a.rad_t[mt + (p & 3)];
      turn = turn + 1u < mine ? turn + 1u : 0u;
      tT_next = (int)a.cols[t0 + (int)(part + turn * parts)];      // (the last turn asks for the first again)
      float s[16];                     // this lane's part of the distance of the sixteen pairs
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] = 0.f;
      for (int k = lane; k < a.d; k += 64) {
        float h[4], c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { h[j] = a.cent_h[(mh + j) * a.d + k]; c[j] = a.cent_t[(mt + j) * a.d + k]; }
        const float sh = a.shift ? ld_elem(a.shift, (int64_t)(a.r0 + rl) * a.d + k, a.dtype) : 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] += fabsf(h[j >> 2] + sh - c[j & 3]);
      }
      // totals by halving exchanges: lane l ends up with pair 8 b5 + 4 b4 + 2 b3 + b2 (bits of l)
      const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4;
      float s8[8], s4[4], s2[2], s1;
#pragma unroll
      for (int j = 0; j < 8; ++j) s8[j] = (b5 ? s[j + 8] : s[j]) + __shfl_xor(b5 ? s[j] : s[j + 8], 32, 64);
#pragma unroll
      for (int j = 0; j < 4; ++j) s4[j] = (b4 ? s8[j + 4] : s8[j]) + __shfl_xor(b4 ? s8[j] : s8[j + 4], 16, 64);
#pragma unroll
      for (int j = 0; j < 2; ++j) s2[j] = (b3 ? s4[j + 2] : s4[j]) + __shfl_xor(b3 ? s4[j] : s4[j + 2], 8, 64);
      s1 = (b2 ? s2[1] : s2[0]) + __shfl_xor(b2 ? s2[0] : s2[1], 4, 64);
      s1 += __shfl_xor(s1, 2, 64);
      s1 += __shfl_xor(s1, 1, 64);
      // (the bound of k_tile_dist's BOUND form; an empty micro-tile has radius -1)
      const bool keep = (lane & 3) == 0 && rh >= 0.f && rt >= 0.f && !(s1 * (1.f - kBoundSlack) - rh - rt > reach);
      const unsigned long long b = __builtin_amdgcn_ballot_w64(keep);
      const int n = __builtin_popcountll(b);
      if (report) {
        if (lane == 0) {
          const unsigned long long s = atomicAdd(a.sample, (1ull << 32) | (unsigned long long)n) + ((1ull << 32) | (unsigned long long)n);
          const unsigned int seen = (unsigned int)(s >> 32);
          if (seen >= kL1SampleTiles && (unsigned int)s > seen * kL1SampleBlocks) atomicMax(a.count, kL1Whole);
        }
        report = false;
      }
      if (qn + n > room) flush();
      if (keep) {
        const int pos = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
        q[0][pos] = a.r0 + rl; q[1][pos] = tH * kL1Tile + (p >> 2) * 32; q[2][pos] = tT * kL1Tile + (p & 3) * 32;
      }
      qn += n;
    }
  }
  // what the four waves still hold, by one atomic (where the batch goes by whole tiles nobody reads it)
  if (lane == 0) qn_s[wave] = qn;
  __syncthreads();
  const int all = qn_s[0] + qn_s[1] + qn_s[2] + qn_s[3];
  if (stop_s || all == 0) return;                                  // (the same for the workgroup)
  if (threadIdx.x == 0) base_s = atomicAdd(a.count, (unsigned int)all);
  __syncthreads();
  unsigned int base = base_s;
  for (int w = 0; w < wave; ++w) base += (unsigned)qn_s[w];
  for (int k = lane; k < qn && base + (unsigned)k < a.cap; k += 64) a.list[base + (unsigned)k] = ExactEntry{q[0][k], q[1][k], q[2][k], 0};
}

}  // namespace kgc
