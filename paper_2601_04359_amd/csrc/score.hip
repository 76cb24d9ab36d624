// pc_score: importance of every cached key = the softmax probability (Eq. 2) it receives,
// summed over the scoring queries and the query heads of its KV group.
//
// Two passes over Q K^T, both on the 32x32x16 bf16 MFMA and both free of atomics so the
// result is bit-reproducible:
//   1. row pass:    log-sum-exp of every scoring query over all keys (keys split over
//                   work-groups, partial (reference, sum) pairs merged in a fixed order; the
//                   reference is refreshed only when a partial sum runs away);
//   2. column pass: p = exp2(c*s - lse2) with the FINAL normaliser, un-rounded, in fp32,
//                   summed down the query axis (queries split over work-groups, partial
//                   sums added in a fixed order).
// A caller that already has the log-sum-exp skips pass 1.  With scale = ln 2 (the caller folded
// scale * log2(e) into the queries, c == 1) the products of pass 2 start from minus the
// normaliser instead of zero, so an element arrives as s - lse2 and costs a bare exp2.
//
// Both passes have the same shape.  One operand is stationary: every wave keeps 64 of its
// rows as MFMA fragments in registers for the whole kernel (queries in pass 1, keys in
// pass 2).  The other operand streams through a four-slot LDS ring in tiles of 64 rows,
// fetched by direct global->LDS loads three tiles ahead, one work-group barrier per tile.
// Each element of the product costs one exponential, so both passes are bound by the vector
// pipe, not the matrix pipe; matrix and vector instructions overlap only inside one wave's
// instruction stream, so every wave interleaves the 16 products of the next half tile with
// the exponentials of the one before.  Small calls take a form of either pass in which the eight
// waves share 64 stationary rows and deal the streamed rows among them.  The scoring rows of a
// KV head are numbered head after head, so a tile of them may span heads.
#include <limits.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "lds_dma.h"

namespace pc {
namespace {

constexpr int kD = 128;
constexpr int kThreads = 512;        // 8 waves, two per SIMD
constexpr int kWaveRows = 64;        // stationary rows per wave (two 32-row MFMA blocks)
constexpr int kBlockRows = 8 * kWaveRows;
constexpr int kTileRows = 64;        // streamed rows per LDS slot
constexpr int kRowBytes = kD * 2;
constexpr int kTileBytes = kTileRows * kRowBytes;
constexpr int kStages = 4;
constexpr size_t kRowSmem = kStages * kTileBytes + 8 * 32 * kRowBytes;   // the ring, 32 stationary rows per wave
constexpr int kPrepTiles = 64;       // tiles whose rows pass 2 prepares in LDS at a time
constexpr int kPrepRows = (kPrepTiles + kStages) * kTileRows;
constexpr size_t kColSmem = kStages * kTileBytes + kPrepRows * 12;
constexpr int kMaxSplits = 32;       // key splits of pass 1
constexpr int kMaxQSplits = 8;       // query splits of pass 2
constexpr float kNoMax = -1e30f;     // finite stand-in for "no key seen yet"

// Every staging point issues kTileLoads direct loads per wave and nothing else is in flight in the loops:
// waiting until at most that many are leaves only the newest point outstanding.
constexpr int kTileLoads = kTileBytes / (kThreads * 16);
static_assert(kTileLoads == 2, "dma_wait_all_but_newest encodes it");
__device__ __forceinline__ void dma_wait_all_but_newest() { asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); }

// Fetch the two 1-KB pieces of a 64-row tile this wave is responsible for; src(row) is the
// global address of streamed row `row` of the tile.
template <class Src>
__device__ __forceinline__ void stage_rows(Src&& src, uint32_t lds_tile, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (wave * 2 + i) * 4 + (lane >> 4);
    const int chunk = k_chunk_pos(row, lane & 15);
    dma_16B(src(row, i) + chunk * 8, lds_tile + (wave * 2 + i) * 1024);
  }
}

// acc[b] = init(b) + (32 streamed rows at `half`) x (stationary block b)^T, 16 products; after
// each product epi(i) runs one sixteenth of the vector work of the previous half tile.
// kInit = false: the products start from zero and init is not called.
// ring holds the first four fragments of `half` on entry (fetched while the phase before ran) and
// the first four of `next_half` on exit, so that no phase starts by waiting for LDS.
template <bool kInit, class Init, class Epi>
__device__ __forceinline__ void stream_phase(const lds_u8* half, const lds_u8* next_half, const int (&a_off)[8],
                                             const bf16x8 (&st)[2][8], f32x16 (&acc)[2], Init&& init, Epi&& epi,
                                             bf16x8 (&ring)[4]) {
  f32x16 zero;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero[i] = 0.f;
  // issue priority over the SIMD neighbour while inside the interleaved block (measured: +2-3 %)
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const bf16x8 a = ring[s & 3];
    ring[s & 3] = s + 4 < 8 ? lds_frag(half + a_off[s + 4]) : lds_frag(next_half + a_off[s - 4]);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (kInit)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, st[b][s], s == 0 ? init(b) : acc[b], 0, 0, 0);
      else
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, st[b][s], s == 0 ? zero : acc[b], 0, 0, 0);
      epi(s * 2 + b);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// ---- pass 1: per-query (max, sum) over a slice of the keys ---------------------------------
// S^T = K Q^T: a lane owns one query column of each stationary block and 16 of the 32 keys
// of the half tile, and keeps its own running (max, sum) over the keys it sees; the two
// halves of the wave are merged once at the end.
struct RowState {
  float m[2], l[2];
};
struct NoInit {
  __device__ const f32x16& operator()(int) const { __builtin_unreachable(); }
};
constexpr float kRowTrigger = 1024.f;  // phase sum that forces a new reference maximum

// Element pair i of the previous half tile: p = exp2(c s - m) against the reference as it
// stands, summed into the phase's partial sums.  No maximum is taken here.  kZeroRef: c is 1 and
// every reference of the wave is 0, so an element is a bare exp2.
template <bool kZeroRef = false>
__device__ __forceinline__ void row_epilogue(int i, const f32x16 (&s)[2], const RowState& st, float (&psum)[2],
                                             float c) {
  const int b = i >> 3, e = (i & 7) * 2;
#pragma unroll
  for (int k = 0; k < 2; ++k)
    psum[b] += __builtin_amdgcn_exp2f(kZeroRef ? s[b][e + k] : fmaf(s[b][e + k], c, -st.m[b]));
}
// After the phase: add the partial sums; if one ran away (a score outgrew the reference, or
// the reference is still the initial sentinel) redo that half tile against its exact maximum.
// kZeroRef: the sums may grow to 2^100 instead; zero_ref is cleared by a redo, and every half tile
// after it is redone until the caller has left the loop for the general one.
template <bool kZeroRef = false>
__device__ __forceinline__ void row_commit(const f32x16 (&s)[2], RowState& st, float (&psum)[2], float c,
                                           bool& zero_ref) {
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    asm volatile("" : "+v"(psum[b]));
    if (kZeroRef ? !zero_ref || __any(!(psum[b] <= 0x1p100f)) : __any(!(psum[b] <= kRowTrigger))) {
      if (kZeroRef) zero_ref = false;
      float mx = fmaxf(s[b][0], s[b][1]);
#pragma unroll
      for (int k = 2; k < 16; k += 2) mx = fmaxf(mx, fmaxf(s[b][k], s[b][k + 1]));
      const float m_new = fmaxf(st.m[b], mx * c);
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < 16; ++k) sum += __builtin_amdgcn_exp2f(fmaf(s[b][k], c, -m_new));
      st.l[b] = st.l[b] * __builtin_amdgcn_exp2f(st.m[b] - m_new) + sum;
      st.m[b] = m_new;
    } else {
      st.l[b] += psum[b];
    }
    psum[b] = 0.f;
  }
}

__device__ __forceinline__ void mask_keys(f32x16 (&s)[2], int k0, int Nk, int g) {
#pragma unroll
  for (int i = 0; i < 16; ++i)
    if (k0 + (i >> 2) * 8 + g * 4 + (i & 3) >= Nk) {
      s[0][i] = -INFINITY;
      s[1][i] = -INFINITY;
    }
}

// kUnitC (c == 1, the caller folded the scale into the queries): as long as no score is large, the
// probabilities are summed against a reference of zero, which takes the multiply-add out of the loop
// (a score's exponential is within fp32's range from 2^-126 to 2^127, so a sum against zero is as good
// as one against the maximum).  The first half tile decides: scores within +-60 there bound the sum
// from below by 2^-60, and a sum above 2^100 later sends the wave to the general loop.  16 heads x 512
// rows x 100,000 keys: 198 -> 185 us.
template <bool kUnitC>
__global__ __launch_bounds__(kThreads, 1) void score_rowpass_bf16(
    const uint16_t* __restrict__ Qs, const int32_t* __restrict__ q_rows, const uint16_t* __restrict__ K,
    float2* __restrict__ part, int rep, Divisor by_qs, int Nk, int64_t q_stride_h, int64_t k_stride_h, float c,
    Divisor by_tiles, Divisor by_heads, int per) {
  extern __shared__ __align__(16) uint8_t smem_raw[];
  lds_u8* smem = (lds_u8*)smem_raw;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  // logical order: split slowest, so the work-groups of one XCD stream the same keys
  const int L = xcd_contiguous_index(blockIdx.x, gridDim.x);
  const int unit = by_tiles.of(L), tile = L - unit * by_tiles.d, Hkv = by_heads.d;
  const int split = by_heads.of(unit), kvh = unit - split * Hkv;
  const int n_rows = rep * by_qs.d;   // scoring rows of the KV head's group, numbered head after head
  const int row0 = tile * kBlockRows + wave * kWaveRows;
  const uint16_t* Kh = K + kvh * k_stride_h;

  const int n_tiles = (Nk + kTileRows - 1) / kTileRows;
  const int t_begin = min(split * per, n_tiles), t_end = min(t_begin + per, n_tiles);
  const int n = t_end - t_begin;
  if (n <= 0) {  // the host never launches an empty split; keep the partials defined anyway
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int rho = row0 + b * 32 + l32;
      if (g == 0 && rho < n_rows) part[(static_cast<int64_t>(split) * Hkv + kvh) * n_rows + rho] = make_float2(kNoMax, 0.f);
    }
    return;
  }

  int a_off[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) a_off[s] = l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  auto stage = [&](int j) {  // tile j of this split (clamped: a repeat of the last tile is never read)
    const RowWindow w = row_window(Kh, (t_begin + min(j, n - 1)) * kTileRows, Nk);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = (wave * 2 + i) * 4 + (lane >> 4);
      dma_16B_at(w.base, row_offset(w, row, k_chunk_pos(row, lane & 15)),
                 lds0 + (j & (kStages - 1)) * kTileBytes + (wave * 2 + i) * 1024);
    }
  };
  auto slot = [&](int j) { return smem + (j & (kStages - 1)) * kTileBytes; };

  RowState st;
  st.m[0] = st.m[1] = kNoMax;
  st.l[0] = st.l[1] = 0.f;
  f32x16 sA[2], sB[2];

  float psum[2] = {0.f, 0.f};
  // The wave's 64 rows come through LDS of its own as whole rows, 32 at a time, between the first fetches (as
  // fragments from memory they were 32 bytes of a row per load, lines evicted between loads).  Lane l finds
  // row l.
  bf16x8 qf[2][8];
  {
    int64_t at;
    {
      const int r = min(row0 + lane, n_rows - 1), in_group = by_qs.of(r);
      int row = r - in_group * by_qs.d;
      if (q_rows) row = q_rows[row];
      asm volatile("" : "+v"(row));
      at = (kvh * rep + in_group) * q_stride_h + static_cast<int64_t>(row) * kD;
    }
    const uint32_t mine = kStages * kTileBytes + wave * 32 * kRowBytes;
    auto fetch = [&](int b) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = i * 4 + (lane >> 4);
        dma_16B(Qs + __shfl(at, b * 32 + row) + k_chunk_pos(row, lane & 15) * 8,
                __builtin_amdgcn_readfirstlane(lds0 + mine + i * 1024));
      }
    };
    auto take = [&](int b) {
#pragma unroll
      for (int s = 0; s < 8; ++s) qf[b][s] = lds_frag(smem + mine + a_off[s]);
#pragma unroll
      for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qf[b][s]));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    fetch(0);
    stage(0);
    asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
    take(0);
    fetch(1);
    stage(1);
    stage(2);
    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    take(1);
  }
  __syncthreads();   // the first tile has landed: it was fetched before the second half of the rows
  bf16x8 ring[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) ring[r] = lds_frag(slot(0) + a_off[r]);
  stream_phase<false>(slot(0), slot(0) + 32 * kRowBytes, a_off, qf, sA, NoInit{}, [](int) {}, ring);
  bool zero_ref = false;  // wave-uniform
  if constexpr (kUnitC) {
    float lo = sA[0][0], hi = sA[0][0];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      float mx = sA[b][0];
#pragma unroll
      for (int k = 1; k < 16; ++k) mx = fmaxf(mx, sA[b][k]);
      lo = b == 0 ? mx : fminf(lo, mx);
      hi = b == 0 ? mx : fmaxf(hi, mx);
    }
    zero_ref = __all(lo >= -60.f && hi <= 60.f);
    if (zero_ref) st.m[0] = st.m[1] = 0.f;
  }
  // Tile j lives in LDS slot j % 4; the loop is unrolled over the slots so that their bases are
  // immediates of the LDS reads.
  auto tile_body = [&](int j, auto slot_tag, auto zero_tag) {
    constexpr int u = decltype(slot_tag)::value;
    constexpr bool kZero = decltype(zero_tag)::value;
    const bool tail = (t_begin + j + 1) * kTileRows > Nk;  // only ever the last tile
    dma_wait_all_but_newest();
    __syncthreads();  // tile j+1 has landed everywhere; slot of tile j-1 is free
    stage(j + 3);
    if (tail) mask_keys(sA, (t_begin + j) * kTileRows, Nk, g);
    stream_phase<false>(smem + u * kTileBytes + 32 * kRowBytes, smem + ((u + 1) & 3) * kTileBytes, a_off, qf, sB, NoInit{},
                        [&](int i) { row_epilogue<kZero>(i, sA, st, psum, c); }, ring);
    row_commit<kZero>(sA, st, psum, c, zero_ref);
    if (tail) mask_keys(sB, (t_begin + j) * kTileRows + 32, Nk, g);
    if (j + 1 < n) {
      stream_phase<false>(smem + ((u + 1) & 3) * kTileBytes, smem + ((u + 1) & 3) * kTileBytes + 32 * kRowBytes, a_off, qf,
                          sA, NoInit{}, [&](int i) { row_epilogue<kZero>(i, sB, st, psum, c); }, ring);
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) row_epilogue<kZero>(i, sB, st, psum, c);
    }
    row_commit<kZero>(sB, st, psum, c, zero_ref);
  };
  // four tiles of either loop; the loops hand over between such groups, where the slots agree
  auto four_tiles = [&](int j0, auto zero_tag) {
    tile_body(j0, std::integral_constant<int, 0>{}, zero_tag);
    if (j0 + 1 >= n) return;
    tile_body(j0 + 1, std::integral_constant<int, 1>{}, zero_tag);
    if (j0 + 2 >= n) return;
    tile_body(j0 + 2, std::integral_constant<int, 2>{}, zero_tag);
    if (j0 + 3 >= n) return;
    tile_body(j0 + 3, std::integral_constant<int, 3>{}, zero_tag);
  };
  int j0 = 0;
  if constexpr (kUnitC)
    for (; j0 < n && zero_ref; j0 += kStages) four_tiles(j0, std::true_type{});
  for (; j0 < n; j0 += kStages) four_tiles(j0, std::false_type{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no direct load may outlive the work-group

#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float m_o = wave_half_swap(st.m[b]), l_o = wave_half_swap(st.l[b]);
    const float m = fmaxf(st.m[b], m_o);
    const float l = st.l[b] * __builtin_amdgcn_exp2f(st.m[b] - m) + l_o * __builtin_amdgcn_exp2f(m_o - m);
    const int rho = row0 + b * 32 + l32;
    if (g == 0 && rho < n_rows) part[(static_cast<int64_t>(split) * Hkv + kvh) * n_rows + rho] = make_float2(m, l);
  }
}

// Negated base-2 normalisers of the scoring rows of KV head kvh (numbered head after head), from one of
// three sources: an array of them (`ready`), the caller's natural-log LSE (`lse`, indexed like the rows
// of Qs), or the row pass's n_splits (reference, sum) pairs, merged in split order: -log2 sum_j
// 2^(c * s_j).  Rows past the last one give -inf: they add nothing.
struct RowNorm {
  const float* ready;        // [Hkv][rep * n_qs], or NULL
  const float* lse;          // the caller's, or NULL
  int64_t lse_stride_h;
  const int32_t* q_rows;
  const float2* part;        // [split][Hkv][rep * n_qs]
  int64_t part_stride;       // Hkv * rep * n_qs
  int n_splits, rep;
  Divisor by_qs;             // by n_qs
};
// v[i]: row rho0 + i * step.  The loads of all of them are in flight together.
template <int kN>
__device__ __forceinline__ void row_norms(const RowNorm& a, int kvh, int rho0, int step, float (&v)[kN]) {
  const int n_rows = a.rep * a.by_qs.d;
  if (a.ready) {
#pragma unroll
    for (int i = 0; i < kN; ++i) v[i] = a.ready[static_cast<int64_t>(kvh) * n_rows + min(rho0 + i * step, n_rows - 1)];
  } else if (a.lse) {
    int head[kN], row[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const int rho = min(rho0 + i * step, n_rows - 1), in_group = a.by_qs.of(rho);
      head[i] = kvh * a.rep + in_group;
      row[i] = rho - in_group * a.by_qs.d;
      if (a.q_rows) row[i] = a.q_rows[row[i]];
    }
#pragma unroll
    for (int i = 0; i < kN; ++i) v[i] = a.lse[head[i] * a.lse_stride_h + row[i]];
#pragma unroll
    for (int i = 0; i < kN; ++i) v[i] *= -1.4426950408889634f;
  } else {
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      if (rho0 - static_cast<int>(threadIdx.x) + i * step >= n_rows) break;   // no thread has a row left
      const float2* p = a.part + static_cast<int64_t>(kvh) * n_rows + min(rho0 + i * step, n_rows - 1);
      constexpr int kBatch = 8;
      float m = -INFINITY, l = 0.f;
      for (int s0 = 0; s0 < a.n_splits; s0 += kBatch) {
        float2 x[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) x[q] = p[min(s0 + q, a.n_splits - 1) * a.part_stride];
        float mb = m;
#pragma unroll
        for (int q = 0; q < kBatch; ++q) mb = fmaxf(mb, x[q].x);
        l *= __builtin_amdgcn_exp2f(m - mb);       // first batch: 0 * exp2(-inf)
        m = mb;
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
          if (s0 + q < a.n_splits && x[q].y > 0.f) l += x[q].y * __builtin_amdgcn_exp2f(x[q].x - m);
      }
      // the logarithm is taken of l's significand: an ulp of it is then far below one of the result
      v[i] = -(m + (static_cast<float>(__builtin_amdgcn_frexp_expf(l)) + log2f(__builtin_amdgcn_frexp_mantf(l))));
    }
  }
#pragma unroll
  for (int i = 0; i < kN; ++i)
    if (rho0 + i * step >= n_rows) v[i] = -INFINITY;
}
// The `ready` array, for calls whose many work-groups would each do the same merging.
__global__ __launch_bounds__(256) void score_row_norms(RowNorm a, float* __restrict__ out) {
  const int rho = blockIdx.x * 256 + threadIdx.x, n_rows = a.rep * a.by_qs.d;
  float v[1];
  row_norms(a, blockIdx.y, rho, 0, v);
  if (rho < n_rows) out[static_cast<int64_t>(blockIdx.y) * n_rows + rho] = v[0];
}

// ---- pass 2: column mass --------------------------------------------------------------------
// S = Q K^T: a lane owns one key column of each stationary block and 16 of the 32 query rows
// of the half tile.  The streamed operand is the scoring rows of the group, head after head, in
// tiles of 64; where they lie and their normalisers are prepared in LDS before the loop.
// nlq: the negated normalisers of the 16 query rows the lane holds.  kUnitC (c == 1): the
// products were started from nlq, so s already holds s - lse2.
template <bool kUnitC>
__device__ __forceinline__ void col_epilogue(int i, const f32x16 (&s)[2], const f32x16& nlq, float (&colsum)[2],
                                             float c) {
  const int b = i >> 3, e = (i & 7) * 2;
  if constexpr (kUnitC) {
    colsum[b] += __builtin_amdgcn_exp2f(s[b][e]);
    colsum[b] += __builtin_amdgcn_exp2f(s[b][e + 1]);
  } else {
    colsum[b] += __builtin_amdgcn_exp2f(fmaf(s[b][e], c, nlq[e]));
    colsum[b] += __builtin_amdgcn_exp2f(fmaf(s[b][e + 1], c, nlq[e + 1]));
  }
}

template <bool kUnitC>
__global__ __launch_bounds__(kThreads, 1) void score_colpass_bf16(
    const uint16_t* __restrict__ Qs, const int32_t* __restrict__ q_rows, const uint16_t* __restrict__ K, RowNorm norm,
    float* __restrict__ out, int64_t out_stride_h, int64_t out_stride_split, int rep, Divisor by_qs, int Nk,
    int64_t q_stride_h, int64_t k_stride_h, float c, Divisor by_blocks, Divisor by_qsplits, int per) {
  extern __shared__ __align__(16) uint8_t smem_raw[];
  lds_u8* smem = (lds_u8*)smem_raw;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  int64_t* s_src = reinterpret_cast<int64_t*>(smem_raw + kStages * kTileBytes);   // element offset of a row in Qs
  float* s_norm = reinterpret_cast<float*>(s_src + kPrepRows);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  // logical order: (kv head, query split) slowest, so the work-groups of one XCD stream the same queries
  const int L = xcd_contiguous_index(blockIdx.x, gridDim.x);
  const int unit = by_blocks.of(L), kb = L - unit * by_blocks.d;
  const int kvh = by_qsplits.of(unit), qsplit = unit - kvh * by_qsplits.d;
  const int key0 = kb * kBlockRows + wave * kWaveRows;
  const uint16_t* Kh = K + kvh * k_stride_h;

  // The wave's 64 keys come through its eighth of the ring as whole rows, 32 at a time (as fragments from
  // memory they were 32 bytes of a row per load, lines evicted between loads): the first half while the
  // row indices are on their way, the second while the normalisers are.
  auto stage_keys = [&](int b) {
    const RowWindow w = row_window(Kh, key0 + b * 32, Nk);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = i * 4 + (lane >> 4);
      dma_16B_at(w.base, row_offset(w, row, k_chunk_pos(row, lane & 15)), lds0 + (wave * 8 + i) * 1024);
    }
  };
  stage_keys(0);

  const int n_rows = rep * by_qs.d, n_vt = (n_rows + kTileRows - 1) / kTileRows;
  const int t_end = min((qsplit + 1) * per, n_vt);

  int a_off[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) a_off[s] = l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  const int my_row = wave * 8 + (lane >> 4);   // this lane fetches rows my_row and my_row + 4 of a tile
  struct Src {
    int64_t at[2];
  };
  auto src_of = [&](int j) {
    const int64_t* p = s_src + j * kTileRows + my_row;
    return Src{{p[0], p[4]}};
  };
  auto stage = [&](int j, const Src& r) {
    stage_rows([&](int, int i) { return Qs + r.at[i]; }, lds0 + (j & (kStages - 1)) * kTileBytes, wave, lane);
  };
  auto slot = [&](int j) { return smem + (j & (kStages - 1)) * kTileBytes; };
  // normalisers of the 16 rows this lane holds in half `half` of tile j
  auto load_lq = [&](int j, int half, f32x16& lq) {
    const float* base = s_norm + j * kTileRows + half * 32 + g * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(base + q * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) lq[q * 4 + e] = v[e];
    }
  };

  float colsum[2] = {0.f, 0.f};
  f32x16 sA[2], sB[2];
  f32x16 lq;            // general path: normalisers of the half tile whose elements the epilogue takes
  f32x16 initA, initB;  // kUnitC: start values of the next sA / sB products, fetched one phase ahead
  auto startA = [&](int) -> const f32x16& { return initA; };
  auto startB = [&](int) -> const f32x16& { return initB; };
  constexpr int kBatch = 4;
  int head[kBatch], row[kBatch];   // where the rows lie that this thread prepares
  auto find_rows = [&](int first) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int rho = min(first + i * kThreads, n_rows - 1), in_group = by_qs.of(rho);
      head[i] = kvh * rep + in_group;
      row[i] = rho - in_group * by_qs.d;
      if (q_rows) row[i] = q_rows[row[i]];
    }
  };
  bf16x8 kf[2][8];
  auto take_keys = [&](int b) {   // all that is in flight has landed
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < 8; ++s) kf[b][s] = lds_frag(smem + wave * 8 * 1024 + a_off[s]);
#pragma unroll
    for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(kf[b][s]));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  bool first_rows = true;
  find_rows(qsplit * per * kTileRows + threadIdx.x);
#pragma unroll
  for (int i = 0; i < kBatch; ++i) asm volatile("" : "+v"(row[i]));
  take_keys(0);
  stage_keys(1);
  for (int t0 = qsplit * per; t0 < t_end; t0 += kPrepTiles) {   // one turn but for thousands of scoring rows
    const int n = min(kPrepTiles, t_end - t0);
    // Sources and normalisers of the turn's rows, and of the kStages tiles after it that are fetched or
    // looked up but never used.  In the loop no load but the direct ones is then in flight: the
    // compiler waits for its own loads in order, which would drain the ring with them.
    // (16/4 heads x 512 rows x 193,792 keys: 377 -> 364 us.)
    for (int r0 = threadIdx.x; r0 < (n + kStages) * kTileRows; r0 += kBatch * kThreads) {
      if (!first_rows) find_rows(t0 * kTileRows + r0);
      first_rows = false;
      float v[kBatch];
      row_norms(norm, kvh, t0 * kTileRows + r0, kThreads, v);
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (r0 + i * kThreads < (n + kStages) * kTileRows) {
          s_src[r0 + i * kThreads] = head[i] * q_stride_h + static_cast<int64_t>(row[i]) * kD;
          s_norm[r0 + i * kThreads] = v[i];
        }
    }
    if (t0 == qsplit * per) take_keys(1);
    __syncthreads();
    stage(0, src_of(0));
    stage(1, src_of(1));
    stage(2, src_of(2));
    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");  // the first tile's pieces
    __syncthreads();
    if constexpr (kUnitC) {
      load_lq(0, 0, initA);
      load_lq(0, 1, initB);
    }
    Src src = src_of(3);
    bf16x8 ring[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) ring[r] = lds_frag(slot(0) + a_off[r]);
    stream_phase<kUnitC>(slot(0), slot(0) + 32 * kRowBytes, a_off, kf, sA, startA, [](int) {}, ring);
    auto tile_body = [&](int j, auto slot_tag) {  // slot j % 4 as a compile-time constant, as in pass 1
      constexpr int u = decltype(slot_tag)::value;
      dma_wait_all_but_newest();
      __syncthreads();  // tile j+1 has landed everywhere; slot of tile j-1 is free
      stage(j + 3, src);
      src = src_of(j + 4);
      if constexpr (kUnitC) load_lq(j + 1, 0, initA); else load_lq(j, 0, lq);
      stream_phase<kUnitC>(smem + u * kTileBytes + 32 * kRowBytes, smem + ((u + 1) & 3) * kTileBytes, a_off, kf, sB, startB,
                           [&](int i) { col_epilogue<kUnitC>(i, sA, lq, colsum, c); }, ring);
      if constexpr (kUnitC) load_lq(j + 1, 1, initB); else load_lq(j, 1, lq);
      if (j + 1 < n) {
        stream_phase<kUnitC>(smem + ((u + 1) & 3) * kTileBytes, smem + ((u + 1) & 3) * kTileBytes + 32 * kRowBytes, a_off, kf,
                             sA, startA, [&](int i) { col_epilogue<kUnitC>(i, sB, lq, colsum, c); }, ring);
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) col_epilogue<kUnitC>(i, sB, lq, colsum, c);
      }
    };
    for (int j0 = 0; j0 < n; j0 += kStages) {
      tile_body(j0, std::integral_constant<int, 0>{});
      if (j0 + 1 >= n) break;
      tile_body(j0 + 1, std::integral_constant<int, 1>{});
      if (j0 + 2 >= n) break;
      tile_body(j0 + 2, std::integral_constant<int, 2>{});
      if (j0 + 3 >= n) break;
      tile_body(j0 + 3, std::integral_constant<int, 3>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no direct load may outlive the turn or the work-group
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float v = wave_half_sum(colsum[b]);
    const int key = key0 + b * 32 + l32;
    if (g == 0 && key < Nk) out[qsplit * out_stride_split + kvh * out_stride_h + key] = v;
  }
}

// ---- both passes, small calls ---------------------------------------------------------------
// A work-group has 64 stationary rows (every wave holds all of them as fragments); its 8 waves take
// the streamed rows in steps of 32 by turns, each through an LDS double buffer of its own, two steps
// ahead and without a barrier in the loop, and are merged through LDS once: the row pass cuts its
// keys less often, and the column pass leaves no partial sums to add up in another launch.  The products
// of a step and the exponentials of the one before are interleaved as in stream_phase.  Bound: latency.
// The stationary rows come through LDS: each wave fetching all 64 as fragments (32 bytes of each of 32 rows
// per load, 128 KB per work-group) was a third of the call.  8/2 heads x 100 rows x 1,804 keys: both
// passes 16.1 -> 10.9 us, the column pass alone 8.6 -> 5.4; 2/1 x 64 x 300 14.7 -> 9.1.
constexpr int kSmallStep = 32;
constexpr int kSmallStepBytes = kSmallStep * kRowBytes;
constexpr int kSmallRing = 8 * 2 * kSmallStepBytes;            // 8 waves x two steps
constexpr int kSmallMaxRows = 2048;                            // scoring rows pass 2 prepares in LDS
constexpr int kSmallMergeRows = 3 * 8 * kSmallStep;            // the same with the row pass's shares to merge
constexpr size_t kSmallRowSmem = kSmallRing + 8 * kWaveRows * 8 + kWaveRows * kRowBytes;
constexpr size_t kSmallColSmem = kSmallRing + kSmallMaxRows * 12 + 8 * kWaveRows * 4;

// The rows of step i of a wave have landed when at most the next step's eight loads are in flight.
// All eight fragments go to registers, so that the buffer can be refilled at once.
__device__ __forceinline__ void small_fragments(const lds_u8* buf, const int (&a_off)[8], bool more_in_flight, bf16x8 (&f)[8]) {
  if (more_in_flight)
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int s = 0; s < 8; ++s) f[s] = lds_frag(buf + a_off[s]);
#pragma unroll
  for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(f[s]));
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
template <bool kInit, class Init, class Epi>
__device__ __forceinline__ void small_phase(const bf16x8 (&f)[8], const bf16x8 (&st)[2][8], f32x16 (&acc)[2], Init&& init,
                                            Epi&& epi) {
  f32x16 zero;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (kInit)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], st[b][s], s == 0 ? init(b) : acc[b], 0, 0, 0);
      else
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], st[b][s], s == 0 ? zero : acc[b], 0, 0, 0);
      epi(s * 2 + b);
      __builtin_amdgcn_sched_barrier(0);
    }
}

__global__ __launch_bounds__(kThreads, 1) void score_rowpass_small(
    const uint16_t* __restrict__ Qs, const int32_t* __restrict__ q_rows, const uint16_t* __restrict__ K,
    float2* __restrict__ part, int rep, Divisor by_qs, int Nk, int64_t q_stride_h, int64_t k_stride_h, float c,
    Divisor by_tiles, Divisor by_heads, int per) {
  extern __shared__ __align__(16) uint8_t smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const lds_u8* ring = (lds_u8*)smem_raw + wave * 2 * kSmallStepBytes;
  const uint32_t ring_w = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ring));
  const int L = xcd_contiguous_index(blockIdx.x, gridDim.x);
  const int unit = by_tiles.of(L), tile = L - unit * by_tiles.d, Hkv = by_heads.d;
  const int split = by_heads.of(unit), kvh = unit - split * Hkv;
  const int n_rows = rep * by_qs.d;
  const uint16_t* Kh = K + kvh * k_stride_h;
  const int steps_all = (Nk + kSmallStep - 1) / kSmallStep;
  const int t_end = min((split + 1) * per, steps_all), t_first = split * per + wave;
  const int n = t_first < t_end ? (t_end - t_first + 7) / 8 : 0;   // steps of this wave
  auto stage = [&](int i) {
    const RowWindow w = row_window(Kh, (t_first + i * 8) * kSmallStep, Nk);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int row = q * 4 + (lane >> 4);
      dma_16B_at(w.base, row_offset(w, row, k_chunk_pos(row, lane & 15)), ring_w + (i & 1) * kSmallStepBytes + q * 1024);
    }
  };
  // The stationary rows go through LDS once (every wave holds all of them: 16 KB instead of 128 from L2),
  // eight per wave; their indices are scalar loads, which direct loads are not waited for.
  const lds_u8* q_tile = (lds_u8*)smem_raw + kSmallRing + 8 * kWaveRows * 8;
  {
    int64_t at[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int rho = min(tile * kWaveRows + wave * 8 + j, n_rows - 1), in_group = by_qs.of(rho);
      int row = rho - in_group * by_qs.d;
      if (q_rows) row = q_rows[row];
      at[j] = (kvh * rep + in_group) * q_stride_h + static_cast<int64_t>(row) * kD;
    }
    if (n > 0) stage(0);
    const uint32_t to = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(q_tile)) + wave * 8 * kRowBytes;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t* four = at + i * 4;
      const int which = lane >> 4, row = wave * 8 + i * 4 + which;
      const int64_t src = which == 0 ? four[0] : which == 1 ? four[1] : which == 2 ? four[2] : four[3];
      dma_16B(Qs + src + k_chunk_pos(row, lane & 15) * 8, to + i * 1024);
    }
  }
  if (n > 1) {
    stage(1);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  int a_off[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) a_off[s] = l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  bf16x8 qf[2][8];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[b][s] = lds_frag(q_tile + b * 32 * kRowBytes + a_off[s]);

  RowState st;
  st.m[0] = st.m[1] = kNoMax;
  st.l[0] = st.l[1] = 0.f;
  float psum[2] = {0.f, 0.f};
  f32x16 sA[2], sB[2];
  bf16x8 f[8];
  auto fetch = [&](int i) {   // fragments of step i; step i + 2 into the buffer they came from
    small_fragments(ring + (i & 1) * kSmallStepBytes, a_off, i + 1 < n, f);
    if (i + 2 < n) stage(i + 2);
  };
  auto mask = [&](f32x16 (&sc)[2], int i) {
    const int k0 = (t_first + i * 8) * kSmallStep;
    if (k0 + kSmallStep > Nk) mask_keys(sc, k0, Nk, g);
  };
  auto body = [&](int i, f32x16 (&cur)[2], f32x16 (&nxt)[2]) {
    mask(cur, i);
    if (i + 1 < n) {
      fetch(i + 1);
      small_phase<false>(f, qf, nxt, NoInit{}, [&](int e) { row_epilogue(e, cur, st, psum, c); });
    } else if (i == 0) {   // the only step: there is no reference yet, so row_commit forms its sums
      psum[0] = psum[1] = INFINITY;
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) row_epilogue(e, cur, st, psum, c);
    }
    bool unused = false;
    row_commit(cur, st, psum, c, unused);
  };
  if (n > 0) {
    fetch(0);
    small_phase<false>(f, qf, sA, NoInit{}, [](int) {});
    for (int i = 0; i < n; i += 2) {
      body(i, sA, sB);
      if (i + 1 < n) body(i + 1, sB, sA);
    }
  }
  // merge: the halves of a wave, then the waves in order
  float2* s_ml = reinterpret_cast<float2*>(smem_raw + kSmallRing);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float m_o = wave_half_swap(st.m[b]), l_o = wave_half_swap(st.l[b]);
    const float m = fmaxf(st.m[b], m_o);
    const float l = st.l[b] * __builtin_amdgcn_exp2f(st.m[b] - m) + l_o * __builtin_amdgcn_exp2f(m_o - m);
    if (g == 0) s_ml[wave * kWaveRows + b * 32 + l32] = make_float2(m, l);
  }
  __syncthreads();
  const int rho = tile * kWaveRows + threadIdx.x;
  if (threadIdx.x >= kWaveRows || rho >= n_rows) return;
  float m = kNoMax, l = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) m = fmaxf(m, s_ml[w * kWaveRows + threadIdx.x].x);
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const float2 v = s_ml[w * kWaveRows + threadIdx.x];
    l += v.y * __builtin_amdgcn_exp2f(v.x - m);
  }
  part[(static_cast<int64_t>(split) * Hkv + kvh) * n_rows + rho] = make_float2(m, l);
}

template <bool kUnitC>
__global__ __launch_bounds__(kThreads, 1) void score_colpass_small(
    const uint16_t* __restrict__ Qs, const int32_t* __restrict__ q_rows, const uint16_t* __restrict__ K, RowNorm norm,
    float* __restrict__ out, int64_t out_stride_h, int rep, Divisor by_qs, int Nk, int64_t q_stride_h, int64_t k_stride_h,
    float c, Divisor by_blocks) {
  extern __shared__ __align__(16) uint8_t smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const lds_u8* ring = (lds_u8*)smem_raw + wave * 2 * kSmallStepBytes;
  const uint32_t ring_w = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ring));
  int64_t* s_src = reinterpret_cast<int64_t*>(smem_raw + kSmallRing);      // element offset of a row in Qs
  float* s_norm = reinterpret_cast<float*>(smem_raw + kSmallRing + kSmallMaxRows * 8);
  float* s_sum = s_norm + kSmallMaxRows;
  const int L = xcd_contiguous_index(blockIdx.x, gridDim.x);
  const int kvh = by_blocks.of(L), key0 = (L - kvh * by_blocks.d) * kWaveRows;
  const uint16_t* Kh = K + kvh * k_stride_h;
  const int n_rows = rep * by_qs.d, n_steps = (n_rows + kSmallStep - 1) / kSmallStep;
  const int n = wave < n_steps ? (n_steps - wave + 7) / 8 : 0;   // steps of this wave: wave, wave + 8, ...

  // The stationary keys go through LDS once (every wave holds all of them), eight per wave: keys 0..31 lie
  // in the second step's buffer of wave 0, 32..63 in that of wave 1, which is filled only behind them.
  auto key_half = [&](int b) { return (lds_u8*)smem_raw + b * 2 * kSmallStepBytes + kSmallStepBytes; };
  {
    const RowWindow w = row_window(Kh, key0, Nk);
    const uint32_t to = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(key_half(wave >> 2))) + (wave & 3) * 8 * kRowBytes;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = wave * 8 + i * 4 + (lane >> 4);
      dma_16B_at(w.base, row_offset(w, row, k_chunk_pos(row, lane & 15)), to + i * 1024);
    }
  }
  // a thread prepares the rows threadIdx.x + 512 i; everything is loaded before anything is waited for
  constexpr int kPrep = kSmallMaxRows / kThreads;
  int head[kPrep], row[kPrep];
#pragma unroll
  for (int i = 0; i < kPrep; ++i) {
    if (i * kThreads >= n_steps * kSmallStep) break;   // uniform
    const int r = min(static_cast<int>(threadIdx.x) + i * kThreads, n_rows - 1);
    const int in_group = by_qs.of(r);
    head[i] = kvh * rep + in_group;
    row[i] = r - in_group * by_qs.d;
    if (q_rows) row[i] = q_rows[row[i]];
  }
  {
    float v[kPrep];
    row_norms(norm, kvh, threadIdx.x, kThreads, v);
#pragma unroll
    for (int i = 0; i < kPrep; ++i) {
      if (i * kThreads >= n_steps * kSmallStep) break;
      s_src[threadIdx.x + i * kThreads] = head[i] * q_stride_h + static_cast<int64_t>(row[i]) * kD;
      s_norm[threadIdx.x + i * kThreads] = v[i];
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  auto stage = [&](int i) {
    const int64_t* src = s_src + (wave + i * 8) * kSmallStep + (lane >> 4);
    int64_t at[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) at[q] = src[q * 4];
#pragma unroll
    for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(at[q]));   // one wait, not one per load
    const uint32_t to = __builtin_amdgcn_readfirstlane(ring_w + (i & 1) * kSmallStepBytes);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      dma_16B(Qs + at[q] + k_chunk_pos(q * 4 + (lane >> 4), lane & 15) * 8, to + q * 1024);
  };
  if (n > 0) stage(0);

  int a_off[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) a_off[s] = l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  bf16x8 kf[2][8];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int s = 0; s < 8; ++s) kf[b][s] = lds_frag(key_half(b) + a_off[s]);
  if (n_steps > 8) {   // second steps: every wave has its keys
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(kf[b][s]));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (n > 1) stage(1);
  }
  auto load_lq = [&](int i, f32x16& lq) {   // normalisers of the 16 rows this lane holds of step i
    const float* base = s_norm + (wave + i * 8) * kSmallStep + g * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(base + q * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) lq[q * 4 + e] = v[e];
    }
  };
  float colsum[2] = {0.f, 0.f};
  f32x16 sA[2], sB[2], lq;
  bf16x8 f[8];
  auto init = [&](int) -> const f32x16& { return lq; };
  auto fetch = [&](int i) {
    small_fragments(ring + (i & 1) * kSmallStepBytes, a_off, i + 1 < n, f);
    if (i + 2 < n) stage(i + 2);
  };
  auto body = [&](int i, f32x16 (&cur)[2], f32x16 (&nxt)[2]) {
    if (!kUnitC) load_lq(i, lq);
    if (i + 1 < n) {
      fetch(i + 1);
      if (kUnitC) load_lq(i + 1, lq);
      small_phase<kUnitC>(f, kf, nxt, init, [&](int e) { col_epilogue<kUnitC>(e, cur, lq, colsum, c); });
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) col_epilogue<kUnitC>(e, cur, lq, colsum, c);
    }
  };
  if (n > 0) {
    fetch(0);
    if (kUnitC) load_lq(0, lq);
    small_phase<kUnitC>(f, kf, sA, init, [](int) {});
    for (int i = 0; i < n; i += 2) {
      body(i, sA, sB);
      if (i + 1 < n) body(i + 1, sB, sA);
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float v = wave_half_sum(colsum[b]);
    if (g == 0) s_sum[wave * kWaveRows + b * 32 + l32] = v;
  }
  __syncthreads();
  const int key = key0 + threadIdx.x;
  if (threadIdx.x >= kWaveRows || key >= Nk) return;
  float v = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) v += s_sum[w * kWaveRows + threadIdx.x];
  out[kvh * out_stride_h + key] = v;
}

// sum over parts p of part[p][h][j], p ascending.  Latency-bound: the parts are loaded together.
__device__ __forceinline__ float parts_sum(const float* part, int n_parts, int64_t split_stride, int64_t at) {
  float v[kMaxQSplits];
#pragma unroll
  for (int p = 0; p < kMaxQSplits; ++p) v[p] = p < n_parts ? part[p * split_stride + at] : 0.f;
  float sum = 0.f;
#pragma unroll
  for (int p = 0; p < kMaxQSplits; ++p) sum += v[p];   // a missing part adds +0: the sum is unchanged
  return sum;
}
// out[h][j] = that sum; with share_heads (n_parts = 1) the heads are summed, head 0 first, into out[j].
__global__ void score_reduce(const float* __restrict__ part, float* __restrict__ out, int64_t out_stride_h,
                             int n_parts, int Hkv, int Nk, int share_heads) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= Nk) return;
  if (share_heads) {
    float s = 0.f;
    for (int h0 = 0; h0 < Hkv; h0 += 8) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = h0 + i < Hkv ? part[static_cast<int64_t>(h0 + i) * Nk + j] : 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[i];
    }
    out[j] = s;
  } else {
    const int h = blockIdx.y;
    out[h * out_stride_h + j] = parts_sum(part, n_parts, static_cast<int64_t>(Hkv) * Nk, static_cast<int64_t>(h) * Nk + j);
  }
}
// The same for share_heads and several parts: a wave per head (eight at most) and 64 keys per work-group, so that
// the loads of a key are in flight together (a thread that goes from head to head waits for each head's).
// Calls fed with log-sum-exps: 16/4 heads x 512 x 7,199 keys (four parts) 20.3 -> 19.0 us, 24/8 x 512 x 2,200 (six)
// 15.2 -> 12.1.  With one part a thread of score_reduce has all loads in flight, and is 0.2-0.5 us faster.
constexpr int kReduceHeads = 8;
__global__ __launch_bounds__(64 * kReduceHeads) void score_reduce_heads(const float* __restrict__ part,
                                                                        float* __restrict__ out, int n_parts, int Hkv,
                                                                        int Nk) {
  __shared__ float s_sum[kReduceHeads][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = blockDim.x >> 6, j = blockIdx.x * 64 + lane;
  float total = 0.f;
  for (int h0 = 0; h0 < Hkv; h0 += waves) {
    if (h0 > 0) __syncthreads();   // the sums before have been read
    if (h0 + wave < Hkv)
      s_sum[wave][lane] = parts_sum(part, n_parts, static_cast<int64_t>(Hkv) * Nk,
                                    static_cast<int64_t>(h0 + wave) * Nk + min(j, Nk - 1));
    __syncthreads();
    if (wave == 0)
      for (int i = 0; i < min(waves, Hkv - h0); ++i) total += s_sum[i][lane];
  }
  if (wave == 0 && j < Nk) out[j] = total;
}

// ---- fp32 tier ------------------------------------------------------------------------------
// Both passes on the 16x16x4 fp32 MFMA (fp32 operands and accumulation), S^T = K Q^T: lane
// (r = l % 16, kg = l / 16) holds dims 16 s + 4 kg .. + 3 of key row r and of query row r as
// 16-byte loads, the four MFMAs of step s contract over (kg, element e), and the result leaves the
// lane with keys 4 kg .. 4 kg + 3 of query column r.  Operands come from global memory (a few
// hundred rows: they live in the caches), nothing is staged.  A work-group is 8 waves that share
// the stationary 16 rows, take the streamed axis by turns and merge through LDS once, in wave
// order: bit-reproducible.  Latency-bound at the sizes this tier runs at, hence the fine cut:
// 2 heads x 64 rows x 336 keys, D = 64: 106 + 79 us with one thread per row / key and plain FMA,
// 6.6 + 4.8 us like this.
constexpr int kF32Waves = 8;
constexpr int kF32Threads = 64 * kF32Waves;

template <int D>
struct F32Frag {  // one row of a 16-row operand, this lane's quarter of it
  f32x4 v[D / 16];
  __device__ __forceinline__ void load(const float* row, int kg) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s) v[s] = load_f32x4(row + s * 16 + kg * 4);
  }
};
// two independent 16x16 products, interleaved: neither waits for its own last MFMA
template <int D>
__device__ __forceinline__ void f32_products(const F32Frag<D>& k0, const F32Frag<D>& q0, const F32Frag<D>& k1,
                                             const F32Frag<D>& q1, f32x4 (&sc)[2]) {
  sc[0] = sc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_sched_barrier(0);  // every load of the step is issued before the first product
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(k0.v[s][e], q0.v[s][e], sc[0], 0, 0, 0);
      sc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(k1.v[s][e], q1.v[s][e], sc[1], 0, 0, 0);
    }
}

// Pass 1: natural-log sum-exp of 16 scoring rows of one head over all keys.
template <int D>
__global__ __launch_bounds__(kF32Threads) void score_rowpass_f32(const float* __restrict__ Qs,
                                                                 const int32_t* __restrict__ q_rows,
                                                                 const float* __restrict__ K,
                                                                 float* __restrict__ lse, int rep, int n_qs,
                                                                 int Nk, int64_t q_stride_h,
                                                                 int64_t k_stride_h, float scale) {
  __shared__ float s_m[kF32Waves][16], s_l[kF32Waves][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int h = blockIdx.y;
  const int row = blockIdx.x * 16 + r;
  int qr = min(row, n_qs - 1);
  if (q_rows) qr = q_rows[qr];
  F32Frag<D> q, k[2];
  q.load(Qs + h * q_stride_h + static_cast<int64_t>(qr) * D, kg);
  const float* Kh = K + (h / rep) * k_stride_h;
  float m = -INFINITY, l = 0.f;
  for (int k0 = wave * 32; k0 < Nk; k0 += kF32Waves * 32) {
#pragma unroll
    for (int t = 0; t < 2; ++t) k[t].load(Kh + static_cast<int64_t>(min(k0 + t * 16 + r, Nk - 1)) * D, kg);
    f32x4 sc[2];
    f32_products<D>(k[0], q, k[1], q, sc);
    float mt = m;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sc[t][e] = k0 + t * 16 + kg * 4 + e < Nk ? sc[t][e] * scale : -INFINITY;
        mt = fmaxf(mt, sc[t][e]);
      }
    // a lane may not have seen a valid key yet: exp(-inf - -inf) is not wanted
    const float m_use = mt == -INFINITY ? 0.f : mt;
    l *= expf(m - m_use);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) l += expf(sc[t][e] - m_use);
    m = mt;
  }
  // the four lanes of a query column, then the waves
#pragma unroll
  for (int x = 16; x <= 32; x *= 2) {
    const float m_o = __shfl_xor(m, x), l_o = __shfl_xor(l, x);
    const float mt = fmaxf(m, m_o), m_use = mt == -INFINITY ? 0.f : mt;
    l = l * expf(m - m_use) + l_o * expf(m_o - m_use);
    m = mt;
  }
  if (kg == 0) {
    s_m[wave][r] = m;
    s_l[wave][r] = l;
  }
  __syncthreads();
  if (threadIdx.x >= 16 || row >= n_qs) return;
  float M = s_m[0][r];  // wave 0 always has keys
#pragma unroll
  for (int w = 1; w < kF32Waves; ++w) M = fmaxf(M, s_m[w][r]);
  float lt = 0.f;
#pragma unroll
  for (int w = 0; w < kF32Waves; ++w) lt += s_l[w][r] * expf(s_m[w][r] - M);
  lse[static_cast<int64_t>(h) * n_qs + row] = M + logf(lt);
}

// Pass 2: column mass of 16 keys over the (query head of the group, 16-row tile) list.  lse: the
// dense [head][n_qs] output of pass 1 (lse_rows NULL), or the caller's array, indexed like Qs.
template <int D>
__global__ __launch_bounds__(kF32Threads) void score_colpass_f32(const float* __restrict__ Qs,
                                                                 const int32_t* __restrict__ q_rows,
                                                                 const float* __restrict__ K,
                                                                 const float* __restrict__ lse, int64_t lse_stride_h,
                                                                 int lse_by_q_row, float* __restrict__ score,
                                                                 int64_t score_stride_h, int rep, int n_qs,
                                                                 int Nk, int64_t q_stride_h,
                                                                 int64_t k_stride_h, float scale) {
  __shared__ f32x4 s_sum[kF32Waves][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kg = lane >> 4;
  const int kvh = blockIdx.y;
  const int key0 = blockIdx.x * 16;
  F32Frag<D> k, q[2];
  k.load(K + kvh * k_stride_h + static_cast<int64_t>(min(key0 + r, Nk - 1)) * D, kg);
  const int tiles = (n_qs + 15) / 16, n_units = rep * tiles;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  for (int u0 = wave * 2; u0 < n_units; u0 += kF32Waves * 2) {
    float ls[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int u = min(u0 + t, n_units - 1);
      const int h = kvh * rep + u / tiles, row = (u % tiles) * 16 + r;
      const int rowc = min(row, n_qs - 1);
      const int qr = q_rows ? q_rows[rowc] : rowc;
      q[t].load(Qs + h * q_stride_h + static_cast<int64_t>(qr) * D, kg);
      const float x = lse[h * lse_stride_h + (lse_by_q_row ? qr : rowc)];
      ls[t] = u0 + t < n_units && row < n_qs ? x : INFINITY;  // padding adds nothing
    }
    f32x4 sc[2];
    f32_products<D>(k, q[0], k, q[1], sc);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[e] += expf(sc[t][e] * scale - ls[t]);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)  // over the 16 query columns
#pragma unroll
    for (int x = 1; x < 16; x *= 2) sum[e] += __shfl_xor(sum[e], x);
  if (r == 0) s_sum[wave][kg] = sum;
  __syncthreads();
  if (threadIdx.x >= 4) return;
  f32x4 tot = s_sum[0][threadIdx.x];
#pragma unroll
  for (int w = 1; w < kF32Waves; ++w) tot += s_sum[w][threadIdx.x];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int key = key0 + threadIdx.x * 4 + e;
    if (key < Nk) score[kvh * score_stride_h + key] = tot[e];
  }
}

// The same with fewer than 16 units of rows, numbered head after head here: only the waves that have one
// are launched (an idle one holds a slot until the work-group ends: 16 heads, 1 row, 30,000 keys, D =
// 64: 105 us with eight waves, 26 with one).
template <int D>
__global__ __launch_bounds__(kF32Threads) void score_colpass_f32_few(const float* __restrict__ Qs,
                                                                     const int32_t* __restrict__ q_rows,
                                                                     const float* __restrict__ K,
                                                                     const float* __restrict__ lse, int64_t lse_stride_h,
                                                                     int lse_by_q_row, float* __restrict__ score,
                                                                     int64_t score_stride_h, int rep, int n_qs,
                                                                     int Nk, int64_t q_stride_h,
                                                                     int64_t k_stride_h, float scale) {
  __shared__ f32x4 s_sum[kF32Waves][4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const int kvh = blockIdx.y;
  const int key0 = blockIdx.x * 16;
  F32Frag<D> k, q[2];
  k.load(K + kvh * k_stride_h + static_cast<int64_t>(min(key0 + r, Nk - 1)) * D, kg);
  const int n_rows = rep * n_qs, u0 = wave * 2;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  float ls[2];
  auto fetch = [&](int t) {
    const int rho = (u0 + t) * 16 + r, in_group = min(rho, n_rows - 1) / n_qs, h = kvh * rep + in_group;
    const int row = min(rho, n_rows - 1) - in_group * n_qs, qr = q_rows ? q_rows[row] : row;
    q[t].load(Qs + h * q_stride_h + static_cast<int64_t>(qr) * D, kg);
    const float x = lse[h * lse_stride_h + (lse_by_q_row ? qr : row)];
    ls[t] = rho < n_rows ? x : INFINITY;  // padding adds nothing
  };
  auto add = [&](const f32x4& sc, int t) {
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] += expf(sc[e] * scale - ls[t]);
  };
  fetch(0);
  if ((u0 + 1) * 16 < n_rows) {  // wave-uniform
    fetch(1);
    f32x4 sc[2];
    f32_products<D>(k, q[0], k, q[1], sc);
    add(sc[0], 0);
    add(sc[1], 1);
  } else {
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(k.v[s][e], q[0].v[s][e], sc, 0, 0, 0);
    add(sc, 0);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)  // over the 16 query columns
#pragma unroll
    for (int x = 1; x < 16; x *= 2) sum[e] += __shfl_xor(sum[e], x);
  if (r == 0) s_sum[wave][kg] = sum;
  __syncthreads();
  if (threadIdx.x >= 4) return;
  f32x4 tot = s_sum[0][threadIdx.x];
  for (int w = 1; w < static_cast<int>(blockDim.x >> 6); ++w) tot += s_sum[w][threadIdx.x];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int key = key0 + threadIdx.x * 4 + e;
    if (key < Nk) score[kvh * score_stride_h + key] = tot[e];
  }
}

// lse (caller's, indexed like Qs) or NULL: pass 1 fills ws_lse.  Scores of the nkr keys at k_r.
template <int D>
void score_f32(const float* q, const int32_t* q_rows, const float* k, const float* k_r, const float* lse,
               int64_t lse_stride_h, float* ws_lse, float* out, int64_t out_stride_h, int Hq, int Hkv, int n_qs, int Nk,
               int nkr, int64_t q_stride_h, int64_t k_stride_h, float scale, hipStream_t s) {
  const int rep = Hq / Hkv;
  if (lse == nullptr)
    score_rowpass_f32<D><<<dim3(ceil_div(n_qs, 16), Hq), kF32Threads, 0, s>>>(q, q_rows, k, ws_lse, rep, n_qs, Nk,
                                                                              q_stride_h, k_stride_h, scale);
  // Two units a wave.  At D = 128 a compute unit has registers for 16 waves, two work-groups of eight or of
  // five to seven: there eight are launched (24/8 heads, 64 rows, 10,000 keys: 87 us against 102 with six).
  const int waves = ceil_div(ceil_div(rep * n_qs, 16), 2);
  const bool few = waves <= (D == 64 ? 7 : 4);
  const auto colpass = few ? score_colpass_f32_few<D> : score_colpass_f32<D>;
  colpass<<<dim3(ceil_div(nkr, 16), Hkv), 64 * (few ? waves : kF32Waves), 0, s>>>(
      q, q_rows, k_r, lse ? lse : ws_lse, lse ? lse_stride_h : n_qs, lse != nullptr, out, out_stride_h, rep, n_qs, nkr,
      q_stride_h, k_stride_h, scale);
}

struct WsLayout {
  size_t lse_off, part_off, col_off, total;
};

int padded_rows(int n_qs) { return ceil_div(n_qs, kTileRows) * kTileRows; }

WsLayout ws_layout(int Hq, int Hkv, int n_qs, int Nk, int /*share_heads*/) {
  WsLayout w;
  size_t at = 0;
  w.lse_off = at;
  at += align_up(sizeof(float) * static_cast<size_t>(Hq) * padded_rows(n_qs), 256);
  w.part_off = at;
  at += align_up(sizeof(float2) * static_cast<size_t>(kMaxSplits) * Hq * n_qs, 256);
  w.col_off = at;
  at += align_up(sizeof(float) * static_cast<size_t>(kMaxQSplits) * Hkv * Nk, 256);
  w.total = at;
  return w;
}

// How the two passes of a bf16 call are cut: their form (512 stationary rows per work-group, or 64) and
// the shares of the streamed axis.  The estimates are microseconds: `start` is what a work-group costs
// beside its steps, a step gets slower as the compute units fill up, a further round costs a new start, and
// pass 2 merges the row pass's shares, itself or behind a launch of 2-5 us that does.
// Row pass: fitted to 63 shapes (100 to 512 scoring rows a head, 8 to 24 heads, 600 to 20,000 keys) in both
// forms with every number of shares that makes 64 to 768 work-groups; 0.9 % off the best on average.  Where the
// line lies (16/4 heads, both passes of the call with 64 rows against 512): 100 rows a head x 4,500 keys 19.4 /
// 25.3 us, 330 x 2,600 24.5 / 27.4, 330 x 12,000 49.7 / 51.5, 512 x 12,000 65.7 / 65.6, 512 x 20,000 98.4 / 96.6.
// Column pass: both forms timed on 191 calls fed with log-sum-exps and 181 without (2 to 24 heads, 64 to 1,000
// rows, 40 to 16,000 keys): 0.13 % and 0.44 % off the better form on average.  Where the line lies (16/4 heads,
// log-sum-exps given, 64 keys against 512): 100 rows a head x 2,500 keys 5.4 / 7.7 us, x 6,000 9.5 / 9.0, 170 x
// 12,300 23.4 / 15.0, 330 x 420 10.0 / 10.1, 330 x 7,300 19.0 / 15.0, 512 x 40 12.5 / 11.5, 512 x 1,300 13.1 /
// 11.8, 512 x 6,500 25.6 / 18.7.  With shares to merge in every work-group the column pass keeps to three
// steps of 64 keys' form: there it gains 2-4 us (8/2 heads, 170 x 1,804 14.3 / 18.2), with 2,048 rows 0.5 or
// nothing (8/2, 512 x 4,500 27.2 / 26.5).
struct PassCost {
  double start, step, step_filled, round;
  double of(int blocks, int steps) const {
    const int rounds = ceil_div(blocks, 256);
    return start + rounds * (step + step_filled * std::min(1.0, blocks / 256.0)) * steps + (rounds - 1) * round;
  }
};
struct RowPlan {
  bool small;
  int n_splits;
};
// Forming the normalisers in the column pass's work-groups, while their keys are on their way: some loads per
// thread, once per compute unit, against a launch in between.  24/8 heads x 512 x 12,608 keys (20 loads) 75.4
// us with the launch, 70.7 without; 16/4 x 100 x 20,000 (18) 34.8 / 32.9; with 32 they were 2-6 us more.
bool merges_in_pass_2(int rows_here, int n_splits) { return ceil_div(rows_here, kThreads) * n_splits <= 24; }
RowPlan plan_rows(int Hkv, int rows, int Nk, bool unit_c) {
  RowPlan best = {false, 1};
  double best_cost = 1e30;
  auto consider = [&](bool small, int block_rows, int share_keys, int steps_per, const PassCost& cost) {
    const int base = Hkv * ceil_div(rows, block_rows), units = ceil_div(Nk, share_keys);
    for (int s = 1; s <= std::min(kMaxSplits, units); ++s) {
      const int per = ceil_div(units, s);
      if (ceil_div(units, per) != s) continue;   // would leave a share empty
      // pass 2 merges the shares, by itself or behind a launch that does
      const double c = cost.of(base * s, ceil_div(per, steps_per)) + std::min(s * (0.04 + 1.5e-4 * rows), 2.0 + 0.09 * s);
      if (c < best_cost) {
        best_cost = c;
        best = {small, s};
      }
    }
  };
  consider(false, kBlockRows, kTileRows, 1, {6.9, unit_c ? 1.29 : 1.40, 0.08, 4.5});
  consider(true, kWaveRows, kSmallStep, 8, {4.5, 0.85, 0.05, 4.3});
  return best;
}
struct ColPlan {
  bool small, prepares;   // prepares: the work-groups form the normalisers of their rows themselves
  int n_qsplits;
};
ColPlan plan_cols(int Hkv, int rows, int nkr, int n_splits) {
  const int n_vt = ceil_div(rows, kTileRows), base = Hkv * ceil_div(nkr, kBlockRows);
  ColPlan best = {false, false, 1};
  double best_cost = 1e30;
  for (int s = 1; s <= std::min(kMaxQSplits, n_vt); ++s) {
    const int per = ceil_div(n_vt, s);
    if (ceil_div(n_vt, per) != s) continue;
    const double reduce = s == 1 ? 0.0 : 2.1 + 4.6e-6 * s * Hkv * nkr;
    const double c = PassCost{3.8, 1.27, 0.24, 4.15}.of(base * s, per) + reduce;
    if (c < best_cost) {
      best_cost = c;
      // several rounds of work-groups would each merge again; a log-sum-exp is just read (24/8 heads x 512 x
      // 9,000 keys, two rounds: 37.5 us behind a launch, 36.4 without; from five rounds on no difference)
      best = {false, base * s <= (n_splits == 1 ? 1024 : 256) && merges_in_pass_2((per + kStages) * kTileRows, n_splits), s};
    }
  }
  if (rows <= (n_splits > 1 ? kSmallMergeRows : kSmallMaxRows)) {
    const double c = PassCost{2.6, 0.91, 0.32, 1.8}.of(Hkv * ceil_div(nkr, kWaveRows), ceil_div(rows, 8 * kSmallStep)) +
                     1.2e-3 * rows;   // the normalisers of all rows, in every work-group
    if (c < best_cost) best = {true, merges_in_pass_2(rows, n_splits), 1};
  }
  return best;
}

}  // namespace
}  // namespace pc

using namespace pc;

extern "C" size_t pc_score_workspace_bytes(int Hq, int Hkv, int n_qs, int Nk, int share_heads) {
  if (Hq <= 0 || Hkv <= 0 || n_qs <= 0 || Nk <= 0) return 0;
  return ws_layout(Hq, Hkv, n_qs, Nk, share_heads).total;
}

extern "C" int pc_score_cut(int Hq, int Hkv, int n_qs, int Nk, int n_scored, float scale, int lse_given, int32_t* cut) {
  PC_REQUIRE(cut, PC_ERR_NULL, "pc_score_cut: cut is NULL");
  PC_REQUIRE(Hq > 0 && Hkv > 0 && Hq % Hkv == 0 && n_qs >= 1 && Nk >= 1 && n_scored >= 1 && n_scored <= Nk, PC_ERR_SHAPE,
             "pc_score_cut: Hq=%d Hkv=%d n_qs=%d Nk=%d n_scored=%d", Hq, Hkv, n_qs, Nk, n_scored);
  const int rows = Hq / Hkv * n_qs;
  const RowPlan row = plan_rows(Hkv, rows, Nk, scale * 1.4426950408889634f == 1.0f);
  const ColPlan col = plan_cols(Hkv, rows, n_scored, lse_given ? 1 : row.n_splits);
  cut[0] = lse_given ? 0 : row.small ? kWaveRows : kBlockRows;
  cut[1] = lse_given ? 0 : row.n_splits;
  cut[2] = col.small ? kWaveRows : kBlockRows;
  cut[3] = col.n_qsplits;
  cut[4] = col.prepares;
  return PC_OK;
}

extern "C" int pc_score(const void* Qs, const void* K, int dtype, int Hq, int Hkv, int n_qs,
                        int Nk, int D, int64_t q_stride_h, int64_t k_stride_h,
                        const int32_t* q_rows, float scale, const float* lse, int64_t lse_stride_h, float* score,
                        int64_t score_stride_h, int share_heads, int key_begin, int key_end,
                        void* ws, size_t ws_bytes, void* stream) {
  PC_REQUIRE(dtype == PC_F32 || dtype == PC_BF16, PC_ERR_DTYPE, "pc_score: dtype %d", dtype);
  PC_REQUIRE(Hq > 0 && Hkv > 0 && Hq % Hkv == 0, PC_ERR_SHAPE,
             "pc_score: Hq=%d must be a positive multiple of Hkv=%d", Hq, Hkv);
  PC_REQUIRE(n_qs >= 1 && Nk >= 1, PC_ERR_SHAPE, "pc_score: n_qs=%d Nk=%d must be >= 1", n_qs, Nk);
  PC_REQUIRE(scale > 0.f && isfinite(scale), PC_ERR_SHAPE, "pc_score: scale %g must be > 0", scale);
  PC_REQUIRE(Qs && K && score, PC_ERR_NULL, "pc_score: Qs, K or score is NULL");
  PC_REQUIRE((q_rows != nullptr || q_stride_h >= static_cast<int64_t>(n_qs) * D || Hq == 1) &&
                 (k_stride_h >= static_cast<int64_t>(Nk) * D || Hkv == 1),
             PC_ERR_SHAPE, "pc_score: a head stride is smaller than rows*D");
  PC_REQUIRE(share_heads || Hkv == 1 || score_stride_h >= Nk, PC_ERR_SHAPE,
             "pc_score: score head stride %lld < Nk", static_cast<long long>(score_stride_h));
  if (key_end <= 0) key_end = Nk;  // 0: up to the last key
  PC_REQUIRE(key_begin >= 0 && key_begin < key_end && key_end <= Nk, PC_ERR_SHAPE,
             "pc_score: key range [%d, %d) outside [0, %d)", key_begin, key_end, Nk);
  // Keys outside the range take part in every normaliser (pass 1 runs over all Nk keys) but get no
  // score: pass 2 simply runs on the sub-range (pointers and counts offset here).
  const int nkr = key_end - key_begin;
  PC_REQUIRE(lse == nullptr || Hq == 1 || lse_stride_h >= n_qs, PC_ERR_SHAPE,
             "pc_score: lse head stride %lld < n_qs", static_cast<long long>(lse_stride_h));
  const WsLayout lay = ws_layout(Hq, Hkv, n_qs, Nk, share_heads);
  PC_REQUIRE(ws != nullptr && ws_bytes >= lay.total, PC_ERR_WORKSPACE,
             "pc_score: workspace %zu bytes, need %zu", ws_bytes, lay.total);
  PC_REQUIRE(reinterpret_cast<uintptr_t>(ws) % 16 == 0, PC_ERR_WORKSPACE, "pc_score: workspace not 16-byte aligned");
  hipStream_t s = static_cast<hipStream_t>(stream);
  uint8_t* wsb = static_cast<uint8_t*>(ws);
  float* ws_lse = reinterpret_cast<float*>(wsb + lay.lse_off);
  float2* ws_part = reinterpret_cast<float2*>(wsb + lay.part_off);
  float* ws_col = reinterpret_cast<float*>(wsb + lay.col_off);
  const int rep = Hq / Hkv;

  if (dtype == PC_BF16) {
    PC_REQUIRE(D == kD, PC_ERR_UNSUPPORTED, "pc_score: bf16 tier needs D=128, got %d", D);
    const uintptr_t al = reinterpret_cast<uintptr_t>(Qs) | reinterpret_cast<uintptr_t>(K);
    PC_REQUIRE(al % 16 == 0 && q_stride_h % 8 == 0 && k_stride_h % 8 == 0, PC_ERR_SHAPE,
               "pc_score: bf16 tensors and head strides must be 16-byte aligned");
    const float c = scale * 1.4426950408889634f;
    // c == 1 (scale = ln 2): the caller folded the softmax scale and log2(e) into the queries, and
    // both passes take the affine step out of their loops
    const bool unit_c = c == 1.0f;
    const uint16_t* q = static_cast<const uint16_t*>(Qs);
    const uint16_t* k = static_cast<const uint16_t*>(K);
    const uint16_t* k_r = k + static_cast<int64_t>(key_begin) * kD;
    float* score_r = score + key_begin;
    static std::atomic<uint64_t> row_ok[3], col_ok[4];
    auto allow = [](auto kernel, size_t bytes, std::atomic<uint64_t>& done) {
      return allow_dynamic_lds(reinterpret_cast<const void*>(kernel), bytes, done, "pc_score");
    };
    const Divisor by_qs(n_qs);
    const RowPlan row = plan_rows(Hkv, rep * n_qs, Nk, unit_c);
    const ColPlan col = plan_cols(Hkv, rep * n_qs, nkr, lse ? 1 : row.n_splits);
    if (lse == nullptr) {
      const int n_row_tiles = ceil_div(rep * n_qs, row.small ? kWaveRows : kBlockRows);
      if (row.small) {
        if (int rc = allow(score_rowpass_small, kSmallRowSmem, row_ok[2])) return rc;
        score_rowpass_small<<<n_row_tiles * Hkv * row.n_splits, kThreads, kSmallRowSmem, s>>>(
            q, q_rows, k, ws_part, rep, by_qs, Nk, q_stride_h, k_stride_h, c, Divisor(n_row_tiles), Divisor(Hkv),
            ceil_div(ceil_div(Nk, kSmallStep), row.n_splits));
      } else {
        const auto kernel = unit_c ? score_rowpass_bf16<true> : score_rowpass_bf16<false>;
        if (int rc = allow(kernel, kRowSmem, row_ok[unit_c])) return rc;
        kernel<<<n_row_tiles * Hkv * row.n_splits, kThreads, kRowSmem, s>>>(
            q, q_rows, k, ws_part, rep, by_qs, Nk, q_stride_h, k_stride_h, c, Divisor(n_row_tiles), Divisor(Hkv),
            ceil_div(ceil_div(Nk, kTileRows), row.n_splits));
      }
      PC_CHECK_LAUNCH("pc_score row pass");
    }
    RowNorm norm = {nullptr, lse, lse_stride_h, q_rows, ws_part, static_cast<int64_t>(Hq) * n_qs, row.n_splits, rep, by_qs};
    const bool direct = col.n_qsplits == 1 && !share_heads;
    float* col_out = direct ? score_r : ws_col;
    const int64_t col_stride = direct ? score_stride_h : nkr;
    if (!col.prepares) {
      score_row_norms<<<dim3(ceil_div(rep * n_qs, 256), Hkv), 256, 0, s>>>(norm, ws_lse);
      PC_CHECK_LAUNCH("pc_score normalisers");
      norm.ready = ws_lse;
    }
    if (col.small) {
      const auto kernel = unit_c ? score_colpass_small<true> : score_colpass_small<false>;
      if (int rc = allow(kernel, kSmallColSmem, col_ok[2 + unit_c])) return rc;
      const int n_key_blocks = ceil_div(nkr, kWaveRows);
      kernel<<<n_key_blocks * Hkv, kThreads, kSmallColSmem, s>>>(q, q_rows, k_r, norm, col_out, col_stride, rep, by_qs, nkr,
                                                                 q_stride_h, k_stride_h, c, Divisor(n_key_blocks));
    } else {
      const auto kernel = unit_c ? score_colpass_bf16<true> : score_colpass_bf16<false>;
      if (int rc = allow(kernel, kColSmem, col_ok[unit_c])) return rc;
      const int n_key_blocks = ceil_div(nkr, kBlockRows);
      kernel<<<n_key_blocks * Hkv * col.n_qsplits, kThreads, kColSmem, s>>>(
          q, q_rows, k_r, norm, col_out, col_stride, static_cast<int64_t>(Hkv) * nkr, rep, by_qs, nkr, q_stride_h,
          k_stride_h, c, Divisor(n_key_blocks), Divisor(col.n_qsplits),
          ceil_div(ceil_div(rep * n_qs, kTileRows), col.n_qsplits));
    }
    PC_CHECK_LAUNCH("pc_score column pass");
    if (!direct) {
      if (share_heads && col.n_qsplits > 1)
        score_reduce_heads<<<ceil_div(nkr, 64), 64 * std::min(Hkv, kReduceHeads), 0, s>>>(ws_col, score_r, col.n_qsplits,
                                                                                         Hkv, nkr);
      else
        score_reduce<<<dim3(ceil_div(nkr, 256), share_heads ? 1 : Hkv), 256, 0, s>>>(
            ws_col, score_r, score_stride_h, col.n_qsplits, Hkv, nkr, share_heads);
      PC_CHECK_LAUNCH("pc_score reduce");
    }
    return PC_OK;
  } else {
    PC_REQUIRE(D == 64 || D == 128, PC_ERR_UNSUPPORTED, "pc_score: fp32 tier needs D=64 or 128, got %d", D);
    float* per_head = share_heads ? ws_col : score + key_begin;
    const int64_t per_head_stride = share_heads ? nkr : score_stride_h;
    const float* q = static_cast<const float*>(Qs);
    const float* k = static_cast<const float*>(K);
    const float* k_r = k + static_cast<int64_t>(key_begin) * D;
    if (D == 64)
      score_f32<64>(q, q_rows, k, k_r, lse, lse_stride_h, ws_lse, per_head, per_head_stride, Hq, Hkv, n_qs, Nk, nkr,
                    q_stride_h, k_stride_h, scale, s);
    else
      score_f32<128>(q, q_rows, k, k_r, lse, lse_stride_h, ws_lse, per_head, per_head_stride, Hq, Hkv, n_qs, Nk, nkr,
                     q_stride_h, k_stride_h, scale, s);
    PC_CHECK_LAUNCH("pc_score passes");
    if (share_heads) {
      score_reduce<<<ceil_div(nkr, 256), 256, 0, s>>>(ws_col, score + key_begin, score_stride_h, 1, Hkv, nkr, 1);
      PC_CHECK_LAUNCH("pc_score head sum");
    }
  }
  return PC_OK;
}
