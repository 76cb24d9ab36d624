// pc_frame_attn: attention of one frame's queries over the keys presented (Eq. 2).
//
// bf16 tier (D = 128): flash-style kernel on the gfx950 32x32x16 bf16 MFMA.
//   * Scores are formed transposed, S^T = K Q^T: in the MFMA result layout a lane then
//     holds ONE query column and 16 keys per 32-key block.  The reference maximum and the
//     running sum of a query are per-lane scalars, and the probabilities are already laid
//     out as the B operand of the second product O^T += V^T P^T, so P never goes through LDS.
//   * K and V tiles are fetched straight from global memory into LDS (no register
//     staging), four tiles deep; V stays row-major in LDS and is transposed by the LDS
//     transposing read on its way into the MFMA A operand.
//   * Softmax in fp32 with base-2 exponentials, interleaved instruction by instruction with
//     the products of the neighbouring half tiles.  No row maximum is taken on the fast path:
//     probabilities are formed against the standing reference, and a half tile is redone
//     (and the accumulators rescaled) only when one of its row sums runs away.
//   * With scale = ln 2 (the caller multiplied Q by scale * log2(e), e.g. while rotating it)
//     the affine step c*s - m is taken out of the loop: see kUnitC below.
// fp32 tier (D = 64 or 128): fp32 MFMA, 16 or 32 query rows per work-group (see attn_f32_kernel).
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "lds_dma.h"

namespace pc {
namespace {

constexpr int kD = 128;
constexpr int kPPThreads = 512;      // 8 waves, two per SIMD
constexpr int kBM = 256;             // query rows per work-group (32 per wave)
constexpr int kBN = 64;              // keys per tile
constexpr int kRowBytes = kD * 2;    // a K or V row in LDS: 256 bytes, unpadded, chunk-swizzled
constexpr int kTileBytes = kBN * kRowBytes;
constexpr int kStages = 4;           // LDS slots per operand: tile t lives in slot t % kStages
constexpr size_t kSmemBytes = 2 * kStages * kTileBytes;
constexpr float kRescaleTrigger = 1024.f;  // row sum of a half tile that forces a new reference maximum
constexpr float kLowestStart = -4096.f;    // lowest reference that products start from (see pipeline_phase)
constexpr int kRing = 4;
// The reference of a query that has seen no key, or only keys of a score -inf: finite, so that such
// keys weigh exp2(-inf) = 0 and what has been summed (zeros) merges like any other share.
constexpr float kNoRef = -3.402823466e38f;

// ---- LDS tile layout ---------------------------------------------------------------------------
// K tiles use the fragment-read swizzle of lds_dma.h.  V is read with transposing loads
// (4 rows x 32 bytes per quarter wave): chunk c of row r is stored at position c ^ (4 (r & 3)).
__device__ __forceinline__ int v_chunk_pos(int row, int chunk) { return chunk ^ ((row & 3) << 2); }

// Wait until at most 4 (kStages - 2) of this wave's direct loads are still in flight: every
// staging point issues exactly four, so all but the newest kStages - 2 points have landed.
__device__ __forceinline__ void dma_wait_older() { asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); }
static_assert(kStages == 4, "dma_wait_older encodes 4 * (kStages - 2)");

// Stage tile rows [k0, k0+64) of K or V: each of the 8 waves issues two 1-KB loads.
template <bool kIsV>
__device__ __forceinline__ void stage_tile(const uint16_t* __restrict__ base_h, int k0, int Nk, uint32_t lds_tile,
                                           int wave, int lane) {
  const RowWindow w = row_window(base_h, k0, Nk);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (wave * 2 + i) * 4 + (lane >> 4);  // 4 rows per load
    const int pos = lane & 15;                          // chunk position inside the row
    const int chunk = kIsV ? v_chunk_pos(row, pos) : k_chunk_pos(row, pos);  // both maps are involutions
    dma_16B_at(w.base, row_offset(w, row, chunk), lds_tile + (wave * 2 + i) * 1024);
  }
}

// The query rows of one KV head are numbered through its `rep` query heads: row rho is row
// rho % Nq of head kvh * rep + rho / Nq.  A tile of rows may span heads, so a frame that is no
// multiple of the tile leaves at most one part-filled tile per KV head instead of one per head.
struct RowAt {
  int head, row;
};
__device__ __forceinline__ RowAt row_at(int rho, int kvh, int rep, const Divisor& by_nq) {
  const int in_group = by_nq.of(rho);
  return {kvh * rep + in_group, rho - in_group * by_nq.d};
}

// The key share of work-group L, shares of n_units work-groups one after another; L becomes the unit.  By
// subtraction: calls that are not cut (L < n_units) pay nothing for it.  A division by a number that is not
// known is 0.2 us at the front of every work-group, and there were four of them (16/4 heads x 4,032 rows x 64
// keys 14.0 us with them, 13.4 without; 8/2 x 17 rows x 64 keys 6.3 and 5.6).
__device__ __forceinline__ int take_share(int& L, int n_units) {
  int share = 0;
  for (; L >= n_units; L -= n_units) ++share;   // at most kMaxKeySplits - 1 times
  return share;
}

// One phase of the software pipeline (see the kernel comment): 8 score products, then 8
// value products, with one element of the probability stage behind each.
// The probabilities are formed against the reference m_ref as it stands; no maximum is
// taken on the fast path.  If any row sum of the half tile comes out above kRescaleTrigger
// (a score outgrew the reference: rare, at most once per 2^10 of growth), the half tile is
// redone against its exact maximum and O, l are rescaled.
// kUnitC: the caller folded scale * log2(e) into Q (c == 1).  The score products then start
// from -m_ref instead of zero (neg_m: the reference in all 16 accumulator registers of the
// lane, which holds one query), so a score arrives as s - m_ref and the probability is a bare
// exp2: one vector instruction per element fewer.  When the reference moves, the scores that
// were started from the old one are shifted by the difference.
// Keys of a score -inf, or of a mask value far below the rest, weigh nothing, and a wave may see a half
// tile of nothing else before its first real key.  c general: a reference of -inf makes the row sum
// NaN or inf, so every half tile is redone until there is a finite one, and a redo without one adds
// zeros.  kUnitC: products must not start from such a reference (inf - inf, or a score lost in the
// rounding of -m_ref: an ulp at kLowestStart is 2^-11): they start from zero instead, and while any
// query of the wave is in that state (low_ref) every half tile is redone.
template <bool kUnitC>
__device__ __forceinline__ void pipeline_phase(
    const lds_u8* k_half, const int (&k_off)[8], const lds_u8* v_half, const int (&v_off)[4],
    const bf16x8 (&qf)[8], f32x16& s_nxt, const bf16x8 (&p_mm)[2], f32x16 (&o)[4], const f32x16& s_cur,
    bf16x8 (&p_cur)[2], float& m_ref, float& l_run, float c, f32x16& neg_m, bool& low_ref) {
  // fragment k: 0..7 -> K rows, contraction step k; 8..15 -> V^T (key step (k-8)/4, block (k-8)%4)
  auto frag = [&](int k) -> bf16x8 {
    if (k < 8) {
      return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(k_half + k_off[k]);
    }
    const int ks = (k - 8) >> 2, db = (k - 8) & 3;
    // keys ks*16 + g*4 + {0..3} and + 8: two transposing reads of 4 keys each
    const lds_u8* p = v_half + v_off[db] + ks * 16 * kRowBytes;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(p)));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(p + 8 * kRowBytes)));
    bf16x8 f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[e] = lo[e];
      f[4 + e] = hi[e];
    }
    return f;
  };
  bf16x8 ring[kRing];
#pragma unroll
  for (int r = 0; r < kRing; ++r) ring[r] = frag(r);
  f32x16 zero;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero[i] = 0.f;
  f32x16 s_acc = zero;
  float psum = 0.f;
  float pv[16];
  // The wave asks for issue priority over its SIMD neighbour while it is inside the interleaved
  // matrix / vector block, and gives it back for the bookkeeping behind it (measured: +0.5 %).
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const bf16x8 f = ring[k % kRing];
    if (k < 8) {
      s_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[k], k == 0 ? (kUnitC ? neg_m : zero) : s_acc, 0, 0, 0);
    } else {
      const int ks = (k - 8) >> 2, db = (k - 8) & 3;
      o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, p_mm[ks], o[db], 0, 0, 0);
    }
    if (k + kRing < 16) ring[k % kRing] = frag(k + kRing);
    pv[k] = kUnitC ? __builtin_amdgcn_exp2f(s_cur[k]) : __builtin_amdgcn_exp2f(fmaf(s_cur[k], c, -m_ref));
    psum += pv[k];
    if (k & 1) {
      p_cur[k >> 3][(k & 7) - 1] = static_cast<__bf16>(pv[k - 1]);
      p_cur[k >> 3][k & 7] = static_cast<__bf16>(pv[k]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(0);
  // keep the vector results in this basic block (otherwise they sink below the next branch)
#pragma unroll
  for (int half = 0; half < 2; ++half) asm volatile("" : "+v"(p_cur[half]));
  asm volatile("" : "+v"(psum));
  if ((kUnitC && low_ref) || __any(!(psum <= kRescaleTrigger))) {  // also catches inf and NaN
    float mx = s_cur[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s_cur[i]);
    mx = wave_half_max(mx);
    // unit c: s_cur holds s - start, and so do the scores just formed; start is the reference or zero
    const float start = kUnitC ? -neg_m[0] : 0.f;
    const float m_new = fmaxf(m_ref, kUnitC ? start + mx : mx * c);
    const bool none = m_new == -INFINITY;   // no key of a finite score yet
    const float alpha = none ? 1.f : __builtin_amdgcn_exp2f(m_ref - m_new);
    const float m_use = none ? 0.f : m_new - start;
    psum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      pv[i] = kUnitC ? __builtin_amdgcn_exp2f(s_cur[i] - m_use) : __builtin_amdgcn_exp2f(fmaf(s_cur[i], c, -m_use));
      psum += pv[i];
    }
    if constexpr (kUnitC) {
      const float start_new = m_new >= kLowestStart ? m_new : 0.f;
      low_ref = __any(!(m_new >= kLowestStart));
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s_acc[i] -= start_new - start;
        neg_m[i] = -start_new;
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) p_cur[i >> 3][i & 7] = static_cast<__bf16>(pv[i]);
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    m_ref = m_new;
  }
  l_run += psum;
  s_nxt = s_acc;
}

// ------------------------------------------------------------------------------------------
// bf16 frame attention.  8 waves (two per SIMD), 32 query rows each, 256 rows per
// work-group; keys in tiles of 64, processed as half tiles A (keys 0..31) and B (32..63).
// On this chip matrix and vector instructions overlap only inside one wave's instruction
// stream, so every wave interleaves, in one basic block per phase,
//     matrix:  S_nxt^T = K_half Q^T (8 products)  and  O^T += V_half^T P_mm^T (8 products)
//     vector:  P_cur = exp2(c S_cur - m_ref), its bf16 packing and its row sum
// where cur is the half tile scored one phase earlier and mm the one before that:
//     phase 1 of tile j:  S_B(j), O += V_B(j-1) P_B(j-1)  |  P_A(j)
//     phase 2 of tile j:  S_A(j+1), O += V_A(j) P_A(j)    |  P_B(j)
// One work-group barrier per tile, after phase 1: behind it K(j+4) and V(j+3) are fetched
// straight into the LDS slots just released (four slots per operand, 128 KB), three tiles
// ahead of their first use.
// ------------------------------------------------------------------------------------------
template <bool kUnitC>
__global__ __launch_bounds__(kPPThreads, 1) void attn_bf16_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ lse, int rep, Divisor by_nq, int Nk, int64_t q_stride_h,
    int64_t kv_stride_h, int64_t o_stride_h, float c, Divisor by_tiles_q, int n_whole, int n_cut, int share_tiles,
    float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t row_whole, int64_t rows_cut) {
  extern __shared__ __align__(16) uint8_t smem_raw[];
  lds_u8* smem = (lds_u8*)smem_raw;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  auto k_slot = [](int t) { return (t & (kStages - 1)) * kTileBytes; };
  auto v_slot = [](int t) { return (kStages + (t & (kStages - 1))) * kTileBytes; };

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  // Row tiles in the order (KV head, tile).  The first n_whole of them (whole rounds of the chip, or all)
  // walk all keys; the other n_cut are cut into shares of share_tiles key tiles, share slowest.
  const bool whole = static_cast<int>(blockIdx.x) < n_whole;
  int unit = whole ? xcd_contiguous_index(blockIdx.x, n_whole)
                   : xcd_contiguous_index(blockIdx.x - n_whole, gridDim.x - n_whole);
  const int split = whole ? 0 : take_share(unit, n_cut);
  if (!whole) unit += n_whole;
  const int kvh = by_tiles_q.of(unit), tile = unit - kvh * by_tiles_q.d;
  const int n_rows = rep * by_nq.d;    // query rows of the KV head
  const int rho = tile * kBM + wave * 32 + l32;   // the row this lane owns
  const bool active = rho - l32 < n_rows;  // wave-uniform

  const uint16_t* Kh = K + kvh * kv_stride_h;
  const uint16_t* Vh = V + kvh * kv_stride_h;

  f32x16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  f32x16 sA, sB;
  bf16x8 pA[2], pB[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pA[ks][e] = static_cast<__bf16>(0.f);
      pB[ks][e] = static_cast<__bf16>(0.f);
    }
  float m_ref = -INFINITY, l_run = 0.f;
  bool low_ref = false;   // wave-uniform
  f32x16 neg_m;
#pragma unroll
  for (int i = 0; i < 16; ++i) neg_m[i] = 0.f;

  // per-lane byte offsets inside a half tile
  int k_off[8];  // K fragment of contraction step s: row l32, chunk 2s+g
#pragma unroll
  for (int s = 0; s < 8; ++s) k_off[s] = l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  int v_off[4];  // V^T fragment of output block db: this lane SUPPLIES row g*4 + r/4, dims db*32 + G*16 + 4(r%4)
  {
    const int r = lane & 15, G = (lane >> 4) & 1;
    const int row = g * 4 + (r >> 2);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      const int dim = db * 32 + G * 16 + 4 * (r & 3);
      v_off[db] = row * kRowBytes + v_chunk_pos(row, dim >> 3) * 16 + (dim & 7) * 2;
    }
  }

  // this work-group's share of the key tiles: n of n_all (the host leaves no share empty)
  const int n_all = (Nk + kBN - 1) / kBN;
  const int per = whole ? n_all : share_tiles;
  const int n = min(per, n_all - split * per);
  const int key0 = split * per * kBN;
  const int n_valid = Nk - key0;   // less than n tiles only where the ragged last tile is in this share

  // the V slot of "tile -1" is read once against zero probabilities: clear it
  for (int e = threadIdx.x; e < kTileBytes / 16; e += kPPThreads)
    reinterpret_cast<__attribute__((address_space(3))) u32x4*>(smem + v_slot(-1))[e] = u32x4{0u, 0u, 0u, 0u};
  // Prologue, in order of need: K(0), V(0), K(1), the queries, then K(2), V(1), K(3), V(2).  Tiles past
  // the end of the cache are fetched too (clamped rows, never read) so that every staging point
  // issues the same number of loads and the in-flight count can be waited on.
  auto stage_k = [&](int j) { stage_tile<false>(Kh, key0 + j * kBN, Nk, lds0 + k_slot(j), wave, lane); };
  auto stage_v = [&](int j) { stage_tile<true>(Vh, key0 + j * kBN, Nk, lds0 + v_slot(j), wave, lane); };
  stage_k(0);
  stage_v(0);
  stage_k(1);
  // The wave's 32 query rows, whole rows through the slots that nothing is staged in yet (those of K(2),
  // K(3), V(1), V(2): half a slot per wave), behind the first fetches: one memory latency covers all of them.
  bf16x8 qf[8];
  {
    constexpr int kFree[4] = {2, 3, kStages + 1, kStages + 2};
    const int slot = (wave >> 1) == 0 ? kFree[0] : (wave >> 1) == 1 ? kFree[1] : (wave >> 1) == 2 ? kFree[2] : kFree[3];
    const int at = slot * kTileBytes + (wave & 1) * 32 * kRowBytes;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = i * 4 + (lane >> 4);
      const RowAt from = row_at(min(rho - l32 + row, n_rows - 1), kvh, rep, by_nq);
      dma_16B(Q + from.head * q_stride_h + static_cast<int64_t>(from.row) * kD + k_chunk_pos(row, lane & 15) * 8,
              __builtin_amdgcn_readfirstlane(lds0 + at + i * 1024));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = lds_frag(smem + at + k_off[s]);
#pragma unroll
    for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qf[s]));
  }
  __syncthreads();   // K(0), V(0), K(1) have landed; every wave has its queries and the slots are free
  stage_k(2);
  stage_v(1);
  stage_k(3);
  stage_v(2);

  auto mask_tail = [&](f32x16& sc, int lim) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if ((i >> 2) * 8 + (i & 3) >= lim) sc[i] = -INFINITY;
  };
  if (active) {  // S_A of tile 0 and the first reference maximum
    f32x16 zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const bf16x8 kf = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(smem + k_slot(0) + k_off[s]);
      sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], s == 0 ? zero : sA, 0, 0, 0);
    }
    float mx = sA[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sA[i]);
    m_ref = wave_half_max(mx) * c;
    if constexpr (kUnitC) {
      const float start = m_ref >= kLowestStart ? m_ref : 0.f;
      low_ref = __any(!(m_ref >= kLowestStart));
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sA[i] -= start;
        neg_m[i] = -start;
      }
    }
    if (n_valid < kBN) mask_tail(sA, n_valid - g * 4);
  }

  // Tile j lives in LDS slot j % 4.  The loop is unrolled four times so that every slot is a
  // compile-time constant and lands in the offset field of the LDS reads instead of costing a
  // vector add per fragment address.
  auto tile_body = [&](int j, auto slot_tag) {
    constexpr int u = decltype(slot_tag)::value;            // j % kStages
    constexpr int k_cur = u * kTileBytes, k_nxt = ((u + 1) & 3) * kTileBytes;
    constexpr int v_prev = (kStages + ((u + 3) & 3)) * kTileBytes, v_cur = (kStages + u) * kTileBytes;
    const int left = n_valid - j * kBN;   // valid keys from this tile on
    // ---- phase 1: S_B(j), O += V_B(j-1) P_B(j-1)  |  P_A(j) ----
    if (active) {
      pipeline_phase<kUnitC>(smem + k_cur + 32 * kRowBytes, k_off, smem + v_prev + 32 * kRowBytes, v_off, qf, sB, pB, o, sA,
                     pA, m_ref, l_run, c, neg_m, low_ref);
      if (left < kBN) mask_tail(sB, left - 32 - g * 4);
    }
    // One barrier per tile: every wave is past K(j) and V(j-1), and K(j+1), V(j) (fetched
    // kStages - 1 tiles ago) have landed: each wave waited for its own share.
    dma_wait_older();
    __syncthreads();
    stage_tile<false>(Kh, key0 + (j + kStages) * kBN, Nk, lds0 + k_cur, wave, lane);
    stage_tile<true>(Vh, key0 + (j + kStages - 1) * kBN, Nk, lds0 + v_prev, wave, lane);
    // ---- phase 2: S_A(j+1), O += V_A(j) P_A(j)  |  P_B(j) ----
    // (after the last tile S_A is formed from a clamped tile and never used)
    if (active) {
      pipeline_phase<kUnitC>(smem + k_nxt, k_off, smem + v_cur, v_off, qf, sA, pA, o, sB, pB, m_ref, l_run, c, neg_m,
                             low_ref);
      if (left < 2 * kBN) mask_tail(sA, left - kBN - g * 4);
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
  // ---- drain: O += V_B(n-1) P_B(n-1) ----
  if (active) {
    const lds_u8* v_half = smem + v_slot(n - 1) + 32 * kRowBytes;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const lds_u8* p = v_half + v_off[db] + ks * 16 * kRowBytes;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(p)));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(p + 8 * kRowBytes)));
        bf16x8 vf;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vf[e] = lo[e];
          vf[4 + e] = hi[e];
        }
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pB[ks], o[db], 0, 0, 0);
      }
  }
  const float l_tot = wave_half_sum(l_run);
  const int64_t at = static_cast<int64_t>(kvh) * n_rows + rho;   // row number over all heads
  // The output leaves through LDS in whole rows: a lane holds 4 dims of its row at a time, 32 rows apart.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // tiles past the end may still be landing
  __syncthreads();
  if (!active) return;
  const int rows_w = min(32, n_rows - (rho - l32));   // rows of this wave that exist
  lds_u8* mine = smem + wave * kTileBytes;
  if (!whole) {  // one of several key shares: un-normalised O, reference and sum for the merge
    const int64_t first = split * rows_cut + at - l32 - row_whole;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = o[db][a * 4 + e];
        *reinterpret_cast<__attribute__((address_space(3))) f32x4*>(mine + l32 * 512 + ((db * 8 + a * 2 + g) ^ l32) * 16) = v;
      }
    wave_lds_sync();   // rows come back from other lanes of the wave
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = i * 2 + g;
      const f32x4 v = *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(mine + row * 512 + l32 * 16);
      if (row < rows_w) *reinterpret_cast<f32x4*>(part_o + (first + row) * kD + (l32 ^ row) * 4) = v;
    }
    if (g == 0 && l32 < rows_w) part_ml[first + l32] = make_float2(m_ref, l_tot);
    return;
  }
  const float inv = 1.f / l_tot;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      u32x2 out;
      out[0] = pack_bf16x2(o[db][a * 4 + 0] * inv, o[db][a * 4 + 1] * inv);
      out[1] = pack_bf16x2(o[db][a * 4 + 2] * inv, o[db][a * 4 + 3] * inv);
      *reinterpret_cast<__attribute__((address_space(3))) u32x2*>(mine + l32 * kRowBytes + k_chunk_pos(l32, db * 4 + a) * 16 + g * 8) = out;
    }
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = i * 4 + (lane >> 4), chunk = k_chunk_pos(row, lane & 15);
    const u32x4 v = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(mine + row * kRowBytes + (lane & 15) * 16);
    if (row < rows_w) {
      const RowAt to = row_at(rho - l32 + row, kvh, rep, by_nq);
      *reinterpret_cast<u32x4*>(O + to.head * o_stride_h + static_cast<int64_t>(to.row) * kD + chunk * 8) = v;
    }
  }
  if (rho < n_rows) {
    if (lse != nullptr && g == 0)
      lse[at] = (m_ref + log2f(l_tot)) * 0.6931471805599453f;
  }
}

// Where the waves of a work-group share rows: wave w holds (O, m, l) of rows 32 (w % kR) .. + 31 over its keys, and
// they are merged in wave order.  A wave's O goes to 16 KB of LDS of its own, piece i = accumulators
// 4 i .. 4 i + 3 of every lane = dims 8 i + 4 g .. + 3 of its row, lanes permuted by i so that the reads
// below use every bank; a thread then adds up eight dims of a row, and a row leaves whole.
constexpr int kWaveOBytes = 32 * kD * 4;
constexpr size_t kMergeBytes = 8 * kWaveOBytes + 8 * 32 * 8;
// kBlocks: blocks of 32 dims that the work-group holds, from dim0 on.
template <int kR, int kBlocks>
__device__ __forceinline__ void merge_waves(lds_u8* smem, const f32x16 (&o)[kBlocks], int dim0, float m, float l, int wave, int lane,
                                            int tile, int kvh, int split, uint16_t* __restrict__ O,
                                            float* __restrict__ lse, int rep, const Divisor& by_nq, int64_t o_stride_h,
                                            float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t rows_all) {
  auto piece = [&](int w, int i, int of_lane) {
    return reinterpret_cast<__attribute__((address_space(3))) f32x4*>(smem + w * kWaveOBytes + i * 1024 + (of_lane ^ i) * 16);
  };
  auto* s_ml = reinterpret_cast<__attribute__((address_space(3))) float*>(smem + 8 * kWaveOBytes);
#pragma unroll
  for (int db = 0; db < kBlocks; ++db)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      *piece(wave, db * 4 + a, lane) = f32x4{o[db][a * 4], o[db][a * 4 + 1], o[db][a * 4 + 2], o[db][a * 4 + 3]};
  if (lane < 32) {
    s_ml[(wave * 32 + lane) * 2] = m;
    s_ml[(wave * 32 + lane) * 2 + 1] = l;
  }
  __syncthreads();
  const int n_rows = rep * by_nq.d;
  const int row = threadIdx.x >> 4, i = threadIdx.x & 15;
  if (i >= 4 * kBlocks) return;
#pragma unroll
  for (int rg = 0; rg < kR; ++rg) {
    const int rho = (tile * kR + rg) * 32 + row;
    float mw[8 / kR], M = -INFINITY, lt = 0.f;
#pragma unroll
    for (int w = 0; w < 8 / kR; ++w) {
      mw[w] = s_ml[((w * kR + rg) * 32 + row) * 2];
      M = fmaxf(M, mw[w]);
    }
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int w = 0; w < 8 / kR; ++w) {
      const float wt = __builtin_amdgcn_exp2f(mw[w] - M);
      lt += wt * s_ml[((w * kR + rg) * 32 + row) * 2 + 1];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const f32x4 v = *piece(w * kR + rg, i, t * 32 + row);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][e] += wt * v[e];
      }
    }
    if (rho >= n_rows) return;
    const int64_t at = static_cast<int64_t>(kvh) * n_rows + rho;
    if (part_o != nullptr) {
      const int64_t at_s = split * rows_all + at;
#pragma unroll
      for (int t = 0; t < 2; ++t) *reinterpret_cast<f32x4*>(part_o + at_s * kD + dim0 + i * 8 + t * 4) = acc[t];
      if (dim0 + i == 0) part_ml[at_s] = make_float2(M, lt);
      continue;
    }
    const float inv = 1.f / lt;
    const RowAt to = row_at(rho, kvh, rep, by_nq);
    u32x4 out;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      out[t * 2] = pack_bf16x2(acc[t][0] * inv, acc[t][1] * inv);
      out[t * 2 + 1] = pack_bf16x2(acc[t][2] * inv, acc[t][3] * inv);
    }
    *reinterpret_cast<u32x4*>(O + to.head * o_stride_h + static_cast<int64_t>(to.row) * kD + dim0 + i * 8) = out;
    if (lse != nullptr && dim0 + i == 0) lse[at] = (M + log2f(lt)) * 0.6931471805599453f;
  }
}

// ------------------------------------------------------------------------------------------
// bf16 frame attention for small calls: 32 query rows per work-group, the 8 waves take the keys in
// steps of 32 by turns, each through LDS of its own (a step's fragments go to registers at once, and
// the next step is fetched behind them), so the loop has no barrier; (O, m, l) of the waves are
// merged through LDS once.  Bound: latency.  Eight times as many work-groups as
// attn_bf16_kernel makes of the same rows, each an eighth as long; K and V come through L2 once per
// 32 rows instead of once per 256, which is why large calls do not take this form (a step of 8 x 32
// keys takes 1.4 us with every compute unit at it: 0.78 PFLOP/s at most).  8/2 heads x 252 rows x
// 1,179 keys: 29.7 us in 8 work-groups of 256 rows, 9.9 us un-split in 64 of these (11.3 before the query rows
// came through LDS; 2/1 x 184 x 900 8.9 -> 7.7).  The loop runs at what a compute unit draws from L2 (128 KB a
// step in 1.17 us).  K straight into registers (32 rows x 32 bytes per load) took 2.2 us a step.
// So where half of the compute units would idle, two or four work-groups take the same rows and keys and divide the
// output's dims (kBlocks of 32 each): each forms all scores, but fetches and adds up only its part of V (96 or
// 80 KB a step, not 128) and merges only its part of O; there is nothing to put together behind them and the
// bits are the same.  8/2 x 252 x 1,179 (64 work-groups of 32 rows) 10.2 us undivided, 8.8 in two, 8.7 in four; 2/1
// x 1,718 x 1,000 (108) 9.4 and 8.2 in two.
// ------------------------------------------------------------------------------------------
constexpr int kSmallRows = 32;
constexpr int kSmallKeys = 32;                                  // keys per wave and step
constexpr int kSmallTileBytes = kSmallKeys * kRowBytes;
constexpr size_t kSmallSmem = kMergeBytes + kSmallRows * kRowBytes;
static_assert(2 * kSmallTileBytes <= kWaveOBytes, "a wave stages K and V in the LDS of its merge piece");

template <int kBlocks>
__global__ __launch_bounds__(kPPThreads, 1) void attn_bf16_small_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ lse, int rep, Divisor by_nq, int Nk, int64_t q_stride_h,
    int64_t kv_stride_h, int64_t o_stride_h, float c, Divisor by_tiles_q, int n_tiles, int share_steps,
    float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t rows_all) {
  extern __shared__ __align__(16) uint8_t smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const lds_u8* lds = (lds_u8*)smem_raw + wave * kWaveOBytes;
  const uint32_t lds_w = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  constexpr int kParts = 4 / kBlocks;           // work-groups that share rows and keys
  constexpr int kVRow = kBlocks * 64, kVChunks = kVRow / 16, kVLoads = 2 * kBlocks;   // a V row in LDS, loads of a step's
  // chunk c of V row r lies where the four rows of a quarter wave's read use different banks
  auto v_pos = [](int row, int chunk) {
    return kBlocks == 4 ? v_chunk_pos(row, chunk) : kBlocks == 2 ? chunk ^ ((row & 2) << 1) : chunk;
  };
  int unit = xcd_contiguous_index(blockIdx.x, gridDim.x);   // n_tiles row tiles per share
  const int dim0 = unit % kParts * kBlocks * 32;
  unit /= kParts;
  const int split = take_share(unit, n_tiles);
  const int kvh = by_tiles_q.of(unit), tile = unit - kvh * by_tiles_q.d;
  const int n_rows = rep * by_nq.d;
  const uint16_t* Kh = K + kvh * kv_stride_h;
  const uint16_t* Vh = V + kvh * kv_stride_h;

  // this share's keys, whole steps but for the very last
  const int k_begin = split * share_steps * kSmallKeys, k_end = min(k_begin + share_steps * kSmallKeys, Nk);

  // a step's 32 rows of K and of V, two 8-KB pieces of the wave's LDS
  auto stage = [&](int k0) {
    const RowWindow wk = row_window(Kh, k0, Nk), wv = row_window(Vh, k0, Nk);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = i * 4 + (lane >> 4);
      dma_16B_at(wk.base, row_offset(wk, row, k_chunk_pos(row, lane & 15)), lds_w + i * 1024);
      if (i < kVLoads) {
        const int v_row = i * (1024 / kVRow) + lane / kVChunks;
        dma_16B_at(wv.base, row_offset(wv, v_row, dim0 / 8 + v_pos(v_row, lane % kVChunks)), lds_w + kSmallTileBytes + i * 1024);
      }
    }
  };
  const int k_first = k_begin + wave * kSmallKeys;
  // The query rows go through LDS once, four per wave: every wave holds all of them, and as fragments from
  // memory (32 bytes of each row per load) they were 64 KB per work-group.
  const lds_u8* q_tile = (lds_u8*)smem_raw + kMergeBytes;
  {
    const int row = wave * 4 + (lane >> 4);
    const RowAt from = row_at(min(tile * kSmallRows + row, n_rows - 1), kvh, rep, by_nq);
    dma_16B(Q + from.head * q_stride_h + static_cast<int64_t>(from.row) * kD + k_chunk_pos(row, lane & 15) * 8,
            static_cast<uint32_t>(reinterpret_cast<uintptr_t>(q_tile)) + wave * 1024);
  }
  stage(k_first);
  int k_off[8], v_off[kBlocks];  // as in attn_bf16_kernel
#pragma unroll
  for (int s = 0; s < 8; ++s) k_off[s] = l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  // this wave's queries: the loads behind them are its first keys
  if constexpr (kBlocks == 4) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  else if constexpr (kBlocks == 2) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
  __syncthreads();
  bf16x8 qf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) qf[s] = lds_frag(q_tile + k_off[s]);
  {
    const int r = lane & 15, G = (lane >> 4) & 1;
    const int row = g * 4 + (r >> 2);
#pragma unroll
    for (int db = 0; db < kBlocks; ++db) {
      const int dim = db * 32 + G * 16 + 4 * (r & 3);
      v_off[db] = kSmallTileBytes + row * kVRow + v_pos(row, dim >> 3) * 16 + (dim & 7) * 2;
    }
  }
  f32x16 o[kBlocks];
#pragma unroll
  for (int db = 0; db < kBlocks; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m = kNoRef, l = 0.f;

  for (int k0 = k_first; k0 < k_end; k0 += 8 * kSmallKeys) {
    // This step's rows have landed (they are all that is in flight): take every fragment into
    // registers, so that the next step's rows can be fetched into the same LDS at once.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bf16x8 kf[8], vf[2][kBlocks];
#pragma unroll
    for (int s = 0; s < 8; ++s) kf[s] = lds_frag(lds + k_off[s]);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < kBlocks; ++db) {
        const lds_u8* src = lds + v_off[db] + ks * 16 * kVRow;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(src)));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(src + 8 * kVRow)));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vf[ks][db][e] = lo[e];
          vf[ks][db][4 + e] = hi[e];
        }
      }
#pragma unroll
    for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(kf[s]));
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < kBlocks; ++db) asm volatile("" : "+v"(vf[ks][db]));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (k0 + 8 * kSmallKeys < k_end) stage(k0 + 8 * kSmallKeys);  // wave-uniform
    f32x16 sc;
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sc, 0, 0, 0);
    if (k0 + kSmallKeys > k_end) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (k0 + (i >> 2) * 8 + g * 4 + (i & 3) >= k_end) sc[i] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
    mx = wave_half_max(mx) * c;
    if (__any(!(mx <= m + 8.f))) {     // the reference lags by at most 2^8
      const float m_new = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int db = 0; db < kBlocks; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
      m = m_new;
    }
    bf16x8 p[2];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float e = __builtin_amdgcn_exp2f(fmaf(sc[i], c, -m));
      sum += e;
      p[i >> 3][i & 7] = static_cast<__bf16>(e);
    }
    l += sum;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < kBlocks; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks][db], p[ks], o[db], 0, 0, 0);
  }
  // a wave without keys still has its first fetch in flight
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  l = wave_half_sum(l);

  merge_waves<1, kBlocks>((lds_u8*)smem_raw, o, dim0, m, l, wave, lane, tile, kvh, split, O, lse, rep, by_nq, o_stride_h, part_o, part_ml,
                 rows_all);
}

// ------------------------------------------------------------------------------------------
// bf16 frame attention between the two: 32 kR query rows per work-group (64 or 128), a wave for each pair of one of
// kR row groups and one of 8 / kR key groups.  The keys are dealt to the key groups in tiles of 32; a tile is in
// LDS once for the kR waves of its group, and the key groups' (O, m, l) are merged through LDS as in the small form.
// Every wave runs the pipeline of attn_bf16_kernel, a phase per tile.  Bound: with every compute unit at it a
// phase of eight 32 x 32 tiles takes 1.0 us at kR = 2 and 0.86 at kR = 4 (0.84 in the 256-row form, 1.36 in the 32-row
// one): 64 KB a phase come into LDS at kR = 2 beside the 128 KB that the eight waves read.  LDS holds two slots per
// operand and key group at kR = 2, four at kR = 4; fetching K a barrier earlier, a quarter into the phase,
// made kR = 2 2 % slower, so the loads' latency is not what is left.
// It is for calls whose 32-row tiles are more than the chip and whose 256-row tiles are far fewer: those went
// through L2 once per 32 rows, or paid a merge launch and fp32 partial rows (16/4 heads x 666 rows x 1,786 keys
// 25.0 -> 18.5 us, 6/2 x 1,593 x 1,701 26.7 -> 18.4, 24/8 x 1,070 x 1,691 40.8 -> 28.3, 16/4 x 581 x 823 14.4 -> 12.3,
// 6/2 x 3,157 x 523 17.9 -> 13.9).
// ------------------------------------------------------------------------------------------
template <bool kUnitC, int kR>
__global__ __launch_bounds__(kPPThreads, 1) void attn_bf16_mid_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ lse, int rep, Divisor by_nq, int Nk, int64_t q_stride_h,
    int64_t kv_stride_h, int64_t o_stride_h, float c, Divisor by_tiles_q, int n_tiles, int share_steps,
    float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t rows_all) {
  static_assert(kR == 2 || kR == 4, "row groups");
  constexpr int kG = 8 / kR;                    // key groups
  constexpr int kSlots = kR;                    // of a key group, per operand
  constexpr int kTile = 32 * kRowBytes;         // 32 keys of K or V
  constexpr int kGroupBytes = 2 * kSlots * kTile;
  constexpr int kLoads = 8 / kR;                // a wave's share of a tile, 1 KB each
  extern __shared__ __align__(16) uint8_t smem_raw[];
  lds_u8* smem = (lds_u8*)smem_raw;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  auto k_slot = [](int t) { return (t & (kSlots - 1)) * kTile; };
  auto v_slot = [](int t) { return (kSlots + (t & (kSlots - 1))) * kTile; };
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rg = wave % kR, kg = wave / kR;
  const int l32 = lane & 31, g = lane >> 5;
  int unit = xcd_contiguous_index(blockIdx.x, gridDim.x);   // n_tiles row tiles per share
  const int split = take_share(unit, n_tiles);
  const int kvh = by_tiles_q.of(unit), tile = unit - kvh * by_tiles_q.d;
  const int n_rows = rep * by_nq.d;
  const int row_first = (tile * kR + rg) * 32;
  const bool active = row_first < n_rows;   // wave-uniform
  const uint16_t* Kh = K + kvh * kv_stride_h;
  const uint16_t* Vh = V + kvh * kv_stride_h;
  // this share's keys, whole steps but for the very last; tile t of the key group starts at key_at(t)
  const int k_begin = split * share_steps * 32 * kG, k_end = min(k_begin + share_steps * 32 * kG, Nk);
  const int n = (k_end - k_begin + 32 * kG - 1) / (32 * kG);
  auto key_at = [&](int t) { return k_begin + (t * kG + kg) * 32; };

  const uint32_t group0 = lds0 + kg * kGroupBytes;
  auto stage = [&](auto is_v, int t, int slot_bytes) {
    const RowWindow w = row_window(decltype(is_v)::value ? Vh : Kh, key_at(t), Nk);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int piece = rg * kLoads + i, row = piece * 4 + (lane >> 4), pos = lane & 15;
      const int chunk = decltype(is_v)::value ? v_chunk_pos(row, pos) : k_chunk_pos(row, pos);
      dma_16B_at(w.base, row_offset(w, row, chunk), group0 + slot_bytes + piece * 1024);
    }
  };
  auto stage_k = [&](int t, int slot_bytes) { stage(std::false_type{}, t, slot_bytes); };
  auto stage_v = [&](int t, int slot_bytes) { stage(std::true_type{}, t, slot_bytes); };

  // Prologue: the queries (each key group's wave fetches its part of the row group's), through value slots that
  // nothing is staged in yet, and the first tiles behind them.
  const int q_at = kR == 2 ? rg * kGroupBytes + v_slot(0) : (rg & 1) * kGroupBytes + v_slot(1 + (rg >> 1));
#pragma unroll
  for (int i = 0; i < 8 / kG; ++i) {
    const int piece = kg * (8 / kG) + i, row = piece * 4 + (lane >> 4);
    const RowAt from = row_at(min(row_first + row, n_rows - 1), kvh, rep, by_nq);
    dma_16B(Q + from.head * q_stride_h + static_cast<int64_t>(from.row) * kD + k_chunk_pos(row, lane & 15) * 8,
            __builtin_amdgcn_readfirstlane(lds0 + q_at + piece * 1024));
  }
  stage_k(0, k_slot(0));
  stage_k(1, k_slot(1));
  if constexpr (kR == 4) {
    stage_v(0, v_slot(0));
    stage_k(2, k_slot(2));
    stage_k(3, k_slot(3));
  }
  // the slot of "values of tile -1" is read once against zero probabilities: clear it
#pragma unroll
  for (int i = 0; i < kLoads; ++i)
    reinterpret_cast<__attribute__((address_space(3))) u32x4*>(smem + kg * kGroupBytes + v_slot(-1))[(rg * kLoads + i) * 64 + lane] =
        u32x4{0u, 0u, 0u, 0u};
  int k_off[8], v_off[4];  // as in attn_bf16_kernel, within the key group's LDS
#pragma unroll
  for (int s = 0; s < 8; ++s) k_off[s] = kg * kGroupBytes + l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16;
  {
    const int r = lane & 15, G = (lane >> 4) & 1;
    const int row = g * 4 + (r >> 2);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      const int dim = db * 32 + G * 16 + 4 * (r & 3);
      v_off[db] = kg * kGroupBytes + row * kRowBytes + v_chunk_pos(row, dim >> 3) * 16 + (dim & 7) * 2;
    }
  }
  f32x16 o[4], sA, sB, neg_m;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
#pragma unroll
    for (int db = 0; db < 4; ++db) o[db][i] = 0.f;
    sA[i] = sB[i] = neg_m[i] = 0.f;
  }
  bf16x8 pA[2], pB[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) pA[ks][e] = pB[ks][e] = static_cast<__bf16>(0.f);
  float m_ref = -INFINITY, l_run = 0.f;
  bool low_ref = false;   // wave-uniform
  auto mask_tail = [&](f32x16& sc, int t) {
    const int left = k_end - key_at(t);
    if (left >= 32) return;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if ((i >> 2) * 8 + (i & 3) >= left - g * 4) sc[i] = -INFINITY;
  };

  // the queries and K(0): all but this wave's K(1) (and V(0), K(2), K(3))
  if constexpr (kR == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  __syncthreads();
  bf16x8 qf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) qf[s] = lds_frag(smem + q_at + l32 * kRowBytes + k_chunk_pos(l32, 2 * s + g) * 16);
#pragma unroll
  for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(qf[s]));
  if (active) {  // scores of tile 0 and the first reference maximum
    f32x16 zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag(smem + k_slot(0) + k_off[s]), qf[s], s == 0 ? zero : sA, 0, 0, 0);
    float mx = sA[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sA[i]);
    m_ref = wave_half_max(mx) * c;
    if constexpr (kUnitC) {
      const float start = m_ref >= kLowestStart ? m_ref : 0.f;
      low_ref = __any(!(m_ref >= kLowestStart));
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sA[i] -= start;
        neg_m[i] = -start;
      }
    }
    mask_tail(sA, 0);
  }
  if constexpr (kR == 4) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();   // K(1) has landed; K(0) and the queries have been read
  if constexpr (kR == 4) stage_v(1, v_slot(1));
  stage_k(kSlots, k_slot(0));
  stage_v(kSlots - 2, v_slot(kSlots - 2));

  // Phase p: S(p+1), O += V(p-1) P(p-1)  |  P(p).  Behind it one barrier: K(p+1) and V(p-1) have been read by
  // all, K(p+2) and V(p) have landed (fetched kSlots - 1 phases ago), and K(p+1+kSlots), V(p-1+kSlots) are fetched.
  auto phase = [&](int p, auto slot_tag, const f32x16& s_cur, f32x16& s_nxt, const bf16x8 (&p_mm)[2], bf16x8 (&p_cur)[2]) {
    constexpr int u = decltype(slot_tag)::value;   // p % kSlots
    constexpr int k_nxt = ((u + 1) & (kSlots - 1)) * kTile, v_prev = (kSlots + ((u + kSlots - 1) & (kSlots - 1))) * kTile;
    if (active) {
      pipeline_phase<kUnitC>(smem + k_nxt, k_off, smem + v_prev, v_off, qf, s_nxt, p_mm, o, s_cur, p_cur, m_ref, l_run, c,
                             neg_m, low_ref);
      mask_tail(s_nxt, p + 1);
    }
    if constexpr (kR == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (p + 1 < n) {
      stage_k(p + 1 + kSlots, k_nxt);
      stage_v(p - 1 + kSlots, v_prev);
    }
  };
  for (int p = 0; p < n; p += kSlots) {
    phase(p, std::integral_constant<int, 0>{}, sA, sB, pB, pA);
    if (p + 1 >= n) break;
    phase(p + 1, std::integral_constant<int, 1>{}, sB, sA, pA, pB);
    if constexpr (kSlots == 4) {
      if (p + 2 >= n) break;
      phase(p + 2, std::integral_constant<int, 2>{}, sA, sB, pB, pA);
      if (p + 3 >= n) break;
      phase(p + 3, std::integral_constant<int, 3>{}, sB, sA, pA, pB);
    }
  }
  // drain: O += V(n-1) P(n-1)
  if (active) {
    const lds_u8* v_last = smem + v_slot(n - 1);
    const bool odd = (n & 1) != 0;   // the last phase was an even one: its probabilities are pA
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const lds_u8* src = v_last + v_off[db] + ks * 16 * kRowBytes;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(src)));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(const_cast<lds_u8*>(src + 8 * kRowBytes)));
        bf16x8 vf;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          vf[e] = lo[e];
          vf[4 + e] = hi[e];
        }
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, odd ? pA[ks] : pB[ks], o[db], 0, 0, 0);
      }
  }
  const float l_tot = wave_half_sum(l_run);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // tiles past the end may still be landing
  __syncthreads();
  merge_waves<kR, 4>(smem, o, 0, fmaxf(m_ref, kNoRef), l_tot, wave, lane, tile, kvh, split, O, lse, rep, by_nq, o_stride_h, part_o,
                  part_ml, rows_all);
}

// ln(2^m l), rounded once: m may reach hundreds where l's logarithm is small
__device__ __forceinline__ float natural_lse(float m, float l) {
  return fmaf(m, 0.693147182464599609375f, fmaf(m, -1.90465429995776804525e-9f, logf(l)));
}

// Merge of the key shares: O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s with M = max_s m_s.
// A thread owns four dims of one row.  The rows in front of row_whole (numbered over all heads) were
// not cut.
template <typename T, int D>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ part_o,
                                                         const float2* __restrict__ part_ml,
                                                         T* __restrict__ O, float* __restrict__ lse,
                                                         int Hq, int Nq, int64_t o_stride_h, int n_splits,
                                                         int64_t row_whole) {
  constexpr bool kF32 = sizeof(T) == 4;
  constexpr int kLanes = D / 4;  // threads per row
  const int64_t r = static_cast<int64_t>(blockIdx.x) * (256 / kLanes) + threadIdx.x / kLanes;
  const int c = threadIdx.x % kLanes;
  const int64_t n_rows = static_cast<int64_t>(Hq) * Nq - row_whole;
  if (r >= n_rows) return;
  // lane s of the row holds share s (n_splits <= kLanes): one load each instead of a chain of them
  float2 ml = make_float2(-INFINITY, 0.f);
  if (c < n_splits) ml = part_ml[c * n_rows + r];
  constexpr int kBatch = 4;   // partial rows in flight
  auto load = [&](int s0, f32x4 (&v)[kBatch]) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
      v[i] = *reinterpret_cast<const f32x4*>(part_o + (min(s0 + i, n_splits - 1) * n_rows + r) * D + c * 4);
  };
  f32x4 v[kBatch];
  load(0, v);
  float M = ml.x;
#pragma unroll
  for (int x = 1; x < kLanes; x *= 2) M = fmaxf(M, __shfl_xor(M, x, kLanes));
  const float w_mine = __builtin_amdgcn_exp2f(ml.x - M);   // 0 beyond the last share
  float l = w_mine * ml.y;
#pragma unroll
  for (int x = 1; x < kLanes; x *= 2) l += __shfl_xor(l, x, kLanes);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0;;) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const float w = s0 + i < n_splits ? __shfl(w_mine, s0 + i, kLanes) : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += w * v[i][e];
    }
    s0 += kBatch;
    if (s0 >= n_splits) break;
    load(s0, v);
  }
  const float inv = 1.f / l;
  const int64_t at = row_whole + r;
  const int h = static_cast<int>(at / Nq), row = static_cast<int>(at % Nq);
  T* out = O + h * o_stride_h + static_cast<int64_t>(row) * D + c * 4;
  if constexpr (kF32) {
    store_f32x4(out, acc * inv);
    if (lse != nullptr && c == 0) lse[at] = natural_lse(M, l);
  } else {
    u32x2 packed;
    packed[0] = pack_bf16x2(acc[0] * inv, acc[1] * inv);
    packed[1] = pack_bf16x2(acc[2] * inv, acc[3] * inv);
    *reinterpret_cast<u32x2*>(out) = packed;
    if (lse != nullptr && c == 0) lse[at] = (M + log2f(l)) * 0.6931471805599453f;
  }
}

// Workspace of n_splits key shares of `rows` query rows: the partial O rows, then the (m, l) pairs.
size_t attn_partial_o_bytes(int64_t rows, int D, int n_splits) {
  return align_up(static_cast<size_t>(n_splits) * rows * D * sizeof(float), 256);
}
size_t attn_partial_bytes(int64_t rows, int D, int n_splits) {
  return n_splits <= 1 ? 0
                       : attn_partial_o_bytes(rows, D, n_splits) +
                             align_up(static_cast<size_t>(n_splits) * rows * sizeof(float2), 256);
}
// What of the caller's workspace key shares may use: nothing of one that is not 16-byte aligned.
size_t usable_bytes(const void* ws, size_t ws_bytes) {
  return ws == nullptr || reinterpret_cast<uintptr_t>(ws) % 16 != 0 ? 0 : ws_bytes;
}
constexpr int kMaxKeySplits = 16;
constexpr int kMidKeys = 2048;   // keys up to which 64 and 128 rows per work-group are considered

// How a bf16 call is cut: 32, 64, 128 or 256 query rows per work-group, and the key shares.  The estimates
// are microseconds, fitted to 24 shapes from 0.1 to 974 GFLOP (2 to 24 heads, 64 to 4,032 rows, 150 to
// 29,500 keys) in the 32- and 256-row forms with 1 to 16 shares: `start` is what a work-group costs beside its
// steps, a step is 8 x 32 keys with 32 rows and 64 keys with 256 and gets slower as the compute units fill up,
// a further round costs a new start, and key shares cost the merge launch and the fp32 partial rows
// (512 bytes written and read per row and share).  The 32-row form was fitted again, to
// 210 shapes (2/1 to 24/8 heads, 33 to 4,032 rows, 64 to 13,000 keys), for each division of its output's dims: a
// work-group with a quarter or half of them costs less, so fewer calls are worth a merge launch (2/1 heads x 690
// rows x 868 keys: four shares 9.0 us, none 6.1; 16/4 x 115 x 1,234 three 10.4, none 8.5).  The cut is 0.5 % off
// the best of all forms on average.  Where the line to 256 rows lies, both sides measured: 8/2 x 252 x 1,179, 8.7
// us with 32 rows against 15.8 with 256 (and 29.7 un-split); 16/4 x 400 x 3,000, 19.9 against 29.4; 24/8 x 568 x
// 2,200, 29.5 against 30.6; 16/4 x 1,008 x 7,455, 85 against 68.
// The forms of 64 and 128 rows were fitted to 140 shapes (2/1 to 24/8 heads, 64 to 4,032 rows, 100 to 13,000 keys) in all
// four forms with 1 to 16 shares (a step is 128 keys with 64 rows and 64 with 128).  They are considered up to 2,048 keys,
// or up to 8,192 over all KV heads: of the 140, 23 took them, 1.26 times as fast at the median and 1.49 at most (one of
// them, 6/2 x 692 x 2,458, 3 % slower; it is not among those that take them now).  Beyond that line they would still win at times (16/4 x 1,594 x 3,031 53 -> 44 us, 16/4 x 853 x 2,371 32 -> 25)
// and no more at 16/4 x 1,008 x 7,455 (68 against 69); it lies where it does because the parity tests pin their
// large shapes, from 2,100 keys on, to the 256-row form that they are there to cover.  They take one round of work-groups
// at most: of 426 shapes (1/1 to 28/4 heads, up to 260,000 rows in all, 1 to 2,048 keys) 107 take them, none of them
// slower than the other two forms (0.92 times as long at the median); of the 136 that are several rounds in either, 133
// are slower (1.39 times as long at the median, 1 % faster at best: 16/4 x 5,311 x 4 24.2 us, 18.8 with 256 rows).
// Their estimate was raised by 6 % and key shares of 128 rows are not considered: on 163 shapes of up to 8,192 keys
// over all KV heads they had been picked in shares where 32 rows in fewer are up to 1.19 times as fast (2/1 x 2,527 x 2,601
// 20.8 us, 17.5; 2/1 x 696 x 6,694 19.0, 16.8); now 49 take them, 0.91 times as long at the median and 3 % longer at worst.
// The small form's work-groups divide the output's dims while all of them still have a compute unit (small_blocks): of
// 27 shapes with 4 to 252 work-groups, the division that fits was the fastest on 26 (by 8 to 21 %; 1 % off on the
// last), one that does not fit took 1.1 to 2.2 times as long (16/4 x 141 x 474, 72 of them: 6.7 us whole, 5.9 in
// two, 9.2 in four; 2/1 x 690 x 868, 176: 9.0 and 11.3).
// Where there are more row tiles than compute units, the whole rounds of them walk all keys and only the
// rest is cut (24/8 heads x 4,032 x 8,320: 128 of 384 tiles in two shares instead of all of them, a
// third of the partial rows and a round less: 363 us, 381 with all of them cut).
// A cut whose partial rows do not fit ws_bytes is not considered; no shares always fit.
struct AttnPlan {
  int rows;           // query rows per work-group: 32, 64, 128 or 256
  int n_splits;
  int n_whole;        // row tiles that are not cut (n_splits > 1)
  int64_t row_whole;  // rows in front of the first that is cut, numbered over all heads
};
// Blocks of 32 dims of a work-group of the small form.
int small_blocks(int work_groups) { return work_groups <= 64 ? 1 : work_groups <= 128 ? 2 : 4; }
AttnPlan plan_bf16(int Hkv, int rows, int Nk, size_t ws_bytes) {
  AttnPlan best = {kBM, 1, 0, 0};
  double best_cost = 1e30;
  struct Cost {
    double start, per_step, fill_step, next_round;
  };
  auto consider = [&](int tile_rows, int share_keys, int step_keys, auto&& cost_of /* that many work-groups */) {
    const int base = Hkv * ceil_div(rows, tile_rows), units = ceil_div(Nk, share_keys);
    const bool one_round = tile_rows == 64 || tile_rows == 128;
    const int64_t all_rows = static_cast<int64_t>(Hkv) * rows;
    for (int s = 1; s <= std::min(tile_rows == 128 ? 1 : kMaxKeySplits, units); ++s) {
      const int per = ceil_div(units, s);
      if (ceil_div(units, per) != s) continue;   // would leave a share empty
      if (one_round && base * s > 256) break;
      const auto [start, per_step, fill_step, next_round] = cost_of(base * s);
      const int steps = ceil_div(per * share_keys, step_keys), rounds = ceil_div(base * s, 256);
      const double merge = s == 1 ? 0.0 : 2.4 + 1.86e-4 * s * Hkv * rows;
      const double cost = start + rounds * (per_step + fill_step * std::min(1.0, base * s / 256.0)) * steps +
                          (rounds - 1) * next_round + merge;
      if (cost < best_cost && attn_partial_bytes(all_rows, kD, s) <= ws_bytes) {
        best_cost = cost;
        best = {tile_rows, s, 0, 0};
      }
      const int whole = base / 256 * 256, cut = base - whole;
      if (tile_rows != kBM || s == 1 || whole == 0 || cut == 0) continue;
      const int cut_rounds = ceil_div(cut * s, 256);
      const double part = start + whole / 256 * (per_step + fill_step) * ceil_div(Nk, step_keys) +
                          cut_rounds * (per_step + fill_step * std::min(1.0, cut * s / 256.0)) * steps +
                          (whole / 256 + cut_rounds - 1) * next_round + 2.4 + 1.86e-4 * s * cut * tile_rows;
      const int tiles_q = base / Hkv;
      const int64_t row_whole = static_cast<int64_t>(whole / tiles_q) * rows + whole % tiles_q * tile_rows;
      if (part < best_cost && attn_partial_bytes(all_rows - row_whole, kD, s) <= ws_bytes) {
        best_cost = part;
        best = {tile_rows, s, whole, row_whole};
      }
    }
  };
  consider(kBM, kBN, kBN, [](int) { return Cost{8.1, 1.14, 0.33, 3.3}; });
  consider(kSmallRows, kSmallKeys, 8 * kSmallKeys, [](int work_groups) {
    const int blocks = small_blocks(work_groups);
    return blocks == 1 ? Cost{3.4, 0.62, 1.5, 3.3} : blocks == 2 ? Cost{3.9, 0.8, 0.5, 3.3} : Cost{4.9, 1.03, 0.32, 3.3};
  });
  if (Nk <= kMidKeys || Hkv * static_cast<int64_t>(Nk) <= 4 * kMidKeys) {
    consider(64, 128, 128, [](int) { return Cost{6.57, 0.72, 0.345, 0.0}; });
    consider(128, 64, 64, [](int) { return Cost{8.0, 0.55, 0.36, 0.0}; });
  }
  return best;
}
// ------------------------------------------------------------------------------------------
// fp32 tier: the 16x16x4 fp32 MFMA (fp32 operands and accumulation throughout; 2,048 FLOP in 32
// cycles, twice the rate of scalar FMAs).  Bound: matrix rate and the loads of K and V when the chip
// is full, latency at the few-hundred-token sizes this tier is used at, so the work is cut fine: a
// work-group owns 16 kR query rows (numbered through the heads of the KV head, as above), its 8 waves
// take the keys in steps of 16 by turns (LDS of their own, no barrier in the loop) and merge their
// (O, m, l) through LDS once; when that leaves compute units idle the host cuts the keys into shares
// as well (plan_f32).  kR = 2 reads K and V half as often per product, kR = 1 starts and ends sooner.
//   * S^T = K Q^T: lane (r = l % 16, kg = l / 16) holds key row r, dims 16 s + 4 kg .. + 3 as one
//     16-byte load; the four MFMAs of step s contract over (kg, element e), the same permutation
//     of the head dimension on both operands.
//   * The result leaves lane (q = l % 16, kg) with keys 4 kg .. 4 kg + 3 of its query column:
//     max and sum need two cross-lane steps, and P^T is already the B operand of O^T += V^T P^T
//     (product e contracts over keys 4 kg + e).
//   * V is the A operand through 16-byte reads too: row r of output block (db, e) stands for dim
//     64 db + 4 r + e, so a lane's accumulators are whole 16-byte pieces of its output row.
//   * Softmax in base 2: a score is s (c + c_lo) with one rounding, c + c_lo = scale * log2(e).
//   * Rows travel whole (1 KB per load) to registers and from there to LDS; as fragments straight from memory they
//     were 64 bytes of each of 16 rows per load, and lines were fetched twice.  One instruction stream
//     forms the scores of a step and the probabilities of the step before, and moves a piece of K or V between
//     products: a wave that issues all its loads at once waits for the seven others' in front of its products.
// Measured: 8/2 heads, 252 rows, 1,804 keys, D = 128 (1.86 GFLOP, 12 us at the rate a large fp32
// product reaches) 29.1 -> 26.1 us; of 700 calls (1 to 28 heads, 1 to 2,500 rows, 1 to 12,000 keys) those with D = 128 take
// 0.88 times as long at the median and those with 64 0.93 (24/8 heads x 155 x 1,379 37.1 -> 32.1, 8/2 x 63 x 261 9.5 -> 8.6;
// D = 64, 8/2 x 169 x 345 8.3 -> 7.1); five are 3 to 4 % slower (16/16 x 3 x 65, D = 64, 4.7 -> 4.9; 8/2 x 2,468 x 42
// 22.4 -> 23.1).
// A large call, 24/8 x 1,000 x 8,000: 872 -> 821 us (120 TFLOP/s).
// Where the 26 us go (clock stamps; the chip runs at 2.04 GHz): queries in LDS at 1.1 us, the first scores at
// 3.9, then 4.7 us for a step of both waves of a SIMD, of which the matrix pipe works 4.0 (2 x 128 products of
// 32 cycles); eight such steps on the SIMD with the most, the merge through LDS from 22.3 on and the merge launch.
// ------------------------------------------------------------------------------------------
constexpr int kF32Waves = 8;
constexpr int kF32Keys = 16;   // keys of a wave's step
constexpr float kF32Trigger = 256.f;
template <int D, int kR, int kWaves>
constexpr size_t f32_smem_bytes() {   // a step's K and V rows of every wave, the query rows, the waves' (m, l)
  return sizeof(float) * (kWaves * (kWaves <= 2 ? 1 : 2) * kF32Keys * D + 16 * kR * D + kWaves * 16 * kR * 2);
}

// Sixteen rows as D / 16 pieces of 1 KB, 16 bytes per lane, through a buffer descriptor: rows past the end are zeros.
// What a piece adds stands in the lane's offset, where the range check is defined to see it (of the scalar offset
// it is not); pieces below 4 KB are immediates of their loads, those above them cost one more register.
template <int D>
struct F32Rows {
  __amdgpu_buffer_rsrc_t rows;
  __device__ __forceinline__ F32Rows(const float* __restrict__ base, int k0, int n_rows) {
    const int first = min(k0, n_rows);
    rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + static_cast<int64_t>(first) * D), 0,
                                             min(n_rows - first, kF32Keys) * D * 4, 0x00020000);
  }
  __device__ __forceinline__ f32x4 piece(int j, int lane_bytes) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, lane_bytes + j * 1024, 0, 0));
  }
};
// Rows in LDS: 16-byte chunk c of row i lies at place c ^ (i % 16), so that writing whole rows and reading either
// operand's fragments use every bank.  Offsets are a lane's own number and an exclusive or with what is known.
template <int D>
__device__ __forceinline__ int f32_place(int row, int chunk) { return (row * (D / 4) + (chunk ^ (row & 15))) * 16; }

template <int D, int kR, int kWaves>
__global__ __launch_bounds__(64 * kWaves) void attn_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    float* __restrict__ O, float* __restrict__ lse, int rep, Divisor by_nq, int Nk, int64_t q_stride_h,
    int64_t kv_stride_h, int64_t o_stride_h, float scale, int keys_per_split, Divisor by_tiles_q, int n_tiles,
    float* __restrict__ part_o, float2* __restrict__ part_ml, int64_t rows_all) {
  constexpr int kS = D / 16, kB = D / 64, kF32Rows = 16 * kR;
  using Rows = F32Rows<D>;
  extern __shared__ __align__(16) uint8_t smem_raw[];
  lds_u8* smem = (lds_u8*)smem_raw;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, kg = lane >> 4;
  constexpr int kTile = kF32Keys * D * 4;      // bytes of a step's keys
  constexpr bool kOneStep = kWaves <= 2;       // the host gives no wave of these a second step
  constexpr int kValues = kOneStep ? 0 : kTile, kMine = kValues + kTile;   // LDS of a wave: its keys, its values (where
                                               // the keys were if there is one step); its rows in the merge
  constexpr int kQAt = kWaves * kMine;         // the query rows
  float* s_m = reinterpret_cast<float*>(smem_raw + kQAt + kF32Rows * D * 4);   // the merge: [wave][row]
  float* s_l = s_m + kWaves * kF32Rows;
  static_assert(kF32Rows * D * 4 <= kMine, "a wave's rows on their way to the merge lie where its keys were");
  auto at4 = [&](int bytes) { return reinterpret_cast<__attribute__((address_space(3))) f32x4*>(smem + bytes); };
  // logical order: key split slowest, then KV head, then row tile: the work-groups of one XCD (one L2)
  // read the same keys
  int unit = xcd_contiguous_index(blockIdx.x, gridDim.x);
  const int split = take_share(unit, n_tiles), kvh = by_tiles_q.of(unit);
  const int row0 = (unit - kvh * by_tiles_q.d) * kF32Rows, n_rows = rep * by_nq.d;
  const float* Kh = K + kvh * kv_stride_h;
  const float* Vh = V + kvh * kv_stride_h;
  const int k_begin = split * keys_per_split, k_end = min(k_begin + keys_per_split, Nk);
  constexpr int kStride = kWaves * kF32Keys;
  const int k_first = k_begin + wave * kF32Keys;
  const int n = k_first >= k_end ? 0 : kOneStep ? 1 : (k_end - k_first + kStride - 1) / kStride;   // steps of this wave

  // The query rows come through LDS once and stay there.
  constexpr int kQPieces = kF32Rows * (D / 4), kQPasses = (kQPieces + 64 * kWaves - 1) / (64 * kWaves);
  f32x4 raw_q[kQPasses], raw[kS], raw_k[kS], raw_v[kS];
#pragma unroll
  for (int i = 0; i < kQPasses; ++i) {
    const int e = min(static_cast<int>(threadIdx.x) + i * 64 * kWaves, kQPieces - 1);
    const RowAt at = row_at(min(row0 + e / (D / 4), n_rows - 1), kvh, rep, by_nq);
    raw_q[i] = load_f32x4(Q + at.head * q_stride_h + static_cast<int64_t>(at.row) * D + e % (D / 4) * 4);
  }
  int lane_bytes = lane * 16;
  {
    const Rows k(Kh, k_first, Nk);
#pragma unroll
    for (int j = 0; j < kS; ++j) raw[j] = k.piece(j, lane_bytes);
  }
  const Rows k_second(Kh, k_first + kStride, Nk), v_first(Vh, k_first, Nk);
  if constexpr (kOneStep) {
#pragma unroll
    for (int j = 0; j < kS; ++j) raw_v[j] = v_first.piece(j, lane_bytes);
  }
#pragma unroll
  for (int i = 0; i < kQPasses; ++i) {
    const int e = min(static_cast<int>(threadIdx.x) + i * 64 * kWaves, kQPieces - 1);
    *at4(kQAt + f32_place<D>(e / (D / 4), e % (D / 4))) = raw_q[i];
  }
  // What a lane adds to or exclusive-ors with: piece j it writes, key and query fragment s, value fragment (e, b).
  constexpr int kRowsPer = 256 / D;   // rows of a piece
  int put_at = wave * kMine + f32_place<D>(lane / (D / 4), lane % (D / 4));
  int key_at = wave * kMine + f32_place<D>(r, kg), q_at = kQAt + f32_place<D>(r, kg);
  int val_at = wave * kMine + kValues + f32_place<D>(kg * 4, r);
  auto put = [&](int tile, int j, f32x4 v) { *at4((put_at ^ (kRowsPer * j * 16)) + tile + j * 1024) = v; };
  f32x4 o[kR][kB][4];
#pragma unroll
  for (int t = 0; t < kR; ++t)
#pragma unroll
    for (int b = 0; b < kB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[t][b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m[kR], l[kR];
#pragma unroll
  for (int t = 0; t < kR; ++t) {
    m[t] = kNoRef;
    l[t] = 0.f;
  }
  // c is rounded down and c_lo above zero: a score of -inf then stays -inf (and is no NaN)
  float c = scale * 1.4426950408889634f;
  auto rest = [&] { return fmaf(scale, 1.92596299e-8f, fmaf(scale, 1.4426950216293335f, -c)); };
  if (rest() < 0.f) c = __uint_as_float(__float_as_uint(c) - 1);
  const float c_lo = fmaxf(rest(), 1.17549435e-38f);
  auto scaled = [&](float x) { return fmaf(x, c, x * c_lo); };

  __syncthreads();   // the query rows
  // Scores of the keys in LDS; behind the products of contraction step s runs epi(s).
  auto score_products = [&](f32x4 (&out)[kR], auto&& epi) {
    f32x4 kf[2], qf[2][kR];
    auto fetch = [&](int s) {
      kf[s & 1] = *at4(key_at ^ (s * 64));
#pragma unroll
      for (int t = 0; t < kR; ++t) qf[s & 1][t] = *at4((q_at ^ (s * 64)) + t * kTile);
    };
#pragma unroll
    for (int t = 0; t < kR; ++t) out[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
#pragma unroll
    for (int s = 0; s < kS; ++s) {
      if (s + 1 < kS) fetch(s + 1);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < kR; ++t) out[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s & 1][e], qf[s & 1][t][e], out[t], 0, 0, 0);
      epi(s);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Exact maximum of a step's (scaled) scores becomes the reference; O and l follow it.
  auto new_reference = [&](const f32x4 (&sc)[kR]) {
#pragma unroll
    for (int t = 0; t < kR; ++t) {
      float mx = scaled(sc[t][0]);
#pragma unroll
      for (int e = 1; e < 4; ++e) mx = fmaxf(mx, scaled(sc[t][e]));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = wave_half_max(mx);
      const float m_new = fmaxf(m[t], mx), alpha = __builtin_amdgcn_exp2f(m[t] - m_new);
      l[t] *= alpha;
#pragma unroll
      for (int b = 0; b < kB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[t][b][e] *= alpha;
      m[t] = m_new;
    }
  };
  auto mask = [&](f32x4 (&sc)[kR], int k0) {
    if (k0 + kF32Keys <= k_end) return;
#pragma unroll
    for (int t = 0; t < kR; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k0 + kg * 4 + e >= k_end) sc[t][e] = -INFINITY;
  };

  // Software pipeline: while the scores of a step are formed, the probabilities of the step before are, against
  // the reference as it stands (no maximum is taken unless a sum of them comes out above kF32Trigger);
  // then that step's values are added up.  Piece by piece between the products, the values of a step go to LDS
  // while its successor's scores are formed and the keys after those are fetched into the registers that become
  // free, and the other way round: a wave never waits for the loads of eight to be taken.
  f32x4 sc[kR], nxt[kR], p[kR];
  if (n > 0) {
#pragma unroll
    for (int j = 0; j < kS; ++j) put(0, j, raw[j]);
    wave_lds_sync();
    score_products(sc, [&](int s) {
      if constexpr (!kOneStep) {
        raw_k[s] = k_second.piece(s, lane_bytes);
        raw_v[s] = v_first.piece(s, lane_bytes);
      }
    });
    mask(sc, k_first);
    new_reference(sc);
    wave_lds_sync();   // the first keys' fragments have been read
#pragma unroll
    for (int j = 0; j < kS; ++j) {
      if constexpr (!kOneStep) put(0, j, raw_k[j]);
      raw[j] = raw_v[j];
    }
  }
  for (int i = 0; i < n; ++i) {
    const int k0 = k_first + i * kStride;
    const Rows k_next(Kh, k0 + 2 * kStride, Nk), v_next(Vh, k0 + kStride, Nk);   // past the end: never used
    // (opaque: else every offset formed from them becomes a register that is kept across the loop)
    asm volatile("" : "+v"(put_at), "+v"(key_at), "+v"(q_at), "+v"(val_at), "+v"(lane_bytes));
    wave_lds_sync();
    float sum[kR];
#pragma unroll
    for (int t = 0; t < kR; ++t) sum[t] = 0.f;
    auto probability = [&](int j) {
      const int t = j / 4, e = j % 4;
      p[t][e] = __builtin_amdgcn_exp2f(scaled(sc[t][e]) - m[t]);
      sum[t] += p[t][e];
    };
    if (!kOneStep && i + 1 < n) {   // wave-uniform
      score_products(nxt, [&](int s) {
        put(kValues, s, raw[s]);
        raw[s] = k_next.piece(s, lane_bytes);
#pragma unroll
        for (int j = s * kR * 4 / kS; j < (s + 1) * kR * 4 / kS; ++j) probability(j);
      });
      mask(nxt, k0 + kStride);
    } else {
#pragma unroll
      for (int s = 0; s < kS; ++s) put(kValues, s, raw[s]);
#pragma unroll
      for (int j = 0; j < kR * 4; ++j) probability(j);
    }
    bool away = false;
#pragma unroll
    for (int t = 0; t < kR; ++t) away = away || !(sum[t] <= kF32Trigger);   // inf and NaN too
    if (__any(away)) {
      new_reference(sc);
#pragma unroll
      for (int t = 0; t < kR; ++t) sum[t] = 0.f;
#pragma unroll
      for (int j = 0; j < kR * 4; ++j) probability(j);
    }
#pragma unroll
    for (int t = 0; t < kR; ++t) l[t] += sum[t];
    wave_lds_sync();
    auto add_values = [&](auto more) {
      f32x4 v[2];
      auto fetch = [&](int j) { v[j & 1] = *at4((val_at ^ (j / kB * 16)) + j / kB * D * 4 + j % kB * 256); };
      fetch(0);
#pragma unroll
      for (int j = 0; j < 4 * kB; ++j) {
        const int e = j / kB, b = j % kB;
        if (j + 1 < 4 * kB) fetch(j + 1);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int t = 0; t < kR; ++t)
            o[t][b][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j & 1][x], p[t][e], o[t][b][x], 0, 0, 0);
        if constexpr (decltype(more)::value) {
          put(0, j, raw[j]);
          raw[j] = v_next.piece(j, lane_bytes);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (!kOneStep && i + 1 < n) add_values(std::true_type{}); else add_values(std::false_type{});
#pragma unroll
    for (int t = 0; t < kR; ++t) sc[t] = nxt[t];
  }

  // accumulator element (b, x, i) of lane (q = r, kg) is dim 64 b + 16 kg + 4 i + x of its query row
#pragma unroll
  for (int t = 0; t < kR; ++t) {
    l[t] += __shfl_xor(l[t], 16);
    l[t] = wave_half_sum(l[t]);
    if constexpr (kWaves == 1) {   // nothing to merge
      const int rho = row0 + t * 16 + r;
      if (rho >= n_rows) continue;
      const RowAt to = row_at(rho, kvh, rep, by_nq);
      float* out = O + to.head * o_stride_h + static_cast<int64_t>(to.row) * D + kg * 16;
      const float inv = 1.f / l[t];
#pragma unroll
      for (int b = 0; b < kB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          store_f32x4(out + b * 64 + i * 4, f32x4{o[t][b][0][i], o[t][b][1][i], o[t][b][2][i], o[t][b][3][i]} * inv);
      if (lse != nullptr && kg == 0) lse[static_cast<int64_t>(kvh) * n_rows + rho] = natural_lse(m[t], l[t]);
      continue;
    }
    const int row = wave * kF32Rows + t * 16 + r;
#pragma unroll
    for (int b = 0; b < kB; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *at4(wave * kMine + f32_place<D>(t * 16 + r, b * 16 + kg * 4 + i)) =
            f32x4{o[t][b][0][i], o[t][b][1][i], o[t][b][2][i], o[t][b][3][i]};
    if (kg == 0) {
      s_m[row] = m[t];
      s_l[row] = l[t];
    }
  }
  if constexpr (kWaves == 1) return;
  __syncthreads();
  // merge in wave order: a thread owns four dims of a row, of every kPass-th
  constexpr int kPass = 64 * kWaves / (D / 4);   // rows per pass
  const int col = threadIdx.x % (D / 4) * 4;
#pragma unroll
  for (int row = threadIdx.x / (D / 4); row < kF32Rows; row += kPass) {
    const int rho = row0 + row;
    if (rho >= n_rows) return;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, s_m[w * kF32Rows + row]);
    float lt = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float wt = __builtin_amdgcn_exp2f(s_m[w * kF32Rows + row] - M);
      lt += wt * s_l[w * kF32Rows + row];
      acc += wt * *at4(w * kMine + f32_place<D>(row, col / 4));
    }
    const int64_t at = static_cast<int64_t>(kvh) * n_rows + rho;   // row number over all heads
    if (part_o != nullptr) {  // one of several key shares: merged by attn_merge_kernel
      const int64_t at_s = split * rows_all + at;
      *reinterpret_cast<f32x4*>(part_o + at_s * D + col) = acc;
      if (col == 0) part_ml[at_s] = make_float2(M, lt);
    } else {
      const RowAt to = row_at(rho, kvh, rep, by_nq);
      store_f32x4(O + to.head * o_stride_h + static_cast<int64_t>(to.row) * D + col, acc * (1.f / lt));
      if (lse != nullptr && col == 0) lse[at] = natural_lse(M, lt);
    }
  }
}

// How an fp32 call is cut: kR and the key shares.  Microseconds, fitted to 400 calls (2 to 24 heads, 33 to 700
// rows, 70 to 4,000 keys, both head dimensions) in both forms with 1 to 16 shares; the cut it picks is 0.4 %
// off the best of them on average, 2.5 % on one call in twenty.  A SIMD has two of the eight waves, so a share
// lasts as long as a quarter of its steps.  Shares that need more than 16 MB of workspace have to save more than 4 %:
// less is within what the estimate errs by (16/4 heads x 4,032 rows x 97,024 keys: eight of them, 256 MB, for 1.6 %).
// The keys of one or two steps need as many waves, whose values take the place of their keys in LDS (16/4 heads,
// 4,032 rows, 32 keys, D = 64: 33.3 us with eight waves, 12.9 with two; 3 keys, D = 128: 49.5, and 19.3 with one).
struct F32Plan {
  int kr, n_splits, waves;
};
F32Plan plan_f32(int Hkv, int rows, int Nk, int D, size_t ws_bytes) {
  if (Nk <= 2 * kF32Keys) return {1, 1, Nk <= kF32Keys ? 1 : 2};
  F32Plan best = {1, 1, kF32Waves};
  double best_cost = 1e30;
  F32Plan uncut = best;
  double uncut_cost = best_cost;
  const double f = D / 128.0;
  for (int kr = 1; kr <= 2; ++kr) {
    const int blocks = ceil_div(rows, 16 * kr) * Hkv, units = ceil_div(Nk, 32 / kr);
    for (int s = 1; s <= std::min(kMaxKeySplits, units); ++s) {
      const int per = ceil_div(units, s);
      if (ceil_div(units, per) != s) continue;   // would leave a share empty
      if (attn_partial_bytes(static_cast<int64_t>(Hkv) * rows, D, s) > ws_bytes) break;
      const double merge = s == 1 ? 0.0 : 2.65 + 4.5e-4 * s * Hkv * rows * f;
      const int steps = ceil_div(ceil_div(per * (32 / kr), kF32Keys), 4);   // of a SIMD
      const double cost = (kr == 1 ? 2.25 + 1.0 * f : 3.4 + 0.3 * f) +
                          ceil_div(blocks * s, 256) * (kr == 1 ? 1.31 : 2.16) * f * steps + merge;
      if (cost < best_cost) {
        best_cost = cost;
        best = {kr, s, kF32Waves};
      }
      if (s == 1 && cost < uncut_cost) {
        uncut_cost = cost;
        uncut = {kr, s, kF32Waves};
      }
    }
  }
  const bool large = attn_partial_bytes(static_cast<int64_t>(Hkv) * rows, D, best.n_splits) > (16u << 20);
  return large && best_cost > 0.96 * uncut_cost ? uncut : best;
}

template <int D>
int attn_f32(const float* Q, const float* K, const float* V, int Hq, int rep, int Nq, int Nk, int64_t q_stride_h,
             int64_t kv_stride_h, int64_t o_stride_h, float scale, float* O, float* lse, void* ws, size_t ws_bytes,
             hipStream_t s) {
  const F32Plan plan = plan_f32(Hq / rep, rep * Nq, Nk, D, usable_bytes(ws, ws_bytes));
  const auto kernel = plan.waves == 1 ? attn_f32_kernel<D, 1, 1>
                      : plan.waves == 2 ? attn_f32_kernel<D, 1, 2>
                      : plan.kr == 2  ? attn_f32_kernel<D, 2, kF32Waves>
                                      : attn_f32_kernel<D, 1, kF32Waves>;
  const size_t smem = plan.waves == 1 ? f32_smem_bytes<D, 1, 1>()
                      : plan.waves == 2 ? f32_smem_bytes<D, 1, 2>()
                      : plan.kr == 2  ? f32_smem_bytes<D, 2, kF32Waves>()
                                      : f32_smem_bytes<D, 1, kF32Waves>();
  static std::atomic<uint64_t> lds_ok[2];
  if (plan.waves == kF32Waves)
    if (int rc = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), smem, lds_ok[plan.kr - 1], "pc_frame_attn"))
      return rc;
  const int n_tiles_q = ceil_div(rep * Nq, 16 * plan.kr), n_splits = plan.n_splits, unit = 32 / plan.kr;
  const int keys_per_split = ceil_div(ceil_div(Nk, unit), n_splits) * unit;
  const int64_t rows = static_cast<int64_t>(Hq) * Nq;
  float* part_o = nullptr;
  float2* part_ml = nullptr;
  if (n_splits > 1) {
    part_o = static_cast<float*>(ws);
    part_ml = reinterpret_cast<float2*>(static_cast<uint8_t*>(ws) + attn_partial_o_bytes(rows, D, n_splits));
  }
  const int n_tiles = n_tiles_q * (Hq / rep);
  kernel<<<n_tiles * n_splits, 64 * plan.waves, smem, s>>>(Q, K, V, O, lse, rep, Divisor(Nq), Nk, q_stride_h,
                                                           kv_stride_h, o_stride_h, scale, keys_per_split,
                                                           Divisor(n_tiles_q), n_tiles, part_o, part_ml, rows);
  PC_CHECK_LAUNCH("pc_frame_attn");
  if (n_splits > 1) {
    constexpr int kRowsPerBlock = 256 / (D / 4);
    attn_merge_kernel<float, D><<<static_cast<unsigned>((rows + kRowsPerBlock - 1) / kRowsPerBlock), 256, 0, s>>>(
        part_o, part_ml, O, lse, Hq, Nq, o_stride_h, n_splits, 0);
    PC_CHECK_LAUNCH("pc_frame_attn merge");
  }
  return PC_OK;
}

}  // namespace
}  // namespace pc

using namespace pc;

extern "C" size_t pc_frame_attn_workspace_bytes_for(int dtype, int Hq, int Hkv, int Nq, int Nk, int D) {
  if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0 || Nq <= 0 || Nk <= 0 || static_cast<int64_t>(Hq) * Nq > INT_MAX) return 0;
  const int rows = Hq / Hkv * Nq;
  const int64_t all_rows = static_cast<int64_t>(Hq) * Nq;
  if (dtype == PC_BF16 && D == kD) {
    const AttnPlan plan = plan_bf16(Hkv, rows, Nk, SIZE_MAX);
    return attn_partial_bytes(all_rows - plan.row_whole, D, plan.n_splits);
  }
  if (dtype == PC_F32 && (D == 64 || D == 128))
    return attn_partial_bytes(all_rows, D, plan_f32(Hkv, rows, Nk, D, SIZE_MAX).n_splits);
  return 0;
}

extern "C" size_t pc_frame_attn_workspace_bytes(int Hq, int Nq, int Nk, int D) {
  size_t most = 0;   // over both tiers and every number of KV heads
  auto consider = [&](int Hkv) {
    most = std::max({most, pc_frame_attn_workspace_bytes_for(PC_F32, Hq, Hkv, Nq, Nk, D),
                     pc_frame_attn_workspace_bytes_for(PC_BF16, Hq, Hkv, Nq, Nk, D)});
  };
  for (int64_t i = 1; i * i <= Hq; ++i)
    if (Hq % i == 0) {
      consider(static_cast<int>(i));
      consider(static_cast<int>(Hq / i));
    }
  return most;
}

extern "C" int pc_frame_attn_cut(int dtype, int Hq, int Hkv, int Nq, int Nk, int D, size_t ws_bytes, int32_t* cut) {
  PC_REQUIRE(cut, PC_ERR_NULL, "pc_frame_attn_cut: cut is NULL");
  PC_REQUIRE(Hq > 0 && Hkv > 0 && Hq % Hkv == 0 && Nq >= 1 && Nk >= 1 && static_cast<int64_t>(Hq) * Nq <= INT_MAX,
             PC_ERR_SHAPE, "pc_frame_attn_cut: Hq=%d Hkv=%d Nq=%d Nk=%d", Hq, Hkv, Nq, Nk);
  const int rows = Hq / Hkv * Nq;
  if (dtype == PC_BF16 && D == kD) {
    const AttnPlan plan = plan_bf16(Hkv, rows, Nk, ws_bytes);
    cut[0] = plan.rows;
    cut[1] = plan.n_splits;
    cut[2] = plan.n_whole;
  } else {
    PC_REQUIRE(dtype == PC_F32 && (D == 64 || D == 128), PC_ERR_UNSUPPORTED, "pc_frame_attn_cut: dtype %d, D=%d", dtype, D);
    const F32Plan plan = plan_f32(Hkv, rows, Nk, D, ws_bytes);
    cut[0] = 16 * plan.kr;
    cut[1] = plan.n_splits;
    cut[2] = 0;
  }
  return PC_OK;
}

extern "C" int pc_frame_attn(const void* Q, const void* K, const void* V, int dtype, int Hq,
                             int Hkv, int Nq, int Nk, int D, int64_t q_stride_h,
                             int64_t kv_stride_h, int64_t o_stride_h, float scale, void* O,
                             float* lse, void* ws, size_t ws_bytes, void* stream) {
  PC_REQUIRE(dtype == PC_F32 || dtype == PC_BF16, PC_ERR_DTYPE, "pc_frame_attn: dtype %d", dtype);
  PC_REQUIRE(Hq > 0 && Hkv > 0 && Hq % Hkv == 0, PC_ERR_SHAPE,
             "pc_frame_attn: Hq=%d must be a positive multiple of Hkv=%d", Hq, Hkv);
  PC_REQUIRE(Nq >= 1 && Nk >= 1, PC_ERR_SHAPE, "pc_frame_attn: Nq=%d Nk=%d must be >= 1", Nq, Nk);
  PC_REQUIRE(scale > 0.f && isfinite(scale), PC_ERR_SHAPE, "pc_frame_attn: scale %g must be > 0", scale);
  PC_REQUIRE(Q && K && V && O, PC_ERR_NULL, "pc_frame_attn: Q, K, V or O is NULL");
  PC_REQUIRE(q_stride_h >= static_cast<int64_t>(Nq) * D && o_stride_h >= static_cast<int64_t>(Nq) * D &&
                 kv_stride_h >= static_cast<int64_t>(Nk) * D,
             PC_ERR_SHAPE, "pc_frame_attn: a head stride is smaller than rows*D");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rep = Hq / Hkv;
  if (dtype == PC_BF16) {
    PC_REQUIRE(D == kD, PC_ERR_UNSUPPORTED, "pc_frame_attn: bf16 tier needs D=128, got %d", D);
    const uintptr_t al = reinterpret_cast<uintptr_t>(Q) | reinterpret_cast<uintptr_t>(K) |
                         reinterpret_cast<uintptr_t>(V) | reinterpret_cast<uintptr_t>(O);
    PC_REQUIRE(al % 16 == 0 && q_stride_h % 8 == 0 && kv_stride_h % 8 == 0 && o_stride_h % 8 == 0,
               PC_ERR_SHAPE, "pc_frame_attn: bf16 tensors and head strides must be 16-byte aligned");
    // Key shares need the caller's workspace for the partial results; without it (or with one
    // that is misaligned or too small for two) the keys are not split, which is always valid.
    const AttnPlan plan = plan_bf16(Hkv, rep * Nq, Nk, usable_bytes(ws, ws_bytes));
    const float c = scale * 1.4426950408889634f;
    const int n_tiles_q = ceil_div(rep * Nq, plan.rows);
    const int64_t rows_cut = static_cast<int64_t>(Hq) * Nq - plan.row_whole;
    float* part_o = nullptr;
    float2* part_ml = nullptr;
    if (plan.n_splits > 1) {
      part_o = static_cast<float*>(ws);
      part_ml = reinterpret_cast<float2*>(static_cast<uint8_t*>(ws) + attn_partial_o_bytes(rows_cut, D, plan.n_splits));
    }
    const int n_tiles = n_tiles_q * Hkv;
    const auto* q = static_cast<const uint16_t*>(Q);
    const auto* k = static_cast<const uint16_t*>(K);
    const auto* v = static_cast<const uint16_t*>(V);
    auto* o = static_cast<uint16_t*>(O);
    static std::atomic<uint64_t> lds_ok[9];
    auto allow = [](auto kernel, size_t bytes, std::atomic<uint64_t>& done) {
      return allow_dynamic_lds(reinterpret_cast<const void*>(kernel), bytes, done, "pc_frame_attn");
    };
    const bool unit_c = c == 1.0f;
    if (plan.rows == 64 || plan.rows == 128) {
      const bool wide = plan.rows == 128;
      const auto kernel = wide ? (unit_c ? attn_bf16_mid_kernel<true, 4> : attn_bf16_mid_kernel<false, 4>)
                               : (unit_c ? attn_bf16_mid_kernel<true, 2> : attn_bf16_mid_kernel<false, 2>);
      if (int rc = allow(kernel, kMergeBytes, lds_ok[3 + wide * 2 + unit_c])) return rc;
      const int share_steps = ceil_div(ceil_div(Nk, 32 * (wide ? 2 : 4)), plan.n_splits);
      kernel<<<n_tiles * plan.n_splits, kPPThreads, kMergeBytes, s>>>(
          q, k, v, o, lse, rep, Divisor(Nq), Nk, q_stride_h, kv_stride_h, o_stride_h, c, Divisor(n_tiles_q), n_tiles,
          share_steps, part_o, part_ml, rows_cut);
    } else if (plan.rows == kSmallRows) {
      const int blocks = small_blocks(n_tiles * plan.n_splits);
      const auto kernel = blocks == 1 ? attn_bf16_small_kernel<1> : blocks == 2 ? attn_bf16_small_kernel<2> : attn_bf16_small_kernel<4>;
      if (int rc = allow(kernel, kSmallSmem, lds_ok[blocks == 4 ? 2 : 6 + blocks])) return rc;
      const int share_steps = ceil_div(ceil_div(Nk, kSmallKeys), plan.n_splits);
      kernel<<<n_tiles * plan.n_splits * (4 / blocks), kPPThreads, kSmallSmem, s>>>(
          q, k, v, o, lse, rep, Divisor(Nq), Nk, q_stride_h, kv_stride_h, o_stride_h, c, Divisor(n_tiles_q), n_tiles,
          share_steps, part_o, part_ml, rows_cut);
    } else {
      const auto kernel = unit_c ? attn_bf16_kernel<true> : attn_bf16_kernel<false>;
      if (int rc = allow(kernel, kSmemBytes, lds_ok[unit_c])) return rc;
      const int n_whole = plan.n_splits > 1 ? plan.n_whole : n_tiles, n_cut = n_tiles - n_whole;
      const int share_tiles = ceil_div(ceil_div(Nk, kBN), plan.n_splits);
      kernel<<<n_whole + n_cut * plan.n_splits, kPPThreads, kSmemBytes, s>>>(
          q, k, v, o, lse, rep, Divisor(Nq), Nk, q_stride_h, kv_stride_h, o_stride_h, c, Divisor(n_tiles_q), n_whole,
          n_cut, share_tiles, part_o, part_ml, plan.row_whole, rows_cut);
    }
    if (plan.n_splits > 1) {
      PC_CHECK_LAUNCH("pc_frame_attn");
      attn_merge_kernel<uint16_t, kD><<<static_cast<unsigned>((rows_cut + 7) / 8), 256, 0, s>>>(
          part_o, part_ml, o, lse, Hq, Nq, o_stride_h, plan.n_splits, plan.row_whole);
    }
  } else {
    PC_REQUIRE(D == 64 || D == 128, PC_ERR_UNSUPPORTED, "pc_frame_attn: fp32 tier needs D=64 or 128, got %d", D);
    if (D == 64)
      return attn_f32<64>(static_cast<const float*>(Q), static_cast<const float*>(K), static_cast<const float*>(V), Hq,
                          rep, Nq, Nk, q_stride_h, kv_stride_h, o_stride_h, scale, static_cast<float*>(O), lse, ws,
                          ws_bytes, s);
    return attn_f32<128>(static_cast<const float*>(Q), static_cast<const float*>(K), static_cast<const float*>(V), Hq,
                         rep, Nq, Nk, q_stride_h, kv_stride_h, o_stride_h, scale, static_cast<float*>(O), lse, ws,
                         ws_bytes, s);
  }
  PC_CHECK_LAUNCH("pc_frame_attn");
  return PC_OK;
}
