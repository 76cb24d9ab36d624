// pc_rope3d: in-place 3D rotary embedding (the operator R of Eq. 2 with the (t, h, w)
// coordinates of Sec. 3.1 / Sec. 3.4).  HBM-bound: every element is read and written
// once; sin/cos of a (token, pair) are computed once and shared by all heads.  bf16, D = 128: 16
// heads x 4,032 tokens (33 MB moved) 8.3 -> 6.9 us, 8 x 252 4.3 -> 3.3 us against 16 tokens per
// work-group and the general fp64 sine and cosine; 6.8 -> 6.3 and 3.3 -> 3.0 with the loads in the order
// below and no divisions by numbers that only the host knows (fp32, 24 x 568 5.3 -> 4.4; 8 x 3 3.3 -> 2.7).
#include <math.h>

#include <algorithm>

#include "common.h"

namespace pc {
namespace {

constexpr int kMaxPairs = 128;    // D <= 256
constexpr int kTokPerBlock = 4;   // tokens per work-group
constexpr int kThreads = 256;
constexpr int kHeadsInFlight = 4;  // loads of several heads are issued before any is used

struct RopeFreq {
  double inv_freq[kMaxPairs];  // base^(-2i/s) of every pair, section by section
  uint8_t axis[kMaxPairs];     // which coordinate (0 = t, 1 = h, 2 = w) turns the pair
};

// The frequencies of the last (sections, base) this host thread asked for: a model uses one set, and
// its pow() calls are a quarter of the host time of a small call.
const RopeFreq& rope_freq(const int (&secs)[3], double base) {
  thread_local RopeFreq fr;
  thread_local int of_secs[3] = {-1, -1, -1};
  thread_local double of_base = 0.0;
  if (secs[0] == of_secs[0] && secs[1] == of_secs[1] && secs[2] == of_secs[2] && base == of_base) return fr;
  int p = 0;
  for (int a = 0; a < 3; ++a)
    for (int i = 0; i < secs[a] / 2; ++i, ++p) {
      fr.inv_freq[p] = pow(base, -2.0 * i / secs[a]);
      fr.axis[p] = static_cast<uint8_t>(a);
    }
  for (; p < kMaxPairs; ++p) {
    fr.inv_freq[p] = 0.0;
    fr.axis[p] = 0;
  }
  for (int a = 0; a < 3; ++a) of_secs[a] = secs[a];
  of_base = base;
  return fr;
}

// sin and cos of x in fp64: Cody-Waite reduction to |r| <= pi/4 (pi/2 in two parts; k has at most 32
// bits here, so x - k pi/2 is good to the last bit of r), then the Taylor series (remainders below
// 1e-13 of the result, which is rounded to fp32).  A quarter of the instructions of the general
// function, which carries a reduction for any x; beyond 2^32 that one is called.
__device__ __forceinline__ void sincos_f64(double x, double* sn, double* cs) {
  if (fabs(x) > 4294967296.0) {
    sincos(x, sn, cs);
    return;
  }
  const double k = rint(x * 0.63661977236758134308);
  double r = fma(-k, 1.57079632679489661923, x);
  r = fma(-k, 6.12323399573676603587e-17, r);
  const double q = r * r;
  double s = fma(q, 1.0 / 6227020800.0, -1.0 / 39916800.0);
  s = fma(q, s, 1.0 / 362880.0);
  s = fma(q, s, -1.0 / 5040.0);
  s = fma(q, s, 1.0 / 120.0);
  s = fma(q, s, -1.0 / 6.0);
  s = fma(q * r, s, r);
  double c = fma(q, -1.0 / 87178291200.0, 1.0 / 479001600.0);
  c = fma(q, c, -1.0 / 3628800.0);
  c = fma(q, c, 1.0 / 40320.0);
  c = fma(q, c, -1.0 / 720.0);
  c = fma(q, c, 1.0 / 24.0);
  c = fma(q, c, -0.5);
  c = fma(q, c, 1.0);
  const int quadrant = static_cast<int>(k - 4.0 * floor(k * 0.25));   // 0..3 (NaN: anything)
  const double a = (quadrant & 1) ? c : s, b = (quadrant & 1) ? s : c;
  *sn = (quadrant & 2) ? -a : a;
  *cs = (quadrant == 1 || quadrant == 2) ? -b : b;
}

// Phase 1: cos/sin of the kTokPerBlock x (D/2) angles of this work-group, angle formed
// and reduced in fp64 (positions reach hundreds of radians), kept as fp32 in LDS: one per thread
// at D = 128.  Four tokens per work-group keep that serial part short and the chip full at small n.
// Phase 2: every thread rotates 16 bytes (8 bf16 = 4 pairs, or 4 fp32 = 2 pairs) of four heads.
// A small call is latency: the first elements are fetched behind the coordinates and in front of the sines, so
// that one memory latency covers both, and all three coordinates of a token are fetched beside the table that
// says which one turns the pair.  kOnce: a thread has at most one angle (D <= 128; with a loop around the
// sines the compiler waits for everything in flight at its head).
template <typename T, bool kOnce>
__global__ __launch_bounds__(kThreads) void rope3d_kernel(T* __restrict__ x, int H, int n, int D,
                                                          int64_t stride_h,
                                                          const int32_t* __restrict__ pos, Divisor by_pairs,
                                                          Divisor by_chunks, RopeFreq fr, double out_scale) {
  __shared__ float2 cs[kTokPerBlock][kMaxPairs];
  const int tok0 = blockIdx.x * kTokPerBlock;
  const int pairs = by_pairs.d, n_angles = kTokPerBlock * pairs;
  const int own = min(static_cast<int>(threadIdx.x), n_angles - 1);   // the angle this thread forms first
  int t_a = by_pairs.of(own), p_a = own - t_a * pairs;
  const int32_t* at_a = pos + static_cast<int64_t>(min(tok0 + t_a, n - 1)) * 3;   // past the end: never used
  int coord_t = at_a[0], coord_h = at_a[1], coord_w = at_a[2], axis = fr.axis[p_a];
  double inv_freq = fr.inv_freq[p_a];

  constexpr int kElems = 16 / sizeof(T);  // elements per 16-byte chunk
  const int chunks_per_row = by_chunks.d;
  const int total = kTokPerBlock * chunks_per_row * ((H + kHeadsInFlight - 1) / kHeadsInFlight);
  struct Place {
    int h0, t, c;
  };
  auto place = [&](int e) {   // four heads of a token's chunk; chunk fastest, then token
    const int r = by_chunks.of(e);
    return Place{r / kTokPerBlock * kHeadsInFlight, r % kTokPerBlock, e - r * chunks_per_row};
  };
  u32x4 raw[kHeadsInFlight];
  auto load = [&](int e) {   // what does not exist is read as what does, and never used
    const Place at = place(min(e, total - 1));
    const T* x0 = x + static_cast<int64_t>(min(tok0 + at.t, n - 1)) * D + at.c * kElems;
#pragma unroll
    for (int i = 0; i < kHeadsInFlight; ++i)
      raw[i] = *reinterpret_cast<const u32x4*>(x0 + min(at.h0 + i, H - 1) * stride_h);
  };
  int e = blockIdx.y * kThreads + threadIdx.x;
  __builtin_amdgcn_sched_barrier(0);   // loads return in order: what the sines wait for is in front
  load(e);
  __builtin_amdgcn_sched_barrier(0);
  for (int i = threadIdx.x;;) {   // (threads past the last angle form that one too)
    const double ang = static_cast<double>(axis == 0 ? coord_t : axis == 1 ? coord_h : coord_w) * inv_freq;
    double s, c;
    sincos_f64(ang, &s, &c);
    // the output scale rides on the rotation: no instruction per element, one rounding of the result
    cs[t_a][p_a] = make_float2(static_cast<float>(c * out_scale), static_cast<float>(s * out_scale));
    i += kThreads;
    if (kOnce || i >= n_angles) break;
    t_a = by_pairs.of(i), p_a = i - t_a * pairs;
    at_a = pos + static_cast<int64_t>(min(tok0 + t_a, n - 1)) * 3;
    coord_t = at_a[0], coord_h = at_a[1], coord_w = at_a[2], axis = fr.axis[p_a];
    inv_freq = fr.inv_freq[p_a];
  }
  __syncthreads();

  while (e < total) {
    const auto [h0, t, c] = place(e);
    const int tok = tok0 + t;
    T* x0 = x + static_cast<int64_t>(tok) * D + c * kElems;
#pragma unroll
    for (int i = 0; i < kHeadsInFlight; ++i) {
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float2 r = cs[t][c * 4 + k];
          const float a0 = bf16_to_f32(static_cast<uint16_t>(raw[i][k] & 0xFFFFu));
          const float a1 = bf16_to_f32(static_cast<uint16_t>(raw[i][k] >> 16));
          raw[i][k] = pack_bf16x2(fmaf(a0, r.x, -(a1 * r.y)), fmaf(a1, r.x, a0 * r.y));
        }
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float2 r = cs[t][c * 2 + k];
          const float a0 = __uint_as_float(raw[i][2 * k]), a1 = __uint_as_float(raw[i][2 * k + 1]);
          raw[i][2 * k] = __float_as_uint(fmaf(a0, r.x, -(a1 * r.y)));
          raw[i][2 * k + 1] = __float_as_uint(fmaf(a1, r.x, a0 * r.y));
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kHeadsInFlight; ++i)
      if (tok < n && h0 + i < H) *reinterpret_cast<u32x4*>(x0 + (h0 + i) * stride_h) = raw[i];
    e += gridDim.y * kThreads;
    if (e < total) load(e);
  }
}

// pc_rebase: every row turns by the same angles, so the host passes cos/sin of the temporal
// pairs (fp64 angles, fp32 values) by value; a thread rewrites one 16-byte chunk of the
// temporal section of one row, the other sections are not touched.
struct RebaseTable {
  float2 cs[kMaxPairs];
};

template <typename T>
__global__ __launch_bounds__(kThreads) void rebase_kernel(T* __restrict__ K, int Hkv, int D, int64_t k_stride_h,
                                                          int32_t* __restrict__ pos, int Hsel,
                                                          int64_t pos_stride_h, int row0, int n_rows, int delta_t,
                                                          int chunks_t, RebaseTable tab) {
  constexpr int kElems = 16 / sizeof(T);
  const int64_t e = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  const int64_t per_head = static_cast<int64_t>(n_rows) * chunks_t;
  if (e >= per_head * Hkv) return;
  const int h = static_cast<int>(e / per_head);
  const int r = static_cast<int>((e % per_head) / chunks_t), c = static_cast<int>(e % chunks_t);
  const int row = row0 + r;
  u32x4* p = reinterpret_cast<u32x4*>(K + h * k_stride_h + static_cast<int64_t>(row) * D + c * kElems);
  u32x4 raw = *p;
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float2 t = tab.cs[c * 4 + k];
      const float x0 = bf16_to_f32(static_cast<uint16_t>(raw[k] & 0xFFFFu));
      const float x1 = bf16_to_f32(static_cast<uint16_t>(raw[k] >> 16));
      raw[k] = pack_bf16x2(x0 * t.x - x1 * t.y, x0 * t.y + x1 * t.x);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float2 t = tab.cs[c * 2 + k];
      const float x0 = __uint_as_float(raw[2 * k]), x1 = __uint_as_float(raw[2 * k + 1]);
      raw[2 * k] = __float_as_uint(x0 * t.x - x1 * t.y);
      raw[2 * k + 1] = __float_as_uint(x0 * t.y + x1 * t.x);
    }
  }
  *p = raw;
  if (c == 0 && h < Hsel) pos[h * pos_stride_h + static_cast<int64_t>(row) * 3] -= delta_t;
}

}  // namespace
}  // namespace pc

using namespace pc;

extern "C" int pc_rope3d(void* x, int dtype, int H, int n, int D, int64_t stride_h,
                         const int32_t* pos, int sec_t, int sec_h, int sec_w, double base,
                         double out_scale, void* stream) {
  PC_REQUIRE(dtype == PC_F32 || dtype == PC_BF16, PC_ERR_DTYPE, "pc_rope3d: dtype %d", dtype);
  PC_REQUIRE(H >= 0 && n >= 0 && D > 0, PC_ERR_SHAPE, "pc_rope3d: H=%d n=%d D=%d", H, n, D);
  const int secs[3] = {sec_t, sec_h, sec_w};
  for (int a = 0; a < 3; ++a)
    PC_REQUIRE(secs[a] >= 0 && secs[a] % 2 == 0, PC_ERR_SHAPE,
               "pc_rope3d: section %d has width %d (must be even, >= 0)", a, secs[a]);
  PC_REQUIRE(sec_t + sec_h + sec_w == D, PC_ERR_SHAPE, "pc_rope3d: sections %d+%d+%d != D=%d",
             sec_t, sec_h, sec_w, D);
  PC_REQUIRE(D <= 2 * kMaxPairs && D % 8 == 0, PC_ERR_SHAPE,
             "pc_rope3d: D=%d must be a multiple of 8 and <= %d", D, 2 * kMaxPairs);
  PC_REQUIRE(base > 0.0, PC_ERR_SHAPE, "pc_rope3d: base %g", base);
  PC_REQUIRE(out_scale > 0.0 && isfinite(out_scale), PC_ERR_SHAPE, "pc_rope3d: out_scale %g must be > 0", out_scale);
  if (H == 0 || n == 0) return PC_OK;
  PC_REQUIRE(x && pos, PC_ERR_NULL, "pc_rope3d: x or pos is NULL");
  PC_REQUIRE(stride_h >= static_cast<int64_t>(n) * D || H == 1, PC_ERR_SHAPE,
             "pc_rope3d: head stride %lld < n*D", static_cast<long long>(stride_h));
  PC_REQUIRE((stride_h * (dtype == PC_BF16 ? 2 : 4)) % 16 == 0 &&
                 reinterpret_cast<uintptr_t>(x) % 16 == 0,
             PC_ERR_SHAPE, "pc_rope3d: x and its head stride must be 16-byte aligned");

  const RopeFreq& fr = rope_freq(secs, base);
  // Few tokens of many heads (a stack's keys): the heads are dealt to grid.y, up to a work-group per compute
  // unit, each forming the angles anew (D = 128, fp32, 3 tokens: 224 heads 29.3 us without, 3.8 with; 16 heads
  // 4.5 and 3.6).
  const int chunks = ceil_div(H, kHeadsInFlight) * kTokPerBlock * (D / (dtype == PC_BF16 ? 8 : 4));
  const int blocks = ceil_div(n, kTokPerBlock);
  const dim3 grid(blocks, std::min(ceil_div(chunks, kThreads), ceil_div(256, blocks)));
  const Divisor by_pairs(D / 2), by_chunks(D / (dtype == PC_BF16 ? 8 : 4));
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto launch = [&](auto kernel, auto* data) {
    kernel<<<grid, kThreads, 0, s>>>(data, H, n, D, stride_h, pos, by_pairs, by_chunks, fr, out_scale);
  };
  const bool once = kTokPerBlock * (D / 2) <= kThreads;
  if (dtype == PC_BF16)
    launch(once ? rope3d_kernel<uint16_t, true> : rope3d_kernel<uint16_t, false>, static_cast<uint16_t*>(x));
  else
    launch(once ? rope3d_kernel<float, true> : rope3d_kernel<float, false>, static_cast<float*>(x));
  PC_CHECK_LAUNCH("pc_rope3d");
  return PC_OK;
}

extern "C" int pc_rebase(void* K, int dtype, int Hkv, int D, int64_t k_stride_h, int32_t* pos, int Hsel,
                         int64_t pos_stride_h, int row0, int n_rows, int delta_t, int sec_t, int sec_h,
                         int sec_w, double base, void* stream) {
  PC_REQUIRE(dtype == PC_F32 || dtype == PC_BF16, PC_ERR_DTYPE, "pc_rebase: dtype %d", dtype);
  PC_REQUIRE(Hkv >= 1 && Hsel >= 1 && Hsel <= Hkv && D > 0 && row0 >= 0 && n_rows >= 0, PC_ERR_SHAPE,
             "pc_rebase: Hkv=%d Hsel=%d D=%d row0=%d n_rows=%d", Hkv, Hsel, D, row0, n_rows);
  PC_REQUIRE(sec_t >= 0 && sec_h >= 0 && sec_w >= 0 && sec_t % 2 == 0 && sec_t + sec_h + sec_w == D, PC_ERR_SHAPE,
             "pc_rebase: sections %d+%d+%d must add up to D=%d, temporal width even", sec_t, sec_h, sec_w, D);
  const int elems = dtype == PC_BF16 ? 8 : 4;  // per 16-byte chunk
  PC_REQUIRE(sec_t % elems == 0 && D % elems == 0 && sec_t <= 2 * kMaxPairs, PC_ERR_UNSUPPORTED,
             "pc_rebase: temporal section of %d elements is not a whole number of 16-byte chunks", sec_t);
  PC_REQUIRE(base > 0.0, PC_ERR_SHAPE, "pc_rebase: base %g", base);
  if (n_rows == 0 || delta_t == 0) return PC_OK;
  PC_REQUIRE(K && pos, PC_ERR_NULL, "pc_rebase: K or pos is NULL");
  PC_REQUIRE((k_stride_h >= static_cast<int64_t>(row0 + n_rows) * D || Hkv == 1) &&
                 (pos_stride_h >= static_cast<int64_t>(row0 + n_rows) * 3 || Hsel == 1),
             PC_ERR_SHAPE, "pc_rebase: a head stride is smaller than the rows it must hold");
  PC_REQUIRE((k_stride_h * (dtype == PC_BF16 ? 2 : 4)) % 16 == 0 && reinterpret_cast<uintptr_t>(K) % 16 == 0,
             PC_ERR_SHAPE, "pc_rebase: K and its head stride must be 16-byte aligned");
  RebaseTable tab = {};
  for (int i = 0; i < sec_t / 2; ++i) {
    const double ang = -static_cast<double>(delta_t) * pow(base, -2.0 * i / sec_t);
    tab.cs[i] = make_float2(static_cast<float>(cos(ang)), static_cast<float>(sin(ang)));
  }
  const int chunks_t = sec_t / elems;
  if (chunks_t == 0) return PC_OK;  // no temporal section: positions only would change nothing the keys encode
  const int64_t total = static_cast<int64_t>(Hkv) * n_rows * chunks_t;
  const dim3 grid(static_cast<unsigned>((total + kThreads - 1) / kThreads));
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (dtype == PC_BF16)
    rebase_kernel<uint16_t><<<grid, kThreads, 0, s>>>(static_cast<uint16_t*>(K), Hkv, D, k_stride_h, pos, Hsel,
                                                      pos_stride_h, row0, n_rows, delta_t, chunks_t, tab);
  else
    rebase_kernel<float><<<grid, kThreads, 0, s>>>(static_cast<float*>(K), Hkv, D, k_stride_h, pos, Hsel,
                                                   pos_stride_h, row0, n_rows, delta_t, chunks_t, tab);
  PC_CHECK_LAUNCH("pc_rebase");
  return PC_OK;
}
