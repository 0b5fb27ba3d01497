// Device arithmetic that exists in a kernel of its own and, for passes of one row, inside the projections: both must give the same bits.
// Device code only (included by .hip files).
#pragma once
#include "goose_internal.h"

// x[0..3] += the S slices at p, in index order, four loads in flight at a time (one load per loop round would make every
// slice its own trip to memory)
static __device__ __forceinline__ void add_slices(float4& a, const float* p, int S, size_t stride) {
  int s = 0;
  for (; s + 4 <= S; s += 4) {
    float4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const float4*>(p + (size_t)(s + k) * stride);
#pragma unroll
    for (int k = 0; k < 4; ++k) { a.x += v[k].x; a.y += v[k].y; a.z += v[k].z; a.w += v[k].w; }
  }
  for (; s < S; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(p + (size_t)s * stride);
    a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
  }
}

// ss + the squares of a, each step rounded as written: y first (the order that every norm here has had; another one moves results in rare places)
static __device__ __forceinline__ float add_squares(float ss, const float4& a) {
  return ss + fmaf(a.w, a.w, fmaf(a.z, a.z, fmaf(a.x, a.x, a.y * a.y)));
}

// (cos, sin) of pos[m] * base^(-2j/d): the angle is reduced in double, then evaluated in float
// (|error| ~ 1e-7 rad at any position).
static __device__ __forceinline__ void rope_entry(const RopeArgs& a, int m, int j) {
  double ang = (double)a.pos[m] * a.inv_freq[j];
  const double two_pi = 6.283185307179586476925286766559;
  ang -= two_pi * rint(ang / two_pi);
  float sn, c;
  sincosf((float)ang, &sn, &c);
  a.cs[(size_t)m * a.half + j] = make_float2(c, sn);
}

// Four columns of a query's attention output from its `nsplit` partial ones: sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s, splits in index
// order, the loads of up to eight in flight together (one load per loop round would make every split a trip to
// memory of its own).  base0: (head, split 0, query) in rows of ml = (m, l) pairs and o (D columns); split s lies s * step rows further.
// after_loads is called once the first loads are on their way.
typedef float fold_f32x4 __attribute__((ext_vector_type(4)));
template <typename F>
static __device__ __forceinline__ fold_f32x4 merge_splits(const float* __restrict__ o, const float* __restrict__ ml_rows, size_t base0,
                                                          size_t step, int nsplit, int D, int c, F after_loads) {
  constexpr int CH = 8;
  constexpr float LOWEST = -1e30f;
  fold_f32x4 num = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f, mmax = LOWEST;
  float2 ml[CH];
  fold_f32x4 ov[CH];
  auto load = [&](int s0) {
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const size_t base = base0 + (size_t)min(s0 + k, nsplit - 1) * step;
      ml[k] = *reinterpret_cast<const float2*>(ml_rows + base * 2);
      ov[k] = *reinterpret_cast<const fold_f32x4*>(o + base * D + c);
    }
  };
  load(0);  // (sums and maxima together: the maxima first would be a second trip to memory)
  after_loads();
#pragma unroll
  for (int k = 0; k < CH; ++k) mmax = fmaxf(mmax, ml[k].x);
  for (int s0 = CH; s0 < nsplit; s0 += CH) {
    float m[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) m[k] = ml_rows[(base0 + (size_t)min(s0 + k, nsplit - 1) * step) * 2];
#pragma unroll
    for (int k = 0; k < CH; ++k) mmax = fmaxf(mmax, m[k]);
  }
  for (int s0 = 0;;) {
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const float w = (s0 + k < nsplit) ? exp2f(ml[k].x - mmax) : 0.f;
      den = fmaf(w, ml[k].y, den);
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] = fmaf(w, ov[k][e], num[e]);
    }
    s0 += CH;
    if (s0 >= nsplit) break;
    load(s0);
  }
  return num / den;
}
