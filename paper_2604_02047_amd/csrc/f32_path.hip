// fp32 kernels for models stored in fp32 (small models).  A pass over one is a chain of short dependent launches, so what
// matters in each is that its loads are issued together instead of one after the other.
#include <math.h>

#include "goose_internal.h"

namespace {

// Exchanges without LDS: within 16 lanes by DPP (quad_perm, row_half_mirror, row_ror), beyond by the row and half swaps.
template <int CTRL>
__device__ inline float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
enum { DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR8 = 0x128 };
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// a and b with the upper half of a and the lower half of b exchanged (HALF), or the odd rows of 16 lanes of a and the even ones of b
template <bool HALF>
__device__ inline void lane_swap(float& a, float& b) {
  const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
  const u32x2 r = HALF ? __builtin_amdgcn_permlane32_swap(x, y, false, false) : __builtin_amdgcn_permlane16_swap(x, y, false, false);
  const unsigned r0 = r[0], r1 = r[1];  // (a bit cast of a vector's element takes the first one)
  a = __builtin_bit_cast(float, r0);
  b = __builtin_bit_cast(float, r1);
}
// op over the 64 lanes, the result in every lane
template <typename Op>
__device__ inline float wave_all(float v, Op op) {
  v = op(v, dpp<DPP_XOR1>(v));
  v = op(v, dpp<DPP_XOR2>(v));
  v = op(v, dpp<DPP_HALF_MIRROR>(v));
  v = op(v, dpp<DPP_ROR8>(v));
  float w = v;
  lane_swap<false>(v, w);
  v = w = op(v, w);
  lane_swap<true>(v, w);
  return op(v, w);
}

// Sums v[0..7] over the wavefront; lane l returns the sum of v[l >> 3].  Three folds that halve the
// number of values a lane carries, then three plain steps: 10 exchanges instead of 48.
// *lo: what the last addition rounded away.
__device__ inline float wave_sum8(const float (&v)[8], int lane, float* lo) {
  float a[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float x = v[i], y = v[4 + i];
    lane_swap<true>(x, y);
    a[i] = x + y;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    float x = a[i], y = a[2 + i];
    lane_swap<false>(x, y);
    c[i] = x + y;
  }
  const bool hi = lane & 8;
  float r = (hi ? c[1] : c[0]) + dpp<DPP_ROR8>(hi ? c[0] : c[1]);
  r += dpp<DPP_XOR1>(r);
  r += dpp<DPP_XOR2>(r);
  const float o = dpp<DPP_HALF_MIRROR>(r), t = r + o, b = t - r;
  *lo = (r - (t - b)) + (o - b);
  return t;
}

// A pass over a small model is as long as its launches (2-3 us each whatever they hold), so a projection takes in what
// lies before and after it:
//   F32_QKV     RMSNorm of the rows, q | k | v, rotary embedding, q to its buffer, k and v into the caches
//   F32_SWIGLU  RMSNorm of the rows, gate and up, h = silu(gate) * up
//   F32_LOGITS  RMSNorm of the rows, out = sums
//   F32_RESID   out += sums (the residual rows)
// A layer is five launches (with norms, rotation, SwiGLU and residual adds as launches of their own it was nine) and the step of
// 8 nodes over two layers 77.2 -> 52.4 us (64 nodes, prefix 512: 109 -> 83).
//
// sum_k A[m][k] * W[n][k]: one wavefront per (n, group of 8 rows), four to a workgroup: lanes stride
// over k, VEC inputs at a time (16 bytes; VEC = 1 where a row length or an address does not allow that),
// so that the weight row is read coalesced, then the 8 sums are reduced across lanes.  Rows beyond M read
// row M-1: the loads of a round are in flight together (behind a branch each they cost 2 us a
// round).  With a norm the wavefront sums x g w and x^2 side by side and scales at the end: every wavefront repeats the
// squares of its rows, which costs arithmetic that idles otherwise.  F32_QKV and F32_SWIGLU
// take two weight rows, (j, j + d/2) of a head or (gate, up) of an output, so that what is combined meets in one wavefront.
enum { F32_QKV, F32_SWIGLU, F32_LOGITS, F32_RESID };
struct F32Proj {
  const float* A;
  const float* W;
  const float* g;  // gain of the norm (F32_RESID: none)
  float* out;      // F32_QKV: the rotated queries
  size_t ldo;
  int lda, N, K, M;  // N: outputs (F32_QKV: head_dim / 2)
  float eps;
  // F32_QKV
  int n_heads, cap;
  const int32_t* pos;
  const int32_t* dP;
  const double* inv_freq;
  float* kc;
  float* vc;
  int32_t* flags;
};
// KW: wavefronts that share an output's inputs (4: one output a workgroup; the down projection then is one round of loads instead of three).
template <int VEC, int MODE, int KW>
__global__ __launch_bounds__(256) void k_proj_f32(const F32Proj p) {
  typedef float fv __attribute__((ext_vector_type(VEC)));
  constexpr bool NORM = MODE != F32_RESID;
  constexpr int NW = MODE == F32_QKV || MODE == F32_SWIGLU ? 2 : 1;  // weight rows
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // F32_QKV: grid (3 heads, pairs / 4, row groups), sections q, k, v of the weights follow each other; else (outputs / 4, row groups)
  const int n = KW == 4 ? (int)blockIdx.x : (MODE == F32_QKV ? blockIdx.y : blockIdx.x) * 4 + wave, m0 = (MODE == F32_QKV ? blockIdx.z : blockIdx.y) * 8;
  if (n >= p.N) return;
  const int K = p.K, M = p.M;
  const float* w0 = p.W + (size_t)(MODE == F32_QKV ? (size_t)blockIdx.x * 2 * p.N + n : n) * K;
  const float* w1 = w0 + (size_t)p.N * K;
  const int m = m0 + (lane >> 3), mc = min(m, M - 1);  // the row whose sum this lane gets in the end
  const bool turn = MODE == F32_QKV && (int)blockIdx.x < 2 * p.n_heads;
  float acc[NW][8], ss[8];
  const float* a[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
#pragma unroll
    for (int u = 0; u < NW; ++u) acc[u][r] = 0.f;
    ss[r] = 0.f;
    a[r] = p.A + (size_t)min(m0 + r, M - 1) * p.lda;
  }
  int slot = 0, position = 0;
  double freq = 0.0;
  if (MODE == F32_QKV) {  // (on their way with the first round)
    slot = *p.dP + m;
    if (turn) {
      position = p.pos[mc];
      freq = p.inv_freq[n];
    }
  }
#pragma unroll 1
  for (int k = (KW == 4 ? threadIdx.x : lane) * VEC; k < K; k += 64 * KW * VEC) {
    fv wv[NW], gv, av[8];
    wv[0] = *reinterpret_cast<const fv*>(w0 + k);
    if constexpr (NW == 2) wv[1] = *reinterpret_cast<const fv*>(w1 + k);
    if constexpr (NORM) gv = *reinterpret_cast<const fv*>(p.g + k);
#pragma unroll
    for (int r = 0; r < 8; ++r) av[r] = *reinterpret_cast<const fv*>(a[r] + k);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if constexpr (VEC == 4) {  // (in pairs: fewer roundings in a row than one after the other)
        if constexpr (NORM) {
          ss[r] += (av[r][0] * av[r][0] + av[r][1] * av[r][1]) + (av[r][2] * av[r][2] + av[r][3] * av[r][3]);
          av[r] *= gv;
        }
#pragma unroll
        for (int u = 0; u < NW; ++u)
          acc[u][r] += (av[r][0] * wv[u][0] + av[r][1] * wv[u][1]) + (av[r][2] * wv[u][2] + av[r][3] * wv[u][3]);
      } else {
        if constexpr (NORM) {
          ss[r] += av[r][0] * av[r][0];
          av[r][0] *= gv[0];
        }
#pragma unroll
        for (int u = 0; u < NW; ++u) acc[u][r] += av[r][0] * wv[u][0];
      }
    }
  }
  float s[NW], s_lo[NW];
#pragma unroll
  for (int u = 0; u < NW; ++u) s[u] = wave_sum8(acc[u], lane, &s_lo[u]);
  if constexpr (NORM) {
    // Scaling at the end must not add a rounding to every result: 1 / sqrt(v) is taken as y + y_lo (one Newton step on y's own error),
    // the sum with its rounding error, and the product rounds once.  (Without: margins 1.0e-7 -> 1.4e-7 from the 64-bit ones.)
    float sq_lo;
    const float sq = wave_sum8(ss, lane, &sq_lo), v = sq / (float)K + p.eps;
    const float y = 1.0f / sqrtf(v), h = v * y, h_lo = fmaf(v, y, -h);
    const float y_lo = 0.5f * y * (fmaf(-h, y, 1.0f) - h_lo * y);
    // A row whose squares or sums leave the range (finite values from about 1e18 on, infinities, NaN) has no such product: it is scaled
    // before it is summed, and squares that overflow scale it to zeros.
    bool beyond = !(v < INFINITY);
#pragma unroll
    for (int u = 0; u < NW; ++u) beyond = beyond || !(fabsf(s[u]) < INFINITY);
#pragma unroll
    for (int u = 0; u < NW; ++u) s[u] = fmaf(s[u], y, fmaf(s[u], y_lo, s_lo[u] * y));
    if (__any(beyond)) {
      float scale[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) scale[r] = __shfl(y, 8 * r, 64);
#pragma unroll
      for (int u = 0; u < NW; ++u)
#pragma unroll
        for (int r = 0; r < 8; ++r) acc[u][r] = 0.f;
#pragma unroll 1
      for (int k = lane; k < K; k += 64) {
        const float gk = p.g[k];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const float xn = a[r][k] * scale[r] * gk;
          acc[0][r] += xn * w0[k];
          if constexpr (NW == 2) acc[1][r] += xn * w1[k];
        }
      }
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        const float scaled = wave_sum8(acc[u], lane, &sq_lo);
        if (beyond) s[u] = scaled;
      }
    }
  }
  if constexpr (KW == 4) {  // (resid only: one sum a row)
    __shared__ float sums[4][8];
    if ((lane & 7) == 0) sums[wave][lane >> 3] = s[0];
    __syncthreads();
    if (wave != 0) return;
    s[0] = (sums[0][lane >> 3] + sums[1][lane >> 3]) + (sums[2][lane >> 3] + sums[3][lane >> 3]);
  }
  const int e = lane & 7;  // (the eight lanes of a row hold the same sums: lane 0 stores the first result, lane 1 the second)
  if (m >= M || e >= (MODE == F32_QKV ? 2 : 1)) return;
  if constexpr (MODE == F32_RESID) {
    p.out[(size_t)m * p.ldo + n] += s[0];
  } else if constexpr (MODE == F32_LOGITS) {
    p.out[(size_t)m * p.ldo + n] = s[0];
  } else if constexpr (MODE == F32_SWIGLU) {
    p.out[(size_t)m * p.ldo + n] = s[0] / (1.0f + expf(-s[0])) * s[1];
  } else {
    // half-split pairing (j, j + d/2), angle pos * base^(-2j/d): reduced in double, then evaluated in float, |error| ~ 1e-7 rad at
    // any position
    float v = e == 0 ? s[0] : s[1];
    if (turn) {
      double ang = (double)position * freq;
      const double two_pi = 6.283185307179586476925286766559;
      ang -= two_pi * rint(ang / two_pi);
      float sn, cs;
      sincosf((float)ang, &sn, &cs);
      v = e == 0 ? s[0] * cs - s[1] * sn : s[1] * cs + s[0] * sn;
    }
    const int d = 2 * p.N, c = n + e * p.N;  // column of the head
    int h = blockIdx.x;
    if (h < p.n_heads) {
      p.out[(size_t)m * p.ldo + (size_t)h * d + c] = v;
    } else if (slot < 0 || slot >= p.cap) {  // no room for this node: say so instead of writing outside the cache
      if (n == 0 && e == 0) atomicOr(p.flags, GOOSE_FLAG_CAPACITY);
    } else if ((h -= p.n_heads) < p.n_heads) {
      p.kc[((size_t)h * p.cap + slot) * d + c] = v;  // K[head][slot][d]
    } else {
      h -= p.n_heads;
      p.vc[((size_t)h * d + c) * p.cap + slot] = v;  // the transposed value cache Vt[head][d][slot]
    }
  }
}

// First launch of a step, one workgroup per node: embedding row, and the node's ancestor bits, depth and position (as
// k_build_mask writes them; the parents are climbed in LDS).  Also keeps the cache length before the step in *P_old, which the commit
// at its end reads.
template <int VEC>
__global__ __launch_bounds__(256) void k_begin_f32(const float* __restrict__ E, const int32_t* __restrict__ tokens, int H, int V,
                                                   float* __restrict__ x, const int32_t* __restrict__ parent, int B,
                                                   const int32_t* __restrict__ dP, uint64_t* __restrict__ mask,
                                                   int32_t* __restrict__ depth, int32_t* __restrict__ pos,
                                                   int32_t* __restrict__ P_old, int32_t* __restrict__ flags, int cap, int P_max) {
  typedef float fv __attribute__((ext_vector_type(VEC)));
  __shared__ int up[GOOSE_MAX_B];
  const int i = blockIdx.x, tid = threadIdx.x;
  const int P = *dP;
  const int tok = min(max(tokens[i], 0), V - 1);
  if (tid < B) up[tid] = parent[tid];
  const float* src = E + (size_t)tok * H;
  float* dst = x + (size_t)i * H;
#pragma unroll 4
  for (int c = tid * VEC; c < H; c += 256 * VEC) *reinterpret_cast<fv*>(dst + c) = *reinterpret_cast<const fv*>(src + c);
  __syncthreads();
  if (tid != 0) return;
  uint64_t w0 = 1, w1 = 0;  // (every path ends at the root)
  int dep = 0;
  bool bad = i == 0 && up[0] != -1;
  for (int v = i; v > 0; ++dep) {
    const uint64_t bit = 1ull << (v & 63);
    w0 |= v < 64 ? bit : 0;
    w1 |= v < 64 ? 0 : bit;
    const int u = up[v];
    const bool off = u < 0 || u >= v;
    bad = bad || off;
    v = off ? 0 : u;  // never index outside the tree
  }
  const int W = (B + 63) >> 6;
  mask[(size_t)i * W] = w0;
  if (W > 1) mask[(size_t)i * W + 1] = w1;
  depth[i] = dep;
  pos[i] = P + dep;
  if (bad) atomicOr(flags, GOOSE_FLAG_BAD_PARENT);
  if (i == 0) {
    if (P < 0 || P > P_max || P + B > cap) atomicOr(flags, GOOSE_FLAG_CAPACITY);
    *P_old = P;
  }
}

// Tree-masked attention for one (query node, head): scores over slots [0,P) and the
// ancestor-or-self slots of the tail, softmax in fp32, weighted sum of V.  What bounds it is a chain of loads and exchanges, and
// the fetch of code that runs once, so the code is compact.  Four lanes share a key (64 contiguous bytes a load; with a thread per
// key every load touches 64 lines); the weighted sum walks the transposed values four
// slots at a time (a wavefront's quarter of the keys each).  8 nodes over 72 slots: 5.0 -> 4.3 us, which a version with its loops
// unrolled (10 KB of code instead of 4) took 6.6 for.
// WIDE: both caches start on a 16-byte boundary (then every key row and every quad of slots does).
template <bool WIDE>
__device__ inline float4 load4(const float* p) {
  return WIDE ? *reinterpret_cast<const float4*>(p) : make_float4(p[0], p[1], p[2], p[3]);
}
template <bool WIDE>
__global__ __launch_bounds__(256) void k_attn_f32(const float* __restrict__ q, int ldq, const float* __restrict__ kc,
                                                  const float* __restrict__ vc, int head_dim, int cap,
                                                  const int32_t* __restrict__ dP, int B,
                                                  const uint64_t* __restrict__ mask, float* __restrict__ o, int ldo,
                                                  int lds_keys, float scale, int32_t* __restrict__ flags) {
  extern __shared__ __attribute__((aligned(16))) float sc[];  // [lds_keys rounded up to 4], then the four partial sums [4][64]
  __shared__ float red[8];                                    // the wavefronts' maxima and sums
  const int i = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int W = (B + 63) >> 6;
  const uint64_t seen0 = mask[(size_t)i * W], seen1 = mask[(size_t)i * W + W - 1];
  const int P = *dP;
  const float* qr = q + (size_t)i * ldq + h * head_dim;  // (rows of q and heads are multiples of eight floats apart)
  const float* kh = kc + (size_t)h * cap * head_dim;
  const float* vh = vc + (size_t)h * head_dim * cap;  // transposed value cache Vt[head][d][slot]
  const int c_lane = 4 * (tid & 3);
  auto col = [&](int c, int u) { return c_lane + min(c + 16 * u, head_dim - 4 - c_lane); };  // (beyond the row: its end once more)
  float4 qv[4], kv[4];  // the first 64 columns of the query, and of the next key (of any slot of the cache: on their way with the length)
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    qv[u] = *reinterpret_cast<const float4*>(qr + col(0, u));
    kv[u] = load4<WIDE>(kh + (size_t)min(tid >> 2, cap - 1) * head_dim + col(0, u));
  }
  int nk = P + B;
  // the launch is sized from the host's upper bound of P: a longer cache is flagged
  // (GOOSE_FLAG_CAPACITY) and the keys beyond the bound are dropped so that nothing is indexed outside LDS
  if ((P < 0 || nk > lds_keys || nk > cap) && i == 0 && h == 0 && tid == 0) atomicOr(flags, GOOSE_FLAG_CAPACITY);
  nk = max(min(nk, min(lds_keys, cap)), 0);
  const int quads = (nk + 3) >> 2, q_lo = quads * wave / 4, q_hi = quads * (wave + 1) / 4;
  float mx = -INFINITY;
#pragma unroll 1
  for (int s = tid >> 2; s < nk; s += 64) {
    float d4[4] = {0.f, 0.f, 0.f, 0.f};
    float4 ka[4], qa[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ka[u] = kv[u];
      qa[u] = qv[u];
      kv[u] = load4<WIDE>(kh + (size_t)min(s + 64, cap - 1) * head_dim + col(0, u));
    }
    for (int c = 0;;) {  // (head_dim is a multiple of 8)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (c + 16 * u + c_lane >= head_dim) break;
        d4[0] += qa[u].x * ka[u].x;
        d4[1] += qa[u].y * ka[u].y;
        d4[2] += qa[u].z * ka[u].z;
        d4[3] += qa[u].w * ka[u].w;
      }
      c += 64;
      if (c >= head_dim) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        ka[u] = load4<WIDE>(kh + (size_t)s * head_dim + col(c, u));
        qa[u] = *reinterpret_cast<const float4*>(qr + col(c, u));
      }
    }
    float d = (d4[0] + d4[1]) + (d4[2] + d4[3]);
    d += dpp<DPP_XOR1>(d);
    d += dpp<DPP_XOR2>(d);
    const int j = s - P;
    const bool vis = s < P || (((j < 64 ? seen0 : seen1) >> (j & 63)) & 1ull);
    d = vis ? d * scale : -INFINITY;  // (an invisible slot may hold anything)
    if (c_lane == 0) sc[s] = d;
    mx = fmaxf(mx, d);
  }
  constexpr int VQ = 5;  // quads of slots whose values (of a column) are in flight; the first ones during the softmax
  float4 v[VQ];
  auto fetch = [&](int c0, int j0) {  // (cap is a multiple of 64: slots 4j .. 4j+3 exist)
    const float* vr = vh + (size_t)min(c0 + lane, head_dim - 1) * cap;
#pragma unroll
    for (int u = 0; u < VQ; ++u) v[u] = load4<WIDE>(vr + 4 * max(min(j0 + u, q_hi - 1), 0));
  };
  fetch(0, q_lo);
  mx = wave_all(mx, [](float a, float b) { return fmaxf(a, b); });
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float sum = 0.f;
#pragma unroll 1
  for (int s = tid; s < 4 * quads; s += 256) {  // (the last quad's slots beyond the keys get zeros)
    const float d = s < nk ? sc[s] : -INFINITY;
    const float p = (d == -INFINITY) ? 0.f : expf(d - mx);
    sc[s] = p;
    sum += p;
  }
  sum = wave_all(sum, [](float a, float b) { return a + b; });
  if (lane == 0) red[4 + wave] = sum;
  __syncthreads();
  sum = (red[4] + red[5]) + (red[6] + red[7]);
  float* part = sc + ((lds_keys + 3) & ~3);
#pragma unroll 1
  for (int c0 = 0; c0 < head_dim; c0 += 64) {
    const int c = c0 + lane;
    float acc = 0.f;
#pragma unroll 1
    for (int j0 = q_lo; j0 < q_hi;) {
#pragma unroll
      for (int u = 0; u < VQ; ++u) {
        if (j0 + u >= q_hi) break;
        const float4 p = *reinterpret_cast<const float4*>(sc + 4 * (j0 + u));
        acc += p.x != 0.f ? p.x * v[u].x : 0.f;
        acc += p.y != 0.f ? p.y * v[u].y : 0.f;
        acc += p.z != 0.f ? p.z * v[u].z : 0.f;
        acc += p.w != 0.f ? p.w * v[u].w : 0.f;
      }
      j0 += VQ;
      if (j0 < q_hi || c0 + 64 < head_dim) fetch(j0 < q_hi ? c0 : c0 + 64, j0 < q_hi ? j0 : q_lo);
    }
    part[tid] = acc;
    __syncthreads();
    if (wave == 0 && c < head_dim)
      o[(size_t)i * ldo + h * head_dim + c] = ((part[lane] + part[64 + lane]) + (part[128 + lane] + part[192 + lane])) / sum;
    if (c0 + 64 < head_dim) __syncthreads();
  }
}

}  // namespace

template <int MODE, int KW = 1>
static int launch_proj_f32(const F32Proj& p, dim3 grid, hipStream_t st) {
  const uintptr_t at = (uintptr_t)p.A | (uintptr_t)p.W | (MODE == F32_RESID ? 0 : (uintptr_t)p.g);
  if (p.K % 4 == 0 && p.lda % 4 == 0 && (at & 15) == 0)
    hipLaunchKernelGGL((k_proj_f32<4, MODE, KW>), grid, dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((k_proj_f32<1, MODE, KW>), grid, dim3(256), 0, st, p);
  return goose_launch_status();
}
static dim3 grid_f32(int N, int M) { return dim3((N + 3) / 4, (M + 7) / 8); }

int launch_qkv_f32(const float* x, int H, const float* g, float eps, const float* W, int n_heads, int head_dim, int M,
                   const int32_t* pos, const double* inv_freq, const int32_t* dP, int cap, float* q, int ldq, float* kc, float* vc,
                   int32_t* flags, hipStream_t st) {
  F32Proj p{x, W, g, q, (size_t)ldq, H, head_dim / 2, H, M, eps, n_heads, cap, pos, dP, inv_freq, kc, vc, flags};
  return launch_proj_f32<F32_QKV>(p, dim3(3 * n_heads, (head_dim / 2 + 3) / 4, (M + 7) / 8), st);
}
int launch_swiglu_f32(const float* x, int H, const float* g, float eps, const float* W, int F, int M, float* h, int ldh, hipStream_t st) {
  F32Proj p{x, W, g, h, (size_t)ldh, H, F, H, M, eps};
  return launch_proj_f32<F32_SWIGLU>(p, grid_f32(F, M), st);
}
int launch_logits_f32(const float* x, int H, const float* g, float eps, const float* W, int V, int M, float* out, size_t ldo,
                      hipStream_t st) {
  F32Proj p{x, W, g, out, ldo, H, V, H, M, eps};
  return launch_proj_f32<F32_LOGITS>(p, grid_f32(V, M), st);
}
int launch_resid_f32(const float* A, int lda, const float* W, int H, int K, int M, float* x, hipStream_t st) {
  F32Proj p{A, W, nullptr, x, (size_t)H, lda, H, K, M, 0.f};
  // (a wavefront takes 256 inputs a round)
  if (K > 256) return launch_proj_f32<F32_RESID, 4>(p, dim3(H, (M + 7) / 8), st);
  return launch_proj_f32<F32_RESID>(p, grid_f32(H, M), st);
}

int launch_begin_f32(const float* E, const int32_t* tokens, int H, int V, float* x, const int32_t* parent, int B, const int32_t* dP,
                     uint64_t* mask, int32_t* depth, int32_t* pos, int32_t* P_old, int32_t* flags, int cap, int P_max,
                     hipStream_t st) {
  if (H % 4 == 0 && (((uintptr_t)E | (uintptr_t)x) & 15) == 0)
    hipLaunchKernelGGL(k_begin_f32<4>, dim3(B), dim3(256), 0, st, E, tokens, H, V, x, parent, B, dP, mask, depth, pos, P_old, flags,
                       cap, P_max);
  else
    hipLaunchKernelGGL(k_begin_f32<1>, dim3(B), dim3(256), 0, st, E, tokens, H, V, x, parent, B, dP, mask, depth, pos, P_old, flags,
                       cap, P_max);
  return goose_launch_status();
}

int launch_attn_f32(const float* q, int ldq, const float* kc, const float* vc, int n_heads, int head_dim, int cap,
                    const int32_t* dP, int B, const uint64_t* mask, float* o, int ldo, int P_max, int32_t* flags,
                    hipStream_t st) {
  const int lds_keys = P_max + B;
  // the fp32 path keeps all scores of a row in LDS (within the limit there has always been)
  if ((size_t)(head_dim + (lds_keys > 4 * head_dim ? lds_keys : 4 * head_dim)) * sizeof(float) > 64 * 1024) return GOOSE_ERR_CAPACITY;
  const size_t smem = (size_t)(round_up(lds_keys, 4) + 256) * sizeof(float);
  const float scale = 1.0f / sqrtf((float)head_dim);
  const bool wide = (((uintptr_t)kc | (uintptr_t)vc) & 15) == 0;
  if (wide)
    hipLaunchKernelGGL(k_attn_f32<true>, dim3(B, n_heads), dim3(256), smem, st, q, ldq, kc, vc, head_dim, cap, dP, B, mask, o,
                       ldo, lds_keys, scale, flags);
  else
    hipLaunchKernelGGL(k_attn_f32<false>, dim3(B, n_heads), dim3(256), smem, st, q, ldq, kc, vc, head_dim, cap, dP, B, mask, o,
                       ldo, lds_keys, scale, flags);
  return goose_launch_status();
}
