// fp32 kernels for models stored in fp32 (small models).  A pass over one is a chain of short dependent launches, so what
// matters in each is that its loads are issued together instead of one after the other.
#include "goose_internal.h"

namespace {

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// Sums v[0..7] over the wavefront; lane l returns the sum of v[l >> 3].  Three folds that halve the
// number of values a lane carries, then three plain steps: 10 exchanges instead of 48.
__device__ inline float wave_sum8(const float (&v)[8], int lane) {
  float a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool hi = lane & 32;
    a[i] = (hi ? v[4 + i] : v[i]) + __shfl_xor(hi ? v[i] : v[4 + i], 32, 64);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool hi = lane & 16;
    b[i] = (hi ? a[2 + i] : a[i]) + __shfl_xor(hi ? a[i] : a[2 + i], 16, 64);
  }
  const bool hi = lane & 8;
  float r = (hi ? b[1] : b[0]) + __shfl_xor(hi ? b[0] : b[1], 8, 64);
#pragma unroll
  for (int off = 4; off > 0; off >>= 1) r += __shfl_xor(r, off, 64);
  return r;
}

// out[m][n] = sum_k A[m][k] * W[n][k].  One wavefront per (n, group of 8 rows), four to a workgroup: lanes stride
// over k, VEC inputs at a time (16 bytes; VEC = 1 where a row length or an address does not allow that),
// so that the weight row is read coalesced, then the 8 sums are reduced across lanes.  Rows beyond M read
// row M-1: nine loads of a round are in flight together (behind a branch each they cost 2 us a
// round: 8 x 768 x 256 took 12 us, 8 x 256 x 688 25 us; now 2.8 and 3.8).
template <int VEC>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ A, int lda, const float* __restrict__ W, int N,
                                                  int K, int M, float* __restrict__ out, size_t ldo) {
  typedef float fv __attribute__((ext_vector_type(VEC)));
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6), m0 = blockIdx.y * 8;
  if (n >= N) return;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const float* w = W + (size_t)n * K;
  const float* a[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) a[r] = A + (size_t)min(m0 + r, M - 1) * lda;
#pragma unroll 2
  for (int k = lane * VEC; k < K; k += 64 * VEC) {
    const fv wv = *reinterpret_cast<const fv*>(w + k);
    fv av[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) av[r] = *reinterpret_cast<const fv*>(a[r] + k);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if constexpr (VEC == 4)  // (in pairs: fewer roundings in a row than one after the other)
        acc[r] += (av[r][0] * wv[0] + av[r][1] * wv[1]) + (av[r][2] * wv[2] + av[r][3] * wv[3]);
      else
        acc[r] += av[r][0] * wv[0];
    }
  }
  const float s = wave_sum8(acc, lane);
  const int m = m0 + (lane >> 3);
  if ((lane & 7) == 0 && m < M) out[(size_t)m * ldo + n] = s;
}

// Tree-masked attention for one (query node, head): scores over slots [0,P) and the
// ancestor-or-self slots of the tail, softmax in fp32, weighted sum of V.  Four wavefronts share the
// keys; a thread reads its key row in 16-byte pieces, and the weighted sum walks the transposed values four
// slots at a time (a wavefront's quarter of the keys each), so that the loads of a key are in flight together
// (one wavefront, one load after the other: 13 us for 8 nodes over 72 slots; now 5.0).
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
                                                  int lds_keys, int32_t* __restrict__ flags) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float* sq = sm;             // [head_dim]: the query, then the wavefronts' maxima and sums (head_dim >= 8)
  float* red = sq;
  float* sc = sm + head_dim;  // [lds_keys], then the four partial sums [4][head_dim]
  const int i = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = (B + 63) >> 6;
  const int P = *dP;
  int nk = P + B;
  // the launch is sized from the host's upper bound of P: a longer cache is flagged
  // (GOOSE_FLAG_CAPACITY) and the keys beyond the bound are dropped so that nothing is indexed outside LDS
  if ((P < 0 || nk > lds_keys || nk > cap) && i == 0 && h == 0 && tid == 0) atomicOr(flags, GOOSE_FLAG_CAPACITY);
  if (nk > lds_keys) nk = lds_keys;
  if (nk > cap) nk = cap;
  if (nk < 0) nk = 0;
  for (int c = tid; c < head_dim; c += 256) sq[c] = q[(size_t)i * ldq + h * head_dim + c];
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)head_dim);
  const float* kh = kc + (size_t)h * cap * head_dim;
  const float* vh = vc + (size_t)h * head_dim * cap;  // transposed value cache Vt[head][d][slot]
  float mx = -INFINITY;
  for (int s = tid; s < nk; s += 256) {
    bool vis = s < P;
    if (!vis) {
      const int j = s - P;
      vis = (mask[(size_t)i * W + (j >> 6)] >> (j & 63)) & 1ull;
    }
    float d = -INFINITY;
    if (vis) {
      float d4[4] = {0.f, 0.f, 0.f, 0.f};
      const float* kr = kh + (size_t)s * head_dim;  // (head_dim is a multiple of 8)
#pragma unroll 8
      for (int c = 0; c < head_dim; c += 4) {
        const float4 kv = load4<WIDE>(kr + c), qv = *reinterpret_cast<const float4*>(sq + c);
        d4[0] += qv.x * kv.x;
        d4[1] += qv.y * kv.y;
        d4[2] += qv.z * kv.z;
        d4[3] += qv.w * kv.w;
      }
      d = ((d4[0] + d4[1]) + (d4[2] + d4[3])) * scale;
    }
    sc[s] = d;
    mx = fmaxf(mx, d);
  }
  mx = wave_max(mx);
  __syncthreads();
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float sum = 0.f;
  for (int s = tid; s < nk; s += 256) {
    const float d = sc[s];
    const float p = (d == -INFINITY) ? 0.f : expf(d - mx);
    sc[s] = p;
    sum += p;
  }
  sum = wave_sum(sum);
  if (lane == 0) red[4 + wave] = sum;
  __syncthreads();
  sum = red[4] + red[5] + red[6] + red[7];
  const int quads = (nk + 3) >> 2, q_lo = quads * wave / 4, q_hi = quads * (wave + 1) / 4;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};  // columns lane, lane + 64, .. (head_dim <= 256)
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = lane + 64 * u;
    if (c >= head_dim) break;
    const float* vr = vh + (size_t)c * cap;  // (cap is a multiple of 64: slots 4j .. 4j+3 exist)
#pragma unroll 4
    for (int j = q_lo; j < q_hi; ++j) {
      const float4 v = load4<WIDE>(vr + 4 * j);
      const float ve[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p = 4 * j + e < nk ? sc[4 * j + e] : 0.f;
        acc[u] += p != 0.f ? p * ve[e] : 0.f;  // (an invisible slot may hold anything)
      }
    }
  }
  __syncthreads();  // every wavefront is done with the probabilities
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (lane + 64 * u < head_dim) sc[wave * head_dim + lane + 64 * u] = acc[u];
  __syncthreads();
  for (int c = tid; c < head_dim; c += 256)
    o[(size_t)i * ldo + h * head_dim + c] =
        ((sc[c] + sc[head_dim + c]) + (sc[2 * head_dim + c] + sc[3 * head_dim + c])) / sum;
}

}  // namespace

int launch_gemm_f32(const float* A, int lda, const float* W, int N, int K, int M, float* out, size_t ldo,
                    hipStream_t st) {
  const dim3 grid((N + 3) / 4, (M + 7) / 8);
  if (K % 4 == 0 && lda % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0)
    hipLaunchKernelGGL(k_gemm_f32<4>, grid, dim3(256), 0, st, A, lda, W, N, K, M, out, ldo);
  else
    hipLaunchKernelGGL(k_gemm_f32<1>, grid, dim3(256), 0, st, A, lda, W, N, K, M, out, ldo);
  return goose_launch_status();
}

int launch_attn_f32(const float* q, int ldq, const float* kc, const float* vc, int n_heads, int head_dim, int cap,
                    const int32_t* dP, int B, const uint64_t* mask, float* o, int ldo, int P_max, int32_t* flags,
                    hipStream_t st) {
  const int lds_keys = P_max + B;
  const size_t smem = (size_t)(head_dim + (lds_keys > 4 * head_dim ? lds_keys : 4 * head_dim)) * sizeof(float);
  if (smem > 64 * 1024) return GOOSE_ERR_CAPACITY;  // the fp32 path keeps all scores of a row in LDS
  const bool wide = (((uintptr_t)kc | (uintptr_t)vc) & 15) == 0;
  if (wide)
    hipLaunchKernelGGL(k_attn_f32<true>, dim3(B, n_heads), dim3(256), smem, st, q, ldq, kc, vc, head_dim, cap, dP, B, mask, o,
                       ldo, lds_keys, flags);
  else
    hipLaunchKernelGGL(k_attn_f32<false>, dim3(B, n_heads), dim3(256), smem, st, q, ldq, kc, vc, head_dim, cap, dP, B, mask, o,
                       ldo, lds_keys, flags);
  return goose_launch_status();
}
