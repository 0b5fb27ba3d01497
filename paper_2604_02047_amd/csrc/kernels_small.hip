// Small kernels of the verification step: ancestor mask, embedding gather, residual +
// RMSNorm, rotary angles, argmax, logit harvest, greedy walk, KV compaction.
#include <limits.h>

#include "fold.h"
#include "goose_internal.h"

namespace {

template <typename T>
__device__ inline float to_f32(T v) { return (float)v; }

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// ------------------------------------------------------------------------------------------
__global__ void k_set_int(int32_t* dst, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = v;
}

// Ancestor-or-self bit rows, depth and position of every node (Sec. 4, tree attention mask).
// One thread per node climbs its own root path; parent[v] < v makes every climb finite.
// A cache length outside what the launch was sized for (P > P_max) or that leaves no room for the
// tree (P + B > cap) raises GOOSE_FLAG_CAPACITY: the later kernels then clamp their indices and the
// step's results are meaningless.
// DEV_P: the length is *dP, else P_max (the host knows it).  The climb is a chain of dependent loads, so what lies between two of
// them counts, and where the length comes from is no choice inside the kernel: with branches around the two words, a counter
// and that choice a chain of 64 / 128 nodes took 11.1 / 20.8 us, a random tree of 64 2.65; now 6.6 / 11.9 and 2.0.
template <bool DEV_P>
__device__ inline void build_mask_body(const int32_t* __restrict__ parent, int B, const int32_t* __restrict__ dP,
                                       uint64_t* __restrict__ mask, int32_t* __restrict__ depth,
                                       int32_t* __restrict__ pos, int32_t* __restrict__ flags, int cap, int P_max) {
  const int i = threadIdx.x;
  if (i == 0) {
    const int P = DEV_P ? *dP : P_max;
    if (P < 0 || P > P_max || P + B > cap) atomicOr(flags, GOOSE_FLAG_CAPACITY);
  }
  if (i >= B) return;
  const int W = (B + 63) >> 6;
  uint64_t w0 = 1, w1 = 0;  // (every path ends at the root)
  int dep = 0;
  bool bad = i == 0 && parent[0] != -1;
  for (int v = i; v > 0; ++dep) {
    const uint64_t bit = 1ull << (v & 63);
    w0 |= v < 64 ? bit : 0;
    w1 |= v < 64 ? 0 : bit;
    const int p = parent[v];
    const bool off = p < 0 || p >= v;
    bad = bad || off;
    v = off ? 0 : p;  // never index outside the tree
  }
  mask[(size_t)i * W] = w0;
  if (W > 1) mask[(size_t)i * W + 1] = w1;
  depth[i] = dep;
  pos[i] = (DEV_P ? *dP : P_max) + dep;
  if (bad) atomicOr(flags, GOOSE_FLAG_BAD_PARENT);
}

template <bool DEV_P>
__global__ __launch_bounds__(128) void k_build_mask(const int32_t* __restrict__ parent, int B,
                                                    const int32_t* __restrict__ dP, uint64_t* __restrict__ mask,
                                                    int32_t* __restrict__ depth, int32_t* __restrict__ pos,
                                                    int32_t* __restrict__ flags, int cap, int P_max) {
  build_mask_body<DEV_P>(parent, B, dP, mask, depth, pos, flags, cap, P_max);
}

// The per-request steps of a batch as single launches: block index = request, taken from a table
// that travels as a kernel argument (rows of request r start at row0 in the stacked buffers).
struct ReqTable { BatchReq r[GOOSE_MAX_REQUESTS]; };

__global__ __launch_bounds__(128) void k_build_mask_batch(const ReqTable t, uint64_t* __restrict__ mask,
                                                          int32_t* __restrict__ depth, int32_t* __restrict__ pos,
                                                          int32_t* __restrict__ flags, int cap) {
  const BatchReq& q = t.r[blockIdx.x];
  build_mask_body<true>(q.parent, q.B, q.dP, mask + (size_t)q.row0 * 2, depth + q.row0, pos + q.row0, flags, cap, q.P_max);
}

// ------------------------------------------------------------------------------------------
// Embedding rows as fp32.  A thread converts VEC columns at once (16 bytes of the table; VEC = 1 where the
// row length or an address does not allow that), a row is spread over workgroups of 256 threads: all
// loads of a pass are in flight together.  Element by element in a loop, 64 rows of 4096 took 5.8 us
// and 80 rows of 6656 12.8 us, most of it waiting for the next round; now 4.0 and 5.7 us.
template <typename T, int VEC>
__device__ inline void embed_row(const T* __restrict__ E, int tok, int H, int V, float* __restrict__ xr) {
  tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
  const int c = (blockIdx.x * 256 + threadIdx.x) * VEC;
  if (c >= H) return;
  struct alignas(VEC * sizeof(T)) Piece { T e[VEC]; };
  const Piece v = *reinterpret_cast<const Piece*>(E + (size_t)tok * H + c);
  if constexpr (VEC == 1) {
    xr[c] = to_f32(v.e[0]);
  } else {
#pragma unroll
    for (int q = 0; q < VEC; q += 4)
      *reinterpret_cast<float4*>(xr + c + q) =
          make_float4(to_f32(v.e[q]), to_f32(v.e[q + 1]), to_f32(v.e[q + 2]), to_f32(v.e[q + 3]));
  }
}

// grid (column groups, rows)
template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_embed(const T* __restrict__ E, const int32_t* __restrict__ tokens, int H,
                                               int V, float* __restrict__ x) {
  embed_row<T, VEC>(E, tokens[blockIdx.y], H, V, x + (size_t)blockIdx.y * H);
}

// grid (column groups, rows, requests)
template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_embed_batch(const T* __restrict__ E, const ReqTable t, int H, int V,
                                                     float* __restrict__ x) {
  const BatchReq& q = t.r[blockIdx.z];
  const int i = blockIdx.y;
  if (i >= q.B) return;
  embed_row<T, VEC>(E, q.tokens[i], H, V, x + (size_t)(q.row0 + i) * H);
}

// ------------------------------------------------------------------------------------------
// x[m] += sum of S partial GEMM outputs; xn[m] = T(x[m] * rsqrt(mean(x[m]^2) + eps) * g).
// One workgroup per row, four columns per thread per pass (H is a multiple of 4), all loads of a
// pass independent so the few rows still pull their partials at full memory parallelism.
template <typename T>
__device__ inline void store4(T* p, float a, float b, float c, float d);
template <>
__device__ inline void store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
  *reinterpret_cast<bf16x4*>(p) = v;
}
template <>
__device__ inline void store4<_Float16>(_Float16* p, float a, float b, float c, float d) {
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  f16x4 v = {(_Float16)a, (_Float16)b, (_Float16)c, (_Float16)d};
  *reinterpret_cast<f16x4*>(p) = v;
}

// TERMS = 2 (16-bit types): xn is written as hi + lo, lo = T(v - hi), in groups of eight columns
// (8 hi values, then their 8 lo values; row length 2 * columns): the operand layout of the projections.
// Tg: type of the gains; T: type of xn (fp16 activations may meet bf16 gains).
// ROPE: the launch also writes the tree's rotary angles (rope_entry), which nothing before the attention
// needs: its workgroups beyond the `rope.rows` rows take NTHR / half of the table's rows each.
template <typename Tg, typename T, int NTHR, int TERMS, bool ROPE>
__global__ __launch_bounds__(NTHR) void k_resid_norm(float* __restrict__ x, int H, const float* __restrict__ part,
                                                     int S, size_t part_stride, size_t part_ld,
                                                     const Tg* __restrict__ g, float eps, T* __restrict__ xn,
                                                     int ldxn, RopeArgs rope) {
  constexpr int MAXV = 4;  // float4 slots per thread kept in registers (H <= 16 * NTHR)
  const int m = blockIdx.x;
  if (ROPE && m >= rope.rows) {
    const int per = NTHR / rope.half, r = (m - rope.rows) * per + (int)threadIdx.x / rope.half;
    if ((int)threadIdx.x < per * rope.half && r < rope.rows) rope_entry(rope, r, threadIdx.x % rope.half);
    return;
  }
  float* xr = x + (size_t)m * H;
  const int nvec = H >> 2;
  float4 v[MAXV];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int c4 = threadIdx.x + i * NTHR;
    if (c4 < nvec) {
      float4 a = *reinterpret_cast<const float4*>(xr + c4 * 4);
      add_slices(a, part + (size_t)m * part_ld + c4 * 4, S, part_stride);
      if (S > 0) *reinterpret_cast<float4*>(xr + c4 * 4) = a;
      ss = add_squares(ss, a);
      v[i] = a;
    }
  }
  if (xn == nullptr) return;
  __shared__ float red[NTHR / 64];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NTHR / 64; ++w) tot += red[w];
  const float rstd = 1.0f / sqrtf(tot / (float)H + eps);
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int c4 = threadIdx.x + i * NTHR;
    if (c4 < nvec) {
      const Tg* gp = g + c4 * 4;
      const float o0 = (v[i].x * rstd) * to_f32(gp[0]), o1 = (v[i].y * rstd) * to_f32(gp[1]);
      const float o2 = (v[i].z * rstd) * to_f32(gp[2]), o3 = (v[i].w * rstd) * to_f32(gp[3]);
      if (TERMS == 1) {
        store4<T>(xn + (size_t)m * ldxn + c4 * 4, o0, o1, o2, o3);
      } else {  // columns 4 c4 .. 4 c4 + 3 lie inside one group of eight
        T* dst = xn + (size_t)m * ldxn + (size_t)(c4 >> 1) * 16 + (c4 & 1) * 4;
        const T h0 = (T)o0, h1 = (T)o1, h2 = (T)o2, h3 = (T)o3;
        store4<T>(dst, to_f32(h0), to_f32(h1), to_f32(h2), to_f32(h3));
        store4<T>(dst + 8, o0 - to_f32(h0), o1 - to_f32(h1), o2 - to_f32(h2), o3 - to_f32(h3));
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
struct Top2 {
  float v1, v2;
  int i1;
};
__device__ inline Top2 top2_merge(Top2 a, Top2 b) {
  const bool a_first = (a.v1 > b.v1) || (a.v1 == b.v1 && a.i1 < b.i1);
  Top2 r;
  if (a_first) { r.v1 = a.v1; r.i1 = a.i1; r.v2 = fmaxf(a.v2, b.v1); }
  else         { r.v1 = b.v1; r.i1 = b.i1; r.v2 = fmaxf(b.v2, a.v1); }
  return r;
}

// Per-row argmax (lowest index on ties) and top-1 minus top-2 margin.
__global__ __launch_bounds__(256) void k_argmax(const float* __restrict__ logits, size_t ld, int V,
                                                int32_t* __restrict__ argmax, float* __restrict__ margin) {
  const int m = blockIdx.x;
  const float* row = logits + (size_t)m * ld;
  Top2 t = {-INFINITY, -INFINITY, INT_MAX};
  for (int c0 = threadIdx.x; c0 < V; c0 += 256 * 4) {  // (four loads in flight)
    float e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = row[min(c0 + 256 * u, V - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (c0 + 256 * u < V) t = top2_merge(t, Top2{e[u], -INFINITY, c0 + 256 * u});
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    Top2 o;
    o.v1 = __shfl_xor(t.v1, off, 64);
    o.v2 = __shfl_xor(t.v2, off, 64);
    o.i1 = __shfl_xor(t.i1, off, 64);
    t = top2_merge(t, o);
  }
  __shared__ Top2 red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    Top2 r = top2_merge(top2_merge(red[0], red[1]), top2_merge(red[2], red[3]));
    argmax[m] = r.i1;
    if (margin) margin[m] = r.v1 - r.v2;
  }
}

// Same from the per-workgroup reductions of the LM-head kernel (groups cover ascending column ranges): NW wavefronts a row, U records
// of a thread in flight at a time.  The kernel is one trip to memory and little else, so it takes as few rounds as the
// records allow, and one wavefront, without the exchange through LDS, where that makes one round: 64 rows of 1002 records took 7.7 us
// with one wavefront and one record after the other, 5.0 with <4, 4>; the head of 64 rows x 1024 columns (8 records, K = 256) takes
// 10.2 us with <1, 1> and 10.6 with <4, 4>, that of 32768 columns (256 records) 11.2 with <1, 4>, 11.3 with <4, 4>.
template <int NW, int U>
__global__ __launch_bounds__(64 * NW) void k_argmax_top2(const float4* __restrict__ top2, int n_groups,
                                                         int32_t* __restrict__ argmax, float* __restrict__ margin) {
  constexpr int NTHR = 64 * NW;
  const int m = blockIdx.x;
  const float4* row = top2 + (size_t)m * n_groups;
  Top2 t = {-INFINITY, -INFINITY, INT_MAX};
  for (int g0 = threadIdx.x; g0 < n_groups; g0 += NTHR * U) {
    float4 e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) e[u] = row[min(g0 + NTHR * u, n_groups - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g0 + NTHR * u < n_groups) t = top2_merge(t, Top2{e[u].x, e[u].y, __float_as_int(e[u].z)});
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    Top2 o;
    o.v1 = __shfl_xor(t.v1, off, 64);
    o.v2 = __shfl_xor(t.v2, off, 64);
    o.i1 = __shfl_xor(t.i1, off, 64);
    t = top2_merge(t, o);
  }
  if constexpr (NW > 1) {
    __shared__ Top2 red[NW];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    t = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = top2_merge(t, red[w]);
  }
  if (threadIdx.x == 0) {
    argmax[m] = t.i1;
    if (margin) margin[m] = t.v1 - t.v2;
  }
}

// ------------------------------------------------------------------------------------------
// Logit harvest (Sec. 4 stage 2; App. C, adjacency table tier 1): row tokens[m] of the dense
// [vocab][K] successor tables receives the K most likely next tokens of node m (ids, ordered by
// decreasing logit, equal logits by increasing id) and their softmax probabilities.  When several
// nodes carry the same token the highest node index writes (the others skip the store).
//
// What bounds it is reading the logits once, so a row is cut into chunks of 8192 columns and every
// (row, chunk) is a workgroup of its own, its values in registers (32 per thread, all loads in flight
// together): 64 rows of 128256 columns are 1024 workgroups.  One workgroup per row, walking it
// twice, left three quarters of the chip idle and took 113 us where this takes 23 (64 x 128256, 33 MB;
// k_harvest_merge included), and a batch ran one such launch per request (16 x 121 us, now 75 us in all).
// k_harvest_part leaves (max, sum of exponentials) and the K best pairs of its chunk;
// k_harvest_merge combines the chunks of a row.
//   tau: every group of four threads knows its best pair; the K-th best of these 64 pairs is a lower
//   bound of the chunk's K-th best.  At most K groups hold pairs at or above it, so the list of such
//   pairs never exceeds K * 4 * 32 = 2048 entries whatever the data (it usually holds K and a few).
// NaNs are no candidates and count in no sum.  Where the largest logit of a row is infinite its softmax is undefined: the
// scores are NaN (the ids are still ordered).
//
// A pair travels as one 64-bit key, larger = earlier: the value's bits made monotonic (-0 counts as +0) over the complement
// of the id; 0 stands for "no pair".  Ranking the 160 pairs of a row by comparing (float, int) took three quarters of the merge.
typedef unsigned long long hkey;
__device__ inline hkey harvest_key(float v, int id) {
  const unsigned b = __float_as_uint(v + 0.f);
  return (hkey)(b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u)) << 32 | (unsigned)~id;
}
__device__ inline float harvest_value(hkey k) {
  const unsigned b = (unsigned)(k >> 32);
  return __uint_as_float(b ^ ((b >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ inline int harvest_id(hkey k) { return (int)~(unsigned)k; }
// exp(v - m) for v <= m, also where both are the same infinity
__device__ inline float exp_below(float v, float m) { return v == m ? 1.f : __expf(v - m); }

constexpr int HARVEST_VPT = 32, HARVEST_CHUNK = 256 * HARVEST_VPT, HARVEST_KMAX = 16;
constexpr int HARVEST_MERGE = 1024;  // pairs a merge round ranks
static_assert(HARVEST_CHUNK == GOOSE_HARVEST_CHUNK && HARVEST_KMAX == GOOSE_HARVEST_KMAX, "the workspace is sized for these");

struct HarvestTable { HarvestReq r[GOOSE_MAX_REQUESTS]; };

// `n` pairs in LDS -> out(0 ..), the best `keep` of them in order.  All 256 threads call it.
template <typename Out>
__device__ inline void rank_pairs(const hkey* list, int n, int keep, Out out) {
  for (int e = threadIdx.x; e < n; e += 256) {
    const hkey mine = list[e];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) rank += list[j] > mine ? 1 : 0;
    if (rank < keep) out(rank, mine);
  }
}

// Grid (chunk, node, request).  pairs: keys [row][chunks][k_pairs]; lse: float2 (max, sum) [row][chunks].
// WHOLE: the row is one chunk (V <= HARVEST_CHUNK), its pairs go straight into the request's tables and nothing is left to merge.
template <bool WHOLE, int VPT>
__global__ __launch_bounds__(256) void k_harvest_part(const float* __restrict__ logits, size_t ld, int V, int k_pairs,
                                                      const HarvestTable t, hkey* __restrict__ pairs,
                                                      float2* __restrict__ lse) {
  __shared__ hkey best[64], list[HARVEST_KMAX * 4 * VPT], tau_s;
  __shared__ float red[8];
  __shared__ int n_s;
  const HarvestReq& q = t.r[blockIdx.z];
  const int m = blockIdx.y, K = WHOLE ? q.K : k_pairs;
  if (m >= q.B) return;
  const int tid = threadIdx.x, c0 = WHOLE ? 0 : blockIdx.x * HARVEST_CHUNK;
  int tok = 0, tok_t = 0;
  if (WHOLE) {
    tok = q.tokens[m];
    tok_t = tid < q.B ? q.tokens[tid] : 0;
  }
  const size_t row = (size_t)q.row0 + m;
  const float* src = logits + row * ld + c0;
  const int nc = min(HARVEST_CHUNK, V - c0);  // columns of this chunk (>= 1)
  float v[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) v[u] = (tid + u * 256 < nc) ? src[tid + u * 256] : NAN;
  if (tid == 0) {
    n_s = 0;
    tau_s = 0;  // (kept if fewer than K groups hold a value: every pair qualifies)
  }
  float bv = -INFINITY;
  int bi = -1;
#pragma unroll
  for (int u = 0; u < VPT; ++u)
    if (v[u] > bv || (v[u] == bv && bi < 0)) { bv = v[u]; bi = c0 + tid + u * 256; }  // (ids ascend: '>' keeps the lowest)
  hkey bk = bi < 0 ? 0 : harvest_key(bv, bi);
#pragma unroll
  for (int off = 1; off < 4; off <<= 1) {
    const hkey o = __shfl_xor(bk, off, 64);
    bk = o > bk ? o : bk;
  }
  if ((tid & 3) == 0) best[tid >> 2] = bk;
  float mx = bv;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  const float M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  if (tid < 64) {  // the rank of a group's best among the 64
    const hkey mine = best[tid];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < 64; ++j) rank += best[j] > mine ? 1 : 0;
    if (rank == K - 1 && mine != 0) tau_s = mine;
  }
  float sm = 0.f;
#pragma unroll
  for (int u = 0; u < VPT; ++u) sm += v[u] == v[u] ? exp_below(v[u], M) : 0.f;
  sm = wave_sum(sm);
  if ((tid & 63) == 0) red[4 + (tid >> 6)] = sm;
  __syncthreads();
  const hkey tau = tau_s;
  const bool all = tau == 0;
  const float tv = harvest_value(tau);
  const int ti = harvest_id(tau);
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const int c = c0 + tid + u * 256;
    if (v[u] == v[u] && (all || v[u] > tv || (v[u] == tv && c <= ti))) list[atomicAdd(&n_s, 1)] = harvest_key(v[u], c);
  }
  if (WHOLE) {
    const bool dup = __syncthreads_or(tid > m && tid < q.B && tok_t == tok);  // a later node carries the same token
    if (tok < 0 || tok >= V || dup) return;
    const int n = n_s;
    const float S = fabsf(M) == INFINITY ? NAN : red[4] + red[5] + red[6] + red[7];
    int32_t* ids = q.ids + (size_t)tok * K;
    float* scores = q.scores + (size_t)tok * K;
    rank_pairs(list, n, K, [&](int k, hkey p) { ids[k] = harvest_id(p); scores[k] = exp_below(harvest_value(p), M) / S; });
    if (tid >= n && tid < K) { ids[tid] = -1; scores[tid] = 0.f; }
    return;
  }
  __syncthreads();
  const size_t slot = row * gridDim.x + blockIdx.x;
  const int n = n_s;
  rank_pairs(list, n, K, [&](int k, hkey p) { pairs[slot * K + k] = p; });
  if (tid >= n && tid < K) pairs[slot * K + tid] = 0;
  if (tid == 0) lse[slot] = make_float2(M, red[4] + red[5] + red[6] + red[7]);
}

// Grid (node, request): the chunks of a row, K pairs each, into the request's tables.
__global__ __launch_bounds__(256) void k_harvest_merge(int chunks, int table_rows, int Kpart, const HarvestTable t,
                                                       const hkey* __restrict__ pairs, const float2* __restrict__ lse) {
  __shared__ hkey list[HARVEST_MERGE], top[HARVEST_KMAX];
  __shared__ float red[8];
  const HarvestReq& q = t.r[blockIdx.y];
  const int m = blockIdx.x, tid = threadIdx.x;
  if (m >= q.B) return;
  const size_t slot0 = ((size_t)q.row0 + m) * chunks;
  const hkey* src = pairs + slot0 * Kpart;
  const int total = chunks * Kpart;
  // everything the row needs is loaded up front: the kernel is a chain of trips to memory and little else
  hkey first[HARVEST_MERGE / 256];
#pragma unroll
  for (int u = 0; u < HARVEST_MERGE / 256; ++u)
    if (tid + 256 * u < total) first[u] = src[tid + 256 * u];
  float2 l0 = make_float2(-INFINITY, 0.f);
  if (tid < chunks) l0 = lse[slot0 + tid];
  const int tok = q.tokens[m], tok_t = tid < q.B ? q.tokens[tid] : 0;
  // (max, sum of exponentials) of the row: every thread's chunks, then across the workgroup
  float mx = l0.x, sm = l0.y;
  for (int c = tid + 256; c < chunks; c += 256) {
    const float2 e = lse[slot0 + c];
    const float nm = fmaxf(mx, e.x);
    sm = sm * exp_below(mx, nm) + e.y * exp_below(e.x, nm);
    mx = nm;
  }
  float M = mx;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
  sm = wave_sum(sm * exp_below(mx, M));
  if ((tid & 63) == 0) { red[tid >> 6] = M; red[4 + (tid >> 6)] = sm; }
#pragma unroll
  for (int u = 0; u < HARVEST_MERGE / 256; ++u)
    if (tid + 256 * u < total) list[tid + 256 * u] = first[u];
  if (tid < HARVEST_KMAX) top[tid] = 0;
  // does this node write?  (a valid token, and no later node with the same token)
  const bool dup = __syncthreads_or(tid > m && tid < q.B && tok_t == tok);
  // rounds of up to HARVEST_MERGE pairs, the best so far among them (zero keys rank after
  // every real pair, and the slots they do not fill are zero already)
  int n = min(total, HARVEST_MERGE), at = n;
  for (;;) {
    rank_pairs(list, n, q.K, [&](int k, hkey p) { top[k] = p; });
    __syncthreads();
    if (at >= total) break;
    const int take = min(HARVEST_MERGE - q.K, total - at);
    if (tid < q.K) list[tid] = top[tid];
    for (int e = tid; e < take; e += 256) list[q.K + e] = src[at + e];
    __syncthreads();
    if (tid < HARVEST_KMAX) top[tid] = 0;
    __syncthreads();
    n = q.K + take;
    at += take;
  }
  M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float S = fabsf(M) == INFINITY ? NAN : 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) S += red[4 + w] * exp_below(red[w], M);
  if (tid < q.K && tok >= 0 && tok < table_rows && !dup) {
    const hkey p = top[tid];
    q.ids[(size_t)tok * q.K + tid] = p != 0 ? harvest_id(p) : -1;
    q.scores[(size_t)tok * q.K + tid] = p != 0 ? exp_below(harvest_value(p), M) / S : 0.f;
  }
}

// ------------------------------------------------------------------------------------------
// Greedy walk (Alg. UnifiedGreedyWalk).  Every node whose own edge matches (its token equals the prediction
// at its parent) bids for its parent with the key (branch?1:0, node index); the lowest key
// wins, i.e. spine children before branch children, lower index first.  Thread 0 then follows
// the winners from the root; node indices grow along any path, so the walk is finite.
// dP (or null): the cache length becomes P + L + 1 here, and its old value goes to *P_old, which the commit that
// follows reads (a kernel of its own for this one word was the last launch of every step).
// `won` and `pred` take B ints of LDS each; nodes of the accepted path -> route[0 .. L] (LDS), *L_out = L, returns the bonus token to
// thread 0.  All threads (at least B) call it.
__device__ inline int walk(const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
                           const uint8_t* __restrict__ is_spine, const int32_t* __restrict__ argmax, int B, int* won, int* pred,
                           int* route, int* L_out) {
  const int i = threadIdx.x;
  int bid_at = -1, token = 0, branch = 0, bonus = 0;
  if (i < B) {
    won[i] = INT_MAX;
    pred[i] = argmax[i];
    bid_at = parent[i];
    token = tokens[i];
    branch = (is_spine != nullptr && is_spine[i] == 0) ? 1 : 0;
  }
  __syncthreads();
  if (i >= 1 && i < B && bid_at >= 0 && bid_at < i && token == pred[bid_at]) atomicMin(&won[bid_at], (branch << 16) | i);
  __syncthreads();
  if (i == 0) {
    int v = 0, L = 0;
    route[0] = 0;
    while (won[v] != INT_MAX && L < B - 1) {
      v = won[v] & 0xFFFF;
      route[++L] = v;
    }
    *L_out = L;
    bonus = pred[v];
  }
  __syncthreads();
  return bonus;
}

// What a walk hands back; p: cache length before the step.
__device__ inline void accept_store(int B, const int* route, int L, int bonus_token, int32_t* __restrict__ accept_len,
                                    int32_t* __restrict__ path, int32_t* __restrict__ bonus, int32_t* __restrict__ next_root,
                                    int32_t* __restrict__ dP, int p, int cap, int32_t* __restrict__ flags) {
  const int i = threadIdx.x;
  if (i < B) path[i] = i <= L ? route[i] : -1;
  if (i != 0) return;
  *accept_len = L;
  *bonus = bonus_token;
  if (next_root) *next_root = bonus_token;
  if (dP) {
    if (p < 0 || p + L + 1 > cap) atomicOr(flags, GOOSE_FLAG_CAPACITY);
    *dP = p + L + 1;
  }
}

__device__ inline void accept_body(const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
                                   const uint8_t* __restrict__ is_spine, const int32_t* __restrict__ argmax, int B,
                                   int32_t* __restrict__ accept_len, int32_t* __restrict__ path,
                                   int32_t* __restrict__ bonus, int32_t* __restrict__ next_root, int32_t* __restrict__ dP,
                                   int32_t* __restrict__ P_old, int cap, int32_t* __restrict__ flags) {
  __shared__ int won[GOOSE_MAX_B], pred[GOOSE_MAX_B], route[GOOSE_MAX_B], L_sh;
  const int p = dP ? *dP : 0;
  const int word = walk(parent, tokens, is_spine, argmax, B, won, pred, route, &L_sh);
  if (dP && threadIdx.x == 0) *P_old = p;
  accept_store(B, route, L_sh, word, accept_len, path, bonus, next_root, dP, p, cap, flags);
}

__global__ __launch_bounds__(128) void k_accept(const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
                                                const uint8_t* __restrict__ is_spine,
                                                const int32_t* __restrict__ argmax, int B,
                                                int32_t* __restrict__ accept_len, int32_t* __restrict__ path,
                                                int32_t* __restrict__ bonus, int32_t* __restrict__ next_root,
                                                int32_t* __restrict__ dP, int32_t* __restrict__ P_old, int cap,
                                                int32_t* __restrict__ flags) {
  accept_body(parent, tokens, is_spine, argmax, B, accept_len, path, bonus, next_root, dP, P_old, cap, flags);
}

__global__ __launch_bounds__(128) void k_accept_batch(const ReqTable t, const int32_t* __restrict__ argmax_all,
                                                      int32_t* __restrict__ P_old, int cap, int32_t* __restrict__ flags) {
  const BatchReq& q = t.r[blockIdx.x];
  accept_body(q.parent, q.tokens, q.is_spine, argmax_all + q.row0, q.B, q.accept_len, q.path, q.bonus, q.next_root, q.dP,
              P_old + blockIdx.x, cap, flags);
}

// ------------------------------------------------------------------------------------------
// Commit of the accepted path: cache slot P + path[j] -> slot P + j, j = 1..L, in every layer and head.
// fp32 caches, one launch: workgroup 2i moves the rows of K[head i][slot][d], a thread four columns
// of all of them (a cache may start on any float: no 16-byte alignment is assumed); workgroup 2i+1 the columns of
// Vt[head i][d][slot], a thread single elements along one d-row.  Either way a thread walks j upward and path[j] >= j, so a
// slot is always read before the same thread can overwrite it.
struct Float4Any { float e[4]; };
__device__ inline void compact_f32_body(float* __restrict__ kall, float* __restrict__ vall, int cap, int head_dim, int P,
                                        const int32_t* __restrict__ path, int L) {
  const int c = threadIdx.x;
  const bool is_v = blockIdx.x & 1;
  if (c >= (is_v ? head_dim : head_dim / 4)) return;
  const size_t base = (size_t)(blockIdx.x >> 1) * cap * head_dim;  // (layer * n_heads + head)
  Float4Any* kb = reinterpret_cast<Float4Any*>(kall + base) + c;
  float* vb = vall + base + (size_t)c * cap;
  if (L > GOOSE_MAX_B - 1) L = GOOSE_MAX_B - 1;
  for (int j = 1; j <= L; ++j) {
    const int src = path[j];
    if (src < j || src >= GOOSE_MAX_B || P + src >= cap) break;  // malformed path: stop, stay in bounds
    if (src == j) continue;
    if (is_v) vb[P + j] = vb[P + src];
    else kb[(size_t)(P + j) * (head_dim / 4)] = kb[(size_t)(P + src) * (head_dim / 4)];
  }
}
__global__ __launch_bounds__(256) void k_compact_f32(float* __restrict__ kall, float* __restrict__ vall, int cap, int head_dim,
                                                     const int32_t* __restrict__ dP, const int32_t* __restrict__ path,
                                                     const int32_t* __restrict__ accept_len) {
  compact_f32_body(kall, vall, cap, head_dim, *dP, path, *accept_len);
}
// Walk and commit of an fp32 step in one launch: every workgroup walks the tree itself (it is a few hundred bytes), the first one
// hands the results back.  The cache length before the step comes from *P_old (k_begin_f32), as the first workgroup replaces *dP.
__global__ __launch_bounds__(256) void k_commit_f32(const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
                                                    const uint8_t* __restrict__ is_spine, const int32_t* __restrict__ argmax, int B,
                                                    int32_t* __restrict__ accept_len, int32_t* __restrict__ path,
                                                    int32_t* __restrict__ bonus, int32_t* __restrict__ next_root,
                                                    int32_t* __restrict__ dP, const int32_t* __restrict__ P_old,
                                                    float* __restrict__ kall, float* __restrict__ vall, int cap, int head_dim,
                                                    int32_t* __restrict__ flags) {
  __shared__ int won[GOOSE_MAX_B], pred[GOOSE_MAX_B], route[GOOSE_MAX_B], L_sh;
  const int P = *P_old;
  const int word = walk(parent, tokens, is_spine, argmax, B, won, pred, route, &L_sh);
  if (blockIdx.x == 0) accept_store(B, route, L_sh, word, accept_len, path, bonus, next_root, dP, P, cap, flags);
  compact_f32_body(kall, vall, cap, head_dim, P, route, L_sh);
}

// The same for bf16 caches in MFMA operand order (32-key blocks; the layouts are spelled out in
// goose.h): thread c moves chunk c of the K row (16 bytes) and column c of the V row (2 bytes).
template <int D>
__device__ inline void compact_tiled_body(bf16_t* __restrict__ kall, bf16_t* __restrict__ vall, int cap,
                                          const int32_t* __restrict__ dP, const int32_t* __restrict__ path,
                                          const int32_t* __restrict__ accept_len) {
  const int c = threadIdx.x;
  bf16_t* kb = kall + (size_t)blockIdx.x * cap * D;  // blockIdx.x = layer * n_heads + head
  bf16_t* vb = vall + (size_t)blockIdx.x * cap * D;
  const int P = *dP;
  int L = *accept_len;
  if (L > GOOSE_MAX_B - 1) L = GOOSE_MAX_B - 1;
  auto k_off = [](int g, int ch) {  // chunk ch = 2*s + hh of slot g
    const int kk = g & 31, i = (((kk >> 2) & 3) << 3) | ((kk >> 4) << 2) | (kk & 3);
    return (((size_t)(g >> 5) * (D / 16) + (ch >> 1)) * 64 + i + 32 * (ch & 1)) * 8;
  };
  auto v_off = [](int g, int col) {
    const int kk = g & 31;
    return ((((size_t)(g >> 5) * (D / 32) + (col >> 5)) * 2 + ((kk >> 3) & 1)) * 64 + (col & 31) + 32 * (kk >> 4)) * 8 +
           (kk & 7);
  };
  for (int j = 1; j <= L; ++j) {
    const int src = path[j];
    if (src < j || src >= GOOSE_MAX_B || P + src >= cap) break;  // malformed path: stop, stay in bounds
    if (src == j) continue;
    if (c < D / 8)
      *reinterpret_cast<uint4*>(kb + k_off(P + j, c)) = *reinterpret_cast<const uint4*>(kb + k_off(P + src, c));
    vb[v_off(P + j, c)] = vb[v_off(P + src, c)];
  }
}

template <int D>
__global__ __launch_bounds__(D) void k_compact_tiled(bf16_t* __restrict__ kall, bf16_t* __restrict__ vall, int cap,
                                                     const int32_t* __restrict__ dP,
                                                     const int32_t* __restrict__ path,
                                                     const int32_t* __restrict__ accept_len) {
  compact_tiled_body<D>(kall, vall, cap, dP, path, accept_len);
}

template <int D>
__global__ __launch_bounds__(D) void k_compact_tiled_batch(const ReqTable t, int cap) {
  const BatchReq& q = t.r[blockIdx.y];
  compact_tiled_body<D>((bf16_t*)q.kall, (bf16_t*)q.vall, cap, q.dP, q.path, q.accept_len);
}

__global__ void k_new_P(const int32_t* dP, const int32_t* accept_len, int32_t* new_P, int cap, int32_t* flags) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const int p = *dP, l = *accept_len;
    if (p < 0 || l < 0 || p + l + 1 > cap) atomicOr(flags, GOOSE_FLAG_CAPACITY);
    *new_P = p + l + 1;
  }
}

}  // namespace

// ============================================================================================
int launch_set_int(int32_t* dst, int v, hipStream_t st) {
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, st, dst, v);
  return goose_launch_status();
}

int launch_build_mask(const int32_t* parent, int B, const int32_t* dP, uint64_t* mask, int32_t* depth, int32_t* pos,
                      int32_t* flags, int cap, int P_max, hipStream_t st) {
  if (dP != nullptr)
    hipLaunchKernelGGL(k_build_mask<true>, dim3(1), dim3(128), 0, st, parent, B, dP, mask, depth, pos, flags, cap, P_max);
  else
    hipLaunchKernelGGL(k_build_mask<false>, dim3(1), dim3(128), 0, st, parent, B, nullptr, mask, depth, pos, flags, cap, P_max);
  return goose_launch_status();
}

// 16-byte pieces where every row of the table and of x starts on a multiple of them
template <typename T>
static bool embed_vec(const void* E, int H, const float* x) {
  return H % (16 / sizeof(T)) == 0 && (((uintptr_t)E | (uintptr_t)x) & 15) == 0;
}
template <typename T>
static void launch_embed_t(const void* E, const int32_t* tokens, int B, int H, int V, float* x, hipStream_t st) {
  constexpr int VEC = 16 / sizeof(T);
  if (embed_vec<T>(E, H, x))
    hipLaunchKernelGGL((k_embed<T, VEC>), dim3((H / VEC + 255) / 256, B), dim3(256), 0, st, (const T*)E, tokens, H, V, x);
  else
    hipLaunchKernelGGL((k_embed<T, 1>), dim3((H + 255) / 256, B), dim3(256), 0, st, (const T*)E, tokens, H, V, x);
}
int launch_embed(int dtype, const void* E, const int32_t* tokens, int B, int H, int V, float* x, hipStream_t st) {
  if (dtype == GOOSE_DTYPE_BF16) launch_embed_t<bf16_t>(E, tokens, B, H, V, x, st);
  else if (dtype == GOOSE_DTYPE_F16) launch_embed_t<_Float16>(E, tokens, B, H, V, x, st);
  else launch_embed_t<float>(E, tokens, B, H, V, x, st);
  return goose_launch_status();
}

struct NormArgs {
  float* x; int H; const float* part; int S; size_t part_stride, part_ld; const void* g; float eps; void* xn; int ldxn, B;
  RopeArgs rope; hipStream_t st;
};
template <typename Tg, typename T, int NTHR, int TERMS>
static void launch_resid_norm_n(const NormArgs& a) {
  if (a.rope.rows > 0) {
    const int per = NTHR / a.rope.half;  // (half <= 128 <= NTHR)
    hipLaunchKernelGGL((k_resid_norm<Tg, T, NTHR, TERMS, true>), dim3(a.B + (a.rope.rows + per - 1) / per), dim3(NTHR), 0, a.st,
                       a.x, a.H, a.part, a.S, a.part_stride, a.part_ld, (const Tg*)a.g, a.eps, (T*)a.xn, a.ldxn, a.rope);
  } else {
    hipLaunchKernelGGL((k_resid_norm<Tg, T, NTHR, TERMS, false>), dim3(a.B), dim3(NTHR), 0, a.st, a.x, a.H, a.part, a.S,
                       a.part_stride, a.part_ld, (const Tg*)a.g, a.eps, (T*)a.xn, a.ldxn, a.rope);
  }
}
template <typename Tg, typename T, int TERMS>
static void launch_resid_norm_t(const NormArgs& a) {
  if (a.H > 4 * 256) launch_resid_norm_n<Tg, T, 1024, TERMS>(a);  // 1024 threads once a row has more than 1024 columns
  else launch_resid_norm_n<Tg, T, 256, TERMS>(a);
}
template <typename Tg, typename T>
static void launch_resid_norm_terms(int terms, const NormArgs& a) {
  if (terms == 2) launch_resid_norm_t<Tg, T, 2>(a);
  else launch_resid_norm_t<Tg, T, 1>(a);
}

int launch_resid_norm(int gain_dtype, int act_dtype, float* x, int H, const float* part, int S, size_t part_stride,
                      size_t part_ld, const void* g, float eps, void* xn, int ldxn, int terms, int B, hipStream_t st,
                      const RopeArgs* rope) {
  if ((H & 3) || H > 16 * 1024 || (terms == 2 && (H & 7))) return GOOSE_ERR_SHAPE;
  if (terms != 1 && terms != 2) return GOOSE_ERR_ARG;
  if (rope != nullptr && (rope->rows != B || rope->half < 1 || rope->half > 128)) return GOOSE_ERR_ARG;
  const NormArgs a{x, H, part, S, part_stride, part_ld, g, eps, xn, ldxn, B, rope != nullptr ? *rope : RopeArgs{}, st};
  if (gain_dtype == GOOSE_DTYPE_BF16 && act_dtype == GOOSE_DTYPE_BF16) launch_resid_norm_terms<bf16_t, bf16_t>(terms, a);
  else if (gain_dtype == GOOSE_DTYPE_BF16 && act_dtype == GOOSE_DTYPE_F16) launch_resid_norm_terms<bf16_t, _Float16>(terms, a);
  else if (gain_dtype == GOOSE_DTYPE_F16 && act_dtype == GOOSE_DTYPE_F16) launch_resid_norm_terms<_Float16, _Float16>(terms, a);
  else return GOOSE_ERR_ARG;
  return goose_launch_status();
}

int launch_argmax(const float* logits, size_t ld, int V, int B, int32_t* argmax, float* margin, hipStream_t st) {
  hipLaunchKernelGGL(k_argmax, dim3(B), dim3(256), 0, st, logits, ld, V, argmax, margin);
  return goose_launch_status();
}

// fp32 rows -> the two-term 16-bit operand layout of the projections (groups of eight columns:
// 8 hi values T(v), then their 8 lo values T(v - hi)); columns beyond `cols` up to ld_dst/2 are zero.
template <typename T>
__global__ __launch_bounds__(256) void k_split_operand(const float* __restrict__ src, int cols, int ld_src,
                                                       T* __restrict__ dst, int ld_dst) {
  const int m = blockIdx.y, c = blockIdx.x * 256 + threadIdx.x;
  if (c >= ld_dst / 2) return;
  const float v = c < cols ? src[(size_t)m * ld_src + c] : 0.f;
  const T hi = (T)v;
  T* d = dst + (size_t)m * ld_dst + (size_t)(c >> 3) * 16 + (c & 7);
  d[0] = hi;
  d[8] = (T)(v - to_f32(hi));
}

int launch_split_operand(int dtype, const float* src, int rows, int cols, int ld_src, void* dst, int ld_dst,
                         hipStream_t st) {
  const dim3 grid((ld_dst / 2 + 255) / 256, rows);
  if (dtype == GOOSE_DTYPE_BF16)
    hipLaunchKernelGGL(k_split_operand<bf16_t>, grid, dim3(256), 0, st, src, cols, ld_src, (bf16_t*)dst, ld_dst);
  else if (dtype == GOOSE_DTYPE_F16)
    hipLaunchKernelGGL(k_split_operand<_Float16>, grid, dim3(256), 0, st, src, cols, ld_src, (_Float16*)dst, ld_dst);
  else
    return GOOSE_ERR_ARG;
  return goose_launch_status();
}

// Plain streaming copy of n 16-byte words (profiling aid: a kernel of exactly known HBM traffic).
__global__ __launch_bounds__(256) void k_copy_probe(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

int launch_copy_probe(const void* src, void* dst, size_t bytes, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_probe, dim3(2048), dim3(256), 0, st, (const uint4*)src, (uint4*)dst, bytes / 16);
  return goose_launch_status();
}

int launch_argmax_top2(const void* top2, int n_groups, int B, int32_t* argmax, float* margin, hipStream_t st) {
  if (n_groups <= 64)
    hipLaunchKernelGGL((k_argmax_top2<1, 1>), dim3(B), dim3(64), 0, st, (const float4*)top2, n_groups, argmax, margin);
  else if (n_groups <= 4 * 64)
    hipLaunchKernelGGL((k_argmax_top2<1, 4>), dim3(B), dim3(64), 0, st, (const float4*)top2, n_groups, argmax, margin);
  else
    hipLaunchKernelGGL((k_argmax_top2<4, 4>), dim3(B), dim3(256), 0, st, (const float4*)top2, n_groups, argmax, margin);
  return goose_launch_status();
}

// A vocabulary of one chunk, in one launch.  What bounds it is a chain of steps of which each goes with the logits that
// a thread holds, so it holds no more than its 256th of the row needs.  With a merge behind it and 32 logits a thread, 64 rows of
// 1024 / 4096 / 8192 columns took 10.8 / 11.6 / 12.2 us for K = 1 and 11.4 / 12.2 / 13.2 for K = 10; now 4.2 / 5.9 / 8.0 and
// 4.6 / 6.4 / 8.5 (the kernel that walked each row twice: 5.9 / 6.9 / 9.9 and 16.7 / 17.9 / 20.8).
static void launch_harvest_whole(const float* logits, size_t ld, int V, const HarvestTable& t, int b, int n, hipStream_t st) {
  const dim3 grid(1, b, n);
  if (V <= 4 * 256)
    hipLaunchKernelGGL((k_harvest_part<true, 4>), grid, dim3(256), 0, st, logits, ld, V, 0, t, nullptr, nullptr);
  else if (V <= 16 * 256)
    hipLaunchKernelGGL((k_harvest_part<true, 16>), grid, dim3(256), 0, st, logits, ld, V, 0, t, nullptr, nullptr);
  else
    hipLaunchKernelGGL((k_harvest_part<true, HARVEST_VPT>), grid, dim3(256), 0, st, logits, ld, V, 0, t, nullptr, nullptr);
}

// One launch of k_harvest_part for all requests.  The tables of different requests are normally distinct and one
// launch of k_harvest_merge fills them all; where two of them overlap (requests that share a table) they are filled one
// request after the other, so that the later request wins.  A vocabulary of one chunk needs no merge: the K best of its rows
// are known in k_harvest_part (launch_harvest_whole).
int launch_harvest_topk(const float* logits, size_t ld, int V, const HarvestReq* reqs, int n, void* ws, hipStream_t st) {
  if (n < 1 || n > GOOSE_MAX_REQUESTS || ws == nullptr || V < 1) return GOOSE_ERR_ARG;
  HarvestTable t{};
  int k_max = 0, b_max = 0;
  size_t rows = 0;
  bool overlap = false;
  for (int r = 0; r < n; ++r) {
    const HarvestReq& q = reqs[r];
    if (q.K < 1 || q.K > HARVEST_KMAX || q.B < 1 || q.row0 < 0) return GOOSE_ERR_ARG;
    t.r[r] = q;
    k_max = q.K > k_max ? q.K : k_max;
    b_max = q.B > b_max ? q.B : b_max;
    rows = (size_t)(q.row0 + q.B) > rows ? (size_t)(q.row0 + q.B) : rows;
    for (int p = 0; p < r; ++p) {
      const size_t a = (size_t)V * q.K, b = (size_t)V * reqs[p].K;
      overlap = overlap || (q.ids < reqs[p].ids + b && reqs[p].ids < q.ids + a) ||
                (q.scores < reqs[p].scores + b && reqs[p].scores < q.scores + a);
    }
  }
  const int chunks = (V + HARVEST_CHUNK - 1) / HARVEST_CHUNK;
  float2* lse = static_cast<float2*>(ws);
  hkey* pairs = reinterpret_cast<hkey*>(lse + rows * chunks);
  int rc = GOOSE_OK;
  if (chunks > 1) {
    hipLaunchKernelGGL((k_harvest_part<false, HARVEST_VPT>), dim3(chunks, b_max, n), dim3(256), 0, st, logits, ld, V, k_max, t,
                       pairs, lse);
    rc = goose_launch_status();
    if (rc != GOOSE_OK) return rc;
  }
  auto fill = [&](const HarvestTable& reqs_of, int b, int n_of) {
    if (chunks > 1)
      hipLaunchKernelGGL(k_harvest_merge, dim3(b, n_of), dim3(256), 0, st, chunks, V, k_max, reqs_of, pairs, lse);
    else
      launch_harvest_whole(logits, ld, V, reqs_of, b, n_of, st);
    return goose_launch_status();
  };
  if (!overlap) return fill(t, b_max, n);
  for (int r = 0; r < n; ++r) {
    HarvestTable one{};
    one.r[0] = reqs[r];
    rc = fill(one, reqs[r].B, 1);
    if (rc != GOOSE_OK) return rc;
  }
  return GOOSE_OK;
}

static ReqTable req_table(const BatchReq* reqs, int n) {
  ReqTable t{};
  for (int r = 0; r < n; ++r) t.r[r] = reqs[r];
  return t;
}

int launch_batch_begin(int dtype, const BatchReq* reqs, int n, int max_B, const void* E, int H, int V,
                       uint64_t* mask, int32_t* depth, int32_t* pos, float* x, int32_t* flags, int cap, hipStream_t st) {
  if (n < 1 || n > GOOSE_MAX_REQUESTS) return GOOSE_ERR_ARG;
  const ReqTable t = req_table(reqs, n);
  hipLaunchKernelGGL(k_build_mask_batch, dim3(n), dim3(128), 0, st, t, mask, depth, pos, flags, cap);
  int rc = goose_launch_status();
  if (rc != GOOSE_OK) return rc;
  if (dtype != GOOSE_DTYPE_BF16 && dtype != GOOSE_DTYPE_F16) return GOOSE_ERR_SHAPE;
  const bool vec = embed_vec<bf16_t>(E, H, x);  // (both types have 2 bytes)
  const dim3 grid(((vec ? H / 8 : H) + 255) / 256, max_B, n);
  if (dtype == GOOSE_DTYPE_BF16) {
    if (vec) hipLaunchKernelGGL((k_embed_batch<bf16_t, 8>), grid, dim3(256), 0, st, (const bf16_t*)E, t, H, V, x);
    else hipLaunchKernelGGL((k_embed_batch<bf16_t, 1>), grid, dim3(256), 0, st, (const bf16_t*)E, t, H, V, x);
  } else {
    if (vec) hipLaunchKernelGGL((k_embed_batch<_Float16, 8>), grid, dim3(256), 0, st, (const _Float16*)E, t, H, V, x);
    else hipLaunchKernelGGL((k_embed_batch<_Float16, 1>), grid, dim3(256), 0, st, (const _Float16*)E, t, H, V, x);
  }
  return goose_launch_status();
}

int launch_batch_end(const BatchReq* reqs, int n, const int32_t* argmax_all, int n_layers, int n_kv_heads, int cap,
                     int head_dim, int32_t* P_old, int32_t* flags, hipStream_t st) {
  if (n < 1 || n > GOOSE_MAX_REQUESTS) return GOOSE_ERR_ARG;
  ReqTable t = req_table(reqs, n);
  hipLaunchKernelGGL(k_accept_batch, dim3(n), dim3(128), 0, st, t, argmax_all, P_old, cap, flags);
  int rc = goose_launch_status();
  if (rc != GOOSE_OK) return rc;
  for (int r = 0; r < n; ++r) t.r[r].dP = P_old + r;  // the walk replaced the lengths
  if (head_dim == 128)
    hipLaunchKernelGGL(k_compact_tiled_batch<128>, dim3(n_layers * n_kv_heads, n), dim3(128), 0, st, t, cap);
  else if (head_dim == 64)
    hipLaunchKernelGGL(k_compact_tiled_batch<64>, dim3(n_layers * n_kv_heads, n), dim3(64), 0, st, t, cap);
  else
    return GOOSE_ERR_SHAPE;
  return goose_launch_status();
}

int launch_accept(const int32_t* parent, const int32_t* tokens, const uint8_t* is_spine, const int32_t* argmax, int B,
                  int32_t* accept_len, int32_t* path, int32_t* bonus, int32_t* next_root, int32_t* dP, int32_t* P_old, int cap,
                  int32_t* flags, hipStream_t st) {
  hipLaunchKernelGGL(k_accept, dim3(1), dim3(128), 0, st, parent, tokens, is_spine, argmax, B, accept_len, path,
                     bonus, next_root, dP, P_old, cap, flags);
  return goose_launch_status();
}

int launch_commit_f32(const int32_t* parent, const int32_t* tokens, const uint8_t* is_spine, const int32_t* argmax, int B,
                      int32_t* accept_len, int32_t* path, int32_t* bonus, int32_t* next_root, int32_t* dP, const int32_t* P_old,
                      float* kall, float* vall, int n_layers, int n_heads, int cap, int head_dim, int32_t* flags, hipStream_t st) {
  hipLaunchKernelGGL(k_commit_f32, dim3(2 * n_layers * n_heads), dim3(head_dim <= 128 && B <= 128 ? 128 : 256), 0, st, parent, tokens,
                     is_spine, argmax, B, accept_len, path, bonus, next_root, dP, P_old, kall, vall, cap, head_dim, flags);
  return goose_launch_status();
}

int launch_compact(int elem_bytes, void* kall, void* vall, int n_layers, int n_heads, int cap, int head_dim,
                   const int32_t* dP, const int32_t* path, const int32_t* accept_len, int32_t* new_P,
                   int32_t* flags, hipStream_t st) {
  int rc;
  if (elem_bytes == 2) {  // bf16 / fp16 (moved as bit patterns): operand-ordered blocks
    if (head_dim == 128)
      hipLaunchKernelGGL(k_compact_tiled<128>, dim3(n_layers * n_heads), dim3(128), 0, st, (bf16_t*)kall, (bf16_t*)vall,
                         cap, dP, path, accept_len);
    else if (head_dim == 64)
      hipLaunchKernelGGL(k_compact_tiled<64>, dim3(n_layers * n_heads), dim3(64), 0, st, (bf16_t*)kall, (bf16_t*)vall,
                         cap, dP, path, accept_len);
    else
      return GOOSE_ERR_SHAPE;
    rc = goose_launch_status();
  } else {  // fp32: K[head][slot][d], Vt[head][d][slot]; head_dim <= 256, a multiple of 8
    hipLaunchKernelGGL(k_compact_f32, dim3(2 * n_layers * n_heads), dim3(head_dim <= 64 ? 64 : 256), 0, st, (float*)kall,
                       (float*)vall, cap, head_dim, dP, path, accept_len);
    rc = goose_launch_status();
  }
  if (rc != GOOSE_OK) return rc;
  if (new_P) {
    hipLaunchKernelGGL(k_new_P, dim3(1), dim3(1), 0, st, dP, accept_len, new_P, cap, flags);
    rc = goose_launch_status();
  }
  return rc;
}
