// The projections of a pass of one row (an autoregressive cycle) for gfx950: out[n] = sum_k A[k] * W[n][k].
// Operands, K ranges and the order of every sum are those of the skinny kernel of gemm_bf16.hip, and so are the results, bit for bit.
//
// With one row a layer is the weight stream and what lies between its launches: the two norms and the
// attention's merge take 10 of 92 us, 3-4 us each for next to no work.  So the operand row, a few KiB, is
// formed by every workgroup itself while its first weights are on their way:
//   ROW_COPY   as an earlier kernel left it
//   ROW_NORM   RMSNorm(x + split-K slices) * g       (k_resid_norm's arithmetic, over all of the row, of which the K range is kept)
//   ROW_MERGE  the attention's key splits combined   (k_attn_merge's)
// It stays in LDS for the whole K range: the loop copies nothing and has no barrier.  A wavefront owns one column
// tile and keeps two stages (64 inputs, 4 KiB each) of its weights in flight.  All that the row is made of is asked for before the first
// weights (with none or four slices to add, which is what contexts of up to 64 rows have at hidden sizes of 4096 and more; other numbers of slices come
// four at a time and column group after column group, and the weights behind the last): loads return in order, and the gains asked for after them cost
// 1.5 us a launch.  For the same reason a second row, whose loads would follow, made a layer of two rows slower than its launches (94.1 against
// 92.7 us), and more weights in flight first make everything wait (four stages of 128 inputs 91.9 us).
// Layers of one row against the launches that it replaces: 7B over 1024 slots 92.6 -> 88.3 us, over 16000 128.2 -> 123.7, 13B 124.6 -> 118.5, 33B
// 209.2 -> 186.1, Qwen3-8B in two terms over 5000 101.0 -> 94.1.  In contexts for trees of 80 nodes (O in eight ranges at a hidden size of 4096), over 1024: 7B
// 98.2 -> 92.9, Llama-3-8B 102.1 -> 96.3, Qwen3-8B 94.3 -> 88.4, 13B 136.6 -> 128.8, 33B 207.2 -> 199.2; of 256 rows 98.4 -> 93.5, 101.6 -> 95.7.
#include "fold.h"
#include "goose_internal.h"
#include "mma16.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define GOOSE_BUFFER_WORD3 0x00020000  // word 3 of a raw buffer descriptor: 32-bit untyped data, range checked

constexpr int LDS_A = 64 * 1024;  // bytes of the operand row

struct RowArgs {
  const u32x4* Wp;
  int ntiles, ksteps_total, stages_per_split, ngroups;
  float out_scale;
  void* out;
  size_t split_stride;
  int32_t* flags;
  OneRow a;
};

// one of four gains loaded together
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
__device__ inline float gain_of(unsigned short bits, int f16) {
  return f16 ? (float)__builtin_bit_cast(_Float16, bits) : __builtin_bit_cast(float, (unsigned)bits << 16);
}

// NI: passes over a row of up to 4096 columns each (ROW_NORM).  Grid: (K range, column group; one group more where the launch also
// writes the rotary angles).
template <int NW, int TERMS, int EPI, bool F16, int PRO, int NI>
__global__ __launch_bounds__(64 * NW) void k_gemm_row(const RowArgs p) {
  typedef typename Mma16<F16>::T T;
  typedef typename Mma16<F16>::v8 op8;
  constexpr int STEPS = 4, D = 2;  // k-steps (16 inputs) of a stage, stages of weights in flight
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_A];
  __shared__ float red[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int by = blockIdx.x, bx = blockIdx.y;
  const OneRow& a = p.a;
  if (PRO == ROW_NORM && bx >= p.ngroups) {  // the rotary angles, which nothing before the attention needs
    const int n = a.rope.rows * a.rope.half;
    for (int it = by * 64 * NW + tid; it < n; it += gridDim.x * 64 * NW) rope_entry(a.rope, it / a.rope.half, it % a.rope.half);
    return;
  }
  const int tile = bx + p.ngroups * wave;
  const bool active = tile < p.ntiles;
  const int s_begin = by * p.stages_per_split;  // (stages of 128 inputs)
  const int n128 = min(p.stages_per_split, p.ksteps_total / 8 - s_begin);
  const int nst = n128 * (8 / STEPS);

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  u32x4 wreg[D][STEPS];
#if defined(__HIP_DEVICE_COMPILE__)
  // (a descriptor over this wavefront's pieces of its K range: loads beyond it return zeros and cost no memory traffic)
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u32x4*>(p.Wp + ((size_t)(active ? tile : 0) * p.ksteps_total + (size_t)s_begin * 8) * 64), 0,
      active ? nst * STEPS * 1024 : 0, GOOSE_BUFFER_WORD3);
#endif
  auto load_w = [&](int i, int slot, int s) {
#if defined(__HIP_DEVICE_COMPILE__)
    wreg[slot][s] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16, (i * STEPS + s) * 1024, 2);
#endif
  };
  auto first_weights = [&]() {
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
      for (int s = 0; s < STEPS; ++s) load_w(i, i, s);
  };
  // four values, columns c .. c + 3 (c a multiple of 4), as the operand holds them; columns outside the K range are left out
  auto put4 = [&](int c, float v0, float v1, float v2, float v3) {
    const int k = c - s_begin * 128;
    if (k < 0 || k >= n128 * 128) return;
    typedef T t4 __attribute__((ext_vector_type(4)));
    const t4 hi = {(T)v0, (T)v1, (T)v2, (T)v3};
    T* dst = reinterpret_cast<T*>(lds) + term_pos(TERMS, k);
    *reinterpret_cast<t4*>(dst) = hi;
    if (TERMS == 2)
      *reinterpret_cast<t4*>(dst + 8) = t4{(T)(v0 - (float)hi[0]), (T)(v1 - (float)hi[1]), (T)(v2 - (float)hi[2]), (T)(v3 - (float)hi[3])};
  };
  if constexpr (PRO == ROW_NORM) {
    // k_resid_norm's threads are 1024 (256 for rows of up to 1024 columns), a thread here stands for four of them
    const float* x = static_cast<const float*>(a.src);
    const int nvec = a.H >> 2;
    float4 v[NI][4];
    u16x4 gain[NI][4];
    float ss[4] = {0.f, 0.f, 0.f, 0.f};
    if (tid < 256) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c4 = min(tid + 256 * j + 1024 * i, nvec - 1);
          v[i][j] = *reinterpret_cast<const float4*>(x + c4 * 4);
          gain[i][j] = reinterpret_cast<const u16x4*>(a.g)[c4];
        }
      if (a.S == 4) {  // (all slices of all columns in flight)
        constexpr int G = NW > 4 ? 1 : NI;  // (five wavefronts have 256 registers each)
#pragma unroll
        for (int i0 = 0; i0 < NI; i0 += G) {
          float4 q[G][4][4];
#pragma unroll
          for (int i = 0; i < G; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int s = 0; s < 4; ++s) {
                const int c4 = min(tid + 256 * j + 1024 * (i0 + i), nvec - 1);
                q[i][j][s] = *reinterpret_cast<const float4*>(a.part + s * a.part_stride + c4 * 4);
              }
          if (i0 + G == NI) first_weights();
#pragma unroll
          for (int i = 0; i < G; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int s = 0; s < 4; ++s) {
                float4& t = v[i0 + i][j];
                t.x += q[i][j][s].x;
                t.y += q[i][j][s].y;
                t.z += q[i][j][s].z;
                t.w += q[i][j][s].w;
              }
        }
      } else {
        if (a.S == 0) first_weights();
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            add_slices(v[i][j], a.part + min(tid + 256 * j + 1024 * i, nvec - 1) * 4, a.S, a.part_stride);
        if (a.S != 0) first_weights();
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (tid + 256 * j + 1024 * i < nvec) ss[j] = add_squares(ss[j], v[i][j]);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int j = 0; j < 4; ++j) ss[j] += __shfl_xor(ss[j], off, 64);
      if (lane < 4) red[4 * lane + wave] = lane == 0 ? ss[0] : (lane == 1 ? ss[1] : (lane == 2 ? ss[2] : ss[3]));
    } else {
      first_weights();
    }
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) tot += red[w];
    const float rstd = 1.0f / sqrtf(tot / (float)a.H + a.eps);
    if (tid < 256) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = (tid + 256 * j + 1024 * i) * 4;
          if (c < a.H)
            put4(c, (v[i][j].x * rstd) * gain_of(gain[i][j][0], a.g_f16), (v[i][j].y * rstd) * gain_of(gain[i][j][1], a.g_f16),
                 (v[i][j].z * rstd) * gain_of(gain[i][j][2], a.g_f16), (v[i][j].w * rstd) * gain_of(gain[i][j][3], a.g_f16));
        }
      const int cp = a.H + tid * 4;  // (the padding of K, less than 128 columns, meets zero weights: any finite value)
      if (cp < p.ksteps_total * 16) put4(cp, 0.f, 0.f, 0.f, 0.f);
    }
  } else if constexpr (PRO == ROW_MERGE) {
    const int total = n128 * 32;  // groups of four columns
    auto item = [&](int it, auto after_loads) {
      const int c = s_begin * 128 + it * 4, cc = min(c, a.H - 4), h = cc / a.head_dim;
      fold_f32x4 f = merge_splits(a.part, a.att_ml, (size_t)h * a.S * a.Bpad, a.Bpad, a.S, a.head_dim, cc - h * a.head_dim, after_loads);
      if (c >= a.H) f = fold_f32x4{0.f, 0.f, 0.f, 0.f};  // (the padding of K)
      put4(c, f[0], f[1], f[2], f[3]);
    };
    item(min(tid, total - 1), first_weights);  // (by all lanes: the weights' loads need them; an item twice gives the same twice)
    for (int it = tid + 64 * NW; it < total; it += 64 * NW) item(it, []() {});
  } else {
    constexpr int U = 4;
    const int total = n128 * 16 * TERMS;  // 16 bytes each
    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const T*>(a.src) + (size_t)s_begin * 128 * TERMS);
    u32x4 v[U];
    auto fetch = [&](int it) {
#pragma unroll
      for (int q = 0; q < U; ++q) v[q] = src[min(it + q * 64 * NW, total - 1)];
    };
    auto store = [&](int it) {
#pragma unroll
      for (int q = 0; q < U; ++q) reinterpret_cast<u32x4*>(lds)[min(it + q * 64 * NW, total - 1)] = v[q];
    };
    fetch(tid);
    first_weights();
    store(tid);
    for (int it = tid + U * 64 * NW; it < total; it += U * 64 * NW) {
      fetch(it);
      store(it);
    }
  }
  __syncthreads();

  // lane l holds the eight inputs 8 * (l / 32) .. of a k-step, of the one row as all 32 of the matrix instruction
  const unsigned char* arow = lds + (lane >> 5) * 16 * TERMS;
  for (int i = 0; i < nst; i += D) {
#pragma unroll
    for (int slot = 0; slot < D; ++slot) {
      const unsigned char* ap = arow + min(i + slot, nst - 1) * (32 * STEPS * TERMS);  // (a stage beyond the range meets zero weights)
      op8 af[STEPS][TERMS];
#pragma unroll
      for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int t = 0; t < TERMS; ++t) af[s][t] = *reinterpret_cast<const op8*>(ap + s * 32 * TERMS + t * 16);
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
#pragma unroll
        for (int t = 0; t < TERMS; ++t) acc = Mma16<F16>::mfma(af[s][t], __builtin_bit_cast(op8, wreg[slot][s]), acc);
        load_w(i + slot + D, slot, s);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // C layout of the 32x32 MFMA: register 0 of lane l < 32 holds row 0, column l
  if (!active) return;
  if (EPI == EPI_PARTIAL) {
    if (lane < 32) static_cast<float*>(p.out)[by * p.split_stride + tile * 32 + lane] = acc[0] * p.out_scale;
  } else {  // columns 0-15 of a tile are the gates, 16-31 the up values of its 16 outputs
    bool clamped = false;
    const float u = __shfl(acc[0], (lane & 15) + 16, 64);
    if (lane < 16) {
      float h = swiglu_f32(acc[0] * p.out_scale, u * p.out_scale);
      if (F16 && fabsf(h) > 65504.0f) {  // beyond fp16: clamp, and say so (GOOSE_FLAG_RANGE)
        h = copysignf(65504.0f, h);
        clamped = true;
      }
      const T hi = (T)h;
      T* dst = static_cast<T*>(p.out) + term_pos(TERMS, tile * 16 + lane);
      dst[0] = hi;
      if (TERMS == 2) dst[8] = (T)(h - (float)hi);
    }
    if (F16 && clamped && p.flags != nullptr) atomicOr(p.flags, GOOSE_FLAG_RANGE);
  }
}

template <int NW, int TERMS, int EPI, bool F16, int PRO>
int launch_ni(const RowArgs& p, dim3 grid, hipStream_t st) {
  if constexpr (PRO == ROW_NORM) {
    if (p.a.H > 4096) {
      hipLaunchKernelGGL((k_gemm_row<NW, TERMS, EPI, F16, PRO, 2>), grid, dim3(64 * NW), 0, st, p);
      return goose_launch_status();
    }
  }
  hipLaunchKernelGGL((k_gemm_row<NW, TERMS, EPI, F16, PRO, 1>), grid, dim3(64 * NW), 0, st, p);
  return goose_launch_status();
}
template <int NW, int TERMS, int EPI, bool F16>
int launch_pro(const RowArgs& p, dim3 grid, hipStream_t st) {
  if (p.a.kind == ROW_NORM) return launch_ni<NW, TERMS, EPI, F16, ROW_NORM>(p, grid, st);
  if constexpr (EPI == EPI_PARTIAL) {
    if (p.a.kind == ROW_MERGE) return launch_ni<NW, TERMS, EPI, F16, ROW_MERGE>(p, grid, st);
    return launch_ni<NW, TERMS, EPI, F16, ROW_COPY>(p, grid, st);
  }
  return GOOSE_ERR_ARG;
}
template <int NW, int EPI>
int launch_type(bool f16, int terms, const RowArgs& p, dim3 grid, hipStream_t st) {
  if (terms == 2) return f16 ? launch_pro<NW, 2, EPI, true>(p, grid, st) : launch_pro<NW, 2, EPI, false>(p, grid, st);
  return f16 ? launch_pro<NW, 1, EPI, true>(p, grid, st) : launch_pro<NW, 1, EPI, false>(p, grid, st);
}

}  // namespace

bool one_row_fits(int Kpad, int ksplit, int terms) {
  const int stages = Kpad / 128, per = (stages + ksplit - 1) / ksplit;
  return per * 128 * terms * 2 <= LDS_A;
}

int launch_gemm_row_16(int dtype, int epi, const OneRow& row, int terms, const void* Wp, int Npad, int Kpad, int ksplit, void* out,
                       size_t out_split_stride, float out_scale, int32_t* flags, hipStream_t st) {
  if (dtype != GOOSE_DTYPE_BF16 && dtype != GOOSE_DTYPE_F16) return GOOSE_ERR_ARG;
  if ((Npad & 31) || (Kpad % 128) || ksplit < 1 || (terms != 1 && terms != 2) || !one_row_fits(Kpad, ksplit, terms)) return GOOSE_ERR_ARG;
  if (epi != EPI_PARTIAL && (epi != EPI_SWIGLU || ksplit != 1 || (Npad & 63))) return GOOSE_ERR_ARG;
  if (row.kind == ROW_NORM && ((row.H & 3) || row.H > ROW_MAX_HIDDEN || Kpad - row.H >= 128)) return GOOSE_ERR_ARG;
  // the same workgroups as the skinny kernel's: enough of them to fill the chip, five wavefronts where that makes one round
  const int ntiles = Npad / 32;
  const int gx5 = 256 / ksplit;
  const bool five = ((ntiles + 3) / 4) * ksplit > 256 && gx5 * 5 >= ntiles;
  const int want = epi == EPI_SWIGLU ? 256 : (256 + ksplit - 1) / ksplit;
  int gx = (ntiles + 3) / 4;
  if (gx < want) gx = want < ntiles ? want : ntiles;
  if (five) gx = gx5;
  const bool rope = row.kind == ROW_NORM && row.rope.rows > 0;
  if (gx + 1 > 65535) return GOOSE_ERR_ARG;
  const int granules = Kpad / 128, gps = (granules + ksplit - 1) / ksplit;
  if (gps * (ksplit - 1) >= granules) return GOOSE_ERR_ARG;
  const RowArgs p{(const u32x4*)Wp, ntiles, Kpad / 16, gps, gx, out_scale, out, out_split_stride, flags, row};
  const dim3 grid(ksplit, gx + (rope ? 1 : 0));
  const bool f16 = dtype == GOOSE_DTYPE_F16;
  if (epi == EPI_SWIGLU) return five ? launch_type<5, EPI_SWIGLU>(f16, terms, p, grid, st) : launch_type<4, EPI_SWIGLU>(f16, terms, p, grid, st);
  return five ? launch_type<5, EPI_PARTIAL>(f16, terms, p, grid, st) : launch_type<4, EPI_PARTIAL>(f16, terms, p, grid, st);
}
