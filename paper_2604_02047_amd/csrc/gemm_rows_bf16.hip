// Many-row GEMM of 16-bit operands (bf16 or fp16) for gfx950: out[m][n] = sum_k A[m][k] * W[n][k] for the stacked rows of a
// batch of requests, 128 < M <= 512 (the batch sweep of App. D).  Same operands and the same
// results, bit for bit, as the skinny kernel of gemm_bf16.hip (each accumulator takes its k-steps
// in ascending order there and here), but organised for the matrix cores rather than for the
// weight stream alone: with hundreds of rows a weight byte is used often enough that the pass
// sits near the ridge between HBM and MFMA, and what limits a kernel there is the operand traffic
// inside the chip (L2 -> compute unit, LDS -> registers) per matrix instruction.
//
//   * A workgroup = 8 wavefronts (two per SIMD) owns 64*MT rows x 256 columns, MT = 2, 3 or 4: the L2
//     traffic of a product falls with both sides of this tile (512 rows, 28672 x 4096: 0.9 GB with
//     256 x 256, 1.4 GB with tiles of 128 x 256), and 256 x 256 fp32 sums are half of a
//     compute unit's registers.  The wavefronts stand 2 x 4, each owning MT x 2 tiles of 32 x 32.
//   * Both operands go global -> LDS without passing registers (global_load_lds), in stages of 64
//     inputs (32 in two terms), through a ring of three slots (MT = 2: 3 x 48 KiB) or two (56, 64 KiB
//     each).  Rows of A are 128 bytes per stage; the unit (16 bytes) at position p of row r is the
//     row's unit p ^ ((r / 2) % 8), arranged by choosing which unit a lane fetches: the lanes
//     that read LDS together then meet all banks.
//   * A stage issues the copies of the stage D-1 ahead into the slot that the barrier before it
//     freed, and reads the operands of every k-step from LDS one k-step ahead of the matrix
//     instructions; one raw s_barrier per stage, behind a wait that leaves the younger copies in flight.
//   Measured (Llama-3-8B shape, by events inside a pass, 512 / 240 rows, on several cards): gate/up 120-131 / 76-78 us
//   (four-wavefront workgroups of 128 x 256 with the weights through registers: 145 / 80), down 65-70 / 42-48 (73 / 40),
//   q|k|v 40-41 / 25-26 (50 / 26), LM head 482-529 / 260-277, and 540-546 / 291-293 where it also writes the logits (the skinny kernel
//   in passes over 128 rows, logits written: 725 / 373).  1.0 PFLOP/s in gate/up at 512 rows; the parts alone: matrix instructions
//   and LDS reads 82 us (1.47 PFLOP/s, what this card sustains on such data), copies 100 us (A 45, W 62-76): the copies,
//   4 MB per compute unit at about 40 GB/s, are what bounds it.  Tried without gain: a ring of four to six slots of 32
//   inputs with the next operands read across the barrier, non-temporal weights, wave priorities, one chunk of
//   256 rows x 128 columns per workgroup (90 at 240 rows).
//   * Row chunks of one column group run on ONE XCD in neighbouring launch slots (workgroups are
//     dealt to the 8 XCDs round-robin), so the later chunks find the weights in that XCD's L2.
//   * Epilogues: fp32 split-K partials; SwiGLU; per-row (max, second, index) of the LM head.
#include <climits>
#include <type_traits>

#include "goose_internal.h"
#include "mma16.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define GOOSE_BUFFER_WORD3 0x00020000  // word 3 of a raw buffer descriptor: 32-bit untyped data, range checked
#define GOOSE_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }  // s_waitcnt vmcnt(n) only

constexpr int LGKM_0 = 15 | (7 << 4) | (3 << 14);  // s_waitcnt lgkmcnt(0) only

constexpr int NT = 2;         // column tiles per wavefront
constexpr int WG_TILES = 8;   // column tiles per workgroup (four wavefronts side by side)
static_assert(WG_TILES == GOOSE_ROWS_TILES, "the LM head's reductions are one per workgroup");

// TERMS: terms of the activation operand (gemm_bf16.hip): with two, every weight operand meets the hi
// and then the lo operand of its rows, as in the skinny kernel
template <int MT, int EPI, bool F16, int TERMS>
__global__ __launch_bounds__(512, 2) void k_gemm_rows(const typename Mma16<F16>::T* __restrict__ A, int lda,
                                                      const u32x4* __restrict__ Wp, int ntiles, int ksteps_total,
                                                      int stages_per_split, int B, void* __restrict__ out, size_t ldo,
                                                      size_t split_stride, float4* __restrict__ top2, int n_valid, int gx,
                                                      int nsplit, int nchunk, float out_scale, int32_t* __restrict__ flags) {
  typedef typename Mma16<F16>::T T;
  typedef typename Mma16<F16>::v8 op8;
  constexpr int KC = 64 / TERMS, STEPS = KC / 16;
  constexpr int ROWS = 64 * MT;                    // rows of the workgroup
  constexpr int A_BYTES = ROWS * 128, W_BYTES = WG_TILES * STEPS * 1024, SLOT = A_BYTES + W_BYTES;
  constexpr int APW = A_BYTES / 1024 / 8;         // copy instructions of A per wavefront and stage
  constexpr int CP = APW + STEPS;                  // all copy instructions of a wavefront per stage (the same for each)
  constexpr int CT_ROW = 65;                       // floats per row of the LM head's column tile (odd: conflict-free row scans)
  constexpr int TAIL = EPI == EPI_SWIGLU ? 4 * NT * 16 * 64 * 4 : (EPI == EPI_TOP2 ? 4 * 32 * CT_ROW * 4 : 0);
  constexpr int RED = EPI == EPI_TOP2 ? 8 * MT * 32 * 16 : 0;
  constexpr int D = 3 * SLOT <= 160 * 1024 ? 3 : 2;  // slots
  // The slots are separate arrays: the compiler then knows that a copy into one does not touch what is
  // read from another.  The epilogues reuse them (TAIL in the first two, RED in the third).
  __shared__ __attribute__((aligned(1024))) unsigned char lds0[SLOT > TAIL ? SLOT : TAIL];
  __shared__ __attribute__((aligned(1024))) unsigned char lds1[SLOT > TAIL ? SLOT : TAIL];
  __shared__ __attribute__((aligned(1024))) unsigned char lds2[D > 2 ? SLOT : (RED > 16 ? RED : 16)];
  auto slot_of = [&](auto slot_c) -> unsigned char* {
    constexpr int b = decltype(slot_c)::value;
    return b == 0 ? lds0 : (b == 1 ? lds1 : lds2);
  };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 2, wc = wave & 3;  // this wavefront's half of the rows, quarter of the columns

  // work item = (column group bx, split-K range by, row chunk); see the XCD note above
  const int xcd = blockIdx.x & 7, slot_id = blockIdx.x >> 3;
  const int j = slot_id / nchunk, chunk = slot_id - j * nchunk;
  const int t = j * 8 + xcd;
  if (t >= gx * nsplit) return;  // the grid is rounded up to whole groups of 8
  const int by = t / gx, bx = t - by * gx;
  const int row_base = chunk * ROWS;
  const int tile0 = bx * WG_TILES + wc * NT;

  const int nstages_total = ksteps_total / STEPS;
  const int s_begin = by * stages_per_split;
  const int s_end = min(s_begin + stages_per_split, nstages_total);
  const int nst = s_end - s_begin;  // a multiple of 2 (ranges are multiples of 128 inputs)

  f32x16 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0.f;

  // ---- copies: A instruction c of a stage fills rows 8 c .. 8 c + 7; wavefront w brings the pieces of column tile w.  Rows beyond B
  // read row B-1 and tiles beyond the last one the last tile: neither is stored.
  const u32x4* a_src[APW];
#pragma unroll
  for (int q = 0; q < APW; ++q) {
    const int c = wave * APW + q;
    const int row = c * 8 + (lane >> 3);
    const int unit = (lane & 7) ^ ((row >> 1) & 7);
    a_src[q] = reinterpret_cast<const u32x4*>(A + (size_t)min(row_base + row, B - 1) * lda) + (size_t)s_begin * 8 + unit;
  }
  const u32x4* w_src = Wp + ((size_t)min(bx * WG_TILES + wave, ntiles - 1) * ksteps_total + (size_t)s_begin * STEPS) * 64 + lane;
  auto copy = [&](int i, auto slot_c) {  // stage i of the range (beyond it: the last one again)
    const int ic = min(i, nst - 1);
    unsigned char* dst = slot_of(slot_c);
#if defined(__HIP_DEVICE_COMPILE__)  // (the host pass knows no such builtin and would silently drop the kernel's stub)
#pragma unroll
    for (int q = 0; q < APW; ++q)
      __builtin_amdgcn_global_load_lds(a_src[q] + (size_t)ic * 8, GOOSE_LDS_PTR(dst + (wave * APW + q) * 1024),
                                       16, 0, 0);
#pragma unroll
    for (int q = 0; q < STEPS; ++q)
      __builtin_amdgcn_global_load_lds(w_src + ((size_t)ic * STEPS + q) * 64,
                                       GOOSE_LDS_PTR(dst + A_BYTES + (wave * STEPS + q) * 1024), 16, 0, 0);
#else
    (void)dst;
    (void)ic;
#endif
  };
  auto barrier = [&]() {  // (raw: __syncthreads would also drain every copy in flight)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // ---- operand reads: lane l holds row l % 32 of a row tile and the eight inputs 8*(l/32).. of a k-step
  const int hh = lane >> 5, a_x = ((lane & 31) >> 1) & 7;
  const int a_row = (wr * 32 * MT + (lane & 31)) * 128;
  op8 af[2][TERMS][MT], bf[2][NT];
  auto read_ops = [&](auto slot_c, auto step_c, auto par_c) {
    constexpr int s = decltype(step_c)::value, par = decltype(par_c)::value;
    const unsigned char* src = slot_of(slot_c);
    // the reads before these were issued a k-step's matrix instructions ago: waiting for them here, by
    // hand, keeps the compiler from waiting for the ones below as well
    __builtin_amdgcn_s_waitcnt(LGKM_0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int tm = 0; tm < TERMS; ++tm) {
      const int pos = ((2 * s + hh) * TERMS + tm) ^ a_x;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) af[par][tm][mt] = *reinterpret_cast<const op8*>(src + a_row + mt * 32 * 128 + pos * 16);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      bf[par][nt] = *reinterpret_cast<const op8*>(src + A_BYTES + ((wc * NT + nt) * STEPS + s) * 1024 + lane * 16);
  };
  const std::integral_constant<int, 0> c0;
  const std::integral_constant<int, 1> c1;
  const std::integral_constant<int, 2> c2;
  const std::integral_constant<int, 3> c3;
  auto stage = [&](auto slot_c, int i) {
    constexpr int slot = decltype(slot_c)::value;
    copy(i + D - 1, std::integral_constant<int, (slot + D - 1) % D>());
    __builtin_amdgcn_sched_barrier(0);
    read_ops(slot_c, c0, c0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s == 0) read_ops(slot_c, c1, c1);
      if constexpr (STEPS == 4) {
        if (s == 1) read_ops(slot_c, c2, c0);
        if (s == 2) read_ops(slot_c, c3, c1);
      }
      if (s == STEPS - 1) __builtin_amdgcn_s_waitcnt(LGKM_0);
      __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink the reads to their use)
#pragma unroll
      for (int tm = 0; tm < TERMS; ++tm)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = Mma16<F16>::mfma(af[s & 1][tm][mt], bf[s & 1][nt], acc[mt][nt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // stage i+1 has landed once at most the copies of the stages after it are pending (copies complete in order)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((D - 2) * CP));
    barrier();
  };
  if (nst > 0) {
    copy(0, c0);
    if constexpr (D > 2) copy(1, c1);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((D - 2) * CP));
    barrier();
    int i = 0;
    for (; i + D <= nst; i += D) {
      stage(c0, i);
      stage(c1, i + 1);
      if constexpr (D > 2) stage(c2, i + 2);
    }
    if constexpr (D > 2) {
      if (i < nst) stage(c0, i);
      if (i + 1 < nst) stage(c1, i + 1);
    }
    // the copies issued by the last stages still target slots that the epilogues reuse
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    barrier();
  }

  // C layout of the 32x32 MFMA: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
  const int row_w = row_base + wr * 32 * MT;  // this wavefront's first row
  // fp32 rows of one tile, through a buffer descriptor over rows [.., B): rows beyond B are dropped
  auto store_tile = [&](float* o, int mt, int nt) {
    const int row0 = row_w + mt * 32, left = min(B - row0, 32);
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        o + (size_t)row0 * ldo, 0, left > 0 && tile0 + nt < ntiles ? (int)((unsigned)left * (unsigned)ldo * 4u) : 0, GOOSE_BUFFER_WORD3);
    const int ldo4 = (int)ldo * 4;
    const int voff = 4 * hh * ldo4 + ((tile0 + nt) * 32 + (lane & 31)) * 4;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, acc[mt][nt][r] * out_scale), rsrc, voff,
                                            (8 * (r >> 2) + (r & 3)) * ldo4, 0);
#else
    (void)o;
    (void)left;
#endif
  };
  if (EPI == EPI_PARTIAL) {
    float* o = reinterpret_cast<float*>(out) + by * split_stride;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) store_tile(o, mt, nt);
  } else if (EPI == EPI_SWIGLU) {  // every tile holds the gate rows (columns 0-15) and the up rows (16-31) of 16 outputs
    // One row tile at a time, the wavefront passes its accumulators through LDS (register r of lane l
    // at [r][l]) and walks the outputs two columns at a time in a rolled loop, as the skinny kernel
    // does: the gate values of columns 2p, 2p+1 sit at lanes 2p, 2p+1 of a half, the up values 16
    // lanes further.  (Unrolled this epilogue is tens of KB of code that runs once, at 40 ns a line.)
    T* hq = reinterpret_cast<T*>(out);
    float* mine = reinterpret_cast<float*>(wr == 0 ? lds0 : lds1) + (size_t)wc * (NT * 16 * 64);
    bool clamped = false;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      __builtin_amdgcn_wave_barrier();  // (LDS operations of one wavefront complete in order)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(nt * 16 + r) * 64 + lane] = acc[mt][nt][r] * out_scale;
      __builtin_amdgcn_wave_barrier();
#pragma unroll 1
      for (int e = lane; e < NT * 16 * 16; e += 64) {
        const int pr = e & 7, half = (e >> 3) & 1, rr = (e >> 4) & 15, nt = e >> 8;  // column pair, lane half, register, tile
        const int row = row_w + mt * 32 + 8 * (rr >> 2) + 4 * half + (rr & 3);
        const int col = (tile0 + nt) * 16 + 2 * pr;
        const float* src = &mine[(nt * 16 + rr) * 64 + half * 32 + 2 * pr];
        const float2 g = *reinterpret_cast<const float2*>(src);
        const float2 u = *reinterpret_cast<const float2*>(src + 16);
        float h0 = swiglu_f32(g.x, u.x), h1 = swiglu_f32(g.y, u.y);
        const bool keep = row < B && tile0 + nt < ntiles;
        if (F16) {  // beyond fp16: clamp, and say so (GOOSE_FLAG_RANGE)
          if (fabsf(h0) > 65504.0f) { h0 = copysignf(65504.0f, h0); clamped = clamped || keep; }
          if (fabsf(h1) > 65504.0f) { h1 = copysignf(65504.0f, h1); clamped = clamped || keep; }
        }
        if (keep) {
          const T a0 = (T)h0, a1 = (T)h1;
          T* dst = hq + (size_t)row * ldo + term_pos(TERMS, col);
          union { T t[2]; unsigned u; } pk;
          pk.t[0] = a0; pk.t[1] = a1;
          *reinterpret_cast<unsigned*>(dst) = pk.u;
          if (TERMS == 2) {
            pk.t[0] = (T)(h0 - (float)a0); pk.t[1] = (T)(h1 - (float)a1);
            *reinterpret_cast<unsigned*>(dst + 8) = pk.u;
          }
        }
      }
    }
    if (F16 && clamped && flags != nullptr) atomicOr(flags, GOOSE_FLAG_RANGE);
  } else {  // EPI_TOP2
    float* o = reinterpret_cast<float*>(out);
    float* ct = reinterpret_cast<float*>(wr == 0 ? lds0 : lds1) + wc * 32 * CT_ROW;
    float4* red = reinterpret_cast<float4*>(lds2);  // [wavefront][row]
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if (o != nullptr) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) store_tile(o, mt, nt);
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          ct[(8 * (r >> 2) + 4 * hh + (r & 3)) * CT_ROW + nt * 32 + (lane & 31)] = acc[mt][nt][r] * out_scale;
      __builtin_amdgcn_wave_barrier();
      // lane = (row, column tile): scan the tile's 32 columns in ascending order (the lowest index wins a tie)
      const int col0 = (tile0 + hh) * 32;
      const int c_end = min(32, n_valid - col0);
      const float* crow = ct + (lane & 31) * CT_ROW + hh * 32;
      float v1 = -INFINITY, v2 = -INFINITY;
      int i1 = INT_MAX;
      for (int c0 = 0; c0 < c_end; c0 += 8) {  // (eight reads in flight: 8 us off 512 x 128256)
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = crow[c0 + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = c0 + e < c_end ? v[e] : -INFINITY;
          if (x > v1) { v2 = v1; v1 = x; i1 = col0 + c0 + e; }
          else v2 = fmaxf(v2, x);
        }
      }
      // the second tile's columns follow the first's
      const float ov1 = __shfl_xor(v1, 32, 64), ov2 = __shfl_xor(v2, 32, 64);
      const int oi1 = __shfl_xor(i1, 32, 64);
      if (hh == 0) {
        if (ov1 > v1) { v2 = fmaxf(v1, ov2); v1 = ov1; i1 = oi1; }
        else v2 = fmaxf(v2, ov1);
        red[(wave * MT + mt) * 32 + (lane & 31)] = make_float4(v1, v2, __int_as_float(i1), 0.f);
      }
    }
    __syncthreads();
    if (tid < ROWS && row_base + tid < B) {
      const int half = tid / (32 * MT), in = tid - half * (32 * MT);
      const float4* e0 = red + (half * 4) * MT * 32 + in;
      float4 best = e0[0];
#pragma unroll
      for (int w = 1; w < 4; ++w) {  // column ranges ascend with w
        const float4 e = e0[w * MT * 32];
        if (e.x > best.x) { best.y = fmaxf(best.x, e.y); best.x = e.x; best.z = e.z; }
        else best.y = fmaxf(best.y, e.x);
      }
      top2[(size_t)(row_base + tid) * gx + bx] = best;
    }
  }
}

struct RowsCall {
  const void* A; int lda; const void* Wp; int Npad, Kpad, B, ksplit; void* out; size_t ldo, split_stride; void* top2; int n_valid;
  float out_scale; int32_t* flags; hipStream_t st;
};

template <int MT, int EPI, bool F16, int TERMS>
int launch_rows(const RowsCall& g) {
  const int ntiles = g.Npad / 32, ksteps = g.Kpad / 16;
  const int gx = (ntiles + WG_TILES - 1) / WG_TILES;
  const int nchunk = (g.B + 64 * MT - 1) / (64 * MT);
  const int granules = g.Kpad / 128;                        // split-K ranges are multiples of 128 inputs,
  const int gps = (granules + g.ksplit - 1) / g.ksplit;     // the same ranges as the skinny kernel's
  const dim3 grid((gx * g.ksplit + 7) / 8 * 8 * nchunk);
  hipLaunchKernelGGL((k_gemm_rows<MT, EPI, F16, TERMS>), grid, dim3(512), 0, g.st, (const typename Mma16<F16>::T*)g.A, g.lda,
                     (const u32x4*)g.Wp, ntiles, ksteps, gps * 2 * TERMS, g.B, g.out, g.ldo, g.split_stride, (float4*)g.top2,
                     g.n_valid, gx, g.ksplit, nchunk, g.out_scale, g.flags);
  return goose_launch_status();
}

template <int EPI, bool F16, int TERMS>
int launch_mt(int MT, const RowsCall& g) {
  return MT == 2 ? launch_rows<2, EPI, F16, TERMS>(g) : (MT == 3 ? launch_rows<3, EPI, F16, TERMS>(g) : launch_rows<4, EPI, F16, TERMS>(g));
}

// Height of the workgroups' tiles: the one that the fewest rounds of 256 workgroups and the least
// work per round favour.  A workgroup's time goes with MT plus about one for what does not shrink
// with it (the weights' share of the operand traffic, barriers, epilogue).
// Measured with every height forced (nine products from 1024 x 2752 to 28672 x 4096, one and two terms, 160 .. 512 rows):
// the rule's choice is the fastest of the three, within 2 %, in all 126.  28672 x 4096, MT = 2 / 3 / 4, us: 256 rows
// 78 / 107 / 108, 320 rows 124 / 103 / 126, 512 rows 135 / 179 / 122; two terms, 320 rows 205 / 170 / 217; 4096 x 14336 in
// eight K ranges, 384 rows 68 / 55 / 63, 512 rows 71 / 92 / 65.
int pick_mt(int B, int Npad, int ksplit) {
  const int groups = (Npad / 32 + WG_TILES - 1) / WG_TILES * ksplit;
  int best = 4, best_cost = INT_MAX;
  for (int mt = 4; mt >= 2; --mt) {
    const int wgs = groups * ((B + 64 * mt - 1) / (64 * mt));
    const int cost = (wgs + 255) / 256 * (mt + 1);
    if (cost < best_cost) { best_cost = cost; best = mt; }
  }
  return best;
}

template <int EPI>
int launch_any(bool f16, int terms, const RowsCall& g) {
  const int mt = pick_mt(g.B, g.Npad, g.ksplit);
  if (terms == 2) return f16 ? launch_mt<EPI, true, 2>(mt, g) : launch_mt<EPI, false, 2>(mt, g);
  return f16 ? launch_mt<EPI, true, 1>(mt, g) : launch_mt<EPI, false, 1>(mt, g);
}

}  // namespace

int launch_gemm_rows_16(int dtype, int epi, const void* A, int lda, int terms, const void* Wp, int Npad, int Kpad, int B,
                        int ksplit, void* out, size_t ldo, size_t out_split_stride, void* top2, int n_valid, float out_scale,
                        int32_t* flags, hipStream_t st) {
  if (dtype != GOOSE_DTYPE_BF16 && dtype != GOOSE_DTYPE_F16) return GOOSE_ERR_ARG;
  const bool f16 = dtype == GOOSE_DTYPE_F16;
  if (B < 1 || B > GOOSE_MAX_ROWS || (Npad & 31) || (Kpad % 128) || ksplit < 1 || (terms != 1 && terms != 2))
    return GOOSE_ERR_ARG;
  const RowsCall g{A, lda, Wp, Npad, Kpad, B, ksplit, out, ldo, out_split_stride, top2, n_valid, out_scale, flags, st};
  switch (epi) {
    case EPI_PARTIAL: return launch_any<EPI_PARTIAL>(f16, terms, g);
    case EPI_SWIGLU: return (ksplit != 1 || (Npad & 63)) ? GOOSE_ERR_ARG : launch_any<EPI_SWIGLU>(f16, terms, g);
    case EPI_TOP2: return (ksplit != 1 || !top2) ? GOOSE_ERR_ARG : launch_any<EPI_TOP2>(f16, terms, g);
  }
  return GOOSE_ERR_ARG;
}
