// Many-row GEMM of 16-bit operands (bf16 or fp16) for gfx950: out[m][n] = sum_k A[m][k] * W[n][k] for the stacked rows of a
// batch of requests, 128 < M <= 512 (the batch sweep of App. D).  Same operands and the same
// results, bit for bit, as the skinny kernel of gemm_bf16.hip (each accumulator takes its k-steps
// in ascending order there and here), but organised for the matrix cores rather than for the
// weight stream alone: with hundreds of rows a weight byte is used often enough that the pass
// sits near the ridge between HBM and MFMA, and what limits a kernel there is the operand traffic
// inside the chip (L2 -> compute unit, LDS -> registers) per matrix instruction.
//
//   * A workgroup = 4 wavefronts (one per SIMD, side by side) owns 32*MT rows x 256 columns, MT = 4, 6 or 8; each
//     wavefront owns all the rows and two column tiles, i.e. MT x 2 tiles of 32 x 32.  The L2 traffic of a product falls
//     with both sides of the workgroup's tile (512 rows, 28672 x 4096: 0.9 GB with 256 x 256, 1.4 GB with 128 x 256).
//     One wavefront per SIMD has 512 registers: up to 256 hold sums, 64 two stages of weights.
//   * The weights go straight to the registers of the one wavefront that uses them (they are stored in operand
//     order), refilled right after the matrix instructions that consumed them.  The rows of A, which all four
//     wavefronts read, go global -> LDS without passing registers (raw buffer loads to LDS) into a ring of four slots
//     of one stage each (64 inputs, 32 in two terms; 128 bytes a row).  The unit (16 bytes) at position p of row r is the row's
//     unit p ^ ((r / 2) % 8), arranged by choosing which unit a lane fetches: the lanes that read LDS together then meet all banks.
//     A and W both through LDS, as eight wavefronts did, is 256 KB of LDS traffic per stage of 64 inputs at 256 rows; this is 160.
//   * Stage j issues the copies of stage j+3 and the weights of stage j+2, and reads the operands of every sub-step
//     (k-step, term) a sub-step ahead, those of stage j+1's first one across the barrier.  One raw s_barrier per stage, behind a
//     wait that leaves the loads of one stage in flight.  Reads, copies and loads are placed between
//     matrix instructions, each of which leaves 28 clocks to issue something else in: with one wavefront per SIMD
//     a burst of them stops the matrix cores (512 rows: 116 -> 108 us for gate/up; at 128 rows a workgroup bursts are 4 % faster).
//   * The sums stand transposed in the registers (weights as the first operand of the matrix instruction): a lane holds four neighbouring
//     columns of one row, and the epilogues are short (below).
//   * The K range is the fastest index of the work items, then the column group, and the row chunks of one
//     item run on ONE XCD in neighbouring launch slots (workgroups are dealt to the 8 XCDs round-robin): an XCD with one
//     of eight K ranges fetches an eighth of A, and later chunks find the weights in its L2.  Column groups fastest, each
//     XCD fetched all of A (7 MB for the down projection at 256 rows, more than its L2).  The order alone, in this kernel:
//     passes of 16 / 8 requests over 8 layers 3206 / 2022 us, column groups fastest 3360 / 2065.
//   Measured (Llama-3-8B shape, kernel trace inside a pass, 512 / 240 rows; in brackets eight wavefronts with both operands through LDS):
//   gate/up 104-106 / 74 us (124 / 75), q|k|v 34 / 23 (38 / 23), LM head with logits 446-466 / 278 (538 / 281).  Whole passes over 8 layers, both
//   kernels in turn on one card: 16 requests of 32 rows 3083 us (3358), 12 2421 (2623), 10 2255 (2535), 8 1874-1956 (0.99-1.02 times as
//   fast), 6 1732 (1768), 5 1700 (1765); six in two terms 2194 (2452).  Cards differ by 5 % with their power limits.
//   What bounds it, 512 rows of gate/up: loop 88-93 us, of which matrix
//   instructions and LDS reads alone are 77 (1.5 PFLOP/s, what this card sustains on such data), prologue 2.4, epilogue 6.
//   256 rows: loop 59, 45 with the weights in L2, 39 with no loads at all: the weight stream (4 TB/s) and the
//   matrix instructions overlap in part only, whatever the depth of the rings (four stages of weights and eight slots: 59).
//   Epilogues: fp32 split-K partials; SwiGLU; per-row (max, second, index) of the LM head.
#include <climits>
#include <type_traits>

#include "goose_internal.h"
#include "mma16.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// (rows of the results start at any multiple of four bytes)
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

#define GOOSE_BUFFER_WORD3 0x00020000  // word 3 of a raw buffer descriptor: 32-bit untyped data, range checked
#define GOOSE_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }  // s_waitcnt vmcnt(n) only

#define GOOSE_C(n) std::integral_constant<int, (n)>()

constexpr int LGKM_0 = 15 | (7 << 4) | (3 << 14);  // s_waitcnt lgkmcnt(0) only

constexpr int NT = 2;         // column tiles per wavefront
constexpr int WAVES = 4;      // wavefronts per workgroup
constexpr int WG_TILES = 8;   // column tiles per workgroup (four wavefronts side by side)
static_assert(WG_TILES == GOOSE_ROWS_TILES, "the LM head's reductions are one per workgroup");

// TERMS: terms of the activation operand (gemm_bf16.hip): with two, every weight operand meets the hi
// and then the lo operand of its rows, as in the skinny kernel
// STREAM: the weights come through non-temporal loads (see launch_rows)
template <int MT, int EPI, bool F16, int TERMS, bool STREAM>
__global__ __launch_bounds__(256, 1) void k_gemm_rows(const typename Mma16<F16>::T* __restrict__ A, int lda,
                                                      const u32x4* __restrict__ Wp, int ntiles, int ksteps_total,
                                                      int stages_per_split, int B, void* __restrict__ out, size_t ldo,
                                                      size_t split_stride, float4* __restrict__ top2, int n_valid, int gx,
                                                      int nsplit, int nchunk, float out_scale, int32_t* __restrict__ flags) {
  typedef typename Mma16<F16>::T T;
  typedef typename Mma16<F16>::v8 op8;
  constexpr int STEPS = 4 / TERMS;                 // k-steps (16 inputs) per stage
  constexpr int ROWS = 32 * MT;                    // rows of the workgroup
  constexpr int SLOT = ROWS * 128;                 // bytes of A per stage
  constexpr int APW = SLOT / 1024 / WAVES;         // copy instructions of A per wavefront and stage
  constexpr int WPS = STEPS * NT;                  // weight loads per wavefront and stage
  constexpr int CT_ROW = 68;                       // floats per row of the epilogues' 32 x 64 tile (16-byte reads of 16 rows meet all banks)
  static_assert(32 * CT_ROW * 4 <= SLOT, "the epilogue's tiles lie in the slots");
  constexpr int D = 4;                             // slots of A
  constexpr int DW = 2;                            // stages of weights in registers
  // The slots are separate arrays: the compiler then knows that a copy into one does not touch what is
  // read from another.  The epilogues reuse them.
  __shared__ __attribute__((aligned(1024))) unsigned char lds0[SLOT];
  __shared__ __attribute__((aligned(1024))) unsigned char lds1[SLOT];
  __shared__ __attribute__((aligned(1024))) unsigned char lds2[SLOT];
  __shared__ __attribute__((aligned(1024))) unsigned char lds3[SLOT];
  auto slot_of = [&](auto slot_c) -> unsigned char* {
    constexpr int b = decltype(slot_c)::value;
    return b == 0 ? lds0 : (b == 1 ? lds1 : (b == 2 ? lds2 : lds3));
  };
  __shared__ float4 red[EPI == EPI_TOP2 ? WAVES * ROWS : 1];  // per-wavefront records of the LM head
  auto slot_of_wave = [&](int w) -> unsigned char* { return w == 0 ? lds0 : (w == 1 ? lds1 : (w == 2 ? lds2 : lds3)); };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // work item = (column group bx, split-K range by, row chunk); see the XCD note above
  const int xcd = blockIdx.x & 7, slot_id = blockIdx.x >> 3;
  const int j = slot_id / nchunk, chunk = slot_id - j * nchunk;
  const int t = j * 8 + xcd;
  if (t >= gx * nsplit) return;  // the grid is rounded up to whole groups of 8
  const int bx = t / nsplit, by = t - bx * nsplit;
  const int row_base = chunk * ROWS;
  const int tile0 = bx * WG_TILES + wave * NT;

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

  // ---- copies: instruction c of a stage fills rows 8 c .. 8 c + 7.  The wavefront's rows are read through a descriptor that ends at row B: rows beyond it are zeros.  (The unit that lane i
  // fetches depends on the parity of c only: two offsets in registers serve all the copies.)
  int a_off[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int row = (wave * APW + q) * 8 + (lane >> 3);
    const int unit = (lane & 7) ^ ((row >> 1) & 7);
    a_off[q] = (int)((unsigned)(lane >> 3) * (unsigned)lda * 2u + (unsigned)unit * 16u);
  }
#if defined(__HIP_DEVICE_COMPILE__)
  const int a_row0 = row_base + wave * APW * 8;
  const long a_bytes = (long)max(min(B - a_row0, APW * 8), 0) * lda * 2;
  const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>(A) + (size_t)a_row0 * lda, 0, (int)(unsigned)min(a_bytes, 0xFFFFFFFFl), GOOSE_BUFFER_WORD3);
#endif
  auto copy = [&](int i, auto slot_c, auto lo_c, auto hi_c) {  // copies lo .. hi - 1 of A of stage i (beyond the range: the last one again)
    constexpr int lo = decltype(lo_c)::value, hi = decltype(hi_c)::value;
    const int ic = min(i, nst - 1);
    unsigned char* dst = slot_of(slot_c);
#if defined(__HIP_DEVICE_COMPILE__)  // (the host pass knows no such builtin and would silently drop the kernel's stub)
#pragma unroll
    for (int q = lo; q < hi; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(arsrc, GOOSE_LDS_PTR(dst + (wave * APW + q) * 1024), 16, a_off[q & 1],
                                               (int)((unsigned)(q * 8) * (unsigned)lda * 2u) + (s_begin + ic) * 128, 0, 0);
#else
    (void)dst;
    (void)ic;
#endif
  };
  // ---- weights: this wavefront's two column tiles, through descriptors that cover its K range only (loads beyond it return
  // zeros and cost no memory traffic).  Tiles beyond the last one read the last tile and are not stored.
  u32x4 wreg[DW][STEPS][NT];
#if defined(__HIP_DEVICE_COMPILE__)
  __amdgpu_buffer_rsrc_t wrsrc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    wrsrc[nt] = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<u32x4*>(Wp + ((size_t)min(tile0 + nt, ntiles - 1) * ksteps_total + (size_t)s_begin * STEPS) * 64), 0,
        (nst > 0 ? nst : 0) * STEPS * 1024, GOOSE_BUFFER_WORD3);
#endif
  const int w_lane = lane * 16;
  auto load_w = [&](int i, int s, auto slot_c) {
    constexpr int slot = decltype(slot_c)::value;
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      wreg[slot][s][nt] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc[nt], w_lane, (i * STEPS + s) * 1024, STREAM ? 2 : 0);
#endif
  };
  auto barrier = [&]() {  // (raw: __syncthreads would also drain every copy in flight)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // ---- operand reads: lane l holds row l % 32 of a row tile and the eight inputs 8*(l/32).. of a k-step
  const int hh = lane >> 5, a_x = ((lane & 31) >> 1) & 7;
  const int a_row = (lane & 31) * 128;
  op8 af[2][MT];
  auto read_ops = [&](auto slot_c, auto sub_c, auto par_c) {  // sub-step = (k-step, term)
    constexpr int sub = decltype(sub_c)::value, par = decltype(par_c)::value;
    const unsigned char* src = slot_of(slot_c);
    const int pos = ((2 * (sub / TERMS) + hh) * TERMS + sub % TERMS) ^ a_x;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) af[par][mt] = *reinterpret_cast<const op8*>(src + a_row + mt * 32 * 128 + pos * 16);
  };
  // Loads complete in order as far as the wait counter goes.  Before the barrier that ends stage j, A of stage j+2 (issued in
  // stage j-1; the last sub-step of stage j+1 reads it) and the weights of stage j+1 (issued in stage j-1) must
  // have landed: everything but the PER loads of stage j itself.
  constexpr int PER = APW + WPS;
  static_assert(D == 4 && DW == 2 && PER <= 63, "wait counter");
  constexpr bool SPREAD = MT > 4;  // copies between the matrix instructions instead of at the start of a stage (see above)
  auto stage = [&](auto slot_c, auto live_c, int i) {  // (not live: what it needs is there, and nothing is issued)
    constexpr int slot = decltype(slot_c)::value, wslot = slot % DW;
    constexpr bool live = decltype(live_c)::value;
    if constexpr (live && !SPREAD) {
      copy(i + D - 1, GOOSE_C((slot + D - 1) % D), GOOSE_C(0), GOOSE_C(APW));
      __builtin_amdgcn_sched_barrier(0);
    }
    auto sub_step = [&](auto u_c) {
      constexpr int u = decltype(u_c)::value, s = u / TERMS;
      constexpr bool load = live && u % TERMS == TERMS - 1;
      // the reads before these were issued a sub-step's matrix instructions ago: waiting for them here, by
      // hand, keeps the compiler from waiting for the ones below as well
      __builtin_amdgcn_s_waitcnt(LGKM_0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (u < 3) read_ops(slot_c, GOOSE_C(u + 1), GOOSE_C((u + 1) & 1));
      else read_ops(GOOSE_C((slot + 1) % D), GOOSE_C(0), GOOSE_C(0));
      constexpr int c_lo = u * APW / 4, c_hi = (u + 1) * APW / 4, NC = live && SPREAD ? c_hi - c_lo : 0;
      if constexpr (NC > 0) copy(i + D - 1, GOOSE_C((slot + D - 1) % D), GOOSE_C(c_lo), GOOSE_C(c_hi));
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][nt] = Mma16<F16>::mfma(__builtin_bit_cast(op8, wreg[wslot][s][nt]), af[u & 1][mt], acc[mt][nt]);
      if constexpr (load) load_w(i + DW, s, GOOSE_C(wslot));
#pragma unroll
      for (int q = 0; q < MT; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      constexpr int NV = SPREAD ? NC + (load ? 1 : 0) : 0;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, MT - NV, 0);
      if constexpr (load) __builtin_amdgcn_sched_group_barrier(0x010, SPREAD ? 1 : 2, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    sub_step(GOOSE_C(0));
    sub_step(GOOSE_C(1));
    sub_step(GOOSE_C(2));
    sub_step(GOOSE_C(3));
    if constexpr (live) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(PER));
      barrier();
    }
  };
  auto copy_stage = [&](int i, auto slot_c) { copy(i, slot_c, GOOSE_C(0), GOOSE_C(APW)); };
  auto load_stage = [&](int i, auto slot_c) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s) load_w(i, s, slot_c);
  };
  const std::true_type yes;
  const std::false_type no;
  int i = 0;
  if (nst >= D) {
    // the rings are filled in the order the stages themselves would have issued these loads
    auto fill = [&](auto v_c) {  // what stage v < 0 issues
      constexpr int v = decltype(v_c)::value;
      if constexpr (v + D - 1 >= 0) copy_stage(v + D - 1, GOOSE_C(v + D - 1));
      if constexpr (v + DW >= 0) load_stage(v + DW, GOOSE_C(v + DW));
      __builtin_amdgcn_sched_barrier(0);
    };
    fill(GOOSE_C(-3));
    fill(GOOSE_C(-2));
    fill(GOOSE_C(-1));
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(PER));
    barrier();
    read_ops(GOOSE_C(0), GOOSE_C(0), GOOSE_C(0));
    do {
      stage(GOOSE_C(0), yes, i);
      stage(GOOSE_C(1), yes, i + 1);
      stage(GOOSE_C(2), yes, i + 2);
      stage(GOOSE_C(3), yes, i + 3);
      i += D;
    } while (i + D <= nst);
  } else if (nst > 0) {  // two stages
    copy_stage(0, GOOSE_C(0));
    copy_stage(1, GOOSE_C(1));
    load_stage(0, GOOSE_C(0));
    load_stage(1, GOOSE_C(1));
  }
  // every copy has landed: what is left of the range (two stages or none) lies in the rings
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  barrier();
  if (i < nst) {
    if (i == 0) read_ops(GOOSE_C(0), GOOSE_C(0), GOOSE_C(0));
    stage(GOOSE_C(0), no, i);
    stage(GOOSE_C(1), no, i + 1);
  }
  barrier();  // (the epilogues reuse the slots)

  // ---- epilogues.  Register r of lane l holds row l%32, column 8*(r/4) + 4*(l/32) + r%4 of its 32 x 32 tile.  One row
  // tile at a time the wavefront leaves its 32 x 64 sums in LDS, row by row, in eight 16-byte writes, and reads them back as the
  // results want them: stores of 16 bytes a lane, 256 contiguous bytes a row.  The loop over the row tiles is rolled: only the
  // eight writes exist once per row tile (their registers are fixed), the rest once.  (Code that runs once is
  // fetched at 40 ns a 64-byte line; unrolled over 256 sums the SwiGLU epilogue took 17 us, this takes 6.  Partial sums stored
  // without LDS, 32 bytes a row at a time: 16-22 us instead of 7.)
  float* ct = reinterpret_cast<float*>(slot_of_wave(wave));
  auto dump = [&](auto mt_c) {
    constexpr int mt = decltype(mt_c)::value;
    if constexpr (mt < MT) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int a = 0; a < 4; ++a)
          *reinterpret_cast<f32x4*>(ct + (lane & 31) * CT_ROW + nt * 32 + 8 * a + 4 * hh) =
              f32x4{acc[mt][nt][4 * a], acc[mt][nt][4 * a + 1], acc[mt][nt][4 * a + 2], acc[mt][nt][4 * a + 3]};
      asm volatile("; row tile %0" ::"n"(mt));  // (keeps the cases apart: merged, the sums would be moved together first)
    }
  };
  bool clamped = false;
#pragma unroll 1
  for (int mt = 0; mt < MT; ++mt) {
    const int row0 = row_base + mt * 32;
    if (row0 >= B) break;
    __builtin_amdgcn_wave_barrier();  // (LDS operations of one wavefront complete in order)
    switch (mt) {
      case 0: dump(GOOSE_C(0)); break;
      case 1: dump(GOOSE_C(1)); break;
      case 2: dump(GOOSE_C(2)); break;
      case 3: dump(GOOSE_C(3)); break;
      case 4: dump(GOOSE_C(4)); break;
      case 5: dump(GOOSE_C(5)); break;
      case 6: dump(GOOSE_C(6)); break;
      case 7: dump(GOOSE_C(7)); break;
    }
    __builtin_amdgcn_wave_barrier();
    if (EPI == EPI_PARTIAL || (EPI == EPI_TOP2 && out != nullptr)) {
      // 16 lanes per row, four rows at a time
      float* o = reinterpret_cast<float*>(out) + by * split_stride + (size_t)tile0 * 32 + (lane & 15) * 4;
      const float* src = ct + (lane >> 4) * CT_ROW + (lane & 15) * 4;
      const bool col_ok = tile0 + ((lane & 15) >> 3) < ntiles;
      f32x4 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = *reinterpret_cast<const f32x4*>(src + q * 4 * CT_ROW);
      __builtin_amdgcn_sched_barrier(0);  // (all reads in flight)
      float* po = o + (size_t)(row0 + (lane >> 4)) * ldo;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (col_ok && row0 + q * 4 + (lane >> 4) < B) *reinterpret_cast<f32x4_a4*>(po) = v[q] * out_scale;
        po += 4 * ldo;
      }
    }
    if (EPI == EPI_SWIGLU) {
      // every tile holds the gate rows (columns 0-15) and the up rows (16-31) of 16 outputs; lane = (row, tile)
      const int row = row0 + (lane & 31), tile = tile0 + hh;
      const float* src = ct + (lane & 31) * CT_ROW + hh * 32;
      const bool keep = row < B && tile < ntiles;
      T* dst = reinterpret_cast<T*>(out) + (size_t)row * ldo + (size_t)tile * 16 * TERMS;
      f32x4 gu[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) gu[q] = *reinterpret_cast<const f32x4*>(src + q * 4);
      __builtin_amdgcn_sched_barrier(0);  // (all reads in flight)
      float h[16], big = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          h[q * 4 + e] = swiglu_f32(gu[q][e] * out_scale, gu[4 + q][e] * out_scale);
          big = fmaxf(big, fabsf(h[q * 4 + e]));
        }
      }
      if (F16 && __builtin_amdgcn_ballot_w64(big > 65504.0f) != 0) {  // beyond fp16: clamp, and say so (GOOSE_FLAG_RANGE)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (fabsf(h[e]) > 65504.0f) h[e] = copysignf(65504.0f, h[e]);
        clamped = clamped || (keep && big > 65504.0f);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // a group of eight columns
        op8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          hi[e] = (T)h[q * 8 + e];
          if (TERMS == 2) lo[e] = (T)(h[q * 8 + e] - (float)(T)h[q * 8 + e]);
        }
        if (keep) {
          *reinterpret_cast<u32x4_a4*>(dst + q * 8 * TERMS) = __builtin_bit_cast(u32x4, hi);
          if (TERMS == 2) *reinterpret_cast<u32x4_a4*>(dst + q * 16 + 8) = __builtin_bit_cast(u32x4, lo);
        }
      }
    }
    if (EPI == EPI_TOP2) {
      // lane = (row, column tile): scan the tile's 32 columns in ascending order (the lowest index wins a tie)
      const int col0 = (tile0 + hh) * 32;
      const int c_end = min(32, n_valid - col0);
      const float* crow = ct + (lane & 31) * CT_ROW + hh * 32;
      float v1 = -INFINITY, v2 = -INFINITY;
      int i1 = INT_MAX;
#pragma unroll 1
      for (int c0 = 0; c0 < c_end; c0 += 16) {  // (sixteen columns in flight)
        f32x4 v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const f32x4*>(crow + c0 + e * 4);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float x = c0 + e < c_end ? v[e >> 2][e & 3] * out_scale : -INFINITY;
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
        red[wave * ROWS + mt * 32 + (lane & 31)] = make_float4(v1, v2, __int_as_float(i1), 0.f);
      }
    }
  }
  if (EPI == EPI_SWIGLU && F16 && clamped && flags != nullptr) atomicOr(flags, GOOSE_FLAG_RANGE);
  if (EPI == EPI_TOP2) {
    __syncthreads();
    if (tid < ROWS && row_base + tid < B) {
      float4 best = red[tid];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) {  // column ranges ascend with w
        const float4 e = red[w * ROWS + tid];
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

template <int MT, int EPI, bool F16, int TERMS, bool STREAM>
int launch_rows_as(const RowsCall& g) {
  const int ntiles = g.Npad / 32, ksteps = g.Kpad / 16;
  const int gx = (ntiles + WG_TILES - 1) / WG_TILES;
  const int nchunk = (g.B + 32 * MT - 1) / (32 * MT);
  const int granules = g.Kpad / 128;                        // split-K ranges are multiples of 128 inputs,
  const int gps = (granules + g.ksplit - 1) / g.ksplit;     // the same ranges as the skinny kernel's
  const dim3 grid((gx * g.ksplit + 7) / 8 * 8 * nchunk);
  hipLaunchKernelGGL((k_gemm_rows<MT, EPI, F16, TERMS, STREAM>), grid, dim3(256), 0, g.st, (const typename Mma16<F16>::T*)g.A, g.lda,
                     (const u32x4*)g.Wp, ntiles, ksteps, gps * 2 * TERMS, g.B, g.out, g.ldo, g.split_stride, (float4*)g.top2,
                     g.n_valid, gx, g.ksplit, nchunk, g.out_scale, g.flags);
  return goose_launch_status();
}

// Non-temporal weights leave the lines of A in the L2 alone, and the chunks of an item run side by side, so the later ones still find
// the weights there.  The loads of 28672 x 4096 at 256 / 512 rows on their own (copies, no arithmetic) take 53.5 / 61.6 us, plain 56.3 / 67.0; the
// product 65.8 / 102.7 (69.4 / 105.6), O, down and q|k|v 0.5-1.5 us less each; passes of 16 / 14 / 12 / 8 / 7 requests over 8 layers, prefix 500, 2764 /
// 2617 / 2318 / 1870 / 1806 us (plain throughout 2776 / 2632 / 2353 / 1894 / 1835), 7 in two terms 2404 (2426).  A short last chunk has little of A to copy and
// runs ahead of the others, whose weights then have left the L2 again: below three quarters of the height they are loaded plainly.  Passes of 5 / 6 /
// 9 / 10 requests and of five of 48 nodes 1682 / 1748 / 2122 / 2203 / 2169 us, non-temporal throughout 1750 / 1765 / 2291 / 2259 / 2225, plain
// throughout 1706 / 1767 / 2124 / 2202 / 2172; 11 requests (352 rows, the last chunk five sixths full) 2263, 2261, 2282.
template <int MT, int EPI, bool F16, int TERMS>
int launch_rows(const RowsCall& g) {
  constexpr int H = 32 * MT;
  const int last = g.B - (g.B - 1) / H * H;
  if (g.B > H && 4 * last < 3 * H) return launch_rows_as<MT, EPI, F16, TERMS, false>(g);
  return launch_rows_as<MT, EPI, F16, TERMS, true>(g);
}

template <int EPI, bool F16, int TERMS>
int launch_mt(int MT, const RowsCall& g) {
  return MT == 2 ? launch_rows<4, EPI, F16, TERMS>(g) : (MT == 3 ? launch_rows<6, EPI, F16, TERMS>(g) : launch_rows<8, EPI, F16, TERMS>(g));
}

// Height of the workgroups' tiles in units of 64 rows: the one that the fewest rounds of 256 workgroups and the least
// work per round favour.  A workgroup's time goes with its height plus about one unit for what does not shrink
// with it (the weights, barriers, epilogue).
// Measured with every height forced, 128 / 192 / 256 rows, us: 28672 x 4096 at 256 rows 72 / 75 / 91, 320 rows 107 / 81 / 94, 512
// rows 115 / 145 / 103; 35840 x 6656, 192 rows 172 / 130 / 133, 384 rows 187 / 233 / 254; LM head of 128256 x 4096, 192 rows
// 279 / 236 / 248, 512 rows 502 / 521 / 473.  Of 54 products (seven shapes, 160 .. 512 rows) the rule's is the fastest in 46; the
// others are split-K products with eight ranges, where several workgroups of 128 rows share a unit (up to 20 % in
// a loop over that product alone).  Inside a pass of 16 requests, where the rule gives O and down 256 rows, 128 rows for
// them make the pass 1.4 % slower (3247 against 3202 us, 8 layers); with 256 rows in all the rule takes 128 for them itself.
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
