// GEMM of the decode, prompt and training-target paths on gfx950 MFMA:
// P_s[m][n] = sum over K chunk s of X[m][k] * W[n][k], W in bfloat16 (packed,
// see below), X as split rows (bf16 hi + lo).
//
// Packed weights.  A weight [N][K] is stored as 64-row tiles times 128-column
// blocks, each block 16 KB in the order in which fragments are read: block
// (t, kb) at element ((t * nkt) + kb) * 8192, inside it
// ((g16 * 4 + c) * 64 + lane) * 8 + e holds W[t*64 + g16*16 + (lane & 15)]
// [kb*128 + 32*(lane >> 4) + 8*c + e].  Rows past N and columns past K are
// zero.  Within one MFMA the K index may be any permutation shared by the two
// operands; the X fragments use the same one.
//
// X arrives split by its producer, x = hi + lo with hi = bf16(x) and
// lo = bf16(x - hi), so W x = W hi + W lo carries about 16 significant bits of
// the activations (one bf16 rounding of every GEMM input, amplified by a deep
// stack of layers, is far larger than the error of the weights' products).
#include <hip/hip_ext.h>

#include <algorithm>

#include "msd_internal.h"

namespace msd {

namespace {

constexpr int KB = 128;        // K elements per packed block
constexpr int TILE_ROWS = 64;  // W rows per packed block
constexpr int BLOCK_ELEMS = TILE_ROWS * KB;
constexpr int BLOCK_BYTES = BLOCK_ELEMS * 2;
constexpr int RSRC_RAW = 0x00020000;  // raw buffer: 32-bit data format, stride 0
constexpr int PAST = (int)0x80000000u;  // a byte offset past every buffer

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// The kernel's arguments (the split: see GemmPlan).
struct GemmArgs {
  const uint16_t *X, *W, *W2;
  int ldx, M, K;
  int n_tiles, nkt;    // 64-row tiles and 128-column blocks of W
  int n_mt, n_nt, nw;  // row tiles, column tiles per weight, weights
  int S, bps;          // K chunks, blocks per chunk
  int fold;            // blocks per sum (see the kernel)
  float* part;
  size_t part_split;
  int ldp, off2;
  ArgmaxOut am;
  // EPI_SUM: columns [0, N) of each weight's products, plus add when given
  // (rows of ldp floats, as part)
  const float* add;
  int N;
  size_t wplane;  // elements between the planes of a weight (TW > 1)
};

// What a workgroup does with its sums: store them as partials, or (K whole in
// one chunk) reduce each row to its best column (the LM head of a verify) or
// store them added to a matrix (the training products).
enum Epilogue { EPI_PART, EPI_ARGMAX, EPI_SUM };

// Products of an operand pair given as TX and TW bf16 terms of falling size:
// term i of X with term (plane) p of W for i + p < TX, the rest being below
// the last bit of the sum's largest terms.
MSD_DEV constexpr int n_products(int TX, int TW) {
  int n = 0;
  for (int p = 0; p < TW; ++p) n += TX - p;
  return n;
}

MSD_DEV constexpr int vmcnt_imm(int n) { return 0x0f70 | (n & 15) | ((n >> 4) << 14); }

// A workgroup of four waves computes 32 MT rows of X against 128 NTW rows of
// W; each wave owns 32 NTW of them.  K runs in half blocks of 64 columns:
//  - W fragments go from the packed layout straight to registers (a 64-row x
//    128-column block holds the 16-byte units of a fragment contiguously, and
//    no two waves of the workgroup share one); a register ring of RD half
//    blocks keeps them in flight, each step refilled once its MFMAs are done;
//  - the X rows of a half block go to LDS by buffer loads with the lds bit,
//    one half block ahead (two buffers), or three ahead (NB = 4) where the
//    weight stream is the bound: loads complete in order, so waiting for X
//    one half ahead also drained the ring's older loads (27 rows, 7B-shaped
//    down 19.9 -> 17.3 us, output 8.7 -> 7.8 us).
//    LDS row m holds eight 16-byte units, unit u at u ^ (m & 7): the eight
//    rows that one quarter of an operand read touches fall into distinct
//    banks.  A load instruction writes 64 consecutive units (eight rows), so
//    the swizzle is in the lanes' source addresses;
//  - the fragments of step c + 1 are read from LDS under the MFMAs of step c,
//    one read between MFMAs.
// The LDS buffers are separate arrays and the loads into them are buffer
// loads: the compiler then knows that the reads of one buffer need not wait
// for the loads into the other (global loads to LDS count as flat accesses
// and make it wait for everything in flight).  One barrier per half block:
// before it every wave waits for its own loads into the next buffer; loads
// issued after them stay in flight.
//
// Addresses.  Raw buffer loads check voffset against the record count less
// soffset, so soffset always stays inside the buffer and whatever may fall
// outside is in voffset: rows past M (the record count ends at row M),
// columns past K and blocks past the chunk (voffset 2^31) read zeros.
//
// Sums.  Every add to a float32 sum rounds at the sum's size, so the error of a
// product grows with the root of the adds that one accumulator takes (2.5e-8 of
// the result's root mean square per root of an add of 16 columns, measured).
// The accumulators therefore take `fold` blocks of 128 columns (sum_blocks) and
// are then added to sums of their own.  Where the registers allow it (tiles of up
// to 32 x 256 or 64 x 128 per workgroup, where K can be as short as a block) the
// lo products, 2^-8 of the hi ones, have accumulators of their own too.
// Against float64, K = 4096, one chunk: 5.7e-7 in one accumulator, 2.0e-7 folded
// every four blocks, 2.6e-7 every seven; K = 256: 1.4e-7 -> 0.7e-7; K = 11008:
// 9.7e-7 -> 2.0e-7 and 2.6e-7.  The fold costs a tile of 128 x 256 (accumulators
// in the upper half of the register file, three moves and an add each) 3 to 6%,
// the smaller ones up to 2%.  Tiles with more sums than 128 registers a lane have
// no room for a second set.
//
// K chunks are summed by the consumer in chunk order.
//
// POL: cache policy of the weight loads.  A weight that only one row tile
// reads is streamed non-temporally (policy 2: 27 rows, 7B-shaped gate+up
// 35 -> 32 us); with more row tiles their reads meet in L2 (policy 0).
//
// Measured (one launch, weights from HBM; us), 7B-shaped q/k/v, output, gate+up,
// down, unfolded (with tiles of up to 128 x 512) -> folded:
//    27 rows    18.9,  8.6,  31.7,  18.0 ->  19.6,  9.1,  32.1,  17.7
//    61 rows    24.1, 10.5,  38.0,  21.5 ->  24.4, 11.5,  38.8,  21.3
//   108 rows    30.5, 11.9,  51.0,  30.2 ->  36.2, 12.2,  55.7,  29.6
//   624 rows   109.9, 41.4, 188.4, 102.9 -> 112.1, 42.2, 208.4,  98.2  (0.99-1.15 PFLOP/s)
//  1600 rows   282,   99,   460,   231   -> 269,  101,   527,   267    (1.06-1.20 PFLOP/s)
// Bound: HBM up to about 100 rows, then the matrix cores.
//
// TX, TW: terms of X and of W.  The decode and prompt paths have TX = 2 (hi and
// lo) and bf16 weights (TW = 1).  The training products have float32 operands
// as three terms each, h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), 24
// bits in all (k_train.hip): X rows of 3K, W as three packed planes, and the
// six products down to 2^-16 of the first; or three terms against the bf16 LM
// head.
template <int MT, int NTW, int OCC, int POL, int RD, int NB, int EPI, int TX = 2, int TW = 1>
__global__ __launch_bounds__(256, OCC) void k_gemm(GemmArgs a) {
  static_assert(NB == 2 || (NB == 4 && RD >= 2), "the first waits count on the ring's loads");
  constexpr int XD = NB - 1;          // half blocks that X is loaded ahead
  constexpr int BM = 32 * MT;
  constexpr int UNITS = TX * BM * 8;  // 16-byte units of a half block of X
  constexpr int ND = UNITS / 256;     // loads to LDS per wave and half block
  static_assert(UNITS % 256 == 0, "X units divide over the waves");
  constexpr int DPS = (ND + 1) / 2;   // of them per step (in steps 0 and 1)
  // the rows of term 0, then of term 1, ..., 8 units each
  __shared__ u32x4 xs0[UNITS];
  __shared__ u32x4 xs1[UNITS];
  __shared__ u32x4 xs2[NB > 2 ? UNITS : 1];
  __shared__ u32x4 xs3[NB > 2 ? UNITS : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroup i runs on XCD i mod 8: every XCD takes a contiguous range of
  // the work items, row tiles innermost, so that the row tiles that read one
  // piece of W run on one XCD and meet in its L2.
  const int items = a.n_mt * a.n_nt * a.nw * a.S;
  const int per = (items + 7) >> 3;
  int t = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (((int)blockIdx.x >> 3) >= per || t >= items) return;
  const int mt = t % a.n_mt;
  t /= a.n_mt;
  const int s = t % a.S;
  t /= a.S;
  const int w = t / a.n_nt, nt = t - w * a.n_nt;
  const int m0 = mt * BM;
  const int kb0 = s * a.bps, kb1 = min(a.nkt, kb0 + a.bps);
  const int K = a.K, nkt = a.nkt;
  __amdgpu_buffer_rsrc_t rw[TW];
#pragma unroll
  for (int p = 0; p < TW; ++p)
    rw[p] = __builtin_amdgcn_make_buffer_rsrc((void*)((w ? a.W2 : a.W) + p * a.wplane), 0,
                                              a.n_tiles * nkt * BLOCK_BYTES, RSRC_RAW);
  const int rowb = a.ldx * 2;
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(a.X + (size_t)m0 * a.ldx), 0, min(a.M - m0, BM) * rowb, RSRC_RAW);
  const int r = lane & 31, h = lane >> 5;
  // MFMA step (sp, c) of a block takes the columns 64 sp + 32 h + 8 c + 0..7
  // from lane half h; the unit of W row r lies at (16-row group, c, row in
  // the group + 16 * column group 2 sp + h)
  const int wvo = ((r >> 4) * 256 + (r & 15) + 16 * h) * 16;
  const int n32 = (nt * 4 + wave) * NTW;  // first 32-row group of the wave
  int wso[NTW];
#pragma unroll
  for (int j = 0; j < NTW; ++j) {
    // groups past the weight (discarded) read its first tile
    const int q = (n32 + j) >> 1 < a.n_tiles ? n32 + j : 0;
    wso[j] = (q >> 1) * nkt * BLOCK_BYTES + (q & 1) * (BLOCK_BYTES / 2);
  }
  const auto load_w = [&](int kb, int sp, int c, int j, int p) {
    const int kc = min(kb, kb1 - 1);
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                         rw[p], kb < kb1 ? wvo : PAST,
                                         wso[j] + kc * BLOCK_BYTES + c * 1024 + sp * 512, POL));
  };
  // Load q of a wave fills the eight rows of group wave ND + q (groups run
  // through the rows of term 0, then of term 1, ...), lane i the unit i & 7 of
  // row i >> 3, i.e. source unit (i & 7) ^ (i >> 3).
  const int xu = (lane & 7) ^ (lane >> 3);
  const int xvo = (lane >> 3) * rowb + xu * 16;
  const auto load_x = [&](u32x4* b, int q, int kb, int sp) {
    const int k0 = min(kb, kb1 - 1) * KB + sp * 64;
    const int g = wave * ND + q, term = g / (BM / 8), rg = g - term * (BM / 8);
    const int vo = (kb < kb1 && k0 + 8 * xu < K) ? xvo + rg * 8 * rowb : PAST;
    // the last half block may begin past K: soffset stays inside the buffer
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rx, (__attribute__((address_space(3))) void*)(b + g * 64), 16, vo,
        2 * (term * K + min(k0, K - 8)), 0, 0);
  };
  constexpr int NW = NTW * TW;  // weight loads per step
  u32x4 wr[RD][4][NW];
  // acc: the running sums; low: those of the products below the first, where
  // they have their own (256 columns of three terms: relative error 2.4e-7 in one
  // sum, 0.8e-7 in two; a float32 GEMM 1.5e-7); sum: what has been folded
  constexpr bool LOW = TX == 3 || MT * NTW <= 2;
  constexpr bool FOLD = EPI != EPI_SUM && TX == 2;
  f32x16 acc[NTW][MT], low[LOW ? NTW : 1][LOW ? MT : 1], sum[FOLD ? NTW : 1][FOLD ? MT : 1];
#pragma unroll
  for (int j = 0; j < NTW; ++j)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[j][m][e] = 0.f;
        if constexpr (LOW) low[j][m][e] = 0.f;
        if constexpr (FOLD) sum[j][m][e] = 0.f;
      }
#pragma unroll
  for (int q = 0; q < ND; ++q) load_x(xs0, q, kb0, 0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (NB > 2) {
#pragma unroll
    for (int q = 0; q < ND; ++q) load_x(xs1, q, kb0, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < ND; ++q) load_x(xs2, q, kb0 + 1, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int d = 0; d < RD; ++d)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < NW; ++j) wr[d][c][j] = load_w(kb0 + d / 2, d & 1, c, j % NTW, j / NTW);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(vmcnt_imm((XD - 1) * ND + 4 * NW * RD));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  u32x4 fx[2][TX][MT];  // X fragments of two steps
  const auto frags = [&](const u32x4* b, int c) {
    const int u = r * 8 + ((4 * h + c) ^ (r & 7));
#pragma unroll
    for (int t = 0; t < TX; ++t)
#pragma unroll
      for (int m = 0; m < MT; ++m) fx[c & 1][t][m] = b[t * BM * 8 + m * 256 + u];
  };
  // Half block sp of block kb (X in b), loading the X of XD halves further
  // into bn and refilling ring half rd with the W of RD halves further.
  const auto half = [&](const u32x4* b, u32x4* bn, int rd, int kb, int sp) {
    const int xkb = kb + (sp + XD) / 2, xsp = (sp + XD) & 1;
    const int wkb = kb + (sp + RD) / 2, wsp = (sp + RD) & 1;
    frags(b, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c < 3) frags(b, c + 1);
#pragma unroll
      for (int q = c * DPS; q < (c + 1) * DPS && q < ND; ++q) load_x(bn, q, xkb, xsp);
      if (c > 0) {
#pragma unroll
        for (int j = 0; j < NW; ++j) wr[rd][c - 1][j] = load_w(wkb, wsp, c - 1, j % NTW, j / NTW);
      }
#pragma unroll
      for (int t = 0; t < TX; ++t)
#pragma unroll
        for (int p = 0; p < TW; ++p) {
          if (t + p >= TX) continue;
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < NTW; ++j) {
              f32x16& to = LOW && t + p > 0 ? low[LOW ? j : 0][LOW ? m : 0] : acc[j][m];
              to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  __builtin_bit_cast(bf16x8, wr[rd][c][p * NTW + j]),
                  __builtin_bit_cast(bf16x8, fx[c & 1][t][m]), to, 0, 0, 0);
            }
        }
      // one LDS read and at most one load between groups of MFMAs
      constexpr int GROUP = n_products(TX, TW) * NTW / TX;
      const int loads = (c < 2 ? DPS : 0) + (c > 0 ? NW : 0);
#pragma unroll
      for (int i = 0; i < TX * MT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, GROUP, 0);
        if (c < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (i < loads) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < NW; ++j) wr[rd][3][j] = load_w(wkb, wsp, 3, j % NTW, j / NTW);
    __builtin_amdgcn_sched_barrier(0);
    // The next half's X was loaded XD - 1 halves ago, by the end of step 1:
    // the refills of steps 2 and 3 and those after step 3 (3 NW loads) and
    // all loads of the halves since came later and may stay in flight.
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * NW + (XD - 1) * (ND + 4 * NW)));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int left = a.fold;  // blocks until the sums are folded
  const auto fold = [&] {
    if constexpr (FOLD) {
      if (--left > 0) return;
      left = a.fold;
#pragma unroll
      for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            if constexpr (LOW) {
              acc[j][m][e] += low[j][m][e];
              low[j][m][e] = 0.f;
            }
            sum[j][m][e] += acc[j][m][e];
            acc[j][m][e] = 0.f;
          }
    }
  };
  if constexpr (NB == 2) {
#pragma unroll 1
    for (int kb = kb0; kb < kb1; ++kb) {
      half(xs0, xs1, 0, kb, 0);
      half(xs1, xs0, 1 % RD, kb, 1);
      fold();
    }
  } else {
#pragma unroll 1
    for (int kb = kb0; kb < kb1; kb += 2) {
      half(xs0, xs3, 0, kb, 0);
      half(xs1, xs0, 1, kb, 1);
      fold();
      if (kb + 1 >= kb1) break;
      half(xs2, xs1, 2 % RD, kb + 1, 0);
      half(xs3, xs2, 3 % RD, kb + 1, 1);
      fold();
    }
  }
  if constexpr (LOW || FOLD) {
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if constexpr (LOW) acc[j][m][e] += low[j][m][e];
          if constexpr (FOLD) acc[j][m][e] += sum[j][m][e];
        }
  }
  // C layout of the 32x32 MFMA: lane holds row m = lane & 31, register e the
  // column 8 (e / 4) + 4 (lane / 32) + e % 4
  if constexpr (EPI == EPI_PART) {
    float* const part = a.part + (size_t)s * a.part_split + (size_t)w * a.off2;
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
      if ((n32 + j) >> 1 >= a.n_tiles) continue;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int row = m0 + m * 32 + r;
        if (row >= a.M) continue;
        float* const d = part + (size_t)row * a.ldp + (n32 + j) * 32 + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(d + 8 * q) = make_float4(
              acc[j][m][4 * q], acc[j][m][4 * q + 1], acc[j][m][4 * q + 2], acc[j][m][4 * q + 3]);
      }
    }
  } else if constexpr (EPI == EPI_SUM) {
    const size_t wo = (size_t)w * a.off2;
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const int row = m0 + m * 32 + r;
        if (row >= a.M) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = (n32 + j) * 32 + 8 * q + 4 * h;  // N is a multiple of 4
          if (n >= a.N) continue;
          const size_t o = (size_t)row * a.ldp + wo + n;
          float4 v = make_float4(acc[j][m][4 * q], acc[j][m][4 * q + 1], acc[j][m][4 * q + 2],
                                 acc[j][m][4 * q + 3]);
          if (a.add) {
            const float4 d = *reinterpret_cast<const float4*>(a.add + o);
            v = make_float4(v.x + d.x, v.y + d.y, v.z + d.z, v.w + d.w);
          }
          *reinterpret_cast<float4*>(a.part + o) = v;
        }
      }
  } else {
    // the best (value, id) of each row over the workgroup's columns, as
    // candidate nt of the row; a NaN ranks as -inf, the lowest id wins ties
    __shared__ float sv[4][BM];
    __shared__ int si[4][BM];
    const int V = a.am.V;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int row = m0 + m * 32 + r;
      float* const lg = a.am.logits && row < a.M ? a.am.logits + (size_t)row * V : nullptr;
      float bv = -INFINITY;
      int bi = NO_ID;
#pragma unroll
      for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = (n32 + j) * 32 + 8 * q + 4 * h;
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[j][m][4 * q + e];
          if (lg && a.am.vec) {  // V and the rows are multiples of 16 bytes
            if (n < V) *reinterpret_cast<float4*>(lg + n) = make_float4(v[0], v[1], v[2], v[3]);
          } else if (lg) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n + e < V) lg[n + e] = v[e];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = v[e] == v[e] ? v[e] : -INFINITY;
            if (n + e < V && better(x, n + e, bv, bi)) {
              bv = x;
              bi = n + e;
            }
          }
        }
      const float ov = __shfl_xor(bv, 32);
      const int oi = __shfl_xor(bi, 32);
      if (better(ov, oi, bv, bi)) {
        bv = ov;
        bi = oi;
      }
      if (h == 0) {
        sv[wave][m * 32 + r] = bv;
        si[wave][m * 32 + r] = bi;
      }
    }
    lds_barrier();
    if ((int)threadIdx.x < BM && m0 + (int)threadIdx.x < a.M) {
      float bv = sv[0][threadIdx.x];
      int bi = si[0][threadIdx.x];
#pragma unroll
      for (int q = 1; q < 4; ++q)
        if (better(sv[q][threadIdx.x], si[q][threadIdx.x], bv, bi)) {
          bv = sv[q][threadIdx.x];
          bi = si[q][threadIdx.x];
        }
      const size_t o = (size_t)(m0 + threadIdx.x) * a.n_nt + nt;
      a.am.cand_v[o] = bv;
      a.am.cand_i[o] = bi;
    }
  }
}

// One thread per 16-byte unit of the packed layout.
__global__ void k_pack(const uint16_t* src, int N, int K, int nkt, size_t units, uint16_t* dst) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= units) return;
  const int lane = (int)(q & 63);
  const size_t r = q >> 6;  // (t * nkt + kb) * 16 + wave * 4 + c
  const int c = (int)(r & 3), wave = (int)((r >> 2) & 3);
  const size_t blk = r >> 4;
  const int kb = (int)(blk % nkt);
  const int t = (int)(blk / nkt);
  const int row = t * TILE_ROWS + wave * 16 + (lane & 15);
  const int col = kb * KB + 32 * (lane >> 4) + 8 * c;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < N && col < K) v = *reinterpret_cast<const uint4*>(src + (size_t)row * K + col);
  *reinterpret_cast<uint4*>(dst + q * 8) = v;
}

// The inverse of k_pack: row-major bf16 [N][K] from the packed layout.
__global__ void k_unpack(const uint16_t* src, int N, int K, int nkt, size_t units, uint16_t* dst) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= units) return;
  const int lane = (int)(q & 63);
  const size_t r = q >> 6;
  const int c = (int)(r & 3), wave = (int)((r >> 2) & 3);
  const size_t blk = r >> 4;
  const int kb = (int)(blk % nkt);
  const int t = (int)(blk / nkt);
  const int row = t * TILE_ROWS + wave * 16 + (lane & 15);
  const int col = kb * KB + 32 * (lane >> 4) + 8 * c;
  if (row < N && col < K)
    *reinterpret_cast<uint4*>(dst + (size_t)row * K + col) =
        *reinterpret_cast<const uint4*>(src + q * 8);
}

MSD_DEV uint4 load_stream(const uint16_t* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Streaming read of a buffer with the weight stream's access pattern: every
// wave instruction reads 1 KB contiguous with nontemporal loads, four in
// flight per lane per step, workgroups striding over 64 KB spans.  The XOR
// of everything read keeps the loads alive; a workgroup writes one word only
// if it equals a value the data never produce here (zero-filled buffers).
__global__ __launch_bounds__(256) void k_stream_read(const uint16_t* buf, size_t spans,
                                                     unsigned* sink) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint4 acc = make_uint4(0, 0, 0, 0);
  for (size_t sp = blockIdx.x; sp < spans; sp += gridDim.x) {
    const uint16_t* b = buf + sp * (size_t)(4 * BLOCK_ELEMS) + (size_t)wave * (BLOCK_ELEMS / 4) +
                        lane * 8;
    uint4 v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = load_stream(b + (q / 4) * BLOCK_ELEMS + (q % 4) * 512);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      acc.x ^= v[q].x;
      acc.y ^= v[q].y;
      acc.z ^= v[q].z;
      acc.w ^= v[q].w;
    }
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u) sink[blockIdx.x] = 1u;
}

// The launch function of one kernel variant.
template <int MT, int NTW, int OCC, int RD, int NB>
void launch_cfg(const GemmArgs& a, int wgs, const GemmScratch& sc, hipStream_t st) {
  const dim3 grid(8 * ((wgs + 7) / 8));
  // with timing events the launch carries them in its dispatch packet, so
  // they bracket the kernel's execution only
  const auto go = [&](void (*k)(GemmArgs)) {
    if (sc.ev_start)
      hipExtLaunchKernelGGL(k, grid, dim3(256), 0, st, sc.ev_start, sc.ev_stop, 0, a);
    else
      hipLaunchKernelGGL(k, grid, dim3(256), 0, st, a);
  };
  constexpr int MANY = MT == 1 ? 2 : 0;  // cache policy with several row tiles
  if (a.am.cand_v)
    go(a.n_mt == 1 ? k_gemm<MT, NTW, OCC, 2, RD, NB, EPI_ARGMAX>
                   : k_gemm<MT, NTW, OCC, MANY, RD, NB, EPI_ARGMAX>);
  else
    go(a.n_mt == 1 ? k_gemm<MT, NTW, OCC, 2, RD, NB, EPI_PART>
                   : k_gemm<MT, NTW, OCC, MANY, RD, NB, EPI_PART>);
}

// The variants.  eff: the share of a CU's matrix peak that one workgroup
// reaches on it, fitted to back-to-back launches of nine weight shapes at 17 row
// counts (1 to 2048); larger tiles wait for less per MFMA, but the folds of the
// largest are not hidden by a second workgroup.
struct Config {
  int MT, NTW;
  float eff;
  void (*launch)(const GemmArgs&, int, const GemmScratch&, hipStream_t);
};
constexpr Config CONFIGS[] = {
    {1, 1, 0.271f, launch_cfg<1, 1, 4, 2, 4>}, {1, 2, 0.37f, launch_cfg<1, 2, 2, 2, 4>},
    {2, 1, 0.511f, launch_cfg<2, 1, 2, 2, 4>}, {2, 2, 0.566f, launch_cfg<2, 2, 2, 2, 2>},
    {2, 4, 0.602f, launch_cfg<2, 4, 1, 1, 2>}, {3, 2, 0.639f, launch_cfg<3, 2, 1, 1, 2>},
    {4, 1, 0.505f, launch_cfg<4, 1, 2, 1, 2>}, {4, 2, 0.652f, launch_cfg<4, 2, 1, 1, 2>}};
constexpr int N_CONFIGS = sizeof(CONFIGS) / sizeof(CONFIGS[0]);
constexpr int CUS = 256;

// Blocks per accumulator: an eighth of K, four to eight for the widest weights
// (1.4e-7 to 2.0e-7 against float64); from 320 rows on, where folds are the least
// hidden, a quarter of K and up to seven (1.8e-7 to 2.7e-7).  The library products
// that prompts of more than 128 rows once ran on kept hi and lo sums apart and cut
// K in slices of 1,024 columns or more: 1.9e-7 (output, 320 rows) to 6.3e-7 (down,
// K = 18,944, 624 rows).
int sum_blocks(const Config& c, int M, int nkt) {
  if (M > 320) return std::clamp(nkt / 4, 1, 7);
  return std::clamp(nkt / 8, 1, c.MT * c.NTW <= 2 ? 8 : 4);
}

}  // namespace

size_t stream_span_bytes() { return (size_t)4 * BLOCK_ELEMS * sizeof(uint16_t); }

void launch_stream_read(const uint16_t* buf, size_t spans, int wgs, unsigned* sink,
                        hipStream_t st) {
  hipLaunchKernelGGL(k_stream_read, dim3(wgs), dim3(256), 0, st, buf, spans, sink);
}

void launch_unpack(const uint16_t* src, int N, int K, uint16_t* dst, hipStream_t st) {
  const int nkt = (K + KB - 1) / KB;
  const size_t units = packed_elems(N, K) / 8;
  hipLaunchKernelGGL(k_unpack, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, src, N, K,
                     nkt, units, dst);
}

size_t packed_elems(int N, int K) {
  return (size_t)((N + TILE_ROWS - 1) / TILE_ROWS) * ((K + KB - 1) / KB) * BLOCK_ELEMS;
}

void launch_pack(const uint16_t* src, int N, int K, uint16_t* dst, hipStream_t st) {
  const int nkt = (K + KB - 1) / KB;
  const size_t units = packed_elems(N, K) / 8;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, src, N, K,
                     nkt, units, dst);
}

// Picks the tile and the number of K chunks with the least estimated time:
// the larger of the busiest CU's time (whole workgroups, each its MFMA cycles
// at 2.4 GHz over the variant's eff plus 1.65 us to fill and drain), the
// matrix rate of the whole chip (about 2 PFLOP/s) and the weight stream,
// plus the partials' writing and their reading by the consumer.  On the 153
// (shape, rows) pairs it was fitted to, its choice costs 0.9% over the best
// variant measured for the pair on average, 10% at worst.
GemmPlan plan_gemm(int M, int N, int K, int nw, size_t max_part) {
  GemmPlan best{};
  float best_us = 0.f;
  const int nkt = (K + KB - 1) / KB, n_tiles = (N + TILE_ROWS - 1) / TILE_ROWS;
  const int ldp = n_tiles * TILE_ROWS * nw;
  const float weight_us = (float)N * K * nw * 2.f / 9.7e6f + 2.5f;
  for (int ci = 0; ci < N_CONFIGS; ++ci) {
    const Config& c = CONFIGS[ci];
    const int n_mt = (M + 32 * c.MT - 1) / (32 * c.MT);
    const int fold = sum_blocks(c, M, nkt);
    // up to 64 rows the one row tile that just holds them, so that the weights
    // pass through a CU once
    const int fit = (M + 31) / 32;
    if (M <= 64 ? c.MT != fit : c.MT < 2) continue;
    // 32-bit byte offsets within a row tile
    if (c.MT > 2 && (size_t)32 * c.MT * 4 * K >= ((size_t)1 << 31)) continue;
    const int n_nt = (n_tiles * TILE_ROWS + 128 * c.NTW - 1) / (128 * c.NTW);
    for (int s = 1; s <= MAX_K_CHUNKS && s <= nkt; ++s) {
      const int bps = (nkt + s - 1) / s, S = (nkt + bps - 1) / bps;
      if (S != s) continue;
      if (s > 1 && (bps < 3 || (size_t)s * M * ldp > max_part)) break;
      const int items = n_mt * n_nt * nw * s;
      const float wg_us = bps * 8 * 2 * c.MT * c.NTW * 32 / (2400.f * c.eff) + 1.65f;
      const float cu_us = (items + CUS - 1) / CUS * wg_us;
      const float chip_us = (float)items * (c.MT * 32) * (c.NTW * 128) * (bps * 128.f) * 4e-6f / 2006.f;
      const float part_us = (float)s * M * ldp * (1.0e-6f + 0.8e-6f) + 0.13f * s;
      const float us = std::max({cu_us, chip_us, weight_us}) + part_us;
      if (best_us == 0.f || us < best_us) {
        best_us = us;
        best = GemmPlan{ci, n_mt, n_nt, n_tiles, nkt, S, bps, fold, items, ldp, n_tiles * TILE_ROWS};
      }
    }
  }
  return best;
}

void launch_gemm(const GemmPlan& pl, const uint16_t* X, int ldx, int M, const uint16_t* W,
                 const uint16_t* W2, int K, float* part, const GemmScratch& sc, hipStream_t st,
                 const ArgmaxOut* am) {
  GemmArgs a{};
  if (am) a.am = *am;
  a.X = X;
  a.ldx = ldx;
  a.M = M;
  a.K = K;
  a.W = W;
  a.W2 = W2;
  a.n_tiles = pl.n_tiles;
  a.nkt = pl.nkt;
  a.n_mt = pl.n_mt;
  a.n_nt = pl.n_nt;
  a.nw = W2 ? 2 : 1;
  a.S = pl.S;
  a.bps = pl.bps;
  a.fold = pl.fold;
  a.part = part;
  a.part_split = (size_t)M * pl.ldp;
  a.ldp = pl.ldp;
  a.off2 = pl.off2;
  CONFIGS[pl.config].launch(a, pl.items, sc, st);
}

namespace {

// C = add + the sum of S partials, four columns per thread.
__global__ __launch_bounds__(256) void k_sum_parts(const float* part, int S, size_t split, int ldp,
                                                   int N, const float* add, float* C, int ldc) {
  const int n = 4 * (blockIdx.x * 256 + threadIdx.x);
  if (n >= N) return;
  const size_t o = (size_t)blockIdx.y * ldc + n;
  float4 v = add ? *reinterpret_cast<const float4*>(add + o) : make_float4(0.f, 0.f, 0.f, 0.f);
  const float* p = part + (size_t)blockIdx.y * ldp + n;
  for (int q = 0; q < S; ++q) {
    const float4 x = *reinterpret_cast<const float4*>(p + q * split);
    v = make_float4(v.x + x.x, v.y + x.y, v.z + x.z, v.w + x.w);
  }
  *reinterpret_cast<float4*>(C + o) = v;
}

template <int MT, int NTW, int TX, int TW>
void launch_sum_cfg(const GemmArgs& a, int items, bool part, hipStream_t st) {
  const dim3 grid(8 * ((items + 7) / 8));
  constexpr int OCC = 1;
  if (part)
    hipLaunchKernelGGL((k_gemm<MT, NTW, OCC, 0, 1, 2, EPI_PART, TX, TW>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_gemm<MT, NTW, OCC, 0, 1, 2, EPI_SUM, TX, TW>), grid, dim3(256), 0, st, a);
}

template <int TX, int TW>
void launch_sum_terms(int MT, const GemmArgs& a, int items, bool part, hipStream_t st) {
  if (MT == 4) launch_sum_cfg<4, 2, TX, TW>(a, items, part, st);
  else launch_sum_cfg<2, 2, TX, TW>(a, items, part, st);
}

}  // namespace

// The training products: two tile heights, K split while the tiles leave CUs
// idle and the partials fit.  The estimate is plan_gemm's, with the eff of kernels
// that do not fold.
void launch_gemm_sum(const SumGemm& g, hipStream_t st) {
  const int nkt = (g.K + KB - 1) / KB;
  // a plane's byte offsets are 32-bit: wider matrices go in column ranges
  const size_t tile_bytes = (size_t)nkt * BLOCK_BYTES;
  const int max_n = (int)std::min<size_t>(((((size_t)1 << 31) - 1) / tile_bytes) * TILE_ROWS, 1 << 30);
  for (int n0 = 0; n0 < g.N; n0 += max_n) {
    const int N = std::min(max_n, g.N - n0);
    const int n_tiles = (N + TILE_ROWS - 1) / TILE_ROWS, ldp = n_tiles * TILE_ROWS;
    int np = 0;
    for (int p = 0; p < g.TW; ++p) np += g.TX - p;
    int best_mt = 4, best_bps = nkt;
    float best_us = 0.f;
    for (int MT : {4, 2}) {
      const int n_mt = (g.M + 32 * MT - 1) / (32 * MT), n_nt = (ldp + 255) / 256;
      for (int s = 1; s <= MAX_K_CHUNKS && s <= nkt; ++s) {
        const int bps = (nkt + s - 1) / s;
        if ((nkt + bps - 1) / bps != s) continue;
        if (s > 1 && (bps < 4 || g.M > 65535 || (size_t)s * g.M * ldp > g.max_part)) break;
        const int items = n_mt * n_nt * s;
        const float wg_us = bps * 8 * np * MT * 2 * 32 / (2400.f * (MT == 4 ? 0.74f : 0.56f)) + 1.9f;
        const float us = (items + CUS - 1) / CUS * wg_us + (s > 1 ? s + 1 : 1) * (float)g.M * ldp * 1.8e-6f;
        if (best_us == 0.f || us < best_us) {
          best_us = us;
          best_mt = MT;
          best_bps = bps;
        }
      }
    }
    GemmArgs a{};
    a.X = g.X;
    a.ldx = g.TX * g.K;
    a.M = g.M;
    a.K = g.K;
    a.W = g.W + (size_t)(n0 / TILE_ROWS) * nkt * BLOCK_ELEMS;
    a.wplane = g.wplane;
    a.n_tiles = n_tiles;
    a.nkt = nkt;
    a.n_mt = (g.M + 32 * best_mt - 1) / (32 * best_mt);
    a.n_nt = (ldp + 255) / 256;
    a.nw = 1;
    a.bps = best_bps;
    a.S = (nkt + best_bps - 1) / best_bps;
    a.N = N;
    const bool parts = a.S > 1;
    a.part = parts ? g.part : g.C + n0;
    a.ldp = parts ? ldp : g.ldc;
    a.part_split = (size_t)g.M * ldp;
    a.add = g.add ? g.add + n0 : nullptr;
    const int items = a.n_mt * a.n_nt * a.S;
    if (g.TW == 3) launch_sum_terms<3, 3>(best_mt, a, items, parts, st);
    else if (g.TX == 3) launch_sum_terms<3, 1>(best_mt, a, items, parts, st);
    else launch_sum_terms<2, 1>(best_mt, a, items, parts, st);
    if (parts)
      hipLaunchKernelGGL(k_sum_parts, dim3((N + 1023) / 1024, g.M), dim3(256), 0, st, g.part, a.S,
                         a.part_split, ldp, N, a.add, g.C + n0, g.ldc);
  }
}

}  // namespace msd
