// Products of the target's pass over a training sequence (its features are
// what the draft trains on), up to 64 rows a launch: partial sums over K chunks
// of X[m][k] * W[n][k] on packed bf16 weights, as k_gemm.hip, with an order of
// summation of their own.
//
// A cached key or value that lies next to a rounding boundary of bfloat16 goes
// either way with the order of the sums before it, and its unit in the last
// place grows through the layers: on 13B-shaped text sequences (4 layers, 60 to
// 700 rows) two orders of the same exactness give gradients 3.0e-3 to 4.6e-3
// apart.  A trainer's gradients shall not move by that when a decode kernel is
// tuned, so this pass keeps its chunks (feature_chunk) and, inside a chunk, one
// float32 sum per element that takes, 32 columns at a time, the hi and then the
// lo product.  Longer launches run on rocBLAS (feature_blas in msd_api.hip).
//
// Bound: the weight stream; X (32 KB a block at 64 rows) goes through LDS once
// per workgroup of two 64-row tiles, so L2 serves as many bytes of X as of W.
// The next block's loads are in flight while this one is used.
// Measured (weights from HBM; us), 7B-shaped q/k/v, output, gate+up, down:
//    32 rows   24.2, 11.4, 41.7, 24.2   (2.9-4.3 TB/s of weights)
//    64 rows   29.4, 16.4, 52.8, 30.1   (2.1-3.4 TB/s)
// k_gemm takes 19.6, 9.1, 32.1, 17.7 at 27 rows and 24.4, 11.5, 38.8, 21.3 at 61; a
// training step of 70 rows (two 7B-shaped layers) takes 5.4 ms as a whole.
#include <algorithm>

#include "msd_internal.h"

namespace msd {

namespace {

constexpr int KB = 128;        // columns per packed block
constexpr int TILE_ROWS = 64;  // rows per packed block: 16 per wave
constexpr int BLOCK_ELEMS = TILE_ROWS * KB;
constexpr int NT = 2;          // tiles per workgroup

struct FeatureArgs {
  const uint16_t *X, *W, *W2;
  int ldx, M, K, n_tiles, nkt, chunk, groups;  // groups: workgroups per weight and chunk
  float* part;
  size_t part_split;
  int ldp;
};

// MT: groups of 16 rows.  Grid (groups * weights, chunks).
template <int MT>
__global__ __launch_bounds__(256) void k_feature(FeatureArgs a) {
  constexpr int UNITS = MT * 16 * 32;  // 16-byte units of a block: row m's 16 hi, then 16 lo
  constexpr int NX = UNITS / 256;
  __shared__ uint4 xs[2][UNITS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int w = blockIdx.x / a.groups, t0 = (blockIdx.x - w * a.groups) * NT;
  const int kb0 = blockIdx.y * a.chunk, kb1 = min(a.nkt, kb0 + a.chunk);
  const uint16_t* const W = w ? a.W2 : a.W;
  const auto load_w = [&](uint4 (&f)[NT][4], int kb) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int t = min(t0 + j, a.n_tiles - 1);
      const uint16_t* const p =
          W + ((size_t)t * a.nkt + kb) * BLOCK_ELEMS + wave * (BLOCK_ELEMS / 4) + lane * 8;
#pragma unroll
      for (int c = 0; c < 4; ++c) f[j][c] = *reinterpret_cast<const uint4*>(p + c * 512);
    }
  };
  const auto load_x = [&](uint4 (&x)[NX], int kb) {
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const int e = threadIdx.x + 256 * q;
      const int m = e >> 5, u = e & 31;
      const int col = kb * KB + 8 * (u & 15);
      x[q] = make_uint4(0, 0, 0, 0);
      if (m < a.M && col < a.K)
        x[q] = *reinterpret_cast<const uint4*>(a.X + (size_t)m * a.ldx + (u >> 4) * a.K + col);
    }
  };
  // unit u of row m at u ^ (m & 15): 16 lanes reading one unit of 16 rows take
  // distinct banks
  const auto store_x = [&](const uint4 (&x)[NX], uint4* s) {
#pragma unroll
    for (int q = 0; q < NX; ++q) {
      const int e = threadIdx.x + 256 * q;
      s[(e & ~31) + ((e & 31) ^ ((e >> 5) & 15))] = x[q];
    }
  };
  f32x4 acc[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 wf[NT][4], wn[NT][4], x[NX];
  load_x(x, kb0);
  load_w(wf, kb0);
  store_x(x, xs[0]);
  __syncthreads();
  for (int kb = kb0; kb < kb1; ++kb) {
    const uint4* const s = xs[(kb - kb0) & 1];
    const int next = min(kb + 1, kb1 - 1);
    load_x(x, next);
    load_w(wn, next);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          const bf16x8 f = as_bf16x8(s[(t * 16 + i) * 32 + ((h * 16 + 4 * g + c) ^ i)]);
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wf[j][c]), f, acc[j][t],
                                                                0, 0, 0);
        }
    store_x(x, xs[(kb - kb0 + 1) & 1]);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) wf[j][c] = wn[j][c];
    __syncthreads();
  }
  // C layout of the 16x16 MFMA: lane holds row m = lane & 15, register r the
  // column 4 (lane / 16) + r
  float* const part =
      a.part + (size_t)blockIdx.y * a.part_split + (size_t)w * a.n_tiles * TILE_ROWS;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    if (t0 + j >= a.n_tiles) continue;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int m = t * 16 + i;
      if (m < a.M)
        *reinterpret_cast<float4*>(part + (size_t)m * a.ldp + (t0 + j) * TILE_ROWS + wave * 16 +
                                   4 * g) =
            make_float4(acc[j][t][0], acc[j][t][1], acc[j][t][2], acc[j][t][3]);
    }
  }
}

template <int MT>
void launch_mt(const FeatureArgs& a, int nw, hipStream_t st) {
  hipLaunchKernelGGL(k_feature<MT>, dim3(a.groups * nw, (a.nkt + a.chunk - 1) / a.chunk), dim3(256),
                     0, st, a);
}

struct Split {
  int per, wgs;  // tiles per workgroup; workgroups over all chunks
};
Split split_tiles(int chunks, int n_tiles, int wgs) {
  int G = std::max(1, std::min((wgs + chunks - 1) / chunks, n_tiles));
  int per = (n_tiles + G - 1) / G;
  G = (n_tiles + per - 1) / per;
  while (chunks * G > wgs && G > 1) {
    ++per;
    G = (n_tiles + per - 1) / per;
  }
  return Split{per, chunks * G};
}

}  // namespace

// Blocks of 128 columns per partial sum of a product of M <= 64 rows: 8 for up
// to 32 rows, 4 above, times the chunks that share a sum (as many as keep 256
// workgroups, `wgs`, in work), or all of them for very wide weights.
int feature_chunk(int M, int N, int K, int nw, int wgs) {
  const bool mid = M > 16, big = M > 32;
  const int nkt = (K + KB - 1) / KB, n_tiles = (N + TILE_ROWS - 1) / TILE_ROWS;
  const int nkb = big ? 4 : 8;
  const int S1 = (nkt + nkb - 1) / nkb;
  int S = S1, nc = 1;
  const Split one = split_tiles(S1, n_tiles, wgs);
  Split cur = one;
  if (mid && S1 >= 2) {
    const Split two = split_tiles((S1 + 1) / 2, n_tiles, wgs);
    const bool busy = big ? 4 * two.wgs >= 3 * wgs
                          : nw == 2 || (two.per >= 4 && 20 * two.wgs >= 19 * one.wgs);
    if (two.per <= 5 && busy) {
      nc = 2;
      S = (S1 + 1) / 2;
      cur = two;
    }
  }
  if (!big) return nkb * nc;
  if (nw == 1) {
    const int nt = ((n_tiles + wgs - 1) / wgs + 1) / 2 * 2;
    if (nt >= 8 && nt <= 10) return nkt;
    if (cur.per <= 2) {
      const int half = feature_chunk(32, N, K, nw, wgs / 2);
      if (half == 8) return half;
    }
  }
  for (int n = 4; n >= 3; --n) {
    const int Sn = (S1 + n - 1) / n;
    if (Sn >= S) continue;
    const Split sn = split_tiles(Sn, n_tiles, wgs);
    const bool keep = nw == 2 ? 4 * sn.wgs >= 3 * wgs : sn.per >= 4 && 20 * sn.wgs >= 19 * cur.wgs;
    if (sn.per <= (nw == 2 ? 4 : 5) && keep) return nkb * n;
  }
  return nkb * nc;
}

size_t feature_part_floats(int M, int N, int K, int nw) {
  const int nkt = (K + KB - 1) / KB, chunk = feature_chunk(M, N, K, nw);
  return (size_t)((nkt + chunk - 1) / chunk) * M * ((N + TILE_ROWS - 1) / TILE_ROWS) * TILE_ROWS * nw;
}

Parts launch_feature_gemm(const uint16_t* X, int ldx, int M, const uint16_t* W, const uint16_t* W2,
                          int N, int K, float* part, hipStream_t st) {
  const int nw = W2 ? 2 : 1;
  FeatureArgs a{};
  a.X = X;
  a.W = W;
  a.W2 = W2;
  a.ldx = ldx;
  a.M = M;
  a.K = K;
  a.n_tiles = (N + TILE_ROWS - 1) / TILE_ROWS;
  a.nkt = (K + KB - 1) / KB;
  a.chunk = feature_chunk(M, N, K, nw);
  a.groups = (a.n_tiles + NT - 1) / NT;
  a.part = part;
  a.ldp = a.n_tiles * TILE_ROWS * nw;
  a.part_split = (size_t)M * a.ldp;
  if (M <= 16) launch_mt<1>(a, nw, st);
  else if (M <= 32) launch_mt<2>(a, nw, st);
  else launch_mt<4>(a, nw, st);
  return Parts{part, (a.nkt + a.chunk - 1) / a.chunk, a.part_split, a.ldp, a.n_tiles * TILE_ROWS};
}

}  // namespace msd
