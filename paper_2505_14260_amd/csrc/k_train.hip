// Kernels of the draft-head training step (Sec. 4.2) in float32: the
// teacher-forced draft layer over a training sequence, its loss (regression
// toward the next target feature plus the token cross-entropy against the
// target's next-token distribution) and the backward pass, and the AdamW
// update.  The contractions over the weights run on the library's bf16 GEMM
// with float32 operands as three bf16 terms (launch_gemm_sum; the terms are made
// here), the per-head attention products on rocBLAS in float32; these kernels do
// everything between them.  Row-major throughout; a training pass has
// R = n - 1 rows (positions 0 .. n-2).
#include <algorithm>

#include "msd_internal.h"

namespace msd {

namespace {

constexpr int TB = 256;

MSD_DEV float bsum(float v, float* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

MSD_DEV float bmax(float v, float* sh) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// The three bf16 terms x = h + m + l of a float (see split8).
MSD_DEV void split3(float v, uint16_t (&t)[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    t[q] = f2bf(v);
    // an infinite or NaN value has no remainder
    v = fabsf(bf2f(t[q])) < INFINITY ? v - bf2f(t[q]) : 0.f;
  }
}
// Element k of a row of three terms, K elements each.
MSD_DEV void put_terms(uint16_t* row, int K, int k, float v) {
  uint16_t t[3];
  split3(v, t);
#pragma unroll
  for (int q = 0; q < 3; ++q) row[(size_t)q * K + k] = t[q];
}

// Row i < n: H[i] = target feature (split row hi + lo); for i < R also
// X0[i] = [h_i | e_{i+1}] and E0[i] = the draft input of a visual row i:
// e_i, or h_i with visual_feature (the Visual Feature variant), where e is
// the token embedding (text) or the visual row vis_idx (visual).  Grid (n),
// block TB.
__global__ __launch_bounds__(TB) void k_tr_inputs(const uint16_t* h, const uint16_t* E,
                                                  const int* tok, const int* vis_idx,
                                                  const uint16_t* visual, int n, int d,
                                                  int visual_feature, float* H, float* X0,
                                                  float* E0, uint16_t* xs) {
  const int i = blockIdx.x;
  const int R = n - 1;
  const uint16_t* hr = h + (size_t)i * 2 * d;
  const int vi = vis_idx[i];
  const uint16_t* er = vi >= 0 ? visual + (size_t)vi * d : E + (size_t)tok[i] * d;
  for (int k = threadIdx.x; k < d; k += TB) {
    const float hv = bf2f(hr[k]) + bf2f(hr[d + k]);
    H[(size_t)i * d + k] = hv;
    if (i < R) {
      X0[(size_t)i * 2 * d + k] = hv;
      put_terms(xs + (size_t)i * 6 * d, 2 * d, k, hv);
      E0[(size_t)i * d + k] = visual_feature ? hv : bf2f(er[k]);
    }
    if (i > 0) {
      X0[(size_t)(i - 1) * 2 * d + d + k] = bf2f(er[k]);
      put_terms(xs + (size_t)(i - 1) * 6 * d, 2 * d, d + k, bf2f(er[k]));
    }
  }
}

// Visual rows take E0 as the draft input (Eq. decouple: their embedding, or
// their target feature in the Visual Feature variant).
__global__ __launch_bounds__(TB) void k_tr_visual_rows(float* F, const float* E0,
                                                       const int* vis_idx, int d) {
  const int i = blockIdx.x;
  if (vis_idx[i] < 0) return;
  for (int k = threadIdx.x; k < d; k += TB) F[(size_t)i * d + k] = E0[(size_t)i * d + k];
}

// Zeroes the rows of dF that are visual (they do not pass through f_down).
__global__ __launch_bounds__(TB) void k_tr_zero_visual(float* dF, const int* vis_idx, int d) {
  const int i = blockIdx.x;
  if (vis_idx[i] < 0) return;
  for (int k = threadIdx.x; k < d; k += TB) dF[(size_t)i * d + k] = 0.f;
}

// Y = x / sqrt(mean(x^2) + eps) * g and its terms, rstd[i] saved.  Grid (R).
__global__ __launch_bounds__(TB) void k_tr_rmsnorm(const float* X, const float* g, float eps,
                                                   int d, float* Y, float* rstd, uint16_t* xs) {
  __shared__ float sh[4];
  const int i = blockIdx.x;
  const float* x = X + (size_t)i * d;
  float s = 0.f;
  for (int k = threadIdx.x; k < d; k += TB) s += x[k] * x[k];
  s = bsum(s, sh);
  const float r = rsqrtf(s / (float)d + eps);
  if (threadIdx.x == 0) rstd[i] = r;
  for (int k = threadIdx.x; k < d; k += TB) {
    const float y = x[k] * r * g[k];
    Y[(size_t)i * d + k] = y;
    put_terms(xs + (size_t)i * 3 * d, d, k, y);
  }
}

// dX = base + the gradient of the RMSNorm input given dY (per row), with
// y = x r g, r = (mean(x^2) + eps)^-1/2: dx = r (g dy) - x r^3 mean(x g dy).
__global__ __launch_bounds__(TB) void k_tr_rmsnorm_bwd(const float* X, const float* g,
                                                       const float* rstd, const float* dY,
                                                       const float* base, int d, float* dX) {
  __shared__ float sh[4];
  const int i = blockIdx.x;
  const float* x = X + (size_t)i * d;
  const float* dy = dY + (size_t)i * d;
  const float r = rstd[i];
  float s = 0.f;
  for (int k = threadIdx.x; k < d; k += TB) s += x[k] * g[k] * dy[k];
  s = bsum(s, sh) / (float)d;
  for (int k = threadIdx.x; k < d; k += TB)
    dX[(size_t)i * d + k] =
        base[(size_t)i * d + k] + (r * g[k] * dy[k] - x[k] * r * r * r * s);
}

// Gain gradient dg[k] = sum over rows of dY[i][k] x[i][k] rstd[i]: GAIN_PARTS
// contiguous row ranges per feature (rows in order), then their sums in order.
// One thread per feature over all rows left 240 of 256 CUs idle: 639 rows of
// 4096 took 162 us, these two kernels 12 us.
constexpr int GAIN_PARTS = 32;
__global__ __launch_bounds__(TB) void k_tr_gain_parts(const float* X, const float* rstd,
                                                      const float* dY, int R, int d,
                                                      float* part) {
  const int k = blockIdx.x * TB + threadIdx.x;
  if (k >= d) return;
  const int per = (R + GAIN_PARTS - 1) / GAIN_PARTS;
  const int i0 = blockIdx.y * per, i1 = min(R, i0 + per);
  float s = 0.f;
  for (int i = i0; i < i1; ++i) s += dY[(size_t)i * d + k] * X[(size_t)i * d + k] * rstd[i];
  part[(size_t)blockIdx.y * d + k] = s;
}
__global__ __launch_bounds__(TB) void k_tr_gain_sum(const float* part, int d, int add, float* dg) {
  const int k = blockIdx.x * TB + threadIdx.x;
  if (k >= d) return;
  float s = add ? dg[k] : 0.f;
#pragma unroll
  for (int q = 0; q < GAIN_PARTS; ++q) s += part[(size_t)q * d + k];
  dg[k] = s;
}

// Rotate-half RoPE of the first nh heads of X's rows (stride ld) at position =
// row, by +angle (dir 1) or -angle (dir -1, the backward of the forward
// rotation).  One thread per rotation pair; grid (R, ceil(nh hd / 2 / TB)).
__global__ __launch_bounds__(TB) void k_tr_rope(float* X, int ld, int nh, int hd,
                                                const float2* tab, int dir) {
  const int i = blockIdx.x, half = hd / 2;
  const int p = blockIdx.y * TB + threadIdx.x;
  const int h = p / half, k = p - h * half;
  if (h >= nh) return;
  float* x = X + (size_t)i * ld + h * hd;
  const float2 t = tab[(size_t)i * half + k];
  const float c = t.x, s = dir > 0 ? t.y : -t.y;
  const float a = x[k], b = x[k + half];
  x[k] = a * c - b * s;
  x[k + half] = b * c + a * s;
}

// Causal softmax of S [R][R] rows (one head): P[i][j] = softmax_j<=i(scale
// S[i][j]), 0 above the diagonal.  Grid (R, heads); S in place.
__global__ __launch_bounds__(TB) void k_tr_softmax(float* S, int R, float scale) {
  __shared__ float sh[4];
  const int i = blockIdx.x;
  float* s = S + ((size_t)blockIdx.y * R + i) * R;
  float m = -INFINITY;
  for (int j = threadIdx.x; j <= i; j += TB) m = fmaxf(m, s[j] * scale);
  m = bmax(m, sh);
  float z = 0.f;
  for (int j = threadIdx.x; j <= i; j += TB) z += __expf(s[j] * scale - m);
  z = bsum(z, sh);
  const float inv = 1.f / z;
  for (int j = threadIdx.x; j < R; j += TB) s[j] = j <= i ? __expf(s[j] * scale - m) * inv : 0.f;
}

// dS = scale P (dP - rowsum(dP P)), in place over dP.  Grid (R, heads).
__global__ __launch_bounds__(TB) void k_tr_softmax_bwd(const float* P, float* dP, int R,
                                                       float scale) {
  __shared__ float sh[4];
  const size_t o = ((size_t)blockIdx.y * R + blockIdx.x) * R;
  float t = 0.f;
  for (int j = threadIdx.x; j < R; j += TB) t += dP[o + j] * P[o + j];
  t = bsum(t, sh);
  for (int j = threadIdx.x; j < R; j += TB) dP[o + j] = scale * P[o + j] * (dP[o + j] - t);
}

// Mx = silu(G) * U and its terms, with G and U the halves of GU's rows; grid
// (F / TB, R).
__global__ __launch_bounds__(TB) void k_tr_silu(const float* GU, int F, float* Mx, uint16_t* xs) {
  const int f = blockIdx.x * TB + threadIdx.x;
  if (f >= F) return;
  const float* row = GU + (size_t)blockIdx.y * 2 * F;
  const float g = row[f];
  const float m = g / (1.f + __expf(-g)) * row[F + f];
  Mx[(size_t)blockIdx.y * F + f] = m;
  put_terms(xs + (size_t)blockIdx.y * 3 * F, F, f, m);
}

// dG = dM U silu'(G), dU = dM silu(G) (silu' = s (1 + g (1 - s)), s = sigmoid).
__global__ __launch_bounds__(TB) void k_tr_silu_bwd(const float* GU, const float* dM, int F,
                                                    float* dGU) {
  const int f = blockIdx.x * TB + threadIdx.x;
  if (f >= F) return;
  const float* row = GU + (size_t)blockIdx.y * 2 * F;
  float* out = dGU + (size_t)blockIdx.y * 2 * F;
  const float g = row[f], s = 1.f / (1.f + __expf(-g));
  const float dm = dM[(size_t)blockIdx.y * F + f];
  out[f] = dm * row[F + f] * s * (1.f + g * (1.f - s));
  out[F + f] = dm * g * s;
}

// Regression term of row i: sum over features of SmoothL1(D[i] - H[i+1])
// divided by d into reg[i], its gradient into dD.  Grid (R).
__global__ __launch_bounds__(TB) void k_tr_reg(const float* D, const float* H, int d,
                                               float* dD, float* reg) {
  __shared__ float sh[4];
  const int i = blockIdx.x;
  float s = 0.f;
  for (int k = threadIdx.x; k < d; k += TB) {
    const float x = D[(size_t)i * d + k] - H[(size_t)(i + 1) * d + k];
    const float a = fabsf(x);
    s += a < 1.f ? 0.5f * x * x : a - 0.5f;
    dD[(size_t)i * d + k] = fminf(fmaxf(x, -1.f), 1.f) / (float)d;
  }
  s = bsum(s, sh);
  if (threadIdx.x == 0) reg[i] = s / (float)d;
}

// Token term of row i: with p = softmax(Ld[i]) (draft) and q =
// softmax(Lt[i]) (target, the row of position i + 1), ce[i] = -sum q log p,
// and Ld[i] <- w (p - q), the gradient of w ce[i].  Grid (R).
__global__ __launch_bounds__(TB) void k_tr_ce(float* Ld, const float* Lt, int V, int ldv,
                                              float w, float* ce) {
  __shared__ float sh[4];
  float* ld = Ld + (size_t)blockIdx.x * ldv;
  const float* lt = Lt + (size_t)blockIdx.x * ldv;
  float md = -INFINITY, mt = -INFINITY;
  for (int v = threadIdx.x; v < V; v += TB) {
    md = fmaxf(md, ld[v]);
    mt = fmaxf(mt, lt[v]);
  }
  md = bmax(md, sh);
  mt = bmax(mt, sh);
  float zd = 0.f, zt = 0.f;
  for (int v = threadIdx.x; v < V; v += TB) {
    zd += __expf(ld[v] - md);
    zt += __expf(lt[v] - mt);
  }
  zd = bsum(zd, sh);
  zt = bsum(zt, sh);
  const float lzd = logf(zd);
  float c = 0.f;
  for (int v = threadIdx.x; v < V; v += TB) {
    const float q = __expf(lt[v] - mt) / zt;
    const float lp = ld[v] - md - lzd;
    c -= q * lp;
    ld[v] = w * (__expf(lp) - q);
  }
  c = bsum(c, sh);
  if (threadIdx.x == 0) ce[blockIdx.x] = c;
}

// w -= lr mhat / (sqrt(vhat) + eps) with g = gsum * gscale (AdamW, no decay),
// and the bfloat16 copy of the new w (round to nearest even).
__global__ __launch_bounds__(TB) void k_tr_adamw(float* w, const float* gsum, float* m, float* v,
                                                 size_t n, float gscale, float lr, float c1,
                                                 float c2, float b1, float b2, float eps,
                                                 uint16_t* wb) {
  const size_t k = (size_t)blockIdx.x * TB + threadIdx.x;
  if (k >= n) return;
  const float g = gsum[k] * gscale;
  const float mk = b1 * m[k] + (1.f - b1) * g;
  const float vk = b2 * v[k] + (1.f - b2) * g * g;
  m[k] = mk;
  v[k] = vk;
  const float wk = w[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  w[k] = wk;
  wb[k] = f2bf(wk);
}

__global__ __launch_bounds__(TB) void k_tr_widen(const uint16_t* src, size_t n, float* dst) {
  const size_t k = (size_t)blockIdx.x * TB + threadIdx.x;
  if (k < n) dst[k] = bf2f(src[k]);
}

__global__ __launch_bounds__(TB) void k_tr_fill(float* p, size_t n, float v) {
  const size_t k = (size_t)blockIdx.x * TB + threadIdx.x;
  if (k < n) p[k] = v;
}

// The three bf16 terms of eight floats, one 16-byte unit each.  An infinite value
// (or a finite one past the largest bf16) is infinite in its first term only, and
// its product with an operand whose lower terms are zero is NaN where one float32
// product would be infinite.  No finite loss reaches that: such a row's RMSNorm is
// NaN, or its regression loss infinite, already.
MSD_DEV void split8(const float (&x)[8], uint4 (&t)[3]) {
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint16_t lo[3], hi[3];
    split3(x[2 * e], lo);
    split3(x[2 * e + 1], hi);
#pragma unroll
    for (int q = 0; q < 3; ++q) w[q][e] = lo[q] | ((uint32_t)hi[q] << 16);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) t[q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
}
MSD_DEV void load8(const float* p, float (&x)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w;
  x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
}

// Rows of three terms; one thread per unit of eight columns.
MSD_DEV void split_rows(const float* src, size_t q, size_t units, int C, uint16_t* dst) {
  if (q >= units) return;
  const int upr = C / 8;
  const size_t row = q / upr;
  const int k = (int)(q - row * upr) * 8;
  float x[8];
  load8(src + row * C + k, x);
  uint4 t[3];
  split8(x, t);
  uint16_t* d = dst + row * 3 * C + k;
#pragma unroll
  for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(d + (size_t)p * C) = t[p];
}
__global__ __launch_bounds__(TB) void k_tr_split(const float* src, size_t units, int C,
                                                 uint16_t* dst) {
  split_rows(src, (size_t)blockIdx.x * TB + threadIdx.x, units, C, dst);
}

// Packed planes of [R][C]; one thread per unit of the packed layout (see
// k_gemm.hip), as k_pack.
constexpr int PKB = 128, PTR = 64;
// The matrices that an update packs again: terms of the masters (planes of
// `plane` elements), or the bf16 copies as they are (src16).  A workgroup finds
// its matrix by its first block: one launch for all of them, which at d_model 256
// are a launch's latency each.
__global__ __launch_bounds__(TB) void k_tr_pack(PackJobs jobs) {
  int j = 0;
  while (j + 1 < jobs.n && (int)blockIdx.x >= jobs.job[j + 1].first) ++j;
  const PackJob& a = jobs.job[j];
  const int nkt = (a.C + PKB - 1) / PKB;
  const size_t units = (size_t)((a.R + PTR - 1) / PTR) * nkt * (PTR * PKB / 8);
  const size_t q = (size_t)((int)blockIdx.x - a.first) * TB + threadIdx.x;
  if (q >= units) return;
  const int lane = (int)(q & 63);
  const size_t r = q >> 6;
  const int c = (int)(r & 3), g16 = (int)((r >> 2) & 3);
  const size_t blk = r >> 4;
  const int kb = (int)(blk % nkt), t = (int)(blk / nkt);
  const int row = t * PTR + g16 * 16 + (lane & 15);
  const int col = kb * PKB + 32 * (lane >> 4) + 8 * c;
  const bool in = row < a.R && col < a.C;
  const size_t o = (size_t)row * a.C + col;
  if (a.src16) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (in) v = *reinterpret_cast<const uint4*>(a.src16 + o);
    *reinterpret_cast<uint4*>(a.dst + q * 8) = v;
    return;
  }
  float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (in) load8(a.src + o, x);
  uint4 u[3];
  split8(x, u);
#pragma unroll
  for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(a.dst + p * a.plane + q * 8) = u[p];
}

// A 128-row x 64-column block of src in LDS (zero past R and C), then a unit
// of eight rows of one column per thread and step.  Rows of 65 floats: the
// lanes of a step read different columns or rows 8 apart, in distinct banks.
constexpr int TLD = 65;
template <typename T>
MSD_DEV void load_tile(float* sh, const T* src, int R, int C, int r0, int c0) {
  for (int q = threadIdx.x; q < 128 * 16; q += TB) {
    const int r = q >> 4, c = (q & 15) * 4;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (r0 + r < R && c0 + c < C) {
      const T* p = src + (size_t)(r0 + r) * C + c0 + c;
      if constexpr (sizeof(T) == 4) {
        const float4 f = *reinterpret_cast<const float4*>(p);
        v[0] = f.x, v[1] = f.y, v[2] = f.z, v[3] = f.w;
      } else {
        const uint2 f = *reinterpret_cast<const uint2*>(p);
        v[0] = bf2f(f.x & 0xFFFF), v[1] = bf2f(f.x >> 16);
        v[2] = bf2f(f.y & 0xFFFF), v[3] = bf2f(f.y >> 16);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sh[r * TLD + c + e] = v[e];
  }
  __syncthreads();
}

// The transpose as rows of three terms [C][3 Rp], rows r0.. and columns c0.. of src.
MSD_DEV void split_tile_t(float* sh, const float* src, int R, int C, int Rp, int r0, int c0,
                          uint16_t* dst) {
  load_tile(sh, src, R, C, r0, c0);
  for (int q = threadIdx.x; q < 64 * 16; q += TB) {
    const int c = q >> 4, u = q & 15;  // 16 threads write one row's 256 bytes
    if (c0 + c >= C || r0 + 8 * u >= Rp) continue;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = sh[(8 * u + e) * TLD + c];
    uint4 t[3];
    split8(x, t);
    uint16_t* d = dst + (size_t)(c0 + c) * 3 * Rp + r0 + 8 * u;
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(d + (size_t)p * Rp) = t[p];
  }
}

// Packed planes of the transpose: block (t, kb), 64 columns x 128 rows of src.
template <typename T>
MSD_DEV void pack_tile_t(float* sh, const T* src, int R, int C, int nkt, int kb, int t,
                         uint16_t* dst, size_t plane) {
  load_tile(sh, src, R, C, kb * PKB, t * PTR);
  uint16_t* const o = dst + ((size_t)t * nkt + kb) * PKB * PTR;
  for (int q = threadIdx.x; q < 1024; q += TB) {
    const int lane = q & 63, c = (q >> 6) & 3, g16 = q >> 8;
    const int n = g16 * 16 + (lane & 15), k = 32 * (lane >> 4) + 8 * c;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = sh[(k + e) * TLD + n];
    uint4 u[3];
    split8(x, u);
#pragma unroll
    for (int p = 0; p < (sizeof(T) == 4 ? 3 : 1); ++p)
      *reinterpret_cast<uint4*>(o + p * plane + q * 8) = u[p];
  }
}

__global__ __launch_bounds__(TB) void k_tr_pack_t16(const uint16_t* src, int R, int C, int nkt,
                                                    uint16_t* dst) {
  __shared__ float sh[128 * TLD];
  pack_tile_t(sh, src, R, C, nkt, blockIdx.x, blockIdx.y, dst, (size_t)0);
}

// k_tr_pack of the masters' transposes.
__global__ __launch_bounds__(TB) void k_tr_pack_t(PackJobs jobs) {
  __shared__ float sh[128 * TLD];
  int j = 0;
  while (j + 1 < jobs.n && (int)blockIdx.x >= jobs.job[j + 1].first) ++j;
  const PackJob& a = jobs.job[j];
  const int nkt = (a.R + PKB - 1) / PKB, b = (int)blockIdx.x - a.first;
  pack_tile_t(sh, a.src, a.R, a.C, nkt, b % nkt, b / nkt, a.dst, a.plane);
}

// The operands of one product's gradients: the terms of dY [R][N] transposed
// (dyt, rows [N][3 Rp]) and of A [R][K] transposed and packed (at) for the weight's,
// and of dY as it is (dy, when given) for the input's.  One launch: the first bt
// workgroups take dyt, the next ba at, the others dy (a 64-row step of d_model 256:
// nine launches fewer).
__global__ __launch_bounds__(TB) void k_tr_operands(const float* dY, const float* A, int R, int N,
                                                    int K, int Rp, int bt, int ba, uint16_t* dyt,
                                                    uint16_t* at, size_t plane, uint16_t* dy) {
  __shared__ float sh[128 * TLD];
  const int nkt = (Rp + PKB - 1) / PKB;
  int b = blockIdx.x;
  if (b < bt) {
    split_tile_t(sh, dY, R, N, Rp, b % nkt * 128, b / nkt * 64, dyt);
    return;
  }
  b -= bt;
  if (b < ba) {
    pack_tile_t(sh, A, R, K, nkt, b % nkt, b / nkt, at, plane);
    return;
  }
  b -= ba;
  split_rows(dY, (size_t)b * TB + threadIdx.x, (size_t)R * (N / 8), N, dy);
}

unsigned blocks(size_t n) { return (unsigned)((n + TB - 1) / TB); }

}  // namespace

void tr_inputs(const uint16_t* h, const uint16_t* E, const int* tok, const int* vis_idx,
               const uint16_t* visual, int n, int d, int visual_feature, float* H, float* X0,
               float* E0, uint16_t* xs, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_inputs, dim3(n), dim3(TB), 0, st, h, E, tok, vis_idx, visual, n, d,
                     visual_feature, H, X0, E0, xs);
}
void tr_visual_rows(float* F, const float* E0, const int* vis_idx, int R, int d, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_visual_rows, dim3(R), dim3(TB), 0, st, F, E0, vis_idx, d);
}
void tr_zero_visual(float* dF, const int* vis_idx, int R, int d, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_zero_visual, dim3(R), dim3(TB), 0, st, dF, vis_idx, d);
}
void tr_rmsnorm(const float* X, const float* g, float eps, int R, int d, float* Y, float* rstd,
                uint16_t* xs, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_rmsnorm, dim3(R), dim3(TB), 0, st, X, g, eps, d, Y, rstd, xs);
}
size_t tr_gain_scratch(int d) { return (size_t)GAIN_PARTS * d; }
void tr_rmsnorm_bwd(const float* X, const float* g, const float* rstd, const float* dY,
                    const float* base, int R, int d, float* dX, float* dg, bool add,
                    float* scratch, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_rmsnorm_bwd, dim3(R), dim3(TB), 0, st, X, g, rstd, dY, base, d, dX);
  hipLaunchKernelGGL(k_tr_gain_parts, dim3(blocks(d), GAIN_PARTS), dim3(TB), 0, st, X, rstd, dY, R,
                     d, scratch);
  hipLaunchKernelGGL(k_tr_gain_sum, dim3(blocks(d)), dim3(TB), 0, st, scratch, d, add ? 1 : 0, dg);
}
void tr_rope(float* X, int R, int ld, int nh, int hd, const float2* tab, int dir, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_rope, dim3(R, blocks((size_t)nh * (hd / 2))), dim3(TB), 0, st, X, ld, nh,
                     hd, tab, dir);
}
void tr_softmax(float* S, int R, int heads, float scale, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_softmax, dim3(R, heads), dim3(TB), 0, st, S, R, scale);
}
void tr_softmax_bwd(const float* P, float* dP, int R, int heads, float scale, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_softmax_bwd, dim3(R, heads), dim3(TB), 0, st, P, dP, R, scale);
}
void tr_silu(const float* GU, int R, int F, float* Mx, uint16_t* xs, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_silu, dim3(blocks(F), R), dim3(TB), 0, st, GU, F, Mx, xs);
}
void tr_silu_bwd(const float* GU, const float* dM, int R, int F, float* dGU, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_silu_bwd, dim3(blocks(F), R), dim3(TB), 0, st, GU, dM, F, dGU);
}
void tr_reg(const float* D, const float* H, int R, int d, float* dD, float* reg, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_reg, dim3(R), dim3(TB), 0, st, D, H, d, dD, reg);
}
void tr_ce(float* Ld, const float* Lt, int R, int V, int ld, float w, float* ce, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_ce, dim3(R), dim3(TB), 0, st, Ld, Lt, V, ld, w, ce);
}
void tr_adamw(float* w, const float* gsum, float* m, float* v, size_t n, float gscale, float lr,
              float c1, float c2, float b1, float b2, float eps, uint16_t* wb, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_adamw, dim3(blocks(n)), dim3(TB), 0, st, w, gsum, m, v, n, gscale, lr,
                     c1, c2, b1, b2, eps, wb);
}
void tr_widen(const uint16_t* src, size_t n, float* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_widen, dim3(blocks(n)), dim3(TB), 0, st, src, n, dst);
}
void tr_fill(float* p, size_t n, float v, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_fill, dim3(blocks(n)), dim3(TB), 0, st, p, n, v);
}

void tr_split(const float* src, int R, int C, uint16_t* dst, hipStream_t st) {
  const size_t units = (size_t)R * (C / 8);
  hipLaunchKernelGGL(k_tr_split, dim3(blocks(units)), dim3(TB), 0, st, src, units, C, dst);
}
void tr_operands(const float* dY, const float* A, int R, int N, int K, int Rp, uint16_t* dyt,
                 uint16_t* at, size_t plane, uint16_t* dy, hipStream_t st) {
  const int nkt = (Rp + PKB - 1) / PKB;
  const int bt = nkt * ((N + 63) / 64), ba = nkt * ((K + PTR - 1) / PTR);
  const unsigned bd = dy ? blocks((size_t)R * (N / 8)) : 0;
  hipLaunchKernelGGL(k_tr_operands, dim3(bt + ba + bd), dim3(TB), 0, st, dY, A, R, N, K, Rp, bt, ba,
                     dyt, at, plane, dy);
}
void PackJobs::add(const float* src, const uint16_t* src16, int R, int C, uint16_t* dst,
                   size_t plane, bool transposed) {
  job[n++] = PackJob{src, src16, R, C, dst, plane, wgs};
  wgs += transposed ? ((R + PKB - 1) / PKB) * ((C + PTR - 1) / PTR)
                    : (int)blocks(packed_elems(R, C) / 8);
}
void tr_pack(const PackJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_pack, dim3(j.wgs), dim3(TB), 0, st, j);
}
void tr_pack_t(const PackJobs& j, hipStream_t st) {
  hipLaunchKernelGGL(k_tr_pack_t, dim3(j.wgs), dim3(TB), 0, st, j);
}
void tr_pack_t16(const uint16_t* src, int R, int C, int Rp, uint16_t* dst, hipStream_t st) {
  const int nkt = (Rp + PKB - 1) / PKB;
  hipLaunchKernelGGL(k_tr_pack_t16, dim3(nkt, (C + PTR - 1) / PTR), dim3(TB), 0, st, src, R, C, nkt,
                     dst);
}

}  // namespace msd
