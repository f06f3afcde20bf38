// Stochastic reconfiguration step (Sec. 3.2, Eq. (12); ridge lambda of
// Sec. 3.4) solved in sample space.
//
// With O_bar = (O - <O>)/sqrt(S) and eps = (E_loc - <E_loc>)/sqrt(S), the
// P x P system (O_bar^H O_bar + lambda) dtheta = -dtau O_bar^H eps has the
// same solution as dtheta = -dtau O_bar^H (O_bar O_bar^H + lambda)^{-1} eps
// (push-through identity), an S x S Hermitian positive definite system:
//  1. column means of O, then O_bar written transposed as separate real and
//     imaginary planes [P][S] (unit-stride sample axis for the MFMA operands);
//  2. Gram T = O_bar O_bar^H + lambda I on 16x16x4 MFMA (FP32 for complex64
//     O, on LDS-staged tiles; FP64 for complex128), complex product
//     as four real products, lower block triangle only, stored in FP64;
//  3. blocked FP64 Cholesky T = L L^H with 32 x 32 blocks in panels of 8 block
//     columns: inside a panel each column takes the updates of the panel's
//     columns before it, then one rank-256 update of the trailing matrix per
//     panel, all on FP64 MFMA; eps^H rides along as one more row, which
//     becomes (L^-1 eps)^H;
//  4. L^H x = y, dtheta = -dtau O_bar^H x.
// S is padded to a multiple of 32 with zero rows (their T block is lambda I
// and their eps is 0, so they drop out of x and dtheta).
#include <algorithm>
#include <cmath>
#include <string>

#include "device_common.h"
#include "nqs_internal.h"

namespace nqs {

namespace {

constexpr int kB = 32;   // Cholesky / Gram block
constexpr int kPanel = 8;  // block columns per Cholesky panel (one trailing update each)

__device__ __forceinline__ f64x4 mma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <typename R> struct AccT;
template <> struct AccT<float> { using type = f32x4; };
template <> struct AccT<double> { using type = f64x4; };
// output row of register r in lane group q (see logical_row in device_common.h)
template <typename R> __device__ __forceinline__ int out_row(int q, int r) {
  return sizeof(R) == 8 ? q + 4 * r : 4 * q + r;
}

// ---------------------------------------------------------------- centring
// Column means, one column per thread, the sum in the order of the samples.
// kMeanAhead samples' loads are in flight per thread, one wavefront per
// workgroup so that the columns spread over the device: 2048 x 40500 complex64
// in 0.13 ms (5.2 TB/s) against 0.85 ms with one load at a time.
constexpr int kMeanAhead = 16;
template <typename RO>
__global__ __launch_bounds__(64) void colmean_kernel(const RO* __restrict__ O, int64_t S, int64_t P,
                                                     double* __restrict__ mean) {
  using V = c2_t<RO>;
  const int64_t k = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (k >= P) return;
  const V* o = reinterpret_cast<const V*>(O) + k;
  double sr = 0.0, si = 0.0;
  int64_t s = 0;
  for (; s + kMeanAhead <= S; s += kMeanAhead) {
    V v[kMeanAhead];
#pragma unroll
    for (int u = 0; u < kMeanAhead; ++u) v[u] = o[(s + u) * P];
#pragma unroll
    for (int u = 0; u < kMeanAhead; ++u) {
      sr += (double)v[u].x;
      si += (double)v[u].y;
    }
  }
  for (; s < S; ++s) {
    const V v = o[s * P];
    sr += (double)v.x;
    si += (double)v.y;
  }
  mean[2 * k] = sr / (double)S;
  mean[2 * k + 1] = si / (double)S;
}

// O_bar transposed: Tre[k][s], Tim[k][s] for k < Pk, s < S32 (zero padding)
template <typename RO, typename RG>
__global__ void center_t_kernel(const RO* __restrict__ O, int64_t S, int64_t P, int64_t Pk,
                                int64_t S32, const double* __restrict__ mean, double inv_sqrt_s,
                                RG* __restrict__ Tre, RG* __restrict__ Tim) {
  __shared__ double tr[32][33], ti[32][33];
  const int64_t s0 = (int64_t)blockIdx.x * 32, k0 = (int64_t)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
  for (int yy = ty; yy < 32; yy += 8) {
    const int64_t s = s0 + yy, k = k0 + tx;
    double vr = 0.0, vi = 0.0;
    if (s < S && k < P) {
      vr = ((double)O[(s * P + k) * 2] - mean[2 * k]) * inv_sqrt_s;
      vi = ((double)O[(s * P + k) * 2 + 1] - mean[2 * k + 1]) * inv_sqrt_s;
    }
    tr[yy][tx] = vr;
    ti[yy][tx] = vi;
  }
  __syncthreads();
  for (int yy = ty; yy < 32; yy += 8) {
    const int64_t k = k0 + yy, s = s0 + tx;
    if (k < Pk && s < S32) {
      Tre[k * S32 + s] = (RG)tr[tx][yy];
      Tim[k * S32 + s] = (RG)ti[tx][yy];
    }
  }
}

// Block row nblk of T: row 0 is eps^H, eps[s] = (E_loc[s] - <E_loc>) / sqrt(S)
// (zero for the padding), the other 31 rows are zero.
__global__ void eps_kernel(const double* __restrict__ el, int64_t S, int64_t S32,
                           double* __restrict__ v) {
  __shared__ double red[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double sr = 0.0, si = 0.0;
  for (int64_t s = tid; s < S; s += blockDim.x) {
    sr += el[2 * s];
    si += el[2 * s + 1];
  }
  sr = wave_sum(sr);
  si = wave_sum(si);
  if (lane == 0) {
    red[0][wv] = sr;
    red[1][wv] = si;
  }
  __syncthreads();
  sr = 0.0;
  si = 0.0;
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) {
    sr += red[0][q];
    si += red[1][q];
  }
  const double mr = sr / (double)S, mi = si / (double)S, f = 1.0 / sqrt((double)S);
  for (int64_t s = tid; s < S32; s += blockDim.x) {
    v[2 * s] = s < S ? (el[2 * s] - mr) * f : 0.0;
    v[2 * s + 1] = s < S ? -(el[2 * s + 1] - mi) * f : 0.0;
  }
  for (int64_t e = tid; e < 31 * S32 * 2; e += blockDim.x) v[2 * S32 + e] = 0.0;
}

// ------------------------------------------------------------------- Gram
__device__ __forceinline__ void tri_index(int64_t t, int64_t& I, int64_t& J) {
  I = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while (I * (I + 1) / 2 > t) --I;
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  J = t - I * (I + 1) / 2;
}

// T[I-block][J-block] (I >= J) = sum_k Ob[s][k] conj(Ob[s'][k]) (+ lambda on the diagonal)
template <typename RG>
__global__ __launch_bounds__(256) void gram_kernel(const RG* __restrict__ Tre,
                                                   const RG* __restrict__ Tim, int64_t Pk,
                                                   int64_t S32, int64_t nblk, double lambda,
                                                   double* __restrict__ T) {
  using Acc = typename AccT<RG>::type;
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= nblk * (nblk + 1) / 2) return;
  int64_t I, J;
  tri_index(t, I, J);
  Acc cr[2][2], ci[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      cr[a][b] = Acc{0, 0, 0, 0};
      ci[a][b] = Acc{0, 0, 0, 0};
    }
  const int64_t ra = I * kB + c, rb = J * kB + c;
  for (int64_t k0 = 0; k0 < Pk; k0 += 4) {
    const int64_t kk = (k0 + q) * S32;
    RG ar[2], ai[2], br[2], bi[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      ar[a] = Tre[kk + ra + 16 * a];
      ai[a] = Tim[kk + ra + 16 * a];
      br[a] = Tre[kk + rb + 16 * a];
      bi[a] = Tim[kk + rb + 16 * a];
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        cr[a][b] = mma(ar[a], br[b], cr[a][b]);
        cr[a][b] = mma(ai[a], bi[b], cr[a][b]);
        ci[a][b] = mma(ai[a], br[b], ci[a][b]);
        ci[a][b] = mma(-ar[a], bi[b], ci[a][b]);
      }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = I * kB + 16 * a + out_row<RG>(q, r);
        const int64_t col = J * kB + 16 * b + c;
        double vr = (double)cr[a][b][r], vi = (double)ci[a][b][r];
        if (row == col) vr += lambda;
        T[(row * S32 + col) * 2] = vr;
        T[(row * S32 + col) * 2 + 1] = vi;
      }
}

// FP32 Gram on GT x GT output tiles (GT = 96 or 64), one workgroup of four
// wavefronts per lower tile, each wavefront a quarter of NA x NA MFMA tiles of
// 16 x 16 for each of the real and imaginary parts.  The two row panels of the
// tile go through LDS in stages of kGK parameters, double-buffered, with
// two stages' global loads in flight.  Per k, a
// panel row holds [half][c][a] (row GT/2 half + 16 a + c, a < NA <= 4), written
// and read as 16-byte units, so that lane (q, c) gets its operands with one
// load; kGP pads the k rows apart.  Only 32 x 32 blocks on or below the block
// diagonal are written.  Each output sums the parameters in the same order,
// whatever GT.
//
// Bound: FP32 MFMA, which VALU work does not overlap: the loop keeps its
// addresses in scalars and per-lane offsets made once (with addresses formed per
// load 7.7 ms, one stage in flight 8.2 ms).  The tile size is the one whose
// rounds of workgroups over the CUs cost least (gram_tile): 2048 rows are 136
// tiles of 128, which leave 120 of 256 CUs idle, or 253 of 96: 11.6 -> 6.6 ms at
// P = 40500 (0.74 of the MFMA rate of the CUs in use).
constexpr int kGK = 16, kGP = 128 + 4;

template <int GT>
__global__ __launch_bounds__(256) void gram_tile_kernel(const float* __restrict__ Tre,
                                                        const float* __restrict__ Tim, int64_t Pk,
                                                        int64_t S32, double lambda,
                                                        double* __restrict__ T) {
  constexpr int NA = GT / 32, GH = GT / 2;
  __shared__ __align__(16) float As[2][2][kGK][kGP];   // [buffer][re, im][k][row slot]
  __shared__ __align__(16) float Bs[2][2][kGK][kGP];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = lane >> 4, c = lane & 15;
  const int wy = wv >> 1, wx = wv & 1;
  int64_t I, J;
  tri_index((int64_t)blockIdx.x, I, J);
  const int64_t rowA = I * GT, rowB = J * GT;

  // stage loader: 2048 units (panel x plane x kGK x half x c) of NA rows, eight
  // per thread: unit i of a thread is (panel i / 4, plane i / 2 % 2,
  // k = 8 (i % 2) + tid / 32, half, c), so that everything but the lane's own
  // offset is scalar (VALU work does not overlap FP32 MFMA).  Rows beyond S32
  // repeat the last one (their outputs are dropped); the planes hold whole
  // stages, and stages past the end repeat the last one (not used).
  const int hf = (tid >> 4) & 1, cc = tid & 15, kq = tid >> 5;
  uint32_t off[2][NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const int64_t r = GH * hf + 16 * a + cc;
    off[0][a] = (uint32_t)(kq * S32 + min(rowA + r, S32 - 1));
    off[1][a] = (uint32_t)(kq * S32 + min(rowB + r, S32 - 1));
  }
  const int64_t nst = Pk / kGK;
  float preA[8][NA], preB[8][NA];          // stages in flight
  auto load_stage = [&](float (&pre)[8][NA], int64_t st) __attribute__((always_inline)) {
    const int64_t k0 = min(st, nst - 1) * kGK;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float* src = ((i >> 1) & 1 ? Tim : Tre) + (k0 + 8 * (i & 1)) * S32;
#pragma unroll
      for (int a = 0; a < NA; ++a) pre[i][a] = src[off[i >> 2][a]];
    }
  };
  auto store_stage = [&](const float (&pre)[8][NA], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float* dst = (i >> 2) ? &Bs[buf][(i >> 1) & 1][8 * (i & 1)][0] : &As[buf][(i >> 1) & 1][8 * (i & 1)][0];
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int a = 0; a < NA; ++a) v[a] = pre[i][a];
      *reinterpret_cast<f32x4*>(dst + kq * kGP + 64 * hf + 4 * cc) = v;
    }
  };

  f32x4 cr[NA][NA], ci[NA][NA];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NA; ++b) {
      cr[a][b] = f32x4{0, 0, 0, 0};
      ci[a][b] = f32x4{0, 0, 0, 0};
    }
  auto compute = [&](int cur) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < kGK; ks += 4) {
      const f32x4 ar = *reinterpret_cast<const f32x4*>(&As[cur][0][ks + q][64 * wy + 4 * c]);
      const f32x4 ai = *reinterpret_cast<const f32x4*>(&As[cur][1][ks + q][64 * wy + 4 * c]);
      const f32x4 br = *reinterpret_cast<const f32x4*>(&Bs[cur][0][ks + q][64 * wx + 4 * c]);
      const f32x4 bi = *reinterpret_cast<const f32x4*>(&Bs[cur][1][ks + q][64 * wx + 4 * c]);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NA; ++b) cr[a][b] = mma(ar[a], br[b], cr[a][b]);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NA; ++b) ci[a][b] = mma(ai[a], br[b], ci[a][b]);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NA; ++b) cr[a][b] = mma(ai[a], bi[b], cr[a][b]);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NA; ++b) ci[a][b] = mma(-ar[a], bi[b], ci[a][b]);
    }
  };
  load_stage(preA, 0);
  store_stage(preA, 0);
  load_stage(preA, 1);
  __syncthreads();
  for (int64_t st = 0; st < nst; st += 2) {
    load_stage(preB, st + 2);
    compute(0);
    store_stage(preA, 1);
    __syncthreads();
    if (st + 1 == nst) break;
    load_stage(preA, st + 3);
    compute(1);
    store_stage(preB, 0);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NA; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = rowA + GH * wy + 16 * a + out_row<float>(q, r);
        const int64_t col = rowB + GH * wx + 16 * b + c;
        if (row >= S32 || col >= S32 || row / kB < col / kB) continue;
        double vr = (double)cr[a][b][r], vi = (double)ci[a][b][r];
        if (row == col) vr += lambda;
        T[(row * S32 + col) * 2] = vr;
        T[(row * S32 + col) * 2 + 1] = vi;
      }
}

// Tile size of the FP32 Gram: rounds of workgroups (one per CU at a time) x
// tile area, for tiles of 64 times 1.15 (they read their rows half as often
// again): 64 up to a few thousand samples where it fills the last round better,
// 96 otherwise.  The whole solve at 10x10 M = 400 with tiles of 128, 96 and 64:
// S = 4096 48, 30.9 and 35.1 ms, 8192 143, 109 and 121, 20000 911, 695 and 770;
// 6x6 M = 72 S = 3000 6.4, 5.8 and 5.6.
inline int gram_tile(int64_t S32, int n_cu) {
  auto cost = [&](int64_t gt) {
    const int64_t nt = (S32 + gt - 1) / gt, rounds = (nt * (nt + 1) / 2 + n_cu - 1) / n_cu;
    return rounds * gt * gt;
  };
  return 23 * cost(64) < 20 * cost(96) ? 64 : 96;
}

// --------------------------------------------------------------- Cholesky
// T has one more block row (block row nblk) than columns: its first row is
// eps^H, so that the factorisation leaves (L^-1 eps)^H there and no forward
// substitution is needed.  Block columns are taken in panels of kPanel; inside a
// panel column k first gets the updates of the panel's columns before it, and
// each panel then updates the trailing matrix at once.
//
// At S = 2048 the chain of 64 block columns is the bound: per column one
// workgroup factors the diagonal block (and inverts its factor), 23 us, then
// one launch updates and solves the blocks below, 11 us.  The earlier form took
// three launches a column (29, 20 and 18 us: a division and three barriers per
// pivot, one thread per row for the solve), and four for the two substitutions
// (32 us): 6.3 ms in all, 2.8 ms now.

// acc (16 x 16 quadrant, rows 16 a of block I against rows 16 b of block J)
// += sum_{col in [c0, c1)} T[I rows][col] conj(T[J rows][col]), 32 columns at a
// time with the next 32 columns' loads in flight
__device__ __forceinline__ void quad_gram(const double2* __restrict__ T, int64_t S32, int64_t rI,
                                          int64_t rJ, int64_t c0, int64_t c1, int q, f64x4& cr,
                                          f64x4& ci) {
  if (c0 >= c1) return;
  const double2* x = T + rI * S32 + q;
  const double2* y = T + rJ * S32 + q;
  double2 u[8], v[8], un[8], vn[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    un[i] = x[c0 + 4 * i];
    vn[i] = y[c0 + 4 * i];
  }
  for (int64_t k0 = c0; k0 < c1; k0 += kB) {
    const int64_t nx = k0 + kB < c1 ? k0 + kB : k0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      u[i] = un[i];
      v[i] = vn[i];
      un[i] = x[nx + 4 * i];
      vn[i] = y[nx + 4 * i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      cr = mma(u[i].x, v[i].x, cr);
      ci = mma(u[i].y, v[i].x, ci);
      cr = mma(u[i].y, v[i].y, cr);
      ci = mma(-u[i].x, v[i].y, ci);
    }
  }
}

// 1 / d from the hardware estimate and two Newton steps (about 1 ulp), d within
// 2^+-1000
__device__ __forceinline__ double rcp_pivot(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  return r;
}

// Diagonal block k: apply the panel's earlier columns [c0, 32 k), factor it
// (lower triangle to T) and write the inverse of the factor to Linv[k].
// Thread (i, lg) holds kDE entries (i, kDE lg + e) of the block and of the
// identity that the same row operations turn into the inverse.  Step j passes
// the unscaled column j and row j of the inverse through LDS (one barrier a
// step; the square roots wait until the end).
// (entries per thread, threads: 1, 2 and 4 entries took 10.2, 9.8 and 10.0 ms for
// the whole solve at S = 2048)
constexpr int kDE = 2, kDT = kB * kB / kDE;
__global__ __launch_bounds__(kDT) void potrf_diag_kernel(double2* __restrict__ T, int64_t S32,
                                                         int64_t k, int64_t c0,
                                                         double2* __restrict__ Linv,
                                                         int* __restrict__ flag) {
  __shared__ double2 blk[kB][kB + 1];
  __shared__ double2 col[2][kB], row[2][kB];
  __shared__ double piv[kB];
  __shared__ double2 rs[kB];                 // sqrt(pivot) and its inverse
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = lane >> 4, c = lane & 15;
  const int64_t kb = k * kB;
  if (wv < 4) {
    const int a = wv >> 1, b = wv & 1;
    f64x4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
    if (a >= b) quad_gram(T, S32, kb + 16 * a + c, kb + 16 * b + c, c0, kb, q, cr, ci);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * a + out_row<double>(q, r), j = 16 * b + c;
      double2 v = make_double2(0.0, 0.0);
      if (i >= j) {
        v = T[(kb + i) * S32 + kb + j];
        v.x -= cr[r];
        v.y -= ci[r];
      }
      blk[i][j] = v;
    }
  }
  __syncthreads();
  const int i = tid / (kB / kDE), lg = tid % (kB / kDE);
  double2 A[kDE], X[kDE];
#pragma unroll
  for (int e = 0; e < kDE; ++e) {
    A[e] = blk[i][kDE * lg + e];
    X[e] = make_double2(i == kDE * lg + e ? 1.0 : 0.0, 0.0);
  }
#pragma unroll 1
  for (int jo = 0; jo < kB / 4; ++jo) {
#pragma unroll
    for (int je = 0; je < 4; ++je) {
      const int j = 4 * jo + je, jb = je & 1;
      if (lg == j / kDE) col[jb][i] = A[je % kDE];
      if (i == j) {
#pragma unroll
        for (int e = 0; e < kDE; ++e) row[jb][kDE * lg + e] = X[e];
      }
      __syncthreads();
      double d = col[jb][j].x;
      const bool bad = !(d > 0.0) || !isfinite(d);
      if (bad) d = 1.0;
      if (tid == 0) {
        piv[j] = d;
        if (bad) flag[0] = 1;
      }
      const double2 cv = col[jb][i];
      double fr = 0.0, fi = 0.0;               // row multiplier
      if (d > 0x1p-1000 && d < 0x1p1000) {
        const double inv = rcp_pivot(d);
        fr = i > j ? cv.x * inv : 0.0;
        fi = i > j ? cv.y * inv : 0.0;
      } else if (i > j) {                      // 1 / d may be out of range where cv / d is not
        fr = cv.x / d;
        fi = cv.y / d;
      }
#pragma unroll
      for (int e = 0; e < kDE; ++e) {
        const int l = kDE * lg + e;
        // A[i][l] -= f conj(column j, row l) for l > j; X[i][l] -= f X[j][l] for l <= j
        double2 w = l > j ? col[jb][l] : row[jb][l];
        double2 z = l > j ? A[e] : X[e];
        if (l > j) w.y = -w.y;
        z.x -= fr * w.x - fi * w.y;
        z.y -= fr * w.y + fi * w.x;
        if (l > j) A[e] = z;
        else X[e] = z;
      }
    }
  }
  __syncthreads();
  if (tid < kB) {
    const double r = sqrt(piv[tid]);
    rs[tid] = make_double2(r, 1.0 / r);
  }
  __syncthreads();
  const double si = rs[i].y;
#pragma unroll
  for (int e = 0; e < kDE; ++e) {
    const int l = kDE * lg + e;
    const double sl = rs[l].y;
    if (i > l) T[(kb + i) * S32 + kb + l] = make_double2(A[e].x * sl, A[e].y * sl);
    if (i == l) T[(kb + i) * S32 + kb + l] = make_double2(rs[l].x, 0.0);
    Linv[(k * kB + i) * kB + l] = make_double2(X[e].x * si, X[e].y * si);
  }
}

// Blocks I > k of block column k (one workgroup each, block row nblk included):
// apply the panel's earlier columns [c0, 32 k), then X = A L_kk^-H.
__global__ __launch_bounds__(256) void trsm_panel_kernel(double2* __restrict__ T, int64_t S32,
                                                         int64_t k, int64_t c0,
                                                         const double2* __restrict__ Linv) {
  __shared__ double2 blk[kB][kB + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, q = lane >> 4, c = lane & 15;
  const int a = wv >> 1, b = wv & 1;
  const int64_t kb = k * kB, ib = (k + 1 + blockIdx.x) * kB;
  f64x4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
  quad_gram(T, S32, ib + 16 * a + c, kb + 16 * b + c, c0, kb, q, cr, ci);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * a + out_row<double>(q, r), j = 16 * b + c;
    const double2 v = T[(ib + i) * S32 + kb + j];
    blk[i][j] = make_double2(v.x - cr[r], v.y - ci[r]);
  }
  __syncthreads();
  // X[i][j] = sum_l blk[i][l] conj(Linv[j][l])
  cr = f64x4{0, 0, 0, 0};
  ci = f64x4{0, 0, 0, 0};
  const double2* y = Linv + (kb + 16 * b + c) * kB + q;
#pragma unroll
  for (int l = 0; l < kB; l += 4) {
    const double2 u = blk[16 * a + c][l + q], v = y[l];
    cr = mma(u.x, v.x, cr);
    ci = mma(u.y, v.x, ci);
    cr = mma(u.y, v.y, cr);
    ci = mma(-u.x, v.y, ci);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * a + out_row<double>(q, r), j = 16 * b + c;
    T[(ib + i) * S32 + kb + j] = make_double2(cr[r], ci[r]);
  }
}

// Trailing update of a panel: T[I][J] -= L[I][K] L[J][K]^H over the nk block
// columns K = kc0 ..., for every block I >= J >= j0 and for block row nblk, one
// wavefront per 32 x 32 output block.
__global__ __launch_bounds__(256) void herk_update_kernel(double* __restrict__ T, int64_t S32,
                                                          int64_t kc0, int nk, int64_t j0,
                                                          int64_t nblk) {
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t m = nblk - j0, ntri = m * (m + 1) / 2;
  if (t >= ntri + m) return;
  int64_t I, J;
  if (t < ntri) {
    tri_index(t, I, J);
    I += j0;
    J += j0;
  } else {
    I = nblk;
    J = j0 + t - ntri;
  }
  const int64_t kb = kc0 * kB;
  f64x4 cr[2][2], ci[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      cr[a][b] = f64x4{0, 0, 0, 0};
      ci[a][b] = f64x4{0, 0, 0, 0};
    }
  for (int k0 = 0; k0 < nk * kB; k0 += 4) {
    double xr[2], xi[2], yr[2], yi[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int64_t ri = I * kB + 16 * a + c, rj = J * kB + 16 * a + c;
      xr[a] = T[(ri * S32 + kb + k0 + q) * 2];
      xi[a] = T[(ri * S32 + kb + k0 + q) * 2 + 1];
      yr[a] = T[(rj * S32 + kb + k0 + q) * 2];
      yi[a] = T[(rj * S32 + kb + k0 + q) * 2 + 1];
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        cr[a][b] = mma(xr[a], yr[b], cr[a][b]);
        cr[a][b] = mma(xi[a], yi[b], cr[a][b]);
        ci[a][b] = mma(xi[a], yr[b], ci[a][b]);
        ci[a][b] = mma(-xr[a], yi[b], ci[a][b]);
      }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = I * kB + 16 * a + out_row<double>(q, r);
        const int64_t col = J * kB + 16 * b + c;
        if (row >= col) {
          T[(row * S32 + col) * 2] -= cr[a][b][r];
          T[(row * S32 + col) * 2 + 1] -= ci[a][b][r];
        }
      }
}

// ------------------------------------------------------------------ solves
// y = L^-1 eps from block row nblk (conjugated)
__global__ void take_y_kernel(const double2* __restrict__ T, int64_t S32,
                              double2* __restrict__ v) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= S32) return;
  const double2 y = T[S32 * S32 + j];
  v[j] = make_double2(y.x, -y.y);
}

// L^H x = v on the block columns K0 .. K0 + nk - 1 (one workgroup): from the
// last block back, x_k = L_kk^-H v_k and v_j -= sum_l conj(L[32 k + l][j]) x_l
// for the panel's columns j before it.
__global__ __launch_bounds__(256) void bsolve_panel_kernel(const double2* __restrict__ T,
                                                           int64_t S32, int64_t K0, int nk,
                                                           const double2* __restrict__ Linv,
                                                           double2* __restrict__ v) {
  __shared__ double2 vs[kPanel * kB], xs[kB];
  const int tid = threadIdx.x;
  const int64_t base = K0 * kB;
  if (tid < nk * kB) vs[tid] = v[base + tid];
  __syncthreads();
  for (int kk = nk - 1; kk >= 0; --kk) {
    const int64_t kb = base + kk * kB;
    // x_t = sum_l conj(Linv[l][t]) v_l, eight lanes per t
    // (the rows of L it needs afterwards are loaded meanwhile)
    const int t = tid >> 3, part = tid & 7;
    double2 Lr[kB], m4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) m4[e] = Linv[(kb + 4 * part + e) * kB + t];
#pragma unroll
    for (int l = 0; l < kB; ++l) Lr[l] = T[(kb + l) * S32 + base + min(tid, max(kk * kB - 1, 0))];
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double2 m = m4[e], w = vs[kk * kB + 4 * part + e];
      sr += m.x * w.x + m.y * w.y;
      si += m.x * w.y - m.y * w.x;
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      sr += __shfl_xor(sr, o, 64);
      si += __shfl_xor(si, o, 64);
    }
    if (part == 0) xs[t] = make_double2(sr, si);
    __syncthreads();
    if (tid < kB) vs[kk * kB + tid] = xs[tid];
    if (tid < kk * kB) {
      double2 w = vs[tid];
#pragma unroll
      for (int l = 0; l < kB; ++l) {
        const double2 m = Lr[l], x = xs[l];
        w.x -= m.x * x.x + m.y * x.y;
        w.y -= m.x * x.y - m.y * x.x;
      }
      vs[tid] = w;
    }
    __syncthreads();
  }
  if (tid < nk * kB) v[base + tid] = vs[tid];
}

// v_j -= sum_l conj(L[32 K0 + l][j]) x_l over the panel's rows l, for the
// columns j before the panel: 64 columns a workgroup, the rows in 16 parts of
// at most 16
__global__ __launch_bounds__(1024) void bsolve_update_kernel(const double2* __restrict__ T,
                                                             int64_t S32, int64_t K0, int nk,
                                                             double2* __restrict__ v) {
  constexpr int kParts = 16, kRows = kPanel * kB / kParts;
  __shared__ double2 xs[kPanel * kB], red[kParts][64];
  const int tid = threadIdx.x, jc = tid & 63, part = tid >> 6;
  const int64_t base = K0 * kB, j = (int64_t)blockIdx.x * 64 + jc;
  if (tid < kPanel * kB) xs[tid] = tid < nk * kB ? v[base + tid] : make_double2(0.0, 0.0);
  __syncthreads();
  double sr = 0.0, si = 0.0;
  if (j < base) {
    const int l0 = part * kRows, last = nk * kB - 1;      // rows past the panel: x = 0
#pragma unroll
    for (int l = 0; l < kRows; ++l) {
      const double2 m = T[(base + min(l0 + l, last)) * S32 + j], x = xs[l0 + l];
      sr += m.x * x.x + m.y * x.y;
      si += m.x * x.y - m.y * x.x;
    }
  }
  red[part][jc] = make_double2(sr, si);
  __syncthreads();
  if (part == 0 && j < base) {
    double2 w = v[j];
    for (int o = 0; o < kParts; ++o) {
      w.x -= red[o][jc].x;
      w.y -= red[o][jc].y;
    }
    v[j] = w;
  }
}

// dtheta[k] = -dtau sum_s conj(Ob[s][k]) x[s]   (one wavefront per parameter)
template <typename RG>
__global__ __launch_bounds__(256) void dtheta_kernel(const RG* __restrict__ Tre,
                                                     const RG* __restrict__ Tim, int64_t P,
                                                     int64_t S32, const double* __restrict__ x,
                                                     double dtau, double* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= P) return;
  double sr = 0.0, si = 0.0;
  for (int64_t s = lane; s < S32; s += 64) {
    const double ar = (double)Tre[k * S32 + s], ai = (double)Tim[k * S32 + s];
    const double xr = x[2 * s], xi = x[2 * s + 1];
    sr += ar * xr + ai * xi;
    si += ar * xi - ai * xr;
  }
  sr = wave_sum(sr);
  si = wave_sum(si);
  if (lane == 0) {
    out[2 * k] = -dtau * sr;
    out[2 * k + 1] = -dtau * si;
  }
}

inline size_t al(size_t v) { return (v + 255) / 256 * 256; }
inline int64_t r32(int64_t v) { return (v + kB - 1) / kB * kB; }
inline int64_t rk(int64_t v) { return (v + kGK - 1) / kGK * kGK; }   // whole Gram stages

template <typename RO, typename RG>
hipError_t sr_run(const nqs_ctx* c, const void* Ov, const double* el, int64_t S, double lambda,
                  double dtau, double* out, void* ws, hipStream_t st, int* flag_host) {
  const RO* O = (const RO*)Ov;
  const int64_t P = c->P, Pk = rk(P), S32 = r32(S), nblk = S32 / kB;
  char* p = (char*)ws;
  double* T = (double*)p;
  p += al((size_t)(S32 + kB) * S32 * 16);
  double2* Linv = (double2*)p;
  p += al((size_t)S32 * kB * 16);
  RG* Tre = (RG*)p;
  p += al((size_t)Pk * S32 * sizeof(RG));
  RG* Tim = (RG*)p;
  p += al((size_t)Pk * S32 * sizeof(RG));
  double* v = (double*)p;
  p += al((size_t)S32 * 16);
  double* mean = (double*)p;
  p += al((size_t)P * 16);
  int* flag = (int*)p;

  hipError_t e = hipMemsetAsync(flag, 0, sizeof(int), st);
  if (e != hipSuccess) return e;
  colmean_kernel<RO><<<(unsigned)((P + 63) / 64), 64, 0, st>>>(O, S, P, mean);
  dim3 gct((unsigned)(S32 / 32), (unsigned)((Pk + 31) / 32));
  center_t_kernel<RO, RG><<<gct, 256, 0, st>>>(O, S, P, Pk, S32, mean, 1.0 / std::sqrt((double)S),
                                               Tre, Tim);
  eps_kernel<<<1, 1024, 0, st>>>(el, S, S32, T + (size_t)S32 * S32 * 2);
  const int64_t ntri = nblk * (nblk + 1) / 2;
  prof_begin(c, K_GRAM, st);
  if constexpr (sizeof(RG) == 4) {
    const int gt = gram_tile(S32, c->n_cu > 0 ? c->n_cu : 256);
    const int64_t ntile = (S32 + gt - 1) / gt;
    auto kernel = gt == 96 ? gram_tile_kernel<96> : gram_tile_kernel<64>;
    kernel<<<(unsigned)(ntile * (ntile + 1) / 2), 256, 0, st>>>((const float*)Tre, (const float*)Tim,
                                                                Pk, S32, lambda, T);
  } else {
    gram_kernel<RG><<<(unsigned)((ntri + 3) / 4), 256, 0, st>>>(Tre, Tim, Pk, S32, nblk, lambda, T);
  }
  prof_end(c, K_GRAM, st);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  prof_begin(c, K_CHOL, st);
  double2* T2 = (double2*)T;
  for (int64_t K0 = 0; K0 < nblk; K0 += kPanel) {
    const int64_t K1 = std::min<int64_t>(K0 + kPanel, nblk);
    for (int64_t k = K0; k < K1; ++k) {
      potrf_diag_kernel<<<1, kDT, 0, st>>>(T2, S32, k, K0 * kB, Linv, flag);
      trsm_panel_kernel<<<(unsigned)(nblk - k), 256, 0, st>>>(T2, S32, k, K0 * kB, Linv);
    }
    if (K1 < nblk) {
      const int64_t m = nblk - K1, nt = m * (m + 1) / 2 + m;
      herk_update_kernel<<<(unsigned)((nt + 3) / 4), 256, 0, st>>>(T, S32, K0, (int)(K1 - K0), K1, nblk);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  take_y_kernel<<<(unsigned)((S32 + 255) / 256), 256, 0, st>>>(T2, S32, (double2*)v);
  for (int64_t K0 = (nblk - 1) / kPanel * kPanel; K0 >= 0; K0 -= kPanel) {
    const int nk = (int)(std::min<int64_t>(K0 + kPanel, nblk) - K0);
    bsolve_panel_kernel<<<1, 256, 0, st>>>(T2, S32, K0, nk, Linv, (double2*)v);
    if (K0 > 0)
      bsolve_update_kernel<<<(unsigned)((K0 * kB + 63) / 64), 1024, 0, st>>>(T2, S32, K0, nk, (double2*)v);
  }
  prof_end(c, K_CHOL, st);
  dtheta_kernel<RG><<<(unsigned)((P + 3) / 4), 256, 0, st>>>(Tre, Tim, P, S32, v, dtau, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(flag_host, flag, sizeof(int), hipMemcpyDeviceToHost, st)) != hipSuccess)
    return e;
  return hipStreamSynchronize(st);
}

}  // namespace

size_t sr_workspace_bytes(const nqs_ctx* c, int64_t S) {
  const int64_t S32 = r32(std::max<int64_t>(S, 1)), Pk = rk(c->P);
  const size_t rg = c->prec == NQS_FP64 ? 8 : 4;
  return al((size_t)(S32 + kB) * S32 * 16) + al((size_t)S32 * kB * 16) + 2 * al((size_t)Pk * S32 * rg) + al((size_t)S32 * 16) +
         al((size_t)c->P * 16) + al(64);
}

}  // namespace nqs

using namespace nqs;

extern "C" nqs_status nqs_sr_solve(nqs_ctx* c, const void* O, const double* eloc, int64_t S,
                                   double lambda, double dtau, double* dtheta_out, void* ws,
                                   size_t ws_bytes, hipStream_t st) {
  if (!c) return NQS_ERR_ARG;
  auto fail = [&](nqs_status s, const std::string& m) {
    c->last_error = m;
    return s;
  };
  if (S < 1 || !O || !eloc || !dtheta_out) return fail(NQS_ERR_ARG, "sr_solve: bad arguments");
  if (!(lambda >= 0.0) || !std::isfinite(lambda) || !std::isfinite(dtau))
    return fail(NQS_ERR_ARG, "sr_solve: lambda must be finite and >= 0, dtau finite");
  const size_t need = sr_workspace_bytes(c, S);
  if (!ws || ws_bytes < need)
    return fail(NQS_ERR_ARG, "sr_solve: workspace too small: need " + std::to_string(need));
  int flag = 0;
  prof_begin(c, K_SR, st);
  const hipError_t e =
      c->prec == NQS_FP64
          ? sr_run<double, double>(c, O, eloc, S, lambda, dtau, dtheta_out, ws, st, &flag)
          : sr_run<float, float>(c, O, eloc, S, lambda, dtau, dtheta_out, ws, st, &flag);
  prof_end(c, K_SR, st);
  if (e != hipSuccess) return fail(NQS_ERR_DEVICE, std::string("sr_solve: ") + hipGetErrorString(e));
  if (flag) return fail(NQS_ERR_NOT_PD, "sr_solve: Gram matrix is not positive definite");
  return NQS_OK;
}
