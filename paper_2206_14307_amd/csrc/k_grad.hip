// Log-derivatives O_k = d log psi / d theta_k (Sec. 3.2, below Eq. (12)).
//
// With the normalised image weights w_kg = chi_g psi_s^(k)(g sigma)/psi(sigma),
// t = tanh(theta) and the images x_g = g sigma:
//   O_W[k][h][j] = sum_g w_kg t_kgh x_gj,  O_b[k][h] = sum_g w_kg t_kgh,
//   O_a[k][j]    = sum_g w_kg x_gj.
// Per sample this is one contraction over the G images,
// (interleaved Re/Im rows of w t, plus rows of w) x (images x [sites | 1]),
// run on 16x16x4 MFMA (FP32 or FP64): an all-ones column yields O_b (where N
// is a multiple of 16, so that the column would need a block of its own, the
// lanes sum their A values instead), extra w rows yield O_a.
//
// A workgroup of four wavefronts takes one sample (or a share of its row tiles,
// for calls too small to fill the device); each wavefront takes every fourth
// 16-row tile with all site-column blocks accumulated side by side.  The images
// are gathered once per workgroup, as sign bits in LDS: one word gives a lane
// its B operands of 16 images.  t and w of the next 16 images are loaded while
// the current ones multiply.
//
// Bound: the FP32 MFMA issue (0.23 ms at 8x8 M = 128, 2003 samples) beside the
// VALU that makes its operands, and the read of t (1.05 GB, 0.22 ms).  nqs_grad
// of those samples, theta and weights included: 1.84 ms with a wavefront per
// (sample, row tile) that gathered every B operand through the permutation and
// the spins, 1.27 ms now; five samples 110 and 61 us; FP64 4x4 M = 64, 5000
// samples 0.62 and 0.47 ms.
#include "device_common.h"
#include "nqs_internal.h"
#include "theta_common.h"

namespace nqs {

namespace {

template <typename R> struct AccOf;
template <> struct AccOf<double> { using type = f64x4; };
template <> struct AccOf<float> { using type = f32x4; };

// +1/2, or -1/2 if bit b of v is set
template <typename R>
__device__ __forceinline__ R half_signed(uint32_t v, int b) {
  const uint32_t sg = (v << (31 - b)) & 0x80000000u;
  if constexpr (sizeof(R) == 4) return __uint_as_float(sg | 0x3f000000u);
  else return __longlong_as_double((long long)((uint64_t)(sg | 0x3fe00000u) << 32));
}

template <typename R, int N>
__global__ __launch_bounds__(256) void grad_kernel(
    const int8_t* __restrict__ spins, const uint8_t* __restrict__ perm, int K, int M, int n_htiles,
    int use_bias, int Prbm, int64_t P, const R* __restrict__ t, const R* __restrict__ w,
    R* __restrict__ O) {
  using Acc = typename AccOf<R>::type;
  using R2 = c2_t<R>;
  constexpr int G = 8 * N, NM = G / 16;
  constexpr bool ONES = N % 16 != 0;                 // the ones column is in the last block
  constexpr int NJB = (N + 15) / 16;
  static_assert(NJB <= 8, "a byte of sign bits per image and column");
  __shared__ uint32_t xb[NM][64];                    // byte e: columns 16 jb + i of image 16 m + 4 e + kq
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int i = lane & 15, kq = lane >> 4;
  const int64_t s = blockIdx.x;
  const SpinBits sb = spin_bits<N>(spins + s * N);
  for (int m = wv; m < NM; m += 4) {
    uint32_t v = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint8_t* prow = perm + (size_t)(16 * m + 4 * e + kq) * N;
#pragma unroll
      for (int jb = 0; jb < NJB; ++jb)
        if (16 * jb + i < N) v |= (x_bits<N>(sb, prow[16 * jb + i]) >> 31) << (8 * e + jb);
    }
    xb[m][lane] = v;
  }
  __syncthreads();
  const int li = logical_row<R>(i);                  // logical A row of this lane
  const int n_rt = n_htiles + (use_bias ? K : 0);
  const int jl = 16 * (NJB - 1) + i;                 // this lane's column of the last block
  const R bl = jl == N ? R(1) : R(0);

  for (int rt = blockIdx.y * 4 + wv; rt < n_rt; rt += 4 * gridDim.y) {
    const bool wrow = rt < n_htiles;
    const int hrow = 8 * rt + li / 2;                // hidden unit of this A row (W tiles)
    const int krow = wrow ? hrow / M : rt - n_htiles;  // RBM of this A row
    const R2* ws = reinterpret_cast<const R2*>(w) + ((size_t)s * K + krow) * G + kq;
    const R2* ts = reinterpret_cast<const R2*>(t) +
                   (((size_t)s * n_htiles + (wrow ? rt : 0)) * G + kq) * 8 + li / 2;
    Acc acc[NJB];
#pragma unroll
    for (int jb = 0; jb < NJB; ++jb) acc[jb] = Acc{0, 0, 0, 0};
    R ob = R(0);
    R2 wn[4], tn[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      wn[e] = ws[4 * e];
      tn[e] = ts[32 * e];
    }
#pragma unroll 1
    for (int m = 0; m < NM; ++m) {
      const uint32_t v = xb[m][lane];
      R2 wc[4], tc[4];
      const int mn = min(m + 1, NM - 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        wc[e] = wn[e];
        tc[e] = tn[e];
        wn[e] = ws[16 * mn + 4 * e];
        tn[e] = ts[128 * mn + 32 * e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const R wr = wc[e].x, wi = wc[e].y;
        R a;
        if (wrow) {
          const R tr = tc[e].x, ti = tc[e].y;
          a = (li & 1) ? (wr * ti + wi * tr) : (wr * tr - wi * ti);
        } else {
          a = li == 0 ? wr : (li == 1 ? wi : R(0));
        }
        if constexpr (!ONES) ob += a;
        R b[NJB];
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) {
          b[jb] = half_signed<R>(v, 8 * e + jb);
          if (ONES && jb == NJB - 1) b[jb] = jl < N ? b[jb] : bl;
        }
#pragma unroll
        for (int jb = 0; jb < NJB; ++jb) acc[jb] = mfma(a, b[jb], acc[jb]);
      }
    }
    // lane (kq, i) holds rows 4 kq .. 4 kq + 3 of column 16 jb + i
    R* Os = O + (size_t)s * P * 2;
#pragma unroll
    for (int jb = 0; jb < NJB; ++jb) {
      const int j = 16 * jb + i;
      if (j > N) continue;
      if (wrow) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int h = 8 * rt + 2 * kq + u;
          const int k = h / M, hh = h % M;
          size_t idx;
          if (j < N) idx = (size_t)k * Prbm + (size_t)hh * N + j;
          else if (use_bias) idx = (size_t)k * Prbm + (size_t)M * N + N + hh;
          else continue;
          Os[2 * idx] = (R)acc[jb][2 * u];
          Os[2 * idx + 1] = (R)acc[jb][2 * u + 1];
        }
      } else if (kq == 0 && j < N) {
        const size_t idx = (size_t)krow * Prbm + (size_t)M * N + j;
        Os[2 * idx] = (R)acc[jb][0];
        Os[2 * idx + 1] = (R)acc[jb][1];
      }
    }
    if constexpr (!ONES) {
      // O_b: A row li summed over the images (4 lanes hold a quarter each)
      ob += __shfl_xor(ob, 16, 64);
      ob += __shfl_xor(ob, 32, 64);
      if (wrow && use_bias && kq == 0) {
        const size_t idx = (size_t)krow * Prbm + (size_t)M * N + N + (hrow - krow * M);
        Os[2 * idx + (li & 1)] = ob;
      }
    }
  }
}

template <typename R, int N>
hipError_t grad_for(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t, const void* w,
                    void* O, hipStream_t st) {
  const int n_rt = c->n_htiles + (c->d.use_bias ? c->K : 0);
  // few samples: their row tiles go to several workgroups (each gathers the images)
  const int64_t n_cu = c->n_cu > 0 ? c->n_cu : 256;
  const int ny = (int)std::max<int64_t>(1, std::min<int64_t>((n_rt + 3) / 4, 4 * n_cu / S));
  grad_kernel<R, N><<<dim3((unsigned)S, (unsigned)ny), 256, 0, st>>>(
      spins, c->dev.perm, c->K, c->M, c->n_htiles, c->d.use_bias, c->P_rbm, c->P, (const R*)t,
      (const R*)w, (R*)O);
  return hipGetLastError();
}

template <typename R>
hipError_t grad_typed(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t,
                      const void* w, void* O, hipStream_t st) {
  switch (c->L) {
    case 4: return grad_for<R, 16>(c, spins, S, t, w, O, st);
    case 6: return grad_for<R, 36>(c, spins, S, t, w, O, st);
    case 8: return grad_for<R, 64>(c, spins, S, t, w, O, st);
    default: return grad_for<R, 100>(c, spins, S, t, w, O, st);
  }
}

}  // namespace

hipError_t launch_grad(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t,
                       const void* w, void* O, hipStream_t st) {
  if (S <= 0) return hipSuccess;
  return c->prec == NQS_FP64 ? grad_typed<double>(c, spins, S, t, w, O, st)
                             : grad_typed<float>(c, spins, S, t, w, O, st);
}

}  // namespace nqs
