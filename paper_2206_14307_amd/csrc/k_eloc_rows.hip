// Bond-exchange sums of E_loc (Sec. 3.2, Eq. (10)) from stored t = tanh(theta)
// and image weights w, FP32, any number of hidden units: the models without a
// register-resident bond kernel.
//
// Same work split as the wide kernel (k_eloc_wide.hip): a workgroup of eight
// wavefronts takes one configuration, a wavefront one 16-image block; lane
// (q, c) holds image c and the bonds q + 4 jb of the antiparallel list; the
// hidden units are walked in chunks of 8, the chunk's rows of the bond table
// T = tanh(D) staged in LDS for all wavefronts (double-buffered through
// registers).  t of the chunk is one 64-byte run per image, read one chunk
// ahead.
//
// Bound: VALU issue of the factors F prod_h (s + t_h T_h), 8 instructions each,
// 130 per pair of bonds and chunk with the two addresses and signs.  At 8x8
// M = 128, 2003 configurations: 4.7 ms (0.73 of the issue bound) where the
// kernel before it, which read every T row from L2 per (image, bond), took
// 18.6 ms; 10x10 M = 104, 500 configurations 2.4 against 8.0 ms.  Every product is
// formed in the order and with the roundings of F prod_h (1 + t_h (+-T_h)).
// Placing the rows by bank group, as the wide kernel does, measured the same.
#include "device_common.h"
#include "nqs_internal.h"

namespace nqs {

namespace {

constexpr int kRowWaves = 8;
typedef __attribute__((address_space(3))) const f32x4* lds_f32x4_ptr;
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const f32x2* lds_f32x2_ptr;
constexpr int kRowBytes = 80;             // staged row: T of 8 units, F_+, F_- (an odd number
                                          // of 16-byte units: rows spread over the bank groups)
constexpr uint32_t kBufStride = 1u << 16;   // bytes between the two staged chunks

// Bond slots per lane (even), four lane groups: they cover the antiparallel bonds of nearly
// every Sz = 0 configuration (mean 2 N N / (N - 1): 34, 74, 130, 202) in one
// pass, at 10x10 in two; each pass reads t and the bond table again.
template <int N>
constexpr int row_bonds() { return N == 16 ? 10 : N == 36 ? 20 : N == 64 ? 36 : 28; }

template <int N>
__global__ __launch_bounds__(64 * kRowWaves) void eloc_rows_kernel(
    const int8_t* __restrict__ spins, int64_t S, int rsplit, int K, int M,
    const int32_t* __restrict__ bonds,
    const int32_t* __restrict__ bmap, const float* __restrict__ t, const float* __restrict__ w, const float* __restrict__ Tpm,
    const float* __restrict__ F, double* __restrict__ partial) {
  constexpr int NB = 4 * N, G = 8 * N, nblk = G / 16, THREADS = 64 * kRowWaves;
  constexpr int WB = row_bonds<N>();
  constexpr int E4 = NB * 4, NSTG = (E4 + THREADS - 1) / THREADS;   // float4 of a chunk
  constexpr int rounds = (nblk + kRowWaves - 1) / kRowWaves;
  static_assert(WB % 2 == 0, "the products run two bonds at a time");
  constexpr int CAP = NB * kRowBytes;        // bytes of a staged chunk
  static_assert(CAP <= (int)kBufStride, "a chunk fits below the second buffer");
  // chunk buffers 64 KiB apart, so that a row's LDS address is (offset | buffer
  // bit) without an addition per bond; the space between holds nothing
  __shared__ __align__(16) unsigned char Tc[kBufStride + CAP];
  __shared__ uint16_t list[NB];
  __shared__ int nc_s;

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int q = lane >> 4, c = lane & 15;
  const int KM = K * M, NCH = KM / 8, CPR = M / 8;

  f32x4 stg[NSTG], sF;
  auto stage_load = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i) {
      const int e = min(tid + THREADS * i, E4 - 1);
      stg[i] = *reinterpret_cast<const f32x4*>(Tpm + (size_t)(e / 4) * 4 * KM + 16 * ch + 4 * (e % 4));
    }
    sF = *reinterpret_cast<const f32x4*>(F + ((size_t)(ch / CPR) * NB + (tid < NB ? tid : 0)) * 4);
  };
  auto stage_store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i) {
      const int e = tid + THREADS * i;
      if (e < E4)
        *reinterpret_cast<f32x4*>(&Tc[buf * kBufStride + kRowBytes * (e / 4) + 16 * (e % 4)]) = stg[i];
    }
    if (tid < NB) *reinterpret_cast<f32x4*>(&Tc[buf * kBufStride + kRowBytes * tid + 64]) = sF;
  };
  stage_load(0);
  stage_store(0);
  const uint32_t tc0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)Tc;
  int gc = 0;                                  // chunks processed by the workgroup so far

  // work items: configurations, or (rsplit) rounds of eight image blocks of them
  const int64_t n_items = rsplit ? S * rounds : S;
  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    const int64_t s = rsplit ? item / rounds : item;
    const int rd0 = rsplit ? (int)(item - s * rounds) : 0, rd1 = rsplit ? rd0 + 1 : rounds;
    const int8_t* srow = spins + s * N;
    __syncthreads();                           // previous configuration done with the list
    if (wv == 0) {
      int n = 0;
      for (int base = 0; base < NB; base += 64) {
        const int b = base + lane;
        bool anti = false;
        int sp = 0;
        if (b < NB) {
          sp = srow[bonds[2 * b]];
          anti = sp != srow[bonds[2 * b + 1]];
        }
        const unsigned long long msk = __ballot(anti);
        const int pos = __popcll(msk & ((1ull << lane) - 1ull));
        if (anti) list[n + pos] = (uint16_t)(b | (sp > 0 ? 0x8000 : 0));
        n += __popcll(msk);
      }
      if (lane == 0) nc_s = n;
    }
    __syncthreads();
    const int nc = nc_s;
    const int npass = nc > 0 ? (nc + 4 * WB - 1) / (4 * WB) : 1;

    for (int rd = rd0; rd < rd1; ++rd) {
      const int blk = rd * kRowWaves + wv;
      const bool active = blk < nblk;
      const int g = (active ? blk : 0) * 16 + c;
      double Qr = 0.0, Qi = 0.0;
      const f32x4* tg = reinterpret_cast<const f32x4*>(t) + ((size_t)s * NCH * G + g) * 4;

      for (int pass = 0; pass < npass; ++pass) {
        uint32_t offs[WB];                     // row offset in bytes, bit 0: s = -1
        const int i0 = pass * 4 * WB + q;
        const int nv = nc > i0 ? min(WB, (nc - i0 + 3) / 4) : 0;
        // bonds of lane group 0 (the most of any group): a partly filled pass
        // skips the empty pairs of slots
        const int p0 = pass * 4 * WB;
        const int nvu = __builtin_amdgcn_readfirstlane(nc > p0 ? min(WB, (nc - p0 + 3) / 4) : 0);
#pragma unroll
        for (int jb = 0; jb < WB; ++jb) {
          const int ii = i0 + 4 * jb;
          const int e = ii < nc ? list[ii] : 0;   // padding entries use bond 0
          const int v = bmap[(size_t)g * NB + (e & 0x7fff)] ^ (e >> 15);
          offs[jb] = (uint32_t)(kRowBytes * (v >> 1)) | (uint32_t)(v & 1);
        }
        float Pr[WB], Pi[WB];
        f32x4 tn[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) tn[e] = tg[e];

        for (int ch = 0; ch < NCH; ++ch, ++gc) {
          const int buf = gc & 1;
          const int nxt = ch + 1 < NCH ? ch + 1 : 0;
          const uint32_t base = tc0 + (buf ? kBufStride : 0u);
          if (ch % CPR == 0) {                 // RBM start: products begin at F_s
#pragma unroll
            for (int jb = 0; jb < WB; ++jb) {
              const f32x2 f = *(lds_f32x2_ptr)((offs[jb] & ~1u) + base + 64u + 8u * (offs[jb] & 1u));
              Pr[jb] = f.x;
              Pi[jb] = f.y;
            }
          }
          f32x4 tv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            tv[e] = tn[e];
            tn[e] = tg[(size_t)nxt * G * 4 + e];
          }
          stage_load(nxt);                     // lands during the bond products
#pragma unroll
          for (int jb = 0; jb < WB; jb += 2) {
            if (jb < nvu) {
              const lds_f32x4_ptr r0 = (lds_f32x4_ptr)((offs[jb] & ~1u) + base);
              const lds_f32x4_ptr r1 = (lds_f32x4_ptr)((offs[jb + 1] & ~1u) + base);
              const float sg0 = __uint_as_float((offs[jb] << 31) | 0x3f800000u);
              const float sg1 = __uint_as_float((offs[jb + 1] << 31) | 0x3f800000u);
              float ar = Pr[jb], ai = Pi[jb], br = Pr[jb + 1], bi = Pi[jb + 1];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const f32x4 x0 = r0[e];
                const f32x4 x1 = r1[e];
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                  const float tr = tv[e][2 * hh], ti = tv[e][2 * hh + 1];
                  float pa = fmaf(tr, x0[2 * hh], fmaf(-ti, x0[2 * hh + 1], sg0));
                  float pb = fmaf(tr, x0[2 * hh + 1], ti * x0[2 * hh]);
                  float nr = fmaf(ar, pa, -(ai * pb));
                  ai = fmaf(ar, pb, ai * pa);
                  ar = nr;
                  pa = fmaf(tr, x1[2 * hh], fmaf(-ti, x1[2 * hh + 1], sg1));
                  pb = fmaf(tr, x1[2 * hh + 1], ti * x1[2 * hh]);
                  nr = fmaf(br, pa, -(bi * pb));
                  bi = fmaf(br, pb, bi * pa);
                  br = nr;
                }
              }
              Pr[jb] = ar; Pi[jb] = ai; Pr[jb + 1] = br; Pi[jb + 1] = bi;
            }
          }
          if (ch % CPR == CPR - 1) {           // RBM k complete: weight and sum
            const float* wk = w + (((size_t)s * K + ch / CPR) * G + g) * 2;
            const float wr = wk[0], wi = wk[1];
#pragma unroll
            for (int jb = 0; jb < WB; ++jb) {
              Qr += jb < nv ? (double)(wr * Pr[jb] - wi * Pi[jb]) : 0.0;
              Qi += jb < nv ? (double)(wr * Pi[jb] + wi * Pr[jb]) : 0.0;
            }
          }
          stage_store(buf ^ 1);
          __syncthreads();
        }
      }
      Qr = wave_sum(Qr);
      Qi = wave_sum(Qi);
      if (active && lane == 0) {
        double* o = partial + ((size_t)s * nblk + blk) * 2;
        o[0] = Qr;
        o[1] = Qi;
      }
    }
  }
}

template <int N>
hipError_t run(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t, const void* w,
               double* partial, hipStream_t st) {
  // few configurations: their rounds of image blocks go to different workgroups
  const int n_cu = c->n_cu > 0 ? c->n_cu : 256, rounds = (c->G / 16 + kRowWaves - 1) / kRowWaves;
  const int rsplit = S < 4 * (int64_t)n_cu && rounds > 1;
  const int64_t blocks = std::min<int64_t>(rsplit ? S * rounds : S, n_cu);
  eloc_rows_kernel<N><<<(unsigned)blocks, 64 * kRowWaves, 0, st>>>(
      spins, S, rsplit, c->K, c->M, c->dev.bonds, c->dev.bmap, (const float*)t, (const float*)w,
       (const float*)c->par.Tpm, (const float*)c->par.F, partial);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_eloc_rows(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t,
                            const void* w, double* partial, hipStream_t st) {
  switch (c->N) {
    case 16: return run<16>(c, spins, S, t, w, partial, st);
    case 36: return run<36>(c, spins, S, t, w, partial, st);
    case 64: return run<64>(c, spins, S, t, w, partial, st);
    case 100: return run<100>(c, spins, S, t, w, partial, st);
    default: return hipErrorNotSupported;
  }
}

}  // namespace nqs
