// Bond-exchange sums of E_loc (Sec. 3.2, Eq. (10)) from stored t = tanh(theta)
// and image weights w, FP32, any number of hidden units: the models without a
// register-resident bond kernel.
//
// Same work split as the wide kernel (k_eloc_wide.hip): a wavefront takes one
// (configuration, 16-image block); lane (q, c) holds image c and the bonds
// q + 4 jb of the antiparallel list; the eight wavefronts of a workgroup walk
// the hidden units in lockstep in chunks of 8, the chunk's rows of the bond
// table T = tanh(D) staged in LDS for all of them (double-buffered through
// registers).  t of the chunk is one 64-byte run per image, read one chunk
// ahead.
//
// Bound: VALU issue of the factors F prod_h (s + t_h T_h), 8 instructions each,
// 132 per pair of bonds and chunk with the two addresses and signs.  At 8x8
// M = 128, 2003 configurations: 4.3 ms (a VALU instruction in 3.9 cycles) where a kernel
// that reads every T row from L2 per (image, bond) took 18.6 ms, and one whose
// eight wavefronts share a configuration 4.7 ms; nqs_eloc at 10x10 M = 104, 500
// configurations 8.4, 2.9 and 2.7 ms; 6x6 K = 3 M = 24, 3000 configurations 4.2,
// 2.1 and 1.6 ms; seven at 6x6 M = 40 117, 59 and 44 us.
// Every product is formed in the order and with the roundings of
// F prod_h (1 + t_h (+-T_h)).  Placing the rows by bank group, as the wide
// kernel does, measured the same.
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

// Bond slots per lane (even), four lane groups: 40, 88, 144 and 224 bonds cover
// the antiparallel bonds of nearly every Sz = 0 configuration (mean
// 2 N N / (N - 1): 34, 74, 130, 202), so t and the bond table are read once.
template <int N>
constexpr int row_bonds() { return N == 16 ? 10 : N == 36 ? 22 : N == 64 ? 36 : 56; }

// Workgroups per compute unit: at 4x4 a walk is short (five pairs of slots a
// chunk), and a second workgroup fills its list building and barriers
// (nqs_eloc at M = 64, 5000 configurations: 0.61 -> 0.47 ms).
template <int N>
constexpr int row_wgs() { return N == 16 ? 2 : 1; }

// LDS, in bytes: the staged chunks lie a power of two apart, so that a row's
// address is (offset | buffer bit); the small arrays lie between them.
template <int N>
struct RowsCfg {
  static constexpr int NB = 4 * N;
  static constexpr uint32_t CAP = NB * kRowBytes;
  static constexpr uint32_t BUF = N == 16 ? 1u << 13 : N == 36 ? 1u << 14 : N == 64 ? 1u << 15 : 1u << 16;
  static constexpr uint32_t LIST = CAP;                        // [waves][NB] uint16
  static constexpr uint32_t BUSY = LIST + kRowWaves * NB * 2;  // [waves] int
  static constexpr uint32_t LDS = BUF + CAP;
  static_assert(BUSY + kRowWaves * 4 <= BUF, "the small arrays fit between the chunks");
};

// per: items of a workgroup in a round (its first `per` wavefronts take them)
template <int N>
__global__ __launch_bounds__(64 * kRowWaves, 2 * row_wgs<N>()) void eloc_rows_kernel(
    const int8_t* __restrict__ spins, int64_t S, int per, int K, int M,
    const int32_t* __restrict__ bonds, const int32_t* __restrict__ bmap,
    const float* __restrict__ t, const float* __restrict__ w, const float* __restrict__ Tpm,
    const float* __restrict__ F, double* __restrict__ partial) {
  using Cfg = RowsCfg<N>;
  constexpr int NB = Cfg::NB, G = 8 * N, nblk = G / 16, THREADS = 64 * kRowWaves;
  constexpr int WB = row_bonds<N>();
  constexpr int E4 = NB * 4, NSTG = (E4 + THREADS - 1) / THREADS;   // float4 of a chunk
  static_assert(WB % 2 == 0, "the products run two bonds at a time");
  constexpr bool PACK = N == 100;              // two bond slots' offsets in a register
  constexpr int OW = PACK ? WB / 2 : WB;
  // aligned to the chunk distance, so that addresses are ORs
  __shared__ __align__(Cfg::BUF) unsigned char lds[Cfg::LDS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, c = lane & 15;
  const int KM = K * M, NCH = KM / 8, CPR = M / 8;
  uint16_t* list = reinterpret_cast<uint16_t*>(lds + Cfg::LIST) + wv * NB;
  int* busy = reinterpret_cast<int*>(lds + Cfg::BUSY);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // staging of chunk ch: float4 e = tid + 512 i -> row e / 4, part e % 4 of
  // tanh(D); thread tid < NB also stages (F_+, F_-) of row tid for its RBM k
  f32x4 stg[NSTG], sF;
  const uint32_t sofs = (uint32_t)(tid >> 2) * 16u * (uint32_t)KM + 16u * (tid & 3);
  auto stage_load = [&](int ch, int k) __attribute__((always_inline)) {
    const char* b = reinterpret_cast<const char*>(Tpm) + (size_t)ch * 64;
#pragma unroll
    for (int i = 0; i < NSTG; ++i)
      if (THREADS * (i + 1) <= E4 || tid + THREADS * i < E4)
        stg[i] = *reinterpret_cast<const f32x4*>(b + (size_t)i * (THREADS / 4) * 16 * KM + sofs);
    if (tid < NB) sF = *reinterpret_cast<const f32x4*>(F + ((size_t)k * NB + tid) * 4);
  };
  auto stage_store = [&](uint32_t buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NSTG; ++i)
      if (THREADS * (i + 1) <= E4 || tid + THREADS * i < E4)
        *reinterpret_cast<f32x4*>(lds + buf + kRowBytes * ((tid + THREADS * i) >> 2) +
                                  16 * (tid & 3)) = stg[i];
    if (tid < NB) *reinterpret_cast<f32x4*>(lds + buf + kRowBytes * tid + 64) = sF;
  };
  stage_load(0, 0);
  stage_store(0);
  uint32_t buf = 0;                            // byte offset of the chunk in use

  const int64_t n_items = S * nblk;
  int64_t item = (int64_t)blockIdx.x * per + wv;
  bool act = wv < per && item < n_items;
  bool first = true;                           // first walk of the item
  int64_t s = 0;
  int blk = 0, e0 = 0, nc = 0;                 // list entries from e0 on in this and later walks
  double Qr = 0.0, Qi = 0.0;

  for (;;) {
    if (lane == 0) busy[wv] = act;
    __syncthreads();                           // also: the walk's first chunk is staged
    if (__ballot(lane < kRowWaves && busy[lane & (kRowWaves - 1)] != 0) == 0ull) break;
    // a walk over the hidden units: bonds e0 + q + 4 jb of the list
    uint32_t offs[OW];                         // row offset in bytes, bit 0: s = -1
    int nv = 0, nvu = 0;                       // slots in use in the lane, and in lane group 0
    const f32x4* tg = reinterpret_cast<const f32x4*>(t);
    f32x4 tn[4];
    if (act) {
      if (first) {
        s = item / nblk;
        blk = (int)(item - s * nblk);
        const int8_t* srow = spins + s * N;
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
        wave_sync_lds();
        nc = n;
        e0 = 0;
        Qr = Qi = 0.0;
      }
      const int g = blk * 16 + c;
      tg += ((size_t)s * NCH * G + g) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) tn[e] = tg[e];
      nv = nc > e0 + q ? min(WB, (nc - e0 - q + 3) / 4) : 0;
      nvu = __builtin_amdgcn_readfirstlane(nv);
#pragma unroll
      for (int jb = 0; jb < WB; ++jb) {
        const int e = jb < nv ? list[e0 + q + 4 * jb] : 0;   // padding entries use bond 0
        const uint32_t v = (uint32_t)(bmap[(size_t)g * NB + (e & 0x7fff)] ^ (e >> 15));
        const uint32_t o = kRowBytes * (v >> 1) | (v & 1u);
        if constexpr (!PACK) offs[jb] = o;
        else if (jb & 1) offs[jb / 2] |= o << 16;
        else offs[jb / 2] = o;
      }
      e0 += 4 * WB;
    } else {
#pragma unroll
      for (int i = 0; i < OW; ++i) offs[i] = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) tn[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    float Pr[WB], Pi[WB];
    int k = 0, cin = 0;                        // RBM, chunk within it
    for (int ch = 0; ch < NCH; ++ch) {
      const bool last = ch + 1 == NCH;
      const uint32_t base = lds0 | buf;
      // keep the comparisons with these in the loop: hoisted, they fill registers
      nvu = __builtin_amdgcn_readfirstlane(nvu);
      asm volatile("" : "+s"(nvu), "+v"(nv));
      if (cin == 0) {                          // RBM start: products begin at F_s
#pragma unroll
        for (int jb = 0; jb < WB; ++jb) {
          const uint32_t o = PACK ? (jb & 1 ? offs[jb / 2] >> 16 : offs[jb / 2]) : offs[jb];
          const f32x2 f = *(lds_f32x2_ptr)(((o & 0xfff0u) | base) + 64u + 8u * (o & 1u));
          Pr[jb] = f.x;
          Pi[jb] = f.y;
        }
      }
      f32x4 tv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) tv[e] = tn[e];
      if (act) {
#pragma unroll
        for (int e = 0; e < 4; ++e) tn[e] = tg[(size_t)(last ? 0 : ch + 1) * G * 4 + e];
      }
      // lands during the bond products
      stage_load(last ? 0 : ch + 1, last ? 0 : cin + 1 == CPR ? k + 1 : k);
#pragma unroll
      for (int jb = 0; jb < WB; jb += 2) {
        if (jb < nvu) {
          uint32_t o0, o1;
          if constexpr (PACK) {
            asm volatile("" : "+v"(offs[jb / 2]));
            o0 = offs[jb / 2];
            o1 = o0 >> 16;
          } else {
            asm volatile("" : "+v"(offs[jb]), "+v"(offs[jb + 1]));
            o0 = offs[jb];
            o1 = offs[jb + 1];
          }
          const lds_f32x4_ptr r0 = (lds_f32x4_ptr)((PACK ? o0 & 0xfff0u : o0 & ~15u) | base);
          const lds_f32x4_ptr r1 = (lds_f32x4_ptr)((o1 & ~15u) | base);
          const float sg0 = __uint_as_float((o0 << 31) | 0x3f800000u);
          const float sg1 = __uint_as_float((o1 << 31) | 0x3f800000u);
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
      if (++cin == CPR) {                      // RBM k complete: weight and sum
        if (act) {
          const float* wk = w + (((size_t)s * K + k) * G + blk * 16 + c) * 2;
          const float wr = wk[0], wi = wk[1];
#pragma unroll
          for (int jb = 0; jb < WB; ++jb) {
            if (jb < nvu) {
              Qr += jb < nv ? (double)(wr * Pr[jb] - wi * Pi[jb]) : 0.0;
              Qi += jb < nv ? (double)(wr * Pi[jb] + wi * Pr[jb]) : 0.0;
            }
          }
        }
        cin = 0;
        ++k;
      }
      buf ^= Cfg::BUF;
      stage_store(buf);
      __syncthreads();
    }

    if (act) {
      first = false;
      if (e0 >= nc) {                          // the item's last walk
        Qr = wave_sum(Qr);
        Qi = wave_sum(Qi);
        if (lane == 0) {
          partial[2 * item] = Qr;
          partial[2 * item + 1] = Qi;
        }
        item += (int64_t)gridDim.x * per;
        act = item < n_items;
        first = true;
      }
    }
  }
}

template <int N>
hipError_t run(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t, const void* w,
               double* partial, hipStream_t st) {
  if (S <= 0) return hipSuccess;
  const int64_t n_wg = (c->n_cu > 0 ? c->n_cu : 256) * row_wgs<N>(), items = S * (c->G / 16);
  // fewer items than wavefront slots: the same number in every workgroup
  const int per = (int)std::min<int64_t>(kRowWaves, (items + n_wg - 1) / n_wg);
  const int64_t blocks = std::min<int64_t>((items + per - 1) / per, n_wg);
  eloc_rows_kernel<N><<<(unsigned)blocks, 64 * kRowWaves, 0, st>>>(
      spins, S, per, c->K, c->M, c->dev.bonds, c->dev.bmap, (const float*)t, (const float*)w,
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
