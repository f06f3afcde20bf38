// Fused log psi + E_loc (Sec. 3.1 Eqs. (2), (6); Sec. 3.2 Eq. (10)) for
// models whose hidden layer does not fit in registers (K*M > 128,
// M a multiple of 16), with theta in FP32 or split BF16.
//
// A work item is one 16-image column block of one configuration (or a share of
// its bond list, for calls too small to fill the device); a wavefront walks
// the hidden units of its item in chunks of kHC, in lockstep with the other
// seven wavefronts of its workgroup, which are at items of their own:
//   * the chunk's rows of the bond table T = tanh(D) (all 4N bonds x kHC units)
//     are staged in LDS for all of them, double-buffered: each thread loads its
//     share of the next chunk into registers before the bond products and
//     stores it after them;
//   * theta of the chunk runs on 16x16 MFMA with the W fragments read from L2,
//     and the log 2cosh / tanh epilogue accumulates log psi of the images;
//   * tanh(theta) of the chunk goes through a small LDS tile so that lane
//     (q, c) holds all kHC values of image c, and the lane multiplies the
//     running products F_s prod_h (s + t_h T_h) of its bonds q + 4 jb
//     (jb < wide_bonds) of the list, the bond rows read from LDS.
// At the end of each RBM the products are weighted with the image weights
// u = chi e^{L - m} (m a running maximum over the RBMs of the wave's images)
// and summed; the wave emits (m, sum u, sum u R) per item in the same format as
// the fused kernel, combined by its finish kernel.  The shares of a small call
// store their products instead, and wide_join_kernel sums and weights a block's
// whole list as an unsplit wavefront does: a configuration's results are the same
// bits whatever the call that holds it.
//
// Bound: VALU issue of the factors, 8 instructions per (image, bond, unit) and
// 4 or 5 per pair of bonds and chunk for the row addresses and signs; counters
// put a SIMD at one VALU instruction in 3.5 cycles.  10x10 M = 400, 1500
// configurations: 20.5 ms, where eight wavefronts on the blocks of one
// configuration (7 rounds for 50 blocks) and 18 bonds a lane, so theta three
// times per image, took 28.3 ms; 8x8 K = 4 M = 256, 1000 configurations 17.3 ->
// 14.9 ms; one 10x10 configuration, its lists in eight shares, 4.4 -> 0.27 ms.
// Every product has the same factors in the same order.  theta of the next
// chunk in half of the wavefronts before the bond products, in the others after
// them, gave 2-4 % at 6x6 and 8x8 and lost 1 % at 10x10 in split BF16 and 3-8 %
// in calls of a few configurations: not used.
#include "theta_common.h"
#include "hops.h"

namespace nqs {

namespace {

constexpr int kWideWaves = 8;
// Bonds per lane and walk over the hidden units (even: the products run two
// bonds at a time; empty pairs are skipped).  The four lane groups cover 88,
// 144 and 224 bonds, nearly every list of a configuration at Sz = 0 (means 74,
// 130, 202), so theta is evaluated once per image.
template <int N>
constexpr int wide_bonds() { return N == 36 ? 22 : N == 64 ? 36 : 56; }
// The list entries whose sums over several RBMs are rescaled as the running
// maximum m rises; those of later entries are weighted once, with the final m.
// The line lies where the first of several walks of 18 (16) bonds a lane ended: the
// sums of K > 1 keep that split's grouping and roundings.  The price is WideRec in
// LDS, two sums a lane and, for K > 4, a walk of the first entries by themselves.
template <int N, bool PAIRS>
constexpr int wide_head() { return N >= 64 && !(PAIRS && N >= 100) ? 72 : 64; }
constexpr int kHC = 8;             // hidden units per chunk
constexpr int kXS = 2 * kHC + 4;   // LDS row stride of the tanh exchange tile (floats)
constexpr int kRecK = kWideLrawK;  // RBMs whose per-image sums are held to the end of a walk
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const f32x4* lds_f32x4_ptr;
typedef __attribute__((address_space(3))) const f32x2* lds_f32x2_ptr;

// An RBM's results in a walk: per image Re L without log|P| and Im a x, per
// lane the joined product P of 2 cosh (its rounding depends on the lane) and
// the lane's sum over the later bonds.
struct WideRec {
  double Er[16], axi[16], dr[64], di[64];
  float pr[64], pi[64];
};

// Partials of a split launch of n blocks (configuration, 16 images): the blocks'
// partials [n][6] (written by the join), the RBMs' results [n][K], the products
// [n][K][list entry][image].
struct WideRaw {
  double Er[16], axi[16];
  float pr[64], pi[64];
};
struct WideSplit {
  double* part;
  WideRaw* raw;
  float2* prod;
  __device__ WideSplit(double* p, int64_t n, int K)
      : part(p), raw(reinterpret_cast<WideRaw*>(p + 6 * n)),
        prod(reinterpret_cast<float2*>(raw + n * K)) {}
};

// The weighting of an RBM's sums, in explicit operations: the kernel and the join
// round alike.  m: the running maximum of Re L over the RBMs of the wave's images.
struct WideSums {
  double m, Qr, Qi, denr, deni;
  __device__ __forceinline__ void init() {
    m = -INFINITY;
    Qr = Qi = denr = deni = 0.0;
  }
  __device__ __forceinline__ void raise(double Er) {
    const double mk = wave_max(Er);
    if (mk > m) {
      const double sc = (double)exp_t((float)(m - mk));   // 0 at the first RBM
      Qr *= sc; Qi *= sc; denr *= sc; deni *= sc;
      m = mk;
    }
  }
  // u = chi e^{Er - m} P e^{i axi}
  __device__ __forceinline__ float2 weight(double Er, double axi, float pr, float pi, float ch) const {
    const float e = ch * exp_t((float)(Er - m));
    float sn, cs;
    sincos_t((float)axi, &sn, &cs);
    return make_float2(e * fmaf(pr, cs, -(pi * sn)), e * fmaf(pr, sn, pi * cs));
  }
  // Q += u (sr + i si)
  __device__ __forceinline__ void add(float2 u, double sr, double si) {
    Qr = fma((double)u.x, sr, fma(-(double)u.y, si, Qr));
    Qi = fma((double)u.x, si, fma((double)u.y, sr, Qi));
  }
  __device__ __forceinline__ void count(float2 u) {
    denr += (double)u.x;
    deni += (double)u.y;
  }
};

// LDS, in bytes: the two staged chunks lie 64 KiB apart, so that a row's
// address is (offset | buffer bit); the small arrays lie between them.
template <int N>
struct WideCfg {
  static constexpr int NB = 4 * N;
  static constexpr uint32_t CAP = wide_cap16(NB) * 16;
  static constexpr uint32_t BUF = 1u << 16;
  static constexpr uint32_t TX = CAP;                                   // [waves][16][kXS] float
  static constexpr uint32_t LIST = TX + kWideWaves * 16 * kXS * 4;      // [waves][NB] uint16
  static constexpr uint32_t ROWS = LIST + kWideWaves * NB * 2;          // [NB] int: row starts
  static constexpr uint32_t BUSY = ROWS + NB * 4;                       // [waves] int
  static constexpr uint32_t REC = BUF + CAP;                            // [waves][kRecK] WideRec
  static constexpr uint32_t LDS = REC + kWideWaves * kRecK * sizeof(WideRec);
  static_assert(BUSY + kWideWaves * 4 <= BUF, "the small arrays fit between the chunks");
};

// Spins of an image as the sign bits of its theta B fragments: dword d of the
// fragments has its two signs at bits d % 16 and 16 + d % 16 of word d / 16.
// At N = 100 the fragments themselves would take 28 or 40 registers.
template <int N, int PREC>
struct XBits {
  static constexpr int ND = 4 * nk_of<N, PREC>(), NW = (ND + 15) / 16;
  uint32_t w[NW];
  __device__ __forceinline__ void load(const int8_t* srow, const uint8_t* prow, int q) {
    const SpinBits m = spin_bits<N>(srow);
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = 0u;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int kap = 32 * (d / 4) + 8 * q + 2 * (d % 4) + h;   // beyond the copies W is 0
        w[d / 16] |= (x_bits<N>(m, prow[kap % N]) >> 31) << (d % 16 + 16 * h);
      }
    }
  }
  __device__ __forceinline__ bf16x8 frag(int kk) const {
    uint32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int d = 4 * kk + e;
      v[e] = ((w[d / 16] << (15 - d % 16)) & 0x80008000u) | 0x3f003f00u;
    }
    return __builtin_bit_cast(bf16x8, v);
  }
};

// Pairs: the rows are exchange neighbours with parent bonds (parent[s]); the
// bond list is the parent's unordered-pair list and pairs counted twice weigh 2.
// Split: shares of the bond lists, part as WideSplit.
// Lout: also write the images' log amplitudes, unreduced (see below).
// per: items of a workgroup in a round (its first `per` wavefronts take them).
// the wavefront's sums to a block's partial
__device__ __forceinline__ void store_partial(const WideSums& w, double* o, int lane) {
  const double Qr = wave_sum(w.Qr), Qi = wave_sum(w.Qi);
  const double denr = wave_sum(w.denr), deni = wave_sum(w.deni);
  if (lane == 0) {
    o[0] = w.m;
    o[1] = denr;
    o[2] = deni;
    o[3] = Qr;
    o[4] = Qi;
    o[5] = 0.0;
  }
}

enum class Wide { Plain, Pairs, Split };
template <int N, int PREC, Wide MODE>
__global__ __launch_bounds__(64 * kWideWaves) void eloc_wide_kernel(
    const int8_t* __restrict__ spins, int64_t S, int nsplit, int per,
    const uint8_t* __restrict__ perm, int K, int M,
    const typename ThetaTraits<PREC>::AFrag* __restrict__ wfrag,
    const float* __restrict__ bias, const float* __restrict__ avec,
    const int32_t* __restrict__ bonds, const int32_t* __restrict__ wmap,
    const int32_t* __restrict__ wrow,
    const double* __restrict__ chi, const float* __restrict__ Tpm, const float* __restrict__ F,
    double* __restrict__ part, const int16_t* __restrict__ parent, double* __restrict__ Lout) {
  using T = ThetaTraits<PREC>;
  using Cfg = WideCfg<N>;
  constexpr int NB = Cfg::NB, G = 8 * N, nblk = G / 16, NK = nk_of<N, PREC>();
  constexpr bool PAIRS = MODE == Wide::Pairs, SPLIT = MODE == Wide::Split;
  constexpr int THREADS = 64 * kWideWaves, E4 = NB * 4, NSTG = (E4 + THREADS - 1) / THREADS;
  constexpr int kWB = wide_bonds<N>(), kHead = wide_head<N, PAIRS>();
  constexpr bool PACK = N == 100;            // two bond slots' offsets in a register
  constexpr bool BITS = N == 100;
  constexpr int kOW = PACK ? kWB / 2 : kWB;
  // aligned to the chunk distance, so that addresses are ORs
  __shared__ __align__(65536) unsigned char lds[Cfg::LDS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, c = lane & 15;
  const int KM = K * M, NCH = KM / kHC, CPR = M / kHC;
  float* tx = reinterpret_cast<float*>(lds + Cfg::TX) + wv * 16 * kXS;
  uint16_t* list = reinterpret_cast<uint16_t*>(lds + Cfg::LIST) + wv * NB;
  int* rows = reinterpret_cast<int*>(lds + Cfg::ROWS);
  int* busy = reinterpret_cast<int*>(lds + Cfg::BUSY);
  WideRec* rec = reinterpret_cast<WideRec*>(lds + Cfg::REC) + wv * kRecK;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // staging of chunk ch: float4 e = tid + 512 i -> row e / 4, part e % 4 of
  // tanh(D); thread tid < NB also stages (F_+, F_-) of row tid for the chunk's
  // RBM into the row's last 16 bytes.
  f32x4 stg[NSTG], sF;
  const uint32_t sofs = (uint32_t)(tid >> 2) * 16u * (uint32_t)KM + 16u * (tid & 3);
  auto stage_load = [&](int ch, int k) __attribute__((always_inline)) {
    const char* b = reinterpret_cast<const char*>(Tpm) + (size_t)ch * (8 * kHC);
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
        *reinterpret_cast<f32x4*>(lds + buf + rows[(tid + THREADS * i) >> 2] + 16 * (tid & 3)) = stg[i];
    if (tid < NB) *reinterpret_cast<f32x4*>(lds + buf + rows[tid] + 8 * kHC) = sF;
  };
  for (int i = tid; i < NB; i += THREADS) rows[i] = 16 * wrow[i];
  __syncthreads();
  stage_load(0, 0);
  stage_store(0);
  uint32_t buf = 0;                            // byte offset of the chunk in use

  const int64_t n_items = S * nblk * (SPLIT ? nsplit : 1);
  int64_t item = (int64_t)blockIdx.x * per + wv;
  bool act = wv < per && item < n_items;

  // state of the wavefront's item, carried from walk to walk
  int64_t s = 0;
  int blk = 0, share = 0, e0 = 0, e1 = 0;      // list entries [e0, e1) of this and later walks
  bool first = true;                           // first walk of the item
  float ch_g = 0.f;
  WideSums sum;
  sum.init();
  typename T::BFrag bx[BITS ? 1 : NK];
  XBits<N, PREC> xb;

  for (;;) {
    if (lane == 0) busy[wv] = act;
    __syncthreads();                           // also: the walk's first chunk is staged
    if (__ballot(lane < kWideWaves && busy[lane & (kWideWaves - 1)] != 0) == 0ull) break;
    // a walk over the hidden units: bonds e0 + q + 4 jb of the list
    uint32_t offs[kOW];                        // row offset in bytes | twice << 1 | (s = -1)
    int nv = 0, nvu = 0;                       // slots in use in the lane, and in lane group 0
    int head = 0;                              // slots of the list's first kHead entries
    if (act) {
      if (first) {
        const int64_t cb = SPLIT ? item / nsplit : item;
        share = SPLIT ? (int)(item - cb * nsplit) : 0;
        s = cb / nblk;
        blk = (int)(cb - s * nblk);
        const int8_t* srow = spins + s * N;
        // with a parent bond b1 (s is the exchange neighbour s0^{b1} of a
        // two-hop sum): the unordered-pair list of the second hops (b1 itself
        // excluded, bonds disjoint from b1 only above it, counted twice: flag 0x4000)
        const int b1 = PAIRS ? (int)parent[s] : -1;
        const int i1 = b1 >= 0 ? bonds[2 * b1] : -1, j1 = b1 >= 0 ? bonds[2 * b1 + 1] : -1;
        int n = 0;
        for (int base = 0; base < NB; base += 64) {
          const int b = base + lane;
          bool anti = false, twice = false;
          int sp = 0;
          if (b < NB) {
            const int bi = bonds[2 * b], bj = bonds[2 * b + 1];
            sp = srow[bi];
            anti = sp != srow[bj];
            if (anti && b1 >= 0) {
              const bool shared = bi == i1 || bi == j1 || bj == i1 || bj == j1;
              anti = b != b1 && (shared || b > b1);
              twice = !shared;
            }
          }
          const unsigned long long msk = __ballot(anti);
          const int pos = __popcll(msk & ((1ull << lane) - 1ull));
          if (anti) list[n + pos] = (uint16_t)(b | (sp > 0 ? 0x8000 : 0) | (twice ? 0x4000 : 0));
          n += __popcll(msk);
        }
        wave_sync_lds();
        if constexpr (SPLIT) {
          const int len = ((n + nsplit - 1) / nsplit + 7) & ~7;
          e0 = min(n, share * len);
          e1 = min(n, e0 + len);
        } else {
          e0 = 0;
          e1 = n;
        }
        const uint8_t* prow = perm + (size_t)(blk * 16 + c) * N;
        if constexpr (BITS) xb.load(srow, prow, q);
        else load_bfrag_gather<N, PREC>(srow, prow, q, bx);
        if constexpr (!SPLIT) {
          ch_g = (float)chi[blk * 16 + c];
          sum.init();
        }
      }
      const int g = blk * 16 + c;
      // more RBMs than the record holds: the first kHead entries take a walk of their own
      const int lim = K > kRecK && e0 < kHead ? min(kWB, (kHead - e0) / 4) : kWB;
      nv = e1 > e0 + q ? min(lim, (e1 - e0 - q + 3) / 4) : 0;
      nvu = __builtin_amdgcn_readfirstlane(nv);
      head = K == 1 || !first || K > kRecK ? kWB : max(0, min(kWB, (kHead - e0) / 4));
#pragma unroll
      for (int jb = 0; jb < kWB; ++jb) {
        const int ii = e0 + q + 4 * jb;
        const int e = jb < nv ? list[ii] : 0;    // padding entries use bond 0
        const uint32_t v = (uint32_t)wmap[(size_t)g * NB + (e & 0x3fff)];   // 2 * floats + flip
        const uint32_t o = 2u * (v & ~1u) | ((v ^ (uint32_t)(e >> 15)) & 1u) |
                           (PAIRS ? (uint32_t)(e >> 13) & 2u : 0u);
        if constexpr (!PACK) offs[jb] = o;
        else if (jb & 1) offs[jb / 2] |= o << 16;
        else offs[jb / 2] = o;
      }
      e0 += 4 * lim;
    } else {
#pragma unroll
      for (int i = 0; i < kOW; ++i) offs[i] = 0u;
    }

    float Pr[kWB], Pi[kWB];
    float lpr = 1.f, lpi = 0.f;
    int lpe = 0;
    uint32_t lpar = 0u;
    double sax = 0.0;
    int k = 0, cin = 0;                        // RBM, chunk within it
    for (int ch = 0; ch < NCH; ++ch) {
      const bool last = ch + 1 == NCH;
      const uint32_t base = lds0 | buf;
      // keep the comparisons with these in the loop: hoisted, they fill registers
      nvu = __builtin_amdgcn_readfirstlane(nvu);
      head = __builtin_amdgcn_readfirstlane(head);
      asm volatile("" : "+s"(nvu), "+v"(nv), "+s"(head));
      if (act) {
        if (cin == 0) {                        // RBM start: products begin at F_s
          // (in halves: the two walks of K > 4 rarely use the upper one, and without
          // the condition took 4-6 % longer at K = 5 M = 40 than 18 bonds a lane did)
          constexpr int kHalf = (kWB / 2 + 1) & ~1;
#pragma unroll
          for (int j0 = 0; j0 < kWB; j0 += kHalf)
            if (j0 < nvu) {
#pragma unroll
              for (int jb = j0; jb < min(j0 + kHalf, kWB); ++jb) {
                const uint32_t o = PACK ? (jb & 1 ? offs[jb / 2] >> 16 : offs[jb / 2]) : offs[jb];
                const f32x2 f = *(lds_f32x2_ptr)(((o & 0xfff0u) | base) + 8u * kHC + 8u * (o & 1u));
                Pr[jb] = f.x;
                Pi[jb] = f.y;
              }
            }
        }
        // theta of the chunk's hidden tile, epilogue, tanh to LDS
        const int h0 = 8 * ch + 2 * q;
        typename T::Acc acc = *reinterpret_cast<const f32x4*>(bias + 2 * h0);   // start from the biases
        if constexpr (BITS) {
#pragma unroll
          for (int i = 0; i < XBits<N, PREC>::NW; ++i) asm volatile("" : "+v"(xb.w[i]));
        }
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
          typename T::BFrag x;
          if constexpr (BITS) x = xb.frag(kk);
          else x = bx[kk];
          acc = mfma(wfrag[((size_t)ch * NK + kk) * 64 + lane], x, acc);
        }
        float axs = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float tr, ti;
          axs += logcosh_step<float, true>(acc[2 * u], acc[2 * u + 1], lpr, lpi, lpar, tr, ti);
          tx[c * kXS + 2 * (2 * q + u)] = tr;
          tx[c * kXS + 2 * (2 * q + u) + 1] = ti;
        }
        sax += (double)axs;
        renorm(lpr, lpi, lpe);
        wave_sync_lds();
      }
      f32x4 t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = *reinterpret_cast<const f32x4*>(&tx[c * kXS + 4 * e]);
      // lands during the bond products
      stage_load(last ? 0 : ch + 1, last ? 0 : cin + 1 == CPR ? k + 1 : k);
#pragma unroll
      for (int jb = 0; jb < kWB; jb += 2) {
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
              const float tr = t[e][2 * hh], ti = t[e][2 * hh + 1];
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
      if (act && cin + 1 == CPR) {             // RBM k complete: weight and sum
        apply_parity(lpr, lpi, lpar);
        int E = lpe;
        float pr = lpr, pi = lpi;
        double sx = sax;
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
          const float orr = __shfl_xor(pr, o, 64), oi = __shfl_xor(pi, o, 64);
          const float nr = pr * orr - pi * oi;
          pi = pr * oi + pi * orr;
          pr = nr;
          E += __shfl_xor(E, o, 64);
          sx += __shfl_xor(sx, o, 64);
        }
        double axr = 0.0, axi = 0.0;
        const float* ak = avec + (size_t)k * N * 2;
        const int8_t* srow = spins + s * N;
        const uint8_t* prow = perm + (size_t)(blk * 16 + c) * N;
        for (int jj = q; jj < N; jj += 4) {
          const double xj = 0.5 * (double)srow[prow[jj]];
          axr += xj * (double)ak[2 * jj];
          axi += xj * (double)ak[2 * jj + 1];
        }
        axr += __shfl_xor(axr, 16, 64);
        axi += __shfl_xor(axi, 16, 64);
        axr += __shfl_xor(axr, 32, 64);
        axi += __shfl_xor(axi, 32, 64);
        const double Er = axr + sx + (double)E * 0.69314718055994530942;
        if constexpr (SPLIT) {
          // the share's one walk began at entry e0 - 4 kWB
          const WideSplit out(part, S * nblk, K);
          const size_t ik = (size_t)(s * nblk + blk) * K + k;
          float2* pk = out.prod + (ik * NB + (e0 - 4 * kWB)) * 16;   // 16 (entry + q) + c
#pragma unroll
          for (int jb = 0; jb < kWB; ++jb)
            if (jb < nv) (pk + 64 * jb)[lane] = make_float2(Pr[jb], Pi[jb]);
          if (share == 0) {
            WideRaw& o = out.raw[ik];
            o.Er[c] = Er;
            o.axi[c] = axi;
            o.pr[lane] = pr;
            o.pi[lane] = pi;
          }
        }
        double sr = 0.0, si = 0.0, dr = 0.0, di = 0.0;
        if constexpr (!SPLIT) {
          sum.raise(Er);
          const float2 u = sum.weight(Er, axi, pr, pi, ch_g);
#pragma unroll
          for (int jb = 0; jb < kWB; ++jb) {
            if (jb < nvu) {
              double wj = 1.0;
              if constexpr (PAIRS) {
                const uint32_t o = PACK ? (jb & 1 ? offs[jb / 2] >> 16 : offs[jb / 2]) : offs[jb];
                wj = o & 2u ? 2.0 : 1.0;
              }
              const double vr = jb < nv ? wj * (double)Pr[jb] : 0.0;
              const double vi = jb < nv ? wj * (double)Pi[jb] : 0.0;
              if (jb < head) {
                sr += vr;
                si += vi;
              } else {
                dr += vr;
                di += vi;
              }
            }
          }
          sum.add(u, sr, si);
          if (first && q == 0) sum.count(u);
        }
        if (first && K <= kRecK) {
          WideRec& o = rec[k];
          o.Er[c] = Er;                        // equal in the four lanes of an image
          o.axi[c] = axi;
          o.pr[lane] = pr;
          o.pi[lane] = pi;
          o.dr[lane] = dr;
          o.di[lane] = di;
        }
        lpr = 1.f; lpi = 0.f; lpe = 0; lpar = 0u; sax = 0.0;
      }
      if (++cin == CPR) {
        cin = 0;
        ++k;
      }
      buf ^= Cfg::BUF;
      stage_store(buf);
      __syncthreads();
    }

    if (act) {
      if (!SPLIT && first && K > 1 && K <= kRecK) {
        // the later entries' sums, weighted with the final m
        wave_sync_lds();
        for (int kk = 0; kk < K; ++kk) {
          const WideRec& o = rec[kk];
          sum.add(sum.weight(o.Er[c], o.axi[c], o.pr[lane], o.pi[lane], ch_g), o.dr[lane],
                  o.di[lane]);
        }
      }
      if (first && Lout != nullptr && share == 0) {
        // the images' log amplitudes L = Er + log|P| + i (Im a x + arg P) to
        // [S][K][G][4], unreduced, for a gradient pass on the same
        // configurations (the log and arg are taken there)
        wave_sync_lds();
        for (int e = lane; e < K * 64; e += 64) {
          const int kk = e >> 6, ci = (e >> 2) & 15, j = e & 3;
          const WideRec& o = rec[kk];
          Lout[(((size_t)s * K + kk) * G + blk * 16 + ci) * 4 + j] =
              j == 0 ? o.Er[ci] : j == 1 ? o.axi[ci] : (double)(j == 2 ? o.pr[ci] : o.pi[ci]);
        }
      }
      first = false;
      if (SPLIT || e0 >= e1) {                 // the item's last walk
        if constexpr (!SPLIT) store_partial(sum, part + item * 6, lane);
        item += (int64_t)gridDim.x * per;
        act = item < n_items;
        first = true;
      }
    }
  }
}

// One workgroup of K wavefronts per (configuration, 16-image block) of a split
// launch: the walks of an unsplit wavefront over the stored products, lane (q, c)
// with the entries q + 4 jb of image c; wavefront k sums RBM k's, the first one
// weights the sums.  Latency bound: the first walk's products are loaded before
// the length of the list is known.
template <int N>
__global__ __launch_bounds__(64 * kRecK) void wide_join_kernel(const int8_t* __restrict__ spins,
                                                               int K,
                                                               const int32_t* __restrict__ bonds,
                                                               const double* __restrict__ chi,
                                                               double* __restrict__ part) {
  constexpr int NB = 4 * N, nblk = N / 2, kWB = wide_bonds<N>();
  static_assert(4 * kWB <= NB, "a walk's entries lie in the block's products");
  __shared__ double2 sums[kRecK][2][64];         // head and later entries
  const int64_t ib = blockIdx.x;
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int k = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t s = ib / nblk;
  const int8_t* srow = spins + s * N;
  const WideSplit in(part, (int64_t)gridDim.x, K);
  const float2* pk = in.prod + (size_t)(ib * K + k) * NB * 16;
  const WideRaw* raw = in.raw + ib * K;
  const float ch_g = (float)chi[(int)(ib - s * nblk) * 16 + c];
  WideSums sum;
  sum.init();
  float2 v[kWB];
#pragma unroll
  for (int jb = 0; jb < kWB; ++jb) v[jb] = (pk + 64 * jb)[lane];
  int n = 0;
#pragma unroll
  for (int base = 0; base < NB; base += 64) {
    const int b = base + lane;
    n += __popcll(__ballot(b < NB && srow[bonds[2 * b]] != srow[bonds[2 * b + 1]]));
  }
  for (int e0 = 0; e0 == 0 || e0 < n; e0 += 4 * kWB) {
    const int nv = n > e0 + q ? min(kWB, (n - e0 - q + 3) / 4) : 0;
    const int head = K == 1 || e0 > 0 ? kWB : wide_head<N, false>() / 4;
    if (e0 > 0) {
#pragma unroll
      for (int jb = 0; jb < kWB; ++jb)
        if (jb < nv) v[jb] = (pk + 16 * e0 + 64 * jb)[lane];
    }
    double2 h = make_double2(0.0, 0.0), t = h;
#pragma unroll
    for (int jb = 0; jb < kWB; ++jb) {
      const double vr = jb < nv ? (double)v[jb].x : 0.0, vi = jb < nv ? (double)v[jb].y : 0.0;
      if (jb < head) {
        h.x += vr;
        h.y += vi;
      } else {
        t.x += vr;
        t.y += vi;
      }
    }
    sums[k][0][lane] = h;
    sums[k][1][lane] = t;
    __syncthreads();
    if (k == 0) {
      for (int kk = 0; kk < K; ++kk) {
        const WideRaw& o = raw[kk];
        sum.raise(o.Er[c]);
        const float2 u = sum.weight(o.Er[c], o.axi[c], o.pr[lane], o.pi[lane], ch_g);
        sum.add(u, sums[kk][0][lane].x, sums[kk][0][lane].y);
        if (e0 == 0 && q == 0) sum.count(u);
      }
      for (int kk = 0; K > 1 && e0 == 0 && kk < K; ++kk) {
        const WideRaw& o = raw[kk];
        sum.add(sum.weight(o.Er[c], o.axi[c], o.pr[lane], o.pi[lane], ch_g), sums[kk][1][lane].x,
                sums[kk][1][lane].y);
      }
    }
    __syncthreads();
  }
  if (k == 0) store_partial(sum, part + ib * 6, lane);
}

size_t split_block_bytes(const nqs_ctx* c) {
  return 48 + (size_t)c->K * (sizeof(WideRaw) + (size_t)c->NB * 16 * sizeof(float2));
}
constexpr size_t kSplitCap = size_t(128) << 20;

// Shares of the bond list per (configuration, column block): as many as leave
// each wavefront slot of the device at most one item, at most eight (every
// share evaluates theta again), if the products fit in cap bytes.
int wide_nsplit(const nqs_ctx* c, int64_t S, size_t cap) {
  const int64_t blocks = std::max<int64_t>(S, 1) * (c->G / 16);
  if (c->K > kRecK || (size_t)blocks * split_block_bytes(c) > std::min(cap, kSplitCap)) return 1;
  return (int)std::max<int64_t>(
      1, std::min<int64_t>(8, (int64_t)fused_max_split_items(c) / blocks));
}

template <int N, int PREC>
hipError_t run(const nqs_ctx* c, const int8_t* spins, int64_t S, double* part, size_t part_cap,
               hipStream_t st, const int16_t* parent, double* Lout) {
  const int nsplit = parent ? 1 : wide_nsplit(c, S, part_cap);
  const int64_t n_cu = c->n_cu > 0 ? c->n_cu : 256, items = S * (c->G / 16) * nsplit;
  // fewer items than wavefront slots: the same number in every workgroup
  const int per = (int)std::min<int64_t>(kWideWaves, (items + n_cu - 1) / n_cu);
  const int64_t blocks = std::min<int64_t>((items + per - 1) / per, n_cu);
  const auto* wf = (const typename ThetaTraits<PREC>::AFrag*)(PREC == kPrecF32X3 ? c->par.wfrag3
                                                                                 : c->par.wfrag);
  auto kernel = parent       ? eloc_wide_kernel<N, PREC, Wide::Pairs>
                : nsplit > 1 ? eloc_wide_kernel<N, PREC, Wide::Split>
                             : eloc_wide_kernel<N, PREC, Wide::Plain>;
  kernel<<<(unsigned)blocks, 64 * kWideWaves, 0, st>>>(
      spins, S, nsplit, per, c->dev.perm, c->K, c->M, wf, (const float*)c->par.bias,
      (const float*)c->par.avec, c->dev.bonds, c->dev.wmap, c->dev.wrow, c->dev.chi,
      (const float*)c->par.Tpm, (const float*)c->par.F, part, parent, Lout);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nsplit == 1) return e;
  wide_join_kernel<N><<<(unsigned)(S * (c->G / 16)), 64 * c->K, 0, st>>>(
      spins, c->K, c->dev.bonds, c->dev.chi, part);
  return hipGetLastError();
}

}  // namespace

bool eloc_wide_supported(const nqs_ctx* c) {
  if (c->prec == NQS_FP64 || c->KM <= 128 || c->M % kHC != 0) return false;
  return c->N == 36 || c->N == 64 || c->N == 100;
}

size_t wide_split_part_bytes(const nqs_ctx* c, int64_t S) {
  if (c->K > kRecK) return 0;
  const int64_t nblk = c->G / 16;
  const int64_t most = std::min<int64_t>((int64_t)fused_max_split_items(c) / 2 / nblk,
                                         (int64_t)(kSplitCap / split_block_bytes(c)) / nblk);
  return (size_t)(std::min<int64_t>(S, most) * nblk) * split_block_bytes(c);
}

namespace {
hipError_t dispatch(const nqs_ctx* c, const int8_t* spins, int64_t S, const int16_t* parent,
                    double* part, size_t cap, double* Lout, hipStream_t st) {
  if (S <= 0) return hipSuccess;
  const bool bf = c->prec == NQS_BF16X2;
  switch (c->N) {
    case 36: return bf ? run<36, NQS_BF16X2>(c, spins, S, part, cap, st, parent, Lout)
                       : run<36, kPrecF32X3>(c, spins, S, part, cap, st, parent, Lout);
    case 64: return bf ? run<64, NQS_BF16X2>(c, spins, S, part, cap, st, parent, Lout)
                       : run<64, kPrecF32X3>(c, spins, S, part, cap, st, parent, Lout);
    case 100: return bf ? run<100, NQS_BF16X2>(c, spins, S, part, cap, st, parent, Lout)
                        : run<100, kPrecF32X3>(c, spins, S, part, cap, st, parent, Lout);
    default: return hipErrorNotSupported;
  }
}
}  // namespace

hipError_t launch_eloc_wide(const nqs_ctx* c, const int8_t* spins, int64_t S, double* part,
                            size_t part_cap, hipStream_t st, double* Lout) {
  return dispatch(c, spins, S, nullptr, part, part_cap, Lout, st);
}

hipError_t launch_eloc_wide_pairs(const nqs_ctx* c, const int8_t* spins, int64_t S,
                                  const int16_t* parent, double* part, hipStream_t st) {
  return dispatch(c, spins, S, parent, part, 0, nullptr, st);
}

}  // namespace nqs
