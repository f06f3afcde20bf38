// Two-hop H^2 terms (Sec. 3.3) on the 4x4 lattice in FP64, one RBM of 8 or 16
// hidden units (the exact evaluations over the Sz = 0 sector).
//
// For exchanges b1 then b2 with signs s1, s2 and T = tanh D (k_eloc_reg.hip):
// the image's ratio is F1 F2 prod_h A_h (s2 + T2_h Q_h), A = s1 + t T1,
// Q = (s1 t + T1) / A.  A wavefront takes 32 images of one configuration, two
// lanes each (halves of the hidden units) with t in registers, and walks a
// share of the first hops; Q and prod A are formed once per first hop.  Each
// first hop leaves a partial of its own, so that e2 is summed in one order
// whatever the shares.  With 64
// bonds the antiparallel bonds and the unordered-pair list are bit masks in
// scalar registers (one vote each), so a pair of second hops costs the lane its
// M factors of 8 instructions and about 30 more.
//
// Bound: FP64 VALU issue (3.4e9 wave instructions for the 12 870 configurations
// of the sector at M = 16, 5.6 ms at four cycles each; with three wavefronts a
// SIMD they issue at about five).  8.3 ms with one partial per share (one per
// first hop costs half a percent: 9.75 -> 9.80 ms on a slower box); the kernel
// before it, which gave a wavefront one first hop and chased list, map and F through
// global memory once per pair of second hops, took 33.7 ms.  Measured alternatives: one lane
// per image (16 units a lane) 12.5 ms without and 9.3 ms with the next table row
// prefetched, at two wavefronts a SIMD; four wavefronts (128 VGPRs) 9.0 ms.
#include "device_common.h"
#include "nqs_internal.h"

namespace nqs {

namespace {

constexpr int kWaves16 = 4;      // wavefronts per workgroup
constexpr int kG16 = 128, kNB16 = 64;

// P <- P (a + i b)
__device__ __forceinline__ void mul_in(double2& p, double a, double b) {
  const double nr = fma(p.x, a, -(p.y * b));
  p.y = fma(p.x, b, p.y * a);
  p.x = nr;
}
__device__ __forceinline__ double rcp64(double v) {      // |v| well inside the FP64 range
  double r = __builtin_amdgcn_rcp(v);
  r = fma(fma(-v, r, 1.0), r, r);
  return fma(fma(-v, r, 1.0), r, r);
}

template <int M>
__global__ __launch_bounds__(64 * kWaves16, 3) void twohop16_kernel(
    const int8_t* __restrict__ spins, int64_t S, const int32_t* __restrict__ bonds,
    const double* __restrict__ bond_J, const int32_t* __restrict__ bmap,
    const double2* __restrict__ t, const double2* __restrict__ w, const double2* __restrict__ Tpm,
    const double2* __restrict__ F, double* __restrict__ part, int lg_parts, int allow_ratio) {
  const int parts = 1 << lg_parts;
  constexpr int MH = M / 2;
  constexpr int ST = M + 1;                               // row stride, complex (bank spread)
  constexpr int BS = kNB16 + 4;                           // byte stride of an image's bond map
  __shared__ double2 Tl[kNB16 * ST];
  __shared__ double2 Fl[kNB16 * 2];
  __shared__ uint8_t bm[kG16 * BS];
  // (loads of a loop in flight together: a small call waits for the tables)
  constexpr int TH = 64 * kWaves16;
  int v[kG16 * kNB16 / TH];
#pragma unroll
  for (int u = 0; u < kG16 * kNB16 / TH; ++u) v[u] = bmap[threadIdx.x + u * TH];
#pragma unroll
  for (int u = 0; u < kNB16 * M / TH; ++u) {
    const int i = threadIdx.x + u * TH;
    Tl[(i / M) * ST + i % M] = Tpm[(size_t)(i / M) * 2 * M + i % M];
  }
  if (threadIdx.x < kNB16 * 2) Fl[threadIdx.x] = F[threadIdx.x];
#pragma unroll
  for (int u = 0; u < kG16 * kNB16 / TH; ++u) {
    const int i = threadIdx.x + u * TH;
    bm[(i / kNB16) * BS + i % kNB16] = (uint8_t)v[u];
  }
  __syncthreads();

  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bi = bonds[2 * lane], bj = bonds[2 * lane + 1];   // lane = bond
  const double J = bond_J[lane];
  const int64_t n_items = S * 4 * parts, stride = (int64_t)gridDim.x * kWaves16;
  for (int64_t item = (int64_t)blockIdx.x * kWaves16 + wv; item < n_items; item += stride) {
    // the shares slowest: those without a first hop (there are 48 at most, often
    // 32) lie at the end, and the others spread over the wavefronts
    const int share = parts == 1 ? 0 : (int)(item / (4 * S));
    const int64_t s = (item >> 2) - share * S;
    const int sub = (int)item & 3;
    // the 16 lanes of a row take the 16 translations of one point-group element:
    // a bond's pre-images under them are the 16 bonds of one kind, rows in
    // distinct bank groups
    const int g = (lane & 15) * 8 + sub * 2 + ((lane >> 4) & 1);
    const uint32_t m =
        (uint32_t)__builtin_amdgcn_ballot_w64(lane < 16 && spins[s * 16 + (lane & 15)] < 0);
    uint64_t l1 = __builtin_amdgcn_ballot_w64(((m >> bi) ^ (m >> bj)) & 1u);
    const uint8_t* bg = bm + g * BS;
    // t of unit h: [s][h / 8][g][h % 8]
    const double2* tg = t + ((size_t)s * (M / 8) + half * MH / 8) * kG16 * 8 + g * 8 + half * MH % 8;
    const double2* Th = Tl + half * MH;
    const double2 wg = w[(size_t)s * kG16 + g];
    double tr[MH], ti[MH];
#pragma unroll
    for (int h = 0; h < MH; ++h) {
      const double2 v = tg[h];
      tr[h] = v.x;
      ti[h] = v.y;
    }
    for (int n = 0; l1 != 0; l1 &= l1 - 1, ++n) {
      if ((n & (parts - 1)) != share) continue;
      const int b1 = __builtin_ctzll(l1);
      const int i1 = __builtin_amdgcn_readlane(bi, b1), j1 = __builtin_amdgcn_readlane(bj, b1);
      const uint32_t m2 = m ^ (1u << i1) ^ (1u << j1);
      const bool anti2 = ((m2 >> bi) ^ (m2 >> bj)) & 1u;
      const bool shared = bi == i1 || bi == j1 || bj == i1 || bj == j1;
      const bool keep = anti2 && lane != b1 && (shared || lane > b1);
      uint64_t l2 = __builtin_amdgcn_ballot_w64(keep);
      const uint64_t once = __builtin_amdgcn_ballot_w64(shared);
      const double diag2 = wave_sum(anti2 ? -0.25 * J : 0.25 * J);
      const double J1 = bond_J[b1];

      const int v1 = bg[b1];
      const bool neg1 = (((m >> i1) & 1u) != 0u) == ((v1 & 1) != 0);   // s1 = -1
      const double s1 = neg1 ? -1.0 : 1.0;
      const double2* T1 = Th + (v1 >> 1) * ST;
      const double2 f1 = Fl[(v1 >> 1) * 2 + (neg1 ? 1 : 0)];
      const double2 g1 = cmul(f1, wg);                     // w F1
      double qr[MH], qi[MH];
      double2 pa = make_double2(1.0, 0.0);
      bool ok = allow_ratio != 0;
#pragma unroll
      for (int h = 0; h < MH; ++h) {
        if (h % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        const double2 T = T1[h];
        const double ar = fma(tr[h], T.x, fma(-ti[h], T.y, s1)), ai = fma(tr[h], T.y, ti[h] * T.x);
        const double br = fma(s1, tr[h], T.x), bb = fma(s1, ti[h], T.y);
        const double a2 = fma(ar, ar, ai * ai);
        ok &= (a2 > 0x1p-60) & (a2 < 0x1p60);
        const double inv = rcp64(a2);
        qr[h] = fma(br, ar, bb * ai) * inv;
        qi[h] = fma(bb, ar, -(br * ai)) * inv;
        mul_in(pa, ar, ai);
      }
      {
        double yr = pa.x, yi = pa.y;                       // prod A over both halves
        swap32(pa.x, yr);
        swap32(pa.y, yi);
        mul_in(pa, yr, yi);
      }
      const bool ratio = __all(ok);
      double sr = 0.0, si = 0.0;                           // sum over the second hops
      // two second hops at a time: the halves' partial products of both are
      // joined by one row swap, after which lane half 0 holds the first hop's
      // product and half 1 the second's
      while (l2 != 0) {
        const int ba = __builtin_ctzll(l2);
        l2 &= l2 - 1;
        const int bb2 = l2 != 0 ? __builtin_ctzll(l2) : ba;
        double mb = l2 != 0 ? ((once >> bb2) & 1u ? 1.0 : 2.0) : 0.0;
        l2 &= l2 - 1;                                      // (0 stays 0)
        const double ma = (once >> ba) & 1u ? 1.0 : 2.0;
        const int va = bg[ba], vb = bg[bb2];
        const bool na = (((m2 >> __builtin_amdgcn_readlane(bi, ba)) & 1u) != 0u) == ((va & 1) != 0);
        const bool nb = (((m2 >> __builtin_amdgcn_readlane(bi, bb2)) & 1u) != 0u) == ((vb & 1) != 0);
        const double sa = na ? -1.0 : 1.0, sb = nb ? -1.0 : 1.0;
        const double2* Ta = Th + (va >> 1) * ST;
        const double2* Tb = Th + (vb >> 1) * ST;
        double2 f2 = Fl[half ? (vb & ~1) + (nb ? 1 : 0) : (va & ~1) + (na ? 1 : 0)];
        double2 pA, pB;
        if (ratio) {
#pragma unroll
          for (int h = 0; h < MH; ++h) {
            const double2 A = Ta[h], B = Tb[h];
            const double ar = fma(A.x, qr[h], fma(-A.y, qi[h], sa)), ai = fma(A.x, qi[h], A.y * qr[h]);
            const double br = fma(B.x, qr[h], fma(-B.y, qi[h], sb)), bi2 = fma(B.x, qi[h], B.y * qr[h]);
            if (h == 0) {
              pA = make_double2(ar, ai);
              pB = make_double2(br, bi2);
            } else {
              mul_in(pA, ar, ai);
              mul_in(pB, br, bi2);
            }
          }
        } else {
          // an A near zero (or a range beyond the check): factors s2 A + T2 B
          pA = pB = make_double2(1.0, 0.0);
#pragma unroll 1
          for (int h = 0; h < MH; ++h) {
            const double2 T = T1[h], A = Ta[h], B = Tb[h], v = tg[h];
            const double ar = fma(v.x, T.x, fma(-v.y, T.y, s1)), ai = fma(v.x, T.y, v.y * T.x);
            const double br = fma(s1, v.x, T.x), bi2 = fma(s1, v.y, T.y);
            mul_in(pA, fma(A.x, br, fma(-A.y, bi2, sa * ar)), fma(A.x, bi2, fma(A.y, br, sa * ai)));
            mul_in(pB, fma(B.x, br, fma(-B.y, bi2, sb * ar)), fma(B.x, bi2, fma(B.y, br, sb * ai)));
          }
        }
        swap32(pA.x, pB.x);
        swap32(pA.y, pB.y);
        mul_in(pA, pB.x, pB.y);
        mul_in(f2, pA.x, pA.y);
        const double mult = half ? mb : ma;
        sr = fma(mult, f2.x, sr);
        si = fma(mult, f2.y, si);
      }
      if (ratio) {
        const double nr = sr * pa.x - si * pa.y;
        si = sr * pa.y + si * pa.x;
        sr = nr;
      }
      // first hop alone and b1 exchanged back (ratio 1), once per image
      const double jj = half ? 0.0 : 0.25 * J1 * J1, dg = half ? 0.0 : diag2;
      sr = fma(dg, pa.x, sr);
      si = fma(dg, pa.y, si);
      double er = fma(g1.x, sr, fma(-g1.y, si, jj * wg.x));
      double ei = fma(g1.x, si, fma(g1.y, sr, jj * wg.y));
      // the sum over the lanes, real part in lanes 0..31 and imaginary in 32..63
      swap32(er, ei);
      er += ei;
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) er += __shfl_xor(er, o, 64);
      if ((lane & 31) == 0) part[2 * ((s * kNB16 + n) * 4 + sub) + half] = er;
    }
  }
}

template <int M>
hipError_t run(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t, const void* w,
               double* part, hipStream_t st) {
  // shares of the first hops, a power of two: enough to give every SIMD four
  // wavefronts, at most one for each bond
  const int64_t n_cu = c->n_cu > 0 ? c->n_cu : 256;
  int parts = 1;
  while (parts < kNB16 && S * 4 * parts < 32 * n_cu) parts *= 2;
  const int64_t items = S * 4 * parts;
  const int64_t blocks = std::min<int64_t>((items + kWaves16 - 1) / kWaves16, 3 * n_cu);
  twohop16_kernel<M><<<(unsigned)blocks, 64 * kWaves16, 0, st>>>(
      spins, S, c->dev.bonds, c->dev.bond_J, c->dev.bmap, (const double2*)t, (const double2*)w,
      (const double2*)c->par.Tpm, (const double2*)c->par.F, part, __builtin_ctz(parts), c->direct_only ? 0 : 1);
  return hipGetLastError();
}

}  // namespace

bool twohop16_supported(const nqs_ctx* c) {
  return c->prec == NQS_FP64 && c->N == 16 && c->K == 1 && (c->M == 8 || c->M == 16);
}

hipError_t launch_twohop16(const nqs_ctx* c, const int8_t* spins, int64_t S, const void* t,
                           const void* w, double* part, hipStream_t st) {
  return c->M == 8 ? run<8>(c, spins, S, t, w, part, st) : run<16>(c, spins, S, t, w, part, st);
}

}  // namespace nqs
