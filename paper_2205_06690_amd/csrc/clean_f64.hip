// Cleaning projection (Eq. 15, linearised) of the FP64 mode on the gfx950
// matrix cores: the coefficients C[f][s] = h^3 sum_r phi_s(r) d_f(r) and the
// update d_f -= sum_s C[f][s] phi_s + c_f E_l.
//
// Both are real GEMMs on v_mfma_f64_16x16x4f64: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] and holds D[4 v + l / 16][l % 16],
// v < 4.  A complex field is two A operands (re, im) against the same B, so
// an interleaved field value is one 16-byte load that feeds two products.
// One product keeps a SIMD's matrix core busy for 64 cycles and takes two
// 8-byte operands per lane, so the operands go from global memory (L1, L2)
// straight to registers: no LDS, no barriers, the next loads in flight.
//
// The sum over points (states) of a product may run in any order, so lane
// group l / 16 takes consecutive ones (a 32-byte piece of an interleaved
// row) instead of the operand's own k.
#include "clean_f64.h"

#include <algorithm>

namespace bse {

typedef double d4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 cm64(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// end of the step for one value: ph (v - i hdt u h)
__device__ __forceinline__ double2 finish64(double2 v, double2 h, double cu, double2 p) {
  return cm64(p, make_double2(v.x + cu * h.y, v.y - cu * h.x));
}

// part[kc][f][s] = sum over chunk kc of phi_s d_f, part[kc][f][S] that of
// conj(E_l) d_f.  A wave owns 16 fields and 16 NS states of one chunk of
// points, eight points at a time (lane l: points 2 (l / 16), 2 (l / 16) + 1
// of field and state l % 16).  Waves are numbered field group fastest, so
// the waves of a block share the states' rows in L1.  64^3, 110 fields, 120
// states: 0.82 ms with the end of the step applied on the fly (0.73 ms
// without), against 1.80 ms for each of two launches of a vector-FMA tile
// whose <E, d> ran on one thread in sixteen, plus 0.15 ms of a pass that
// applied the end of the step; 24^3, 80 fields, 8 states: 1125 us -> 13 us.
// The matrix cores' share of the 0.82 ms is 0.22 ms; the rest is load
// latency that two waves per SIMD do not cover.
template <int NS, bool MID>
__global__ void __launch_bounds__(256, 2) k_coef_f64(const double2* __restrict__ d, int F,
                                                     const double* __restrict__ phi, int S,
                                                     const double2* __restrict__ E, int L, size_t ng, size_t chunk,
                                                     int nfg, int nct, unsigned nwave, MidArgs64 mid,
                                                     double2* __restrict__ part) {
  const unsigned wv = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wv >= nwave) return;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int fg = (int)(wv % nfg), ct = (int)((wv / nfg) % nct), kc = (int)(wv / ((unsigned)nfg * nct));
  const size_t k0 = (size_t)kc * chunk, k1 = min(ng, k0 + chunk);
  const int FT = F + L;
  const int f = min(fg * 16 + lr, FT - 1);      // rows past the last: a copy of it, never stored
  const int l = f < F ? f % L : f - F;
  // an unperturbed field enters as its mid-step state H_l with u = 0
  const double2* src = f < F ? d + (size_t)f * ng : (MID ? mid.H : E) + (size_t)l * ng;
  const double2* hp = (MID ? mid.H : E) + (size_t)l * ng;
  const double* up = MID ? mid.u + (size_t)(f < F ? f / L : 0) * ng : nullptr;
  const bool edot = ct == 0;
  const double* pr[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) pr[j] = phi + (size_t)min((ct * NS + j) * 16 + lr, S - 1) * ng;
  d4v re[NS], im[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) re[j] = im[j] = d4v{0.0, 0.0, 0.0, 0.0};
  double2 nd[2], nh[2], np[2], nu = make_double2(0.0, 0.0), nb[NS];
  auto load = [&](size_t kb) {
    const size_t r = kb + 2 * lk;
    nd[0] = src[r];
    nd[1] = src[r + 1];
    if (MID || edot) {
      nh[0] = hp[r];
      nh[1] = hp[r + 1];
    }
    if (MID) {
      np[0] = mid.ph[r];
      np[1] = mid.ph[r + 1];
      nu = *reinterpret_cast<const double2*>(up + r);
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) nb[j] = *reinterpret_cast<const double2*>(pr[j] + r);
  };
  double ex = 0, ey = 0;
  if (k0 < k1) load(k0);
  for (size_t kb = k0; kb < k1; kb += 8) {
    double2 v[2], b[NS];
    // (not half_dt = 0: a non-finite u of a failed pair must not reach them)
    const double cu[2] = {f < F ? mid.half_dt * nu.x : 0.0, f < F ? mid.half_dt * nu.y : 0.0};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      double2 e = nh[t];
      v[t] = nd[t];
      if (MID) {
        v[t] = finish64(nd[t], nh[t], cu[t], np[t]);
        e = cm64(np[t], nh[t]);
      }
      if (edot) {
        ex += e.x * v[t].x + e.y * v[t].y;
        ey += e.x * v[t].y - e.y * v[t].x;
      }
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) b[j] = nb[j];
    if (kb + 8 < k1) load(kb + 8);
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      re[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0].x, b[j].x, re[j], 0, 0, 0);
      im[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0].y, b[j].x, im[j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      re[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1].x, b[j].y, re[j], 0, 0, 0);
      im[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1].y, b[j].y, im[j], 0, 0, 0);
    }
  }
  double2* out = part + (size_t)kc * FT * (S + 1);
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int s = (ct * NS + j) * 16 + lr;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = fg * 16 + 4 * q + lk;
      if (row < FT && s < S) out[(size_t)row * (S + 1) + s] = make_double2(re[j][q], im[j][q]);
    }
  }
  if (edot) {
    // the four lane groups hold the same fields at different points
    ex += __shfl_xor(ex, 16, 64);
    ey += __shfl_xor(ey, 16, 64);
    ex += __shfl_xor(ex, 32, 64);
    ey += __shfl_xor(ey, 32, 64);
    if (lk == 0 && fg * 16 + lr < FT) out[(size_t)f * (S + 1) + S] = make_double2(ex, ey);
  }
}

// coef[i] = dv sum_k part[k][i]: a block sums 32 outputs in eight slices of
// the chunks (slice j: k = j, j + 8, ...) and adds the slices in order
constexpr int C64_SL = 8;
__global__ void __launch_bounds__(256) k_coef64_reduce(const double2* __restrict__ part, int nchunk, int FS, double dv,
                                                       double2* __restrict__ coef) {
  __shared__ double2 red[C64_SL][32];
  const int o = threadIdx.x & 31, j = threadIdx.x >> 5;
  const int i = blockIdx.x * 32 + o;
  double x = 0, y = 0;
  if (i < FS) {
#pragma unroll 4
    for (int k = j; k < nchunk; k += C64_SL) {
      const double2 v = part[(size_t)k * FS + i];
      x += v.x;
      y += v.y;
    }
  }
  red[j][o] = make_double2(x, y);
  __syncthreads();
  if (j == 0 && i < FS) {
    double sx = 0, sy = 0;
#pragma unroll
    for (int q = 0; q < C64_SL; ++q) {
      sx += red[q][o].x;
      sy += red[q][o].y;
    }
    coef[i] = make_double2(sx * dv, sy * dv);
  }
}

// The update: a wave owns 16 NF fields and 32 points (two column tiles) and
// walks the states four at a time: A = C[f][s] (16 bytes: re and im), B =
// phi_s at 16 consecutive points.  The waves of a block take the same fields
// at different points, so the coefficients come from L1.  64^3, 110 fields,
// 120 states: 0.57 ms, against 1.19 ms for vector FMA on LDS tiles of 16
// fields (which re-read the orbitals for each of them).
template <int NF, bool MID>
__global__ void __launch_bounds__(256, 2) k_update_f64(double2* __restrict__ d, int F, const double* __restrict__ phi,
                                                       int S, const double2* __restrict__ E, int L, size_t ng,
                                                       const double2* __restrict__ coef, MidArgs64 mid) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const size_t r0 = ((size_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32;
  if (r0 >= ng) return;
  const int f0 = blockIdx.y * 16 * NF;
  size_t rc[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) rc[p] = min(r0 + 16 * p + lr, ng - 1);
  const double2* cr[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) cr[i] = coef + (size_t)min(f0 + 16 * i + lr, F - 1) * (S + 1);
  d4v re[NF][2], im[NF][2];
#pragma unroll
  for (int i = 0; i < NF; ++i)
#pragma unroll
    for (int p = 0; p < 2; ++p) re[i][p] = im[i][p] = d4v{0.0, 0.0, 0.0, 0.0};
  double2 nc[NF];
  double nb[2];
  // states past the last: coefficient and orbital both zero
  auto load = [&](int sb) {
    const int s = sb + lk;
    const bool live = s < S;
#pragma unroll
    for (int i = 0; i < NF; ++i) nc[i] = live ? cr[i][s] : make_double2(0.0, 0.0);
#pragma unroll
    for (int p = 0; p < 2; ++p) nb[p] = live ? phi[(size_t)s * ng + rc[p]] : 0.0;
  };
  load(0);
  for (int sb = 0; sb < S; sb += 4) {
    double2 c[NF];
    double b[2];
#pragma unroll
    for (int i = 0; i < NF; ++i) c[i] = nc[i];
    b[0] = nb[0];
    b[1] = nb[1];
    if (sb + 4 < S) load(sb + 4);
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        re[i][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[i].x, b[p], re[i][p], 0, 0, 0);
        im[i][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[i].y, b[p], im[i][p], 0, 0, 0);
      }
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const size_t r = r0 + 16 * p + lr;
    if (r >= ng) continue;
    const double2 ph = MID ? mid.ph[r] : make_double2(1.0, 0.0);
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = f0 + 16 * i + 4 * q + lk;
        if (f >= F) continue;
        const int l = f % L;
        double2 v = d[(size_t)f * ng + r], e;
        if (MID) {
          const double2 h = mid.H[(size_t)l * ng + r];
          v = finish64(v, h, mid.half_dt * mid.u[(size_t)(f / L) * ng + r], ph);
          e = cm64(ph, h);
        } else {
          e = E[(size_t)l * ng + r];
        }
        const double c = coef[(size_t)f * (S + 1) + S].x;
        v.x -= re[i][p][q] + c * e.x;
        v.y -= im[i][p][q] + c * e.y;
        d[(size_t)f * ng + r] = v;
      }
  }
}

// The split of the coefficient GEMM: column tiles of up to 64 states, evenly
// filled, and chunks of points for about 2048 waves (two per SIMD: the
// registers' limit), each at least 64 points; more chunks only add partial
// sums (64^3, 120 fields, 120 states: 30 MB of them).  At most 4096 points: one
// accumulator over 88000 (112^3, 42 pairs, 260 states) left W after 600 steps
// 5.6e-14 from the oracle, 4096 leave 3.2e-14 (vector FMA chains of 4096: 3.6e-14)
// and shorter blocks fill the chip more evenly (15.0 -> 14.3 s a call).
struct Coef64Plan {
  int ns, nct, nfg, nchunk;
  size_t chunk;
};
static Coef64Plan coef64_plan(int FT, int S, size_t ng) {
  Coef64Plan p;
  const int t = (S + 15) / 16;
  p.nct = (t + 3) / 4;
  p.ns = (t + p.nct - 1) / p.nct;
  p.nfg = (FT + 15) / 16;
  const size_t tiles = (size_t)p.nct * p.nfg;
  const size_t want = std::max<size_t>(1, (2048 + tiles - 1) / tiles);
  p.chunk = std::min<size_t>(4096, std::max<size_t>(64, ((ng + want - 1) / want + 7) / 8 * 8));
  p.nchunk = (int)((ng + p.chunk - 1) / p.chunk);
  return p;
}

size_t coef64_part_entries(int F, int L, int S, size_t ng) {
  size_t m = 0;
  for (int f = L; f <= F; f += L) m = std::max(m, (size_t)coef64_plan(f + L, S, ng).nchunk * (f + L) * (S + 1));
  return m;
}

template <int NS>
static void coef64_go(const Coef64Plan& p, const double2* d, int F, const double* phi, int S, const double2* E, int L,
                      size_t ng, double2* part, hipStream_t st, const MidArgs64& mid) {
  const unsigned nwave = (unsigned)p.nfg * p.nct * p.nchunk;
  const dim3 g((nwave + 3) / 4), b(256);
  if (mid.on)
    hipLaunchKernelGGL((k_coef_f64<NS, true>), g, b, 0, st, d, F, phi, S, E, L, ng, p.chunk, p.nfg, p.nct, nwave, mid,
                       part);
  else
    hipLaunchKernelGGL((k_coef_f64<NS, false>), g, b, 0, st, d, F, phi, S, E, L, ng, p.chunk, p.nfg, p.nct, nwave, mid,
                       part);
}

hipError_t launch_coef_f64(const double2* d, int F, const double* phi, int S, const double2* E, int L, size_t ng,
                           double dv, double2* part, double2* coef, hipStream_t st, const MidArgs64& mid) {
  if (F <= 0 || L <= 0 || S <= 0 || ng % 8) return hipErrorInvalidValue;
  const Coef64Plan p = coef64_plan(F + L, S, ng);
  switch (p.ns) {
    case 1: coef64_go<1>(p, d, F, phi, S, E, L, ng, part, st, mid); break;
    case 2: coef64_go<2>(p, d, F, phi, S, E, L, ng, part, st, mid); break;
    case 3: coef64_go<3>(p, d, F, phi, S, E, L, ng, part, st, mid); break;
    case 4: coef64_go<4>(p, d, F, phi, S, E, L, ng, part, st, mid); break;
    default: return hipErrorInvalidValue;
  }
  const int FS = (F + L) * (S + 1);
  hipLaunchKernelGGL(k_coef64_reduce, dim3((FS + 31) / 32), dim3(256), 0, st, part, p.nchunk, FS, dv, coef);
  return hipGetLastError();
}

template <int NF>
static void update64_go(double2* d, int F, const double* phi, int S, const double2* E, int L, size_t ng,
                        const double2* coef, hipStream_t st, const MidArgs64& mid) {
  const dim3 g((unsigned)((ng + 127) / 128), (F + 16 * NF - 1) / (16 * NF)), b(256);
  if (mid.on)
    hipLaunchKernelGGL((k_update_f64<NF, true>), g, b, 0, st, d, F, phi, S, E, L, ng, coef, mid);
  else
    hipLaunchKernelGGL((k_update_f64<NF, false>), g, b, 0, st, d, F, phi, S, E, L, ng, coef, mid);
}

// Fields per wave: up to 64 (the orbitals are then re-read once per 64
// fields), fewer where 64 would leave fewer than about 1024 waves
hipError_t launch_update_f64(double2* d, int F, const double* phi, int S, const double2* E, int L, size_t ng,
                             const double2* coef, hipStream_t st, const MidArgs64& mid) {
  if (F <= 0 || L <= 0 || S <= 0) return hipErrorInvalidValue;
  const size_t np = (ng + 31) / 32;
  const int t = (F + 15) / 16;
  const int groups = (int)std::max<size_t>((t + 3) / 4, std::min<size_t>(t, (1024 + np - 1) / np));
  switch ((t + groups - 1) / groups) {
    case 1: update64_go<1>(d, F, phi, S, E, L, ng, coef, st, mid); break;
    case 2: update64_go<2>(d, F, phi, S, E, L, ng, coef, st, mid); break;
    case 3: update64_go<3>(d, F, phi, S, E, L, ng, coef, st, mid); break;
    case 4: update64_go<4>(d, F, phi, S, E, L, ng, coef, st, mid); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace bse
