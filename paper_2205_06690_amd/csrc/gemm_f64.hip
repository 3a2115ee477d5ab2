// FP64 contractions over the grid on the gfx950 matrix cores
// (v_mfma_f64_16x16x4f64: lane l supplies A[l % 16][l / 16] and B[l / 16][l %
// 16] and holds D[4 v + l / 16][l % 16], v < 4).  A product keeps the matrix
// core busy for 64 cycles and takes two 8-byte operands per lane, so operands
// go from memory (L1, L2) straight to registers; the contraction index may be
// permuted alike in A and B, so each lane reads 16 consecutive bytes.
#include "gemm_f64.h"

#include <algorithm>

namespace bse {

typedef double g4v __attribute__((ext_vector_type(4)));

// part[kc][m][n] = sum over chunk kc: a wave owns 16 MT x 16 NT outputs of one
// chunk, 16 values of r at a time (lane l: r = 4 (l / 16) .. + 3, so that a
// row's loads take whole 128-byte lines; with eight values, half a line at a
// time, 124 us).  Bound by reading the operands: 30 fields on 120 orbitals at
// 64^3, 315 MB in 99 us, against 3 x 77 us for one set of 10 at a time on
// vector FMA and LDS tiles.  MT and NT are what M and N fill: a product of a
// padded tile takes as long as any other (1 field on 5 orbitals at 16^3: 8.0 us
// with MT 2 and NT 4, 3.2; 6 on 30 at 48^3: 14 and 8).
template <int GM_MT, int GM_NT>
__global__ void __launch_bounds__(256, 2) k_gemm_f64(const double* __restrict__ A, int M, const double* __restrict__ B,
                                                     int N, size_t K, size_t chunk, int nmt, int nnt, unsigned nwave,
                                                     double* __restrict__ part) {
  const unsigned wv = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wv >= nwave) return;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int mt = (int)(wv % nmt), nt = (int)((wv / nmt) % nnt), kc = (int)(wv / ((unsigned)nmt * nnt));
  const size_t k0 = (size_t)kc * chunk, k1 = min(K, k0 + chunk);
  // rows past the last: a copy of it, never stored
  const double* pa[GM_MT];
  const double* pb[GM_NT];
#pragma unroll
  for (int i = 0; i < GM_MT; ++i) pa[i] = A + (size_t)min((mt * GM_MT + i) * 16 + lr, M - 1) * K + 4 * lk;
#pragma unroll
  for (int j = 0; j < GM_NT; ++j) pb[j] = B + (size_t)min((nt * GM_NT + j) * 16 + lr, N - 1) * K + 4 * lk;
  g4v acc[GM_MT][GM_NT];
#pragma unroll
  for (int i = 0; i < GM_MT; ++i)
#pragma unroll
    for (int j = 0; j < GM_NT; ++j) acc[i][j] = g4v{0.0, 0.0, 0.0, 0.0};
  // stages in flight: with one row tile the registers hold two (8 fields on 120
  // orbitals at 64^3: 83 -> 77 us; four no more, nor 1024 or 4096 waves)
  constexpr int PF = GM_MT == 1 ? 2 : 1;
  g4v na[PF][GM_MT], nb[PF][GM_NT];
  auto load = [&](int q, size_t r) {
#pragma unroll
    for (int i = 0; i < GM_MT; ++i) na[q][i] = *reinterpret_cast<const g4v*>(pa[i] + r);
#pragma unroll
    for (int j = 0; j < GM_NT; ++j) nb[q][j] = *reinterpret_cast<const g4v*>(pb[j] + r);
  };
#pragma unroll
  for (int q = 0; q < PF; ++q)
    if (k0 + 16 * q < k1) load(q, k0 + 16 * q);
  for (size_t rb = k0; rb < k1; rb += 16 * PF) {
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      const size_t r = rb + 16 * q;
      if (r >= k1) break;
      g4v a[GM_MT], b[GM_NT];
#pragma unroll
      for (int i = 0; i < GM_MT; ++i) a[i] = na[q][i];
#pragma unroll
      for (int j = 0; j < GM_NT; ++j) b[j] = nb[q][j];
      if (r + 16 * PF < k1) load(q, r + 16 * PF);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < GM_MT; ++i)
#pragma unroll
          for (int j = 0; j < GM_NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][t], b[j][t], acc[i][j], 0, 0, 0);
    }
  }
  double* out = part + (size_t)kc * M * N;
#pragma unroll
  for (int i = 0; i < GM_MT; ++i)
#pragma unroll
    for (int j = 0; j < GM_NT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = (mt * GM_MT + i) * 16 + 4 * q + lk, n = (nt * GM_NT + j) * 16 + lr;
        if (m < M && n < N) out[(size_t)m * N + n] = acc[i][j][q];
      }
}

// C[i] = scale sum_k part[k][i]: a block sums 256 / SL outputs in SL slices of
// the chunks and adds the slices in order.  32 slices below 1024 outputs, where
// eight leave most of the chip idle (180 outputs of 1728 chunks: 19.5 -> 7 us;
// 3600 of 1024: no difference to the call).
template <int SL>
__global__ void __launch_bounds__(256) k_gemm_reduce(const double* __restrict__ part, int nchunk, size_t MN,
                                                     double scale, double* __restrict__ C) {
  constexpr int W = 256 / SL;
  __shared__ double red[SL][W];
  const int o = threadIdx.x % W, j = threadIdx.x / W;
  const size_t i = (size_t)blockIdx.x * W + o;
  double s = 0;
  if (i < MN)
#pragma unroll 4
    for (int k = j; k < nchunk; k += SL) s += part[(size_t)k * MN + i];
  red[j][o] = s;
  __syncthreads();
  if (j == 0 && i < MN) {
    double t = 0;
#pragma unroll
    for (int q = 0; q < SL; ++q) t += red[q][o];
    C[i] = t * scale;
  }
}

// chunks for about 2048 waves (two per SIMD), each at least 64 points and, for
// short sums, at most 4096; of large products more, so that the partial sums
// stay below 4096 tiles of 64 x 64 (134 MB)
struct GemmPlan {
  int mt, nt, nmt, nnt, nchunk;
  size_t chunk;
};
static GemmPlan gemm_plan(int M, int N, size_t K) {
  GemmPlan p;
  const int tn = (N + 15) / 16, gn = (tn + 3) / 4;
  p.mt = M <= 16 ? 1 : 2;
  p.nt = (tn + gn - 1) / gn;
  p.nmt = (M + 16 * p.mt - 1) / (16 * p.mt);
  p.nnt = (tn + p.nt - 1) / p.nt;
  const size_t tiles = (size_t)p.nmt * p.nnt, want = std::max<size_t>(1, (2048 + tiles - 1) / tiles);
  const size_t t64 = (size_t)((M + 63) / 64) * ((N + 63) / 64);
  size_t most = 4096;
  while (t64 * ((K + most - 1) / most) > 4096 && most < K) most *= 2;
  p.chunk = std::min(most, std::max<size_t>(64, ((K + want - 1) / want + 15) / 16 * 16));
  p.nchunk = (int)((K + p.chunk - 1) / p.chunk);
  return p;
}
size_t gemm_part_elems(int M, int N, size_t K) { return (size_t)gemm_plan(M, N, K).nchunk * M * N; }

template <int MT>
static void gemm_go(const GemmPlan& p, const double* A, int M, const double* B, int N, size_t K, double* part,
                    hipStream_t st) {
  const unsigned nwave = (unsigned)p.nmt * p.nnt * p.nchunk;
  auto k = p.nt == 1 ? k_gemm_f64<MT, 1> : p.nt == 2 ? k_gemm_f64<MT, 2> : p.nt == 3 ? k_gemm_f64<MT, 3>
                                                                                  : k_gemm_f64<MT, 4>;
  hipLaunchKernelGGL(k, dim3((nwave + 3) / 4), dim3(256), 0, st, A, M, B, N, K, p.chunk, p.nmt, p.nnt, nwave, part);
}
hipError_t launch_gemm_f64(const double* A, int M, const double* B, int N, size_t K, double scale,
                           double* part, double* C, hipStream_t st) {
  if (M < 1 || N < 1 || K % 16) return hipErrorInvalidValue;
  const GemmPlan p = gemm_plan(M, N, K);
  if (p.mt == 1) gemm_go<1>(p, A, M, B, N, K, part, st);
  else gemm_go<2>(p, A, M, B, N, K, part, st);
  const size_t MN = (size_t)M * N;
  if (MN < 1024)
    hipLaunchKernelGGL(k_gemm_reduce<32>, dim3((unsigned)((MN + 7) / 8)), dim3(256), 0, st, part, p.nchunk, MN, scale, C);
  else
    hipLaunchKernelGGL(k_gemm_reduce<8>, dim3((unsigned)((MN + 31) / 32)), dim3(256), 0, st, part, p.nchunk, MN, scale, C);
  return hipGetLastError();
}

// The projection: a wave owns 16 MF fields and 64 points (four column tiles)
// and walks the orbitals four at a time, A = C[j][s], B = phi_s at 16
// consecutive points.  phi is read once per 16 MF fields, which bounds it.
// With the Chebyshev step in the epilogue the projected field is never stored:
// 64^3, 30 fields, 120 orbitals: 503 MB in 100 us (4.99 TB/s), against 3 x (87
// + 15) us for sets of 10 and a pass of its own for the step.
struct ChebStep {
  const double *fc, *fp;
  double* fn;
  double ia, b, dv;
  int first, n_o;
  double* part;          // [blocks][6], nullable: no sums
};
constexpr int PJ_PT = 4;
template <int MF, bool CHEB>
__global__ void __launch_bounds__(256, 2) k_project_f64(double* __restrict__ out, int nf,
                                                        const double* __restrict__ phi, int S,
                                                        const double* __restrict__ C, size_t ng, ChebStep ch) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, w = threadIdx.x >> 6;
  const size_t r0 = ((size_t)blockIdx.x * 4 + w) * 16 * PJ_PT;
  const int f0 = blockIdx.y * 16 * MF;
  size_t rc[PJ_PT];
#pragma unroll
  for (int p = 0; p < PJ_PT; ++p) rc[p] = min(r0 + 16 * p + lr, ng - 1);
  const double* cr[MF];
#pragma unroll
  for (int i = 0; i < MF; ++i) cr[i] = C + (size_t)min(f0 + 16 * i + lr, nf - 1) * S;
  g4v acc[MF][PJ_PT];
#pragma unroll
  for (int i = 0; i < MF; ++i)
#pragma unroll
    for (int p = 0; p < PJ_PT; ++p) acc[i][p] = g4v{0.0, 0.0, 0.0, 0.0};
  double nc[MF], nb[PJ_PT];
  // orbitals past the last: coefficient and orbital both zero
  auto load = [&](int sb) {
    const int s = sb + lk;
    const bool live = s < S;
#pragma unroll
    for (int i = 0; i < MF; ++i) nc[i] = live ? cr[i][s] : 0.0;
#pragma unroll
    for (int p = 0; p < PJ_PT; ++p) nb[p] = live ? phi[(size_t)s * ng + rc[p]] : 0.0;
  };
  load(0);
#pragma unroll 2
  for (int sb = 0; sb < S; sb += 4) {
    double c[MF], b[PJ_PT];
#pragma unroll
    for (int i = 0; i < MF; ++i) c[i] = nc[i];
#pragma unroll
    for (int p = 0; p < PJ_PT; ++p) b[p] = nb[p];
    if (sb + 4 < S) load(sb + 4);
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int p = 0; p < PJ_PT; ++p) acc[i][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[i], b[p], acc[i][p], 0, 0, 0);
  }
  __shared__ double red[4][16 * MF][2];
#pragma unroll
  for (int i = 0; i < MF; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int fl = 16 * i + 4 * q + lk, f = f0 + fl;
      double s0 = 0, s1 = 0;
      if (f < nf)
#pragma unroll
        for (int p = 0; p < PJ_PT; ++p) {
          const size_t r = r0 + 16 * p + lr, e = (size_t)f * ng + r;
          if (r >= ng) continue;
          const double x = out[e] - acc[i][p][q];
          if (!CHEB) {
            out[e] = x;
          } else {
            const double cur = ch.fc[e];
            const double t = (x - ch.b * cur) * ch.ia;
            const double nx = ch.first ? t : 2.0 * t - ch.fp[e];
            ch.fn[e] = nx;
            s0 += cur * cur;
            s1 += nx * cur;
          }
        }
      if (CHEB && ch.part) {
        for (int o = 8; o > 0; o >>= 1) {
          s0 += __shfl_xor(s0, o, 16);
          s1 += __shfl_xor(s1, o, 16);
        }
        if (lr == 0) {
          red[w][fl][0] = s0;
          red[w][fl][1] = s1;
        }
      }
    }
  if (CHEB && ch.part) {
    // six sums of the block: its fields of each set, waves in order
    __syncthreads();
    if (threadIdx.x < 6) {
      const int p = threadIdx.x % 3, v = threadIdx.x / 3;
      double t = 0;
      for (int fl = 0; fl < 16 * MF; ++fl)
        if (f0 + fl < nf && (f0 + fl) / ch.n_o == p)
          for (int k = 0; k < 4; ++k) t += red[k][fl][v];
      ch.part[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 6 + threadIdx.x] = t * ch.dv;
    }
  }
}

// S[q] = sum_k part[k][q], q < 6: one block, a fixed tree
__global__ void __launch_bounds__(384) k_project_sums(const double* __restrict__ part, int nblk,
                                                      double* __restrict__ S) {
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double s = 0;
#pragma unroll 8
  for (int k = lane; k < nblk; k += 64) s += part[(size_t)k * 6 + q];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) S[q] = s;
}

// fields a wave takes: all of them up to 48 (phi is then read once), groups of
// 48 beyond; with four column tiles 48 are what 256 registers hold
static dim3 project_grid(int nf, size_t ng, int* mf) {
  const int t = (nf + 15) / 16, groups = (t + 2) / 3;
  *mf = (t + groups - 1) / groups;
  return dim3((unsigned)((ng + 64 * PJ_PT - 1) / (64 * PJ_PT)), (unsigned)((t + *mf - 1) / *mf));
}
template <bool CHEB>
static hipError_t project_go(double* out, int nf, const double* phi, int S, const double* C, size_t ng,
                             const ChebStep& ch, hipStream_t st) {
  int mf;
  const dim3 g = project_grid(nf, ng, &mf), b(256);
  if (mf == 1) hipLaunchKernelGGL((k_project_f64<1, CHEB>), g, b, 0, st, out, nf, phi, S, C, ng, ch);
  else if (mf == 2) hipLaunchKernelGGL((k_project_f64<2, CHEB>), g, b, 0, st, out, nf, phi, S, C, ng, ch);
  else hipLaunchKernelGGL((k_project_f64<3, CHEB>), g, b, 0, st, out, nf, phi, S, C, ng, ch);
  return hipGetLastError();
}

hipError_t launch_project_out(double* out, int nf, const double* phi, int S, const double* C, size_t ng,
                              hipStream_t st) {
  if (nf < 1 || S < 1) return hipErrorInvalidValue;
  return project_go<false>(out, nf, phi, S, C, ng, ChebStep{}, st);
}
size_t project_part_elems(int nf, size_t ng) {
  int mf;
  const dim3 g = project_grid(nf, ng, &mf);
  return (size_t)g.x * g.y * 6;
}
hipError_t launch_project_cheb(const double* af, int n_o, int n_pol, const double* phi, int S, const double* C,
                               size_t ng, const double* fc, const double* fp, double* fn, double a, double b,
                               int first, double dv, double* part, double* Sk, hipStream_t st) {
  if (n_o < 1 || n_pol < 1 || n_pol > 3 || S < 1 || !part != !Sk) return hipErrorInvalidValue;
  const int nf = n_o * n_pol;
  const ChebStep ch{fc, fp, fn, 1.0 / a, b, dv, first, n_o, part};
  // (CHEB reads af only)
  const hipError_t e = project_go<true>(const_cast<double*>(af), nf, phi, S, C, ng, ch, st);
  if (e != hipSuccess || !part) return e;
  hipLaunchKernelGGL(k_project_sums, dim3(1), dim3(384), 0, st, part, (int)(project_part_elems(nf, ng) / 6), Sk);
  return hipGetLastError();
}

}  // namespace bse
