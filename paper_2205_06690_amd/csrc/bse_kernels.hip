// Tamm-Dancoff matrix (Eq. 1) assembly, dipoles, the FP64 contractions,
// the Lanczos and Chebyshev spectra (Eqs. 7-8), the matrix-free A f of the
// mixed representation (Eq. 6) and the surrogate's features, for gfx950.
//
// The exchange 2(ia|jb) and direct (ab|W|ij) terms are grid contractions
// C[m][n] = h^3 sum_r A_m(r) B_n(r) with K = n_g in the thousands to
// millions and small M, N: split-K GEMMs.  FP64 mode runs them here with
// FP64 FMA; mixed precision on the BF16 matrix cores (contract_mfma.hip).
#include <hip/hip_runtime.h>

#include "bse_kernels.h"

#include <algorithm>

namespace bse {


// flags[b] |= 1 if row b of w has a non-finite value (flags are not cleared)
__global__ void k_finite_check(const double* __restrict__ w, size_t ng, int* __restrict__ flags) {
  const int b = blockIdx.y;
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  int mine = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < ng; i += (size_t)gridDim.x * blockDim.x)
    if (!isfinite(w[(size_t)b * ng + i])) mine = 1;
  if (mine) atomicOr(&bad, 1);
  __syncthreads();
  if (threadIdx.x == 0 && bad) atomicOr(&flags[b], 1);
}

__global__ void k_fill_nan(double* __restrict__ w, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) w[i] = __builtin_nan("");
}

// out[k][r] = phi_p[r] phi_q[r] for (p, q) = pq[k]
template <typename T>
__global__ void k_products(const double* __restrict__ phi, const int* __restrict__ pq, int K,
                           size_t ng, T* __restrict__ out) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (r >= ng || k >= K) return;
  const int p = pq[2 * k], q = pq[2 * k + 1];
  out[(size_t)k * ng + r] = (T)(phi[(size_t)p * ng + r] * phi[(size_t)q * ng + r]);
}

// A[(ia),(jb)] = (e_a - e_i + Delta) d_ij d_ab + 2 X[(ia),(jb)] - D[ab][ij]
// with D packed over a <= b and i <= j (row-major upper triangles).
__device__ __forceinline__ int upack(int a, int b, int n) {
  if (a > b) { const int t = a; a = b; b = t; }
  return a * n - a * (a - 1) / 2 + (b - a);
}
__global__ void k_assemble_a(const double* __restrict__ X, const double* __restrict__ D, int no,
                             int nc, int nij, const double* __restrict__ eps_v,
                             const double* __restrict__ eps_c, double scissors,
                             double* __restrict__ A) {
  const int n = no * nc;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  const int row = idx / n, col = idx % n;
  const int i = row / nc, a = row % nc, j = col / nc, b = col % nc;
  // (ia|jb) = (jb|ia): the two computed copies are averaged, so A is
  // symmetric to the last bit whatever the rounding of the contraction
  double v = (X[idx] + X[(size_t)col * n + row]) - D[(size_t)upack(a, b, nc) * nij + upack(i, j, no)];
  if (row == col) v += eps_c[a] - eps_v[i] + scissors;
  A[idx] = v;
}

// f0[k][ax] = h^3 sum_r phi_p phi_q (r_ax - centre) for (p, q) = pq[k]
// A product's DIP_NB blocks leave part[k][block][3], k_dipole_sums adds them in
// order (64^3, 200 products: one block each 436 us).
constexpr int DIP_NB = 16;
__global__ void __launch_bounds__(256) k_dipoles(const double* __restrict__ phi,
                                                 const int* __restrict__ pq, int n, double h,
                                                 double* __restrict__ part) {
  const int k = blockIdx.x;
  const int p = pq[2 * k], q = pq[2 * k + 1];
  const size_t ng = (size_t)n * n * n;
  const size_t per = (ng + DIP_NB - 1) / DIP_NB, r0 = blockIdx.y * per, r1 = min(ng, r0 + per);
  const double c = 0.5 * n * h;
  double sx = 0, sy = 0, sz = 0;
#pragma unroll 4
  for (size_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const double v = phi[(size_t)p * ng + r] * phi[(size_t)q * ng + r];
    const unsigned xy = (unsigned)(r / n), x = xy / n, y = xy % n, z = (unsigned)(r % n);
    sx += v * (x * h - c);
    sy += v * (y * h - c);
    sz += v * (z * h - c);
  }
  __shared__ double red[3][256];
  red[0][threadIdx.x] = sx;
  red[1][threadIdx.x] = sy;
  red[2][threadIdx.x] = sz;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s)
      for (int a = 0; a < 3; ++a) red[a][threadIdx.x] += red[a][threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x < 3) part[((size_t)k * DIP_NB + blockIdx.y) * 3 + threadIdx.x] = red[threadIdx.x][0];
}
__global__ void __launch_bounds__(64) k_dipole_sums(const double* __restrict__ part, int n, double h3,
                                                    double* __restrict__ f0) {
  const int i = blockIdx.x * 64 + threadIdx.x;   // product, axis
  if (i >= n) return;
  const double* p = part + (size_t)(i / 3) * DIP_NB * 3 + i % 3;
  double s = 0;
#pragma unroll
  for (int k = 0; k < DIP_NB; ++k) s += p[3 * k];
  f0[i] = s * h3;
}

// ---------------------------------------------------------------------------
// Lanczos helpers (FP64): y = A v; c = V^T w; w -= V c; scalars on the host.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_gemv(const double* __restrict__ A, int n,
                                              const double* __restrict__ v, double* __restrict__ y) {
  const int row = blockIdx.x;
  double s = 0;
  for (int j = threadIdx.x; j < n; j += 256) s += A[(size_t)row * n + j] * v[j];
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) y[row] = red[0];
}

// c[k] = sum_i V[k][i] w[i], k < m; c[m-1] also goes to *last when given
__global__ void __launch_bounds__(256) k_vt_w(const double* __restrict__ V, int n, int m,
                                              const double* __restrict__ w, double* __restrict__ c,
                                              double* __restrict__ last) {
  const int k = blockIdx.x;
  if (k >= m) return;
  double s = 0;
  for (int i = threadIdx.x; i < n; i += 256) s += V[(size_t)k * n + i] * w[i];
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int q = 128; q > 0; q >>= 1) {
    if (threadIdx.x < q) red[threadIdx.x] += red[threadIdx.x + q];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    c[k] = red[0];
    if (last && k == m - 1) *last = red[0];
  }
}

// Lanczos iterations k0 .. k1-1 in one workgroup (n <= LZ_T, so the vectors
// live in LDS): w = A v_k, two passes of classical Gram-Schmidt against
// v_0 .. v_k (alpha_k = the first pass's coefficient on v_k), bq[k] = |w|^2
// and v_{k+1} = w / |w|; the steps of the launch-per-operation path in one
// launch.  One CU is latency bound here, so every sum is split so that many
// independent loads are in flight: A v reads columns (A is symmetric) and
// V^T c reads V's rows, both coalesced, each thread summing every P-th term
// of one element (P = LZ_T / n parts, added through LDS); the dot products
// V w take LZ_R rows per wave at a time.
constexpr int LZ_T = 1024, LZ_R = 4;
__global__ void __launch_bounds__(LZ_T) k_lanczos_steps(const double* __restrict__ A, int n,
                                                       double* __restrict__ V, int k0, int k1,
                                                       double* __restrict__ al, double* __restrict__ bq) {
  extern __shared__ double lz[];
  double* v = lz;                // [n]
  double* w = lz + n;            // [n]
  double* c = lz + 2 * n;        // [n]
  double* part = lz + 3 * n;     // [P][n]
  __shared__ double red[LZ_T / 64];
  constexpr int NW = LZ_T / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int P = LZ_T / n, i = tid % n, p = tid / n;
  for (int k = k0; k < k1; ++k) {
    if (tid < n) v[tid] = V[(size_t)k * n + tid];
    __syncthreads();
    if (p < P) {
      double t = 0;
#pragma unroll 8
      for (int j = p; j < n; j += P) t += A[(size_t)j * n + i] * v[j];
      part[p * n + i] = t;
    }
    __syncthreads();
    if (tid < n) {
      double t = 0;
      for (int q = 0; q < P; ++q) t += part[q * n + tid];
      w[tid] = t;
    }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      for (int j0 = LZ_R * wv; j0 <= k; j0 += LZ_R * NW) {
        double t[LZ_R];
#pragma unroll
        for (int q = 0; q < LZ_R; ++q) t[q] = 0;
        const int nj = min(LZ_R, k + 1 - j0);
        for (int e = lane; e < n; e += 64) {
          const double we = w[e];
#pragma unroll
          for (int q = 0; q < LZ_R; ++q)
            if (q < nj) t[q] += V[(size_t)(j0 + q) * n + e] * we;
        }
#pragma unroll
        for (int q = 0; q < LZ_R; ++q)
          for (int off = 32; off > 0; off >>= 1) t[q] += __shfl_down(t[q], off, 64);
        if (lane == 0)
          for (int q = 0; q < nj; ++q) {
            c[j0 + q] = t[q];
            if (pass == 0 && j0 + q == k) al[k] = t[q];
          }
      }
      __syncthreads();
      if (p < P) {
        double t = 0;
#pragma unroll 8
        for (int j = p; j <= k; j += P) t += c[j] * V[(size_t)j * n + i];
        part[p * n + i] = t;
      }
      __syncthreads();
      if (tid < n) {
        double t = 0;
        for (int q = 0; q < P; ++q) t += part[q * n + tid];
        w[tid] -= t;
      }
      __syncthreads();
    }
    double t = tid < n ? w[tid] * w[tid] : 0.0;
    for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
    if (lane == 0) red[wv] = t;
    __syncthreads();
    double b2 = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) b2 += red[q];
    if (tid == 0) bq[k] = b2;
    if (k + 1 < n && tid < n) V[(size_t)(k + 1) * n + tid] = w[tid] * (b2 > 0.0 ? 1.0 / sqrt(b2) : 0.0);
    __syncthreads();   // v_{k+1} in global memory before the next iteration reads it
  }
}

// w[i] -= sum_k c[k] V[k][i]
__global__ void k_w_minus_vc(const double* __restrict__ V, int n, int m,
                             const double* __restrict__ c, double* __restrict__ w) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0;
  for (int k = 0; k < m; ++k) s += c[k] * V[(size_t)k * n + i];
  w[i] -= s;
}

// out[q][j] = sum_k V[k][j] S[q][k]  (Ritz vectors q < nq), k < m
__global__ void k_vt_s(const double* __restrict__ V, int n, int m, const double* __restrict__ S,
                       double* __restrict__ out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int q = blockIdx.y;
  if (j >= n) return;
  double acc = 0;
  for (int k = 0; k < m; ++k) acc += V[(size_t)k * n + j] * S[(size_t)q * m + k];
  out[(size_t)q * n + j] = acc;
}

// out = w / sqrt(*bsq) (zero after a breakdown, which the host truncates)
__global__ void k_scale_norm(const double* __restrict__ w, int n, const double* __restrict__ bsq,
                             double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const double b = *bsq;
  const double s = b > 0.0 ? 1.0 / sqrt(b) : 0.0;
  if (i < n) out[i] = w[i] * s;
}

// ---------------------------------------------------------------------------
// Chebyshev spectrum (Eqs. 7-8), FP64.  Vectors are [3][n], one row per
// polarisation.  With A~ = (A - b)/a the recursion f^{n+1} = 2 A~ f^n -
// f^{n-1} (f^1 = A~ f^0) runs K = n_mom/2 steps; step n also yields
// S_nn = <f^n|f^n> and S_n1n = <f^{n+1}|f^n>, from which the doubling
// identities T_2n = 2 T_n^2 - T_0 and T_2n+1 = 2 T_n+1 T_n - T_1 give the
// residues mu_2n = 2 S_nn - mu_0 and mu_2n+1 = 2 S_n1n - mu_1.
// ---------------------------------------------------------------------------
// row i: lo = A_ii - sum_{j != i} |A_ij|, hi = A_ii + sum_{j != i} |A_ij|
__global__ void __launch_bounds__(256) k_gershgorin(const double* __restrict__ A, int n,
                                                    double* __restrict__ lohi) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  double r = 0;
  for (int j = lane; j < n; j += 64)
    if (j != row) r += fabs(A[(size_t)row * n + j]);
  for (int off = 32; off > 0; off >>= 1) r += __shfl_down(r, off, 64);
  if (lane == 0) {
    const double d = A[(size_t)row * n + row];
    lohi[row] = d - r;
    lohi[n + row] = d + r;
  }
}

// [n][3] electron-hole dipoles -> the three start vectors [3][n]
__global__ void k_cheb_start(const double* __restrict__ f0, int n, double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
#pragma unroll
  for (int p = 0; p < 3; ++p) out[(size_t)p * n + i] = f0[(size_t)i * 3 + p];
}

// mm[0] = min_i lohi[i], mm[1] = max_i lohi[n + i]: one block
__global__ void __launch_bounds__(256) k_interval(const double* __restrict__ lohi, int n,
                                                  double* __restrict__ mm) {
  __shared__ double lo_s[256], hi_s[256];
  double lo = lohi[0], hi = lohi[n];
  for (int i = threadIdx.x; i < n; i += 256) {
    lo = fmin(lo, lohi[i]);
    hi = fmax(hi, lohi[n + i]);
  }
  lo_s[threadIdx.x] = lo;
  hi_s[threadIdx.x] = hi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      lo_s[threadIdx.x] = fmin(lo_s[threadIdx.x], lo_s[threadIdx.x + w]);
      hi_s[threadIdx.x] = fmax(hi_s[threadIdx.x], hi_s[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    mm[0] = lo_s[0];
    mm[1] = hi_s[0];
  }
}

// one recursion step, one wave per row; part[blk][0..2] = <fc|fc>,
// part[blk][3..5] = <fn|fc> over the block's rows
__global__ void __launch_bounds__(256) k_cheb_step(const double* __restrict__ A, int n,
                                                   const double* __restrict__ fc,
                                                   const double* __restrict__ fp,
                                                   double* __restrict__ fn, double ia, double b,
                                                   int first, double* __restrict__ part) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = blockIdx.x * 4 + w;
  double s0 = 0, s1 = 0, s2 = 0;
  if (row < n) {
    const double* a = A + (size_t)row * n;
    for (int j = lane; j < n; j += 64) {
      const double v = a[j];
      s0 += v * fc[j];
      s1 += v * fc[n + j];
      s2 += v * fc[2 * n + j];
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_down(s0, off, 64);
    s1 += __shfl_down(s1, off, 64);
    s2 += __shfl_down(s2, off, 64);
  }
  __shared__ double red[4][6];
  if (lane == 0) {
    double c[6] = {0, 0, 0, 0, 0, 0};
    if (row < n) {
      const double sp[3] = {s0, s1, s2};
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const double cur = fc[(size_t)p * n + row];
        const double t = (sp[p] - b * cur) * ia;
        const double nx = first ? t : 2.0 * t - fp[(size_t)p * n + row];
        fn[(size_t)p * n + row] = nx;
        c[p] = cur * cur;
        c[3 + p] = nx * cur;
      }
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) red[w][q] = c[q];
  }
  __syncthreads();
  if (threadIdx.x < 6)
    part[(size_t)blockIdx.x * 6 + threadIdx.x] =
        red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// part[k][0][q] = sum over the blocks of part[k][blk][q]: one wave per (k, q),
// lanes over the blocks, a fixed shuffle tree
__global__ void __launch_bounds__(256) k_cheb_part_sum(double* __restrict__ part, int K, int nblk) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= 6 * K) return;
  double* p = part + (size_t)(w / 6) * nblk * 6 + w % 6;
  double s = 0;
  for (int i = lane; i < nblk; i += 64) s += p[(size_t)i * 6];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) p[0] = s;
}

// the residues mu[p][m], m < 2K, from S[k][q] = part[k][0][q] (rows nblk apart)
__global__ void k_cheb_moments(const double* __restrict__ part, int K, int nblk,
                               double* __restrict__ mu) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (m >= 2 * K) return;
  auto S = [&](int k, int q) { return part[(size_t)k * nblk * 6 + q]; };
  const double mu0 = S(0, p), mu1 = S(0, 3 + p);
  double v;
  if (m == 0) v = mu0;
  else if (m == 1) v = mu1;
  else if (m % 2 == 0) v = 2.0 * S(m / 2, p) - mu0;
  else v = 2.0 * S(m / 2, 3 + p) - mu1;
  mu[(size_t)p * 2 * K + m] = v;
}

// The node sums D_p(k) = (1/M) (2 sum_{m<N} mu[p][m] T_m(x_k) - mu[p][0]), x_k =
// cos(pi (k+1/2)/M), by Clenshaw's recurrence, the three polarisations' chains
// side by side: DE[k] = D_0 + D_1 + D_2 and DE[M + k] = a x_k + b, the node's
// energy.  The residues come from LDS eight at a time: 37 us at N = 976 against
// 58 us for one chain a thread reading them from global memory.
constexpr int CN_CH = 512;
__global__ void __launch_bounds__(64) k_cheb_nodes(const double* __restrict__ mu, int N, int M, double a, double b,
                                                   double* __restrict__ DE) {
  __shared__ double sm[3][CN_CH];
  const int k = blockIdx.x * 64 + threadIdx.x;
  const double x = cos(M_PI * (k + 0.5) / M), x2 = 2.0 * x;
  double b1[3] = {0, 0, 0}, b2[3] = {0, 0, 0};
  for (int hi = N; hi > 0;) {
    const int lo = (hi - 1) / CN_CH * CN_CH;
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * (hi - lo); e += 64) {
      const int p = e / (hi - lo), j = e % (hi - lo);
      sm[p][j] = mu[(size_t)p * N + lo + j];
    }
    __syncthreads();
#pragma unroll 8
    for (int j = hi - 1; j >= max(lo, 1); --j) {
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const double b0 = x2 * b1[p] + (sm[p][j - lo] - b2[p]);
        b2[p] = b1[p];
        b1[p] = b0;
      }
    }
    hi = lo;
  }
  if (k >= M) return;
  double d[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double m0 = sm[p][0];                       // the last chunk starts at m = 0
    const double sum = m0 + x * b1[p] - b2[p];        // sum_j mu_j T_j(x)
    d[p] = (2.0 * sum - m0) / M;
  }
  DE[k] = d[0] + d[1] + d[2];
  DE[M + k] = a * x + b;
}

// sum over the 256 threads of a block, in every thread (red: 4 doubles)
__device__ __forceinline__ double block_sum4(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double t = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return t;
}

// sigma(omega_q) = omega_q sum_k G(E_k - omega_q) D(k): a block per frequency
// (6 us at 600 frequencies and 1952 nodes; one thread per frequency left the
// chip idle for 693 us)
__global__ void __launch_bounds__(256) k_cheb_sigma(const double* __restrict__ DE, int M,
                                                    const double* __restrict__ w, double sig,
                                                    double* __restrict__ out) {
  __shared__ double red[4];
  const double om = w[blockIdx.x];
  double acc = 0;
  for (int k = threadIdx.x; k < M; k += 256) {
    const double z = (DE[M + k] - om) / sig;
    acc += exp(-0.5 * z * z) * DE[k];
  }
  acc = block_sum4(acc, red);
  if (threadIdx.x == 0) out[blockIdx.x] = om * (1.0 / (sig * sqrt(2.0 * M_PI))) * acc;
}

// ---------------------------------------------------------------------------
// Frequency-resolved exciton states (Eq. 8): F_q = sum_{m < N} g_m(omega_q)
// T_m(A~) f^0 for the three dipole start vectors, accumulated during the
// full three-term recursion, and their exciton densities
// 2 sum_ia F_ia phi_i phi_a on the grid.
// ---------------------------------------------------------------------------
// g[q][m] = (2 - delta_m0)/M sum_k G(a x_k + b - omega_q) cos(m th_k), th_k =
// pi (k + 1/2)/M: the node Gaussians gk[q][k] and angles first, then a block
// per m, threads over the nodes, all frequencies (n_w <= 8) at once.  With a
// thread per (m, omega) the cosines ran on 16 of 256 CUs and once per omega
// (376 us at N = 800, 4 frequencies; 20 us now).
__global__ void __launch_bounds__(256) k_cheb_tables(const double* __restrict__ w, int n_w, int M, double a, double b,
                                                     double sig, double* __restrict__ th, double* __restrict__ gk) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_w * M) return;
  const int k = i % M;
  const double t = M_PI * (k + 0.5) / M;
  const double z = (a * cos(t) + b - w[i / M]) / sig;
  gk[i] = 1.0 / (sig * sqrt(2.0 * M_PI)) * exp(-0.5 * z * z);
  if (i < M) th[i] = t;
}
constexpr int CC_W = 8;
__global__ void __launch_bounds__(256) k_cheb_coef(const double* __restrict__ th, const double* __restrict__ gk,
                                                   int n_w, int N, int M, double* __restrict__ g) {
  __shared__ double red[4];
  const int m = blockIdx.x;
  double acc[CC_W];
#pragma unroll
  for (int q = 0; q < CC_W; ++q) acc[q] = 0;
  for (int k = threadIdx.x; k < M; k += 256) {
    const double c = cos(m * th[k]);
#pragma unroll
    for (int q = 0; q < CC_W; ++q)
      if (q < n_w) acc[q] += gk[(size_t)q * M + k] * c;
  }
#pragma unroll
  for (int q = 0; q < CC_W; ++q) {
    if (q >= n_w) break;
    const double t = block_sum4(acc[q], red);
    if (threadIdx.x == 0) g[(size_t)q * N + m] = (m == 0 ? 1.0 : 2.0) * t / M;
  }
}

// F[q][p][i] = g[q][0] f0[p][i]
__global__ void k_cheb_acc_init(const double* __restrict__ f0, int n, const double* __restrict__ g,
                                int N, int n_w, double* __restrict__ F) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 3 * n) return;
  for (int q = 0; q < n_w; ++q) F[(size_t)q * 3 * n + i] = g[(size_t)q * N] * f0[i];
}

// one recursion step (one wave per row), fn = f^{m_next}, and
// F[q][p][row] += g[q][m_next] fn[p][row]
__global__ void __launch_bounds__(256) k_cheb_step_acc(const double* __restrict__ A, int n,
                                                       const double* __restrict__ fc,
                                                       const double* __restrict__ fp,
                                                       double* __restrict__ fn, double ia, double b,
                                                       int first, const double* __restrict__ g, int N,
                                                       int m_next, int n_w, double* __restrict__ F) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int row = blockIdx.x * 4 + w;
  if (row >= n) return;
  const double* ar = A + (size_t)row * n;
  double s0 = 0, s1 = 0, s2 = 0;
  for (int j = lane; j < n; j += 64) {
    const double v = ar[j];
    s0 += v * fc[j];
    s1 += v * fc[n + j];
    s2 += v * fc[2 * n + j];
  }
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_down(s0, off, 64);
    s1 += __shfl_down(s1, off, 64);
    s2 += __shfl_down(s2, off, 64);
  }
  if (lane == 0) {
    const double sp[3] = {s0, s1, s2};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const double cur = fc[(size_t)p * n + row];
      const double t = (sp[p] - b * cur) * ia;
      const double nx = first ? t : 2.0 * t - fp[(size_t)p * n + row];
      fn[(size_t)p * n + row] = nx;
      for (int q = 0; q < n_w; ++q)
        F[((size_t)q * 3 + p) * n + row] += g[(size_t)q * N + m_next] * nx;
    }
  }
}

// dens[k][r] = 2 sum_e F[k][e] phi_{v0+i}(r) phi_{c0+a}(r), e = i n_c + a < n_o
// n_c, on the FP64 matrix cores (v_mfma_f64_16x16x4f64: lane l supplies A[l %
// 16][l / 16] and B[l / 16][l % 16], holds D[4 v + l / 16][l % 16]): 16 outputs
// x 16 points a wave, contraction over e in steps of 4, the pair products
// formed on the fly.  32^3, 800 pairs, 12 outputs: 78 us (11 us of matrix core
// time, the rest load latency), against 426 us for a thread per point.
typedef double dm4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256) k_exciton_density(const double* __restrict__ phi, int v0, int c0,
                                                         int n_o, int n_c, size_t ng,
                                                         const double* __restrict__ F, int n_out,
                                                         double* __restrict__ dens) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const size_t r = ((size_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + lr;
  const size_t rc = min(r, ng - 1);
  const int k0 = blockIdx.y * 16, n = n_o * n_c;
  // outputs past the last: a copy of it, never stored
  const double* fk = F + (size_t)min(k0 + lr, n_out - 1) * n;
  const double* pv = phi + (size_t)v0 * ng + rc;
  const double* pc = phi + (size_t)c0 * ng + rc;
  dm4 acc = {0.0, 0.0, 0.0, 0.0};
  int i = lk / n_c, a = lk % n_c;
  for (int e = 0; e < n; e += 4) {
    const bool live = e + lk < n;
    const double f = live ? fk[e + lk] : 0.0;
    const double t = live ? pv[(size_t)i * ng] * pc[(size_t)a * ng] : 0.0;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f, t, acc, 0, 0, 0);
    a += 4;
    while (a >= n_c) {
      a -= n_c;
      ++i;
    }
  }
  if (r >= ng) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int k = k0 + 4 * v + lk;
    if (k < n_out) dens[(size_t)k * ng + r] = 2.0 * acc[v];
  }
}

// F[q][i] = g[q][m] f[i] (init) or F[q][i] += g[q][m] f[i], i < len: the
// Eq. 8 sum over grid vectors of the mixed representation
__global__ void __launch_bounds__(256) k_states_acc(double* __restrict__ F, const double* __restrict__ f,
                                                   const double* __restrict__ g, int N, int m, int n_w,
                                                   size_t len, int init) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < len; i += (size_t)gridDim.x * 256) {
    const double v = f[i];
    for (int q = 0; q < n_w; ++q) {
      const double c = g[(size_t)q * N + m] * v;
      double* d = F + (size_t)q * len + i;
      *d = init ? c : *d + c;
    }
  }
}

// ---------------------------------------------------------------------------
// matrix-free A f in the mixed hole-grid representation (Eq. 6), FP64: f, Tf
// and out are [n_o][ng] real fields of the valence window; W_ij comes from
// the [n_ij][ng] stack of pairs i <= j in row order.
// ---------------------------------------------------------------------------
// rho_v = 2 sum_i phi_i f_i of set v = blockIdx.y
__global__ void k_mixed_density(const double* __restrict__ phv, const double* __restrict__ f,
                                int n_o, size_t ng, double* __restrict__ rho) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= ng) return;
  f += (size_t)blockIdx.y * n_o * ng;
  double acc = 0;
#pragma unroll 4
  for (int i = 0; i < n_o; ++i) acc += phv[(size_t)i * ng + r] * f[(size_t)i * ng + r];
  rho[(size_t)blockIdx.y * ng + r] = 2.0 * acc;
}

// out_j = Tf_j + (V + Delta - eps_j) f_j + dv phi_j - sum_i f_i W_ij for NV sets of
// NO fields: one thread per point holds every f and every sum, so that each
// W_ij (i <= j) is read once for all of them.  Bound by reading W, f and Tf and
// writing out: 64^3, 3 sets of 10, 325 MB in 57 us (5.7 TB/s, W partly from the
// Infinity Cache), against 3 x 59 us for a thread per point and field.
template <int NO, int NV>
__global__ void __launch_bounds__(256) k_mixed_combine_all(const double* __restrict__ f, const double* __restrict__ tf,
                                                           const double* __restrict__ vext,
                                                           const double* __restrict__ eps_v, double scissors,
                                                           const double* __restrict__ dv,
                                                           const double* __restrict__ phv,
                                                           const double* __restrict__ wij, size_t ng,
                                                           double* __restrict__ out) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= ng) return;
  double x[NV][NO], s[NV][NO], d[NV];
  const double v0 = vext[r] + scissors;
#pragma unroll
  for (int v = 0; v < NV; ++v) d[v] = dv[(size_t)v * ng + r];
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    const double ph = phv[(size_t)j * ng + r], vj = v0 - eps_v[j];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const size_t e = ((size_t)v * NO + j) * ng + r;
      x[v][j] = f[e];
      s[v][j] = tf[e] + vj * x[v][j] + d[v] * ph;
    }
  }
  size_t p = r;
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int j = i; j < NO; ++j, p += ng) {
      const double w = wij[p];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        s[v][j] -= x[v][i] * w;
        if (i != j) s[v][i] -= x[v][j] * w;
      }
    }
#pragma unroll
  for (int j = 0; j < NO; ++j)
#pragma unroll
    for (int v = 0; v < NV; ++v) out[((size_t)v * NO + j) * ng + r] = s[v][j];
}

// the same for any n_o: a thread per point and field, NV sets at once
template <int NV>
__global__ void __launch_bounds__(256) k_mixed_combine(const double* __restrict__ f, const double* __restrict__ tf,
                                                       const double* __restrict__ vext,
                                                       const double* __restrict__ eps_v, double scissors,
                                                       const double* __restrict__ dv, const double* __restrict__ phv,
                                                       const double* __restrict__ wij, int n_o, size_t ng,
                                                       double* __restrict__ out) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (r >= ng) return;
  const size_t set = (size_t)n_o * ng, e = (size_t)j * ng + r;
  const double vj = vext[r] + scissors - eps_v[j], ph = phv[e];
  double s[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) s[v] = tf[v * set + e] + vj * f[v * set + e] + dv[(size_t)v * ng + r] * ph;
  for (int i = 0; i < n_o; ++i) {
    const int lo = i < j ? i : j, hi = i < j ? j : i;
    const double w = wij[(size_t)(lo * n_o - lo * (lo - 1) / 2 + (hi - lo)) * ng + r];
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] -= f[v * set + (size_t)i * ng + r] * w;
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) out[v * set + e] = s[v];
}

// f0_j(r) = (r_axis - centre) phi_j(r), before the occupied-space projection
__global__ void k_mixed_dipole(const double* __restrict__ phv, int n_o, int n, double h, int axis,
                               double* __restrict__ f) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  const size_t ng = (size_t)n * n * n;
  if (r >= ng) return;
  const int ix = (int)(r / ((size_t)n * n)), iy = (int)((r / n) % n), iz = (int)(r % n);
  const int c = axis == 0 ? ix : (axis == 1 ? iy : iz);
  const double x = c * h - 0.5 * n * h;
  f[(size_t)j * ng + r] = x * phv[(size_t)j * ng + r];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
__global__ void k_fill_zero_words(unsigned int* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// zero a device buffer with a kernel (graph-capture safe, unlike a memset node)
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(k_fill_zero_words, dim3(blocks), dim3(256), 0, st,
                     reinterpret_cast<unsigned int*>(p), n);
  return hipGetLastError();
}

hipError_t launch_finite_check(const double* w, int B, size_t ng, int* flags, hipStream_t st) {
  hipLaunchKernelGGL(k_finite_check, dim3(64, B), dim3(256), 0, st, w, ng, flags);
  return hipGetLastError();
}

hipError_t launch_fill_nan(double* w, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_nan, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, n);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_products(const double* phi, const int* pq, int K, size_t ng, T* out, hipStream_t st) {
  hipLaunchKernelGGL((k_products<T>), dim3((unsigned)((ng + 255) / 256), K), dim3(256), 0, st, phi,
                     pq, K, ng, out);
  return hipGetLastError();
}
template hipError_t launch_products<double>(const double*, const int*, int, size_t, double*, hipStream_t);

hipError_t launch_assemble_a(const double* X, const double* D, int no, int nc, int nij,
                             const double* eps_v, const double* eps_c, double scissors, double* A,
                             hipStream_t st) {
  const int n = no * nc;
  hipLaunchKernelGGL(k_assemble_a, dim3((n * n + 255) / 256), dim3(256), 0, st, X, D, no, nc, nij,
                     eps_v, eps_c, scissors, A);
  return hipGetLastError();
}

size_t dipoles_part_elems(int K) { return (size_t)K * DIP_NB * 3; }
hipError_t launch_dipoles(const double* phi, const int* pq, int K, int n, double h, double* part, double* f0,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_dipoles, dim3(K, DIP_NB), dim3(256), 0, st, phi, pq, n, h, part);
  hipLaunchKernelGGL(k_dipole_sums, dim3((3 * K + 63) / 64), dim3(64), 0, st, part, 3 * K, h * h * h, f0);
  return hipGetLastError();
}

hipError_t launch_gemv(const double* A, int n, const double* v, double* y, hipStream_t st) {
  hipLaunchKernelGGL(k_gemv, dim3(n), dim3(256), 0, st, A, n, v, y);
  return hipGetLastError();
}
hipError_t launch_mixed_density(const double* phv, const double* f, int n_o, int n_vec, size_t ng, double* rho,
                                hipStream_t st) {
  hipLaunchKernelGGL(k_mixed_density, dim3((unsigned)((ng + 255) / 256), n_vec), dim3(256), 0, st, phv, f, n_o,
                     ng, rho);
  return hipGetLastError();
}
template <int NV>
static hipError_t combine_go(int n_o, hipStream_t st, const double* f, const double* tf, const double* vext,
                             const double* eps_v, double scissors, const double* dv, const double* phv,
                             const double* wij, size_t ng, double* out) {
  const dim3 g((unsigned)((ng + 255) / 256)), b(256);
#define BSE_COMBINE(NO)                                                                                          \
  case NO:                                                                                                       \
    hipLaunchKernelGGL((k_mixed_combine_all<NO, NV>), g, b, 0, st, f, tf, vext, eps_v, scissors, dv, phv, wij,   \
                       ng, out);                                                                                 \
    break;
  // one thread per point up to 12 fields (three sets of 12 are 144 registers
  // of values), a thread per point and field beyond
  switch (n_o) {
    BSE_COMBINE(1) BSE_COMBINE(2) BSE_COMBINE(3) BSE_COMBINE(4) BSE_COMBINE(5) BSE_COMBINE(6)
    BSE_COMBINE(7) BSE_COMBINE(8) BSE_COMBINE(9) BSE_COMBINE(10) BSE_COMBINE(11) BSE_COMBINE(12)
    default:
      hipLaunchKernelGGL(k_mixed_combine<NV>, dim3(g.x, n_o), b, 0, st, f, tf, vext, eps_v, scissors, dv, phv, wij,
                         n_o, ng, out);
  }
#undef BSE_COMBINE
  return hipGetLastError();
}
hipError_t launch_mixed_combine(const double* f, const double* tf, const double* vext,
                                const double* eps_v, double scissors, const double* dv,
                                const double* phv, const double* wij, int n_o, int n_vec, size_t ng,
                                double* out, hipStream_t st) {
  if (n_vec == 1) return combine_go<1>(n_o, st, f, tf, vext, eps_v, scissors, dv, phv, wij, ng, out);
  if (n_vec == 3) return combine_go<3>(n_o, st, f, tf, vext, eps_v, scissors, dv, phv, wij, ng, out);
  return hipErrorInvalidValue;
}
hipError_t launch_mixed_dipole(const double* phv, int n_o, int n, double h, int axis, double* f,
                               hipStream_t st) {
  const size_t ng = (size_t)n * n * n;
  hipLaunchKernelGGL(k_mixed_dipole, dim3((unsigned)((ng + 255) / 256), n_o), dim3(256), 0, st, phv, n_o,
                     n, h, axis, f);
  return hipGetLastError();
}
hipError_t launch_gershgorin(const double* A, int n, double* lohi, hipStream_t st) {
  hipLaunchKernelGGL(k_gershgorin, dim3((n + 3) / 4), dim3(256), 0, st, A, n, lohi);
  return hipGetLastError();
}
int cheb_blocks(int n) { return (n + 3) / 4; }
hipError_t launch_cheb_start(const double* f0, int n, double* out, hipStream_t st) {
  if (n <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cheb_start, dim3((n + 255) / 256), dim3(256), 0, st, f0, n, out);
  return hipGetLastError();
}
hipError_t launch_interval(const double* lohi, int n, double* mm, hipStream_t st) {
  if (n <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_interval, dim3(1), dim3(256), 0, st, lohi, n, mm);
  return hipGetLastError();
}
hipError_t launch_cheb_step(const double* A, int n, const double* fc, const double* fp, double* fn,
                            double a, double b, int first, double* part, hipStream_t st) {
  hipLaunchKernelGGL(k_cheb_step, dim3(cheb_blocks(n)), dim3(256), 0, st, A, n, fc, fp, fn, 1.0 / a, b,
                     first, part);
  return hipGetLastError();
}
hipError_t launch_cheb_spectrum(double* part, int K, int nblk, double* mu, int M, double* DE,
                                double a, double b, const double* w, int n_w, double sig,
                                double* out, hipStream_t st) {
  if (nblk > 1) hipLaunchKernelGGL(k_cheb_part_sum, dim3((6 * K + 3) / 4), dim3(256), 0, st, part, K, nblk);
  hipLaunchKernelGGL(k_cheb_moments, dim3((2 * K + 255) / 256, 3), dim3(256), 0, st, part, K, nblk, mu);
  if (n_w > 0) {
    hipLaunchKernelGGL(k_cheb_nodes, dim3((M + 63) / 64), dim3(64), 0, st, mu, 2 * K, M, a, b, DE);
    hipLaunchKernelGGL(k_cheb_sigma, dim3(n_w), dim3(256), 0, st, DE, M, w, sig, out);
  }
  return hipGetLastError();
}
size_t cheb_coef_scratch(int n_w, int M) { return (size_t)(1 + n_w) * M; }
hipError_t launch_cheb_coef(const double* w, int n_w, int N, int M, double a, double b, double sig,
                            double* scratch, double* g, hipStream_t st) {
  if (n_w <= 0 || n_w > CC_W || N <= 0 || M <= 0) return hipErrorInvalidValue;
  double* gk = scratch + (size_t)M;
  const unsigned nt = (unsigned)(((size_t)n_w * M + 255) / 256);
  hipLaunchKernelGGL(k_cheb_tables, dim3(nt), dim3(256), 0, st, w, n_w, M, a, b, sig, scratch, gk);
  hipLaunchKernelGGL(k_cheb_coef, dim3(N), dim3(256), 0, st, scratch, gk, n_w, N, M, g);
  return hipGetLastError();
}
hipError_t launch_cheb_acc_init(const double* f0, int n, const double* g, int N, int n_w, double* F,
                                hipStream_t st) {
  hipLaunchKernelGGL(k_cheb_acc_init, dim3((3 * n + 255) / 256), dim3(256), 0, st, f0, n, g, N, n_w, F);
  return hipGetLastError();
}
hipError_t launch_cheb_step_acc(const double* A, int n, const double* fc, const double* fp, double* fn,
                                double a, double b, int first, const double* g, int N, int m_next,
                                int n_w, double* F, hipStream_t st) {
  hipLaunchKernelGGL(k_cheb_step_acc, dim3(cheb_blocks(n)), dim3(256), 0, st, A, n, fc, fp, fn, 1.0 / a,
                     b, first, g, N, m_next, n_w, F);
  return hipGetLastError();
}
hipError_t launch_states_acc(double* F, const double* f, const double* g, int N, int m, int n_w,
                             size_t len, int init, hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((len + 255) / 256, 4096);
  hipLaunchKernelGGL(k_states_acc, dim3(blocks), dim3(256), 0, st, F, f, g, N, m, n_w, len, init);
  return hipGetLastError();
}
hipError_t launch_exciton_density(const double* phi, int v0, int c0, int n_o, int n_c, size_t ng,
                                  const double* F, int n_out, double* dens, hipStream_t st) {
  if (n_out <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_exciton_density, dim3((unsigned)((ng + 63) / 64), (n_out + 15) / 16), dim3(256), 0,
                     st, phi, v0, c0, n_o, n_c, ng, F, n_out, dens);
  return hipGetLastError();
}
// One CU streams A once per step (about 4.6e-4 n^2 us measured: 18 us at
// n = 200, 290 us at n = 800) where the chip-wide path pays about 70 us of
// launches per step: the single workgroup wins up to n ~ 390.
constexpr int LZ_MAX = 384;
static_assert(LZ_MAX <= LZ_T, "one element of every vector per thread");
int lanczos_fused_max() { return LZ_MAX; }
hipError_t launch_lanczos_steps(const double* A, int n, double* V, int k0, int k1, double* al, double* bq,
                                hipStream_t st) {
  if (n < 1 || n > lanczos_fused_max() || k0 < 0 || k1 > n || k0 >= k1) return hipErrorInvalidValue;
  const size_t sm = sizeof(double) * (3 * (size_t)n + (size_t)(LZ_T / n) * n);
  hipLaunchKernelGGL(k_lanczos_steps, dim3(1), dim3(LZ_T), sm, st, A, n, V, k0, k1, al, bq);
  return hipGetLastError();
}
hipError_t launch_reorth(const double* V, int n, int m, double* c, double* w, hipStream_t st,
                         double* last) {
  hipLaunchKernelGGL(k_vt_w, dim3(m), dim3(256), 0, st, V, n, m, w, c, last);
  hipLaunchKernelGGL(k_w_minus_vc, dim3((n + 255) / 256), dim3(256), 0, st, V, n, m, c, w);
  return hipGetLastError();
}
hipError_t launch_dot(const double* a, const double* b, int n, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_vt_w, dim3(1), dim3(256), 0, st, a, n, 1, b, out, (double*)nullptr);
  return hipGetLastError();
}
hipError_t launch_ritz(const double* V, int n, int m, const double* S, int nq, double* out,
                       hipStream_t st) {
  hipLaunchKernelGGL(k_vt_s, dim3((n + 255) / 256, nq), dim3(256), 0, st, V, n, m, S, out);
  return hipGetLastError();
}
hipError_t launch_scale_norm(const double* w, int n, const double* bsq, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_scale_norm, dim3((n + 255) / 256), dim3(256), 0, st, w, n, bsq, out);
  return hipGetLastError();
}

}  // namespace bse

namespace bse {

// ---------------------------------------------------------------------------
// surrogate features and acceptance checks
// ---------------------------------------------------------------------------
// n0(r) = 2 sum_{s < n_occ} phi_s(r)^2 (ground-state density)
__global__ void k_ground_density(const double* __restrict__ phi, int n_occ, size_t ng,
                                 double* __restrict__ n0) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= ng) return;
  double acc = 0;
  for (int s = 0; s < n_occ; ++s) {
    const double v = phi[(size_t)s * ng + r];
    acc += v * v;
  }
  n0[r] = 2.0 * acc;
}

// per-row sums: out[b][0] = sum a*a, out[b][1] = sum a*c (c nullable), out[b][2] = sum a*d
// A row's ROW_NB blocks leave their partial sums in part[b][block][3], which
// k_row_sums adds in order.  One block per row took 2.26 ms for 21 rows of
// 112^3 (5 GB/s a block); their 236 MB at the memory's rate are 48 us.
constexpr int ROW_NB = 64;
__global__ void __launch_bounds__(256) k_row_dots(const double* __restrict__ a,
                                                  const double* __restrict__ c,
                                                  const double* __restrict__ d, size_t ng,
                                                  double* __restrict__ part) {
  const int b = blockIdx.y;
  const size_t per = (ng + ROW_NB - 1) / ROW_NB, r0 = blockIdx.x * per, r1 = min(ng, r0 + per);
  double s0 = 0, s1 = 0, s2 = 0;
  for (size_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const double v = a[(size_t)b * ng + r];
    s0 += v * v;
    if (c) s1 += v * c[(size_t)b * ng + r];
    if (d) s2 += v * d[(size_t)b * ng + r];
  }
  __shared__ double red[3][256];
  red[0][threadIdx.x] = s0;
  red[1][threadIdx.x] = s1;
  red[2][threadIdx.x] = s2;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k)
      for (int j = 0; j < 3; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x < 3) part[((size_t)b * ROW_NB + blockIdx.x) * 3 + threadIdx.x] = red[threadIdx.x][0];
}
__global__ void __launch_bounds__(64) k_row_sums(const double* __restrict__ part, int n, double* __restrict__ out) {
  const int i = blockIdx.x * 64 + threadIdx.x;   // row, sum
  if (i >= n) return;
  const double* p = part + (size_t)(i / 3) * ROW_NB * 3 + i % 3;
  double s = 0;
#pragma unroll 16
  for (int k = 0; k < ROW_NB; ++k) s += p[3 * k];
  out[i] = s;
}

// x[b][0] = q_b / s_b, x[b][1] = n0 * n0_scale, x[b][2] = V * v_scale
__global__ void k_features(const double* __restrict__ q, const double* __restrict__ scale,
                           const double* __restrict__ n0, double n0s, const double* __restrict__ v,
                           double vs, size_t ng, float* __restrict__ x) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (r >= ng) return;
  float* xb = x + (size_t)b * 3 * ng;
  xb[r] = (float)(q[(size_t)b * ng + r] / scale[b]);
  xb[ng + r] = (float)(n0[r] * n0s);
  xb[2 * ng + r] = (float)(v[r] * vs);
}

// t[b] = wpol_b / s_b (FP32)
__global__ void k_targets(const double* __restrict__ wpol, const double* __restrict__ scale, size_t ng,
                          float* __restrict__ t) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (r >= ng) return;
  t[(size_t)b * ng + r] = (float)(wpol[(size_t)b * ng + r] / scale[b]);
}

// wpol_b = s_b y_b (FP64), w_b = q_b + wpol_b
// The surrogate's judge: for judged pair k, out[2k] = sum_r (a[rows[k]] - b[k])^2
// and out[2k+1] = sum_r b[k]^2 (one block per pair, fixed reduction order).
__global__ void __launch_bounds__(256) k_diff_norms(const double* __restrict__ a, const int* __restrict__ rows,
                                                    const double* __restrict__ b, size_t ng,
                                                    double* __restrict__ out) {
  const int k = blockIdx.x;
  const double* x = a + (size_t)rows[k] * ng;
  const double* y = b + (size_t)k * ng;
  double s0 = 0, s1 = 0;
  for (size_t r = threadIdx.x; r < ng; r += 256) {
    const double d = x[r] - y[r];
    s0 += d * d;
    s1 += y[r] * y[r];
  }
  __shared__ double red[2][256];
  red[0][threadIdx.x] = s0;
  red[1][threadIdx.x] = s1;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      red[0][threadIdx.x] += red[0][threadIdx.x + w];
      red[1][threadIdx.x] += red[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * k] = red[0][0];
    out[2 * k + 1] = red[1][0];
  }
}

__global__ void k_assemble_w(const double* __restrict__ q, const double* __restrict__ scale,
                             const float* __restrict__ y, size_t ng, double* __restrict__ wpol,
                             double* __restrict__ w) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (r >= ng) return;
  const size_t i = (size_t)b * ng + r;
  const double p = scale[b] * (double)y[i];
  wpol[i] = p;
  w[i] = q[i] + p;
}

// ---------------------------------------------------------------------------
// Boundary potential of the finite-box W(k->0) correction (Results
// section): v_bndry = mean of V = V_ext + v_H over the points with a zero
// index (the three faces through the origin corner; the far faces are
// their periodic images) minus its mean over the cell.  Each block sums a
// fixed range of BND_T * BND_PER points; the block sums are added in block
// order by one block, so the result does not depend on scheduling.
// ---------------------------------------------------------------------------
constexpr int BND_T = 256, BND_PER = 16;
__global__ void __launch_bounds__(BND_T) k_boundary_partial(const double* __restrict__ vext,
                                                            const double* __restrict__ vh, int n,
                                                            double* __restrict__ part) {
  __shared__ double red[BND_T / 64];
  const size_t ng = (size_t)n * n * n;
  const size_t r0 = (size_t)blockIdx.x * BND_T * BND_PER;
  double all = 0, bnd = 0;
  for (int q = 0; q < BND_PER; ++q) {
    const size_t r = r0 + (size_t)q * BND_T + threadIdx.x;
    if (r < ng) {
      const double v = vext[r] + vh[r];
      const int k = (int)(r % n), j = (int)((r / n) % n), i = (int)(r / ((size_t)n * n));
      all += v;
      if (i == 0 || j == 0 || k == 0) bnd += v;
    }
  }
  all = block_sum4(all, red);
  bnd = block_sum4(bnd, red);
  if (threadIdx.x == 0) {
    part[2 * (size_t)blockIdx.x] = all;
    part[2 * (size_t)blockIdx.x + 1] = bnd;
  }
}

__global__ void __launch_bounds__(BND_T) k_boundary_final(const double* __restrict__ part, int nblk, int n,
                                                          double* __restrict__ out) {
  __shared__ double red[BND_T / 64];
  double all = 0, bnd = 0;
  for (int b = threadIdx.x; b < nblk; b += BND_T) {
    all += part[2 * (size_t)b];
    bnd += part[2 * (size_t)b + 1];
  }
  all = block_sum4(all, red);
  bnd = block_sum4(bnd, red);
  if (threadIdx.x == 0) {
    const double nb = 3.0 * n * n - 3.0 * n + 1.0, ng = (double)n * n * n;
    out[0] = bnd / nb - all / ng;
  }
}

size_t boundary_part_elems(int n) {
  const size_t ng = (size_t)n * n * n;
  return 2 * ((ng + (size_t)BND_T * BND_PER - 1) / ((size_t)BND_T * BND_PER));
}

hipError_t launch_boundary_average(const double* vext, const double* vh, int n, double* part, double* out,
                                   hipStream_t st) {
  if (n < 1) return hipErrorInvalidValue;
  const int nblk = (int)(boundary_part_elems(n) / 2);
  hipLaunchKernelGGL(k_boundary_partial, dim3(nblk), dim3(BND_T), 0, st, vext, vh, n, part);
  hipLaunchKernelGGL(k_boundary_final, dim3(1), dim3(BND_T), 0, st, part, nblk, n, out);
  return hipGetLastError();
}

hipError_t launch_ground_density(const double* phi, int n_occ, size_t ng, double* n0, hipStream_t st) {
  hipLaunchKernelGGL(k_ground_density, dim3((unsigned)((ng + 255) / 256)), dim3(256), 0, st, phi, n_occ,
                     ng, n0);
  return hipGetLastError();
}
// scale[b] = sqrt(dots[b][0] / ng) (the RMS of a row), 1 for a zero row
__global__ void k_rms_scales(const double* __restrict__ dots, int B, size_t ng, double* __restrict__ scale) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const double r = sqrt(dots[(size_t)b * 3] / (double)ng);
  scale[b] = r > 0.0 ? r : 1.0;
}
hipError_t launch_rms_scales(const double* dots, int B, size_t ng, double* scale, hipStream_t st) {
  hipLaunchKernelGGL(k_rms_scales, dim3((unsigned)((B + 63) / 64)), dim3(64), 0, st, dots, B, ng, scale);
  return hipGetLastError();
}
size_t row_dots_part_elems(int B) { return (size_t)B * ROW_NB * 3; }
hipError_t launch_row_dots(const double* a, const double* c, const double* d, int B, size_t ng,
                           double* part, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_row_dots, dim3(ROW_NB, B), dim3(256), 0, st, a, c, d, ng, part);
  hipLaunchKernelGGL(k_row_sums, dim3((3 * B + 63) / 64), dim3(64), 0, st, part, 3 * B, out);
  return hipGetLastError();
}
hipError_t launch_features(const double* q, const double* scale, const double* n0, double n0s,
                           const double* v, double vs, int B, size_t ng, float* x, hipStream_t st) {
  hipLaunchKernelGGL(k_features, dim3((unsigned)((ng + 255) / 256), B), dim3(256), 0, st, q, scale, n0,
                     n0s, v, vs, ng, x);
  return hipGetLastError();
}
hipError_t launch_targets(const double* wpol, const double* scale, int B, size_t ng, float* t,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_targets, dim3((unsigned)((ng + 255) / 256), B), dim3(256), 0, st, wpol, scale,
                     ng, t);
  return hipGetLastError();
}
hipError_t launch_diff_norms(const double* a, const int* rows, const double* b, int K, size_t ng, double* out,
                             hipStream_t st) {
  if (K <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_diff_norms, dim3(K), dim3(256), 0, st, a, rows, b, ng, out);
  return hipGetLastError();
}
hipError_t launch_assemble_w(const double* q, const double* scale, const float* y, int B, size_t ng,
                             double* wpol, double* w, hipStream_t st) {
  hipLaunchKernelGGL(k_assemble_w, dim3((unsigned)((ng + 255) / 256), B), dim3(256), 0, st, q, scale,
                     y, ng, wpol, w);
  return hipGetLastError();
}

}  // namespace bse
