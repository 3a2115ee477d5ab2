// The recursions of the electron-hole spectra with A in registers and LDS: the
// Chebyshev recursion (Eqs. 7-8) as one launch per CHEB_SEG steps, and the
// Lanczos steps up to a convergence check.
//
// A step is a matrix-vector product whose result the next step needs: as a
// launch per step it costs a launch and a walk of A through one wave per row
// (n = 200: 4.4 us and a 1 us gap, n = 800: 10.8 us) for 0.1 - 2 us of
// arithmetic.  The three polarisations never meet, so each gets workgroups of
// its own, and a workgroup holds 32 NI rows of A for the whole launch: one
// workgroup per polarisation up to n = 256 (nothing but its own barrier
// between steps), ceil(n / 32 NI) of them beyond, which exchange the vector
// through memory.
//
// Exchange: every f^k has a slot of its own, filled with a NaN bit pattern
// that no arithmetic produces before the launch.  A workgroup publishes its
// rows with agent-scope atomic stores and polls the others' values until they
// differ from the pattern: one trip through the memory side per step, no
// flags, no slot reused within a launch, no ordering between locations
// needed.  A poll that runs out of tries raises err and every workgroup
// leaves; the host then takes the launch-per-step path.
//
// Per step: n = 200 0.88 us (was 4.4 us and the gap to the next launch), bound
// by its dependent chain of LDS read, 104 FMAs a thread, row sums and barrier;
// n = 800 3.1 us (was 10.8 us), of which the exchange is about 2.5.
#include "cheb_f64.h"

#include <algorithm>

namespace bse {

constexpr unsigned long long CHEB_EMPTY = 0x7FF8C0DEFEEDBEEFull;
constexpr unsigned CHEB_SPIN = 1u << 21;   // polls of about a microsecond
constexpr int CR_T = 512;
// elements of A a thread keeps in registers (the rest in LDS): what 256
// registers leave beside NI sums
constexpr int cr_reg(int NI) { return NI == 8 ? 92 : 96; }

// the value of lane (l ^ B) of the same 16-lane row, by DPP: quad
// permutations for 1 and 2, the row rotation for 8, and for 4 the half-row
// mirror (l ^ 7) of the quad reversal (l ^ 3)
template <int CTRL> __device__ __forceinline__ int dpp(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}
template <int B> __device__ __forceinline__ double xor16(double v) {
  int2 w = __builtin_bit_cast(int2, v);
  if constexpr (B == 8) w = make_int2(dpp<0x128>(w.x), dpp<0x128>(w.y));
  else if constexpr (B == 4) w = make_int2(dpp<0x1B>(dpp<0x141>(w.x)), dpp<0x1B>(dpp<0x141>(w.y)));
  else if constexpr (B == 2) w = make_int2(dpp<0x4E>(w.x), dpp<0x4E>(w.y));
  else w = make_int2(dpp<0xB1>(w.x), dpp<0xB1>(w.y));
  return __builtin_bit_cast(double, w);
}
// Sums of H rows over the 16 lanes: while there are several, lanes l and
// l ^ B exchange halves and each keeps half of the rows; then plain sums.
template <int H, int B> __device__ __forceinline__ void rows16(double* s, int c16) {
  if constexpr (B > 0) {
    if constexpr (H > 1) {
      const bool up = (c16 & B) != 0;
#pragma unroll
      for (int i = 0; i < H / 2; ++i) {
        const double keep = up ? s[i + H / 2] : s[i], give = up ? s[i] : s[i + H / 2];
        s[i] = keep + xor16<B>(give);
      }
      rows16<H / 2, B / 2>(s, c16);
    } else {
      s[0] += xor16<B>(s[0]);
      rows16<1, B / 2>(s, c16);
    }
  }
}

// Thread (g, c16) of 32 groups of 16 lanes: rows r0 + g + 32 i (i < NI),
// columns c16 + 16 j (j < NJ).
template <int NI, int NJ, bool MULTI>
__global__ void __launch_bounds__(CR_T) k_cheb_res(const double* __restrict__ A, int n, const double* __restrict__ fc,
                                                   const double* __restrict__ fp, double* out, int steps, int first,
                                                   double ia, double b, int nwg, int* err) {
  constexpr int E = NI * NJ, ER = E < cr_reg(NI) ? E : cr_reg(NI), EL = E - ER;
  extern __shared__ double cr_lds[];
  double* f = cr_lds;                       // [2][16 NJ], zero past n
  double* al = cr_lds + 2 * 16 * NJ;        // [EL][CR_T]
  __shared__ int stop[2];                   // by step parity: a wave may still read the last step's
  const int tid = threadIdx.x, c16 = tid & 15, g = tid >> 4;
  const int p = blockIdx.x / nwg, r0 = (blockIdx.x % nwg) * 32 * NI;
  double ar[ER];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e % NI, j = e / NI, r = r0 + g + 32 * i, c = c16 + 16 * j;
    const double v = (r < n && c < n) ? A[(size_t)r * n + c] : 0.0;
    if (e < ER) ar[e < ER ? e : 0] = v;
    else al[(e - ER) * CR_T + tid] = v;
  }
  for (int c = tid; c < 16 * NJ; c += CR_T) {
    f[c] = c < n ? fc[(size_t)p * n + c] : 0.0;
    f[16 * NJ + c] = 0.0;
  }
  if (tid < 2) stop[tid] = 0;
  // the row this lane owns after the reduction: bits 3, 2, .. of c16 pick it
  int own = 0;
#pragma unroll
  for (int h = NI / 2, bit = 8; h > 0; h >>= 1, bit >>= 1)
    if (c16 & bit) own += h;
  const int r = r0 + g + 32 * own;
  constexpr int LOW = 16 / NI - 1;          // lanes that end with the same row
  const bool owner = (c16 & LOW) == 0 && r < n;
  double cur = r < n ? fc[(size_t)p * n + r] : 0.0;
  double prev = (!first && r < n) ? fp[(size_t)p * n + r] : 0.0;
  __syncthreads();
  for (int k = 0; k < steps; ++k) {
    const double* fk = f + (k & 1) * 16 * NJ;
    double* fn = f + ((k + 1) & 1) * 16 * NJ;
    double s[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) s[i] = 0.0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const double x = fk[c16 + 16 * j];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int e = j * NI + i;
        s[i] += (e < ER ? ar[e < ER ? e : 0] : al[(e - ER) * CR_T + tid]) * x;
      }
    }
    rows16<NI, 8>(s, c16);
    const double t = (s[0] - b * cur) * ia;
    const double nx = (first && k == 0) ? t : 2.0 * t - prev;
    prev = cur;
    cur = nx;
    double* row = out + ((size_t)k * 3 + p) * n;
    if (!MULTI) {
      if (owner) {
        row[r] = nx;
        fn[r] = nx;
      }
    } else {
      if (owner) __hip_atomic_store(row + r, nx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int c = tid; c < n; c += CR_T) {
        unsigned tries = 0;
        double v;
        while (true) {
          v = __hip_atomic_load(row + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (__builtin_bit_cast(unsigned long long, v) != CHEB_EMPTY) break;
          ++tries;
          if (tries == CHEB_SPIN) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((tries & 1023u) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            stop[k & 1] = 1;
            break;
          }
        }
        fn[c] = v;
      }
    }
    __syncthreads();
    if (MULTI && stop[k & 1]) return;
  }
}

__global__ void k_cheb_empty(unsigned long long* __restrict__ p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = CHEB_EMPTY;
}

// sum over the 16 lanes of a row, in every lane
__device__ __forceinline__ double sum16(double v) {
  v += xor16<8>(v);
  v += xor16<4>(v);
  v += xor16<2>(v);
  v += xor16<1>(v);
  return v;
}

// Lanczos iterations k0 .. k1-1 in one workgroup: w = A v_k, two passes of
// classical Gram-Schmidt against v_0 .. v_k (alpha_k = the first pass's
// coefficient on v_k), bq[k] = |w|^2, v_{k+1} = w / |w|.  A step reads A once and
// V four times, so V is what stays on the CU: group g of 16 lanes owns the
// vectors g + 32 q, the first 128 in registers, the rest in LDS; a group forms
// its coefficients and its share of V c without a barrier, and the shares meet
// in LDS.  A streams from L2 through registers.  n = 200: 11.5 us a step on
// average over 140 steps (21 us with A and V read from L2 by every step; 14 us
// with A in registers and V in LDS and L2).
constexpr int LZ_QR = 4;                    // vectors a group keeps in registers
template <int NJ>
__global__ void __launch_bounds__(CR_T) k_lanczos_res(const double* __restrict__ A, int n, double* __restrict__ V,
                                                      int k0, int k1, double* __restrict__ alpha,
                                                      double* __restrict__ bq) {
  constexpr int NP = 16 * NJ, NI = (NP + 31) / 32, NW = CR_T / 64;
  extern __shared__ double cr_lds[];
  double* f = cr_lds;                       // [NP] v_k, zero past n
  double* w = f + NP;                       // [NP]
  double* part = w + NP;                    // [NW][NP]
  double* red = part + NW * NP;             // [NW]
  double* vl = red + NW;                    // [.][NP] vectors 32 LZ_QR ..
  const int tid = threadIdx.x, c16 = tid & 15, g = tid >> 4, wv = tid >> 6;
  double vr[LZ_QR][NJ];
#pragma unroll
  for (int q = 0; q < LZ_QR; ++q)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int row = g + 32 * q, col = c16 + 16 * j;
      vr[q][j] = (row <= k0 && col < n) ? V[(size_t)row * n + col] : 0.0;
    }
  for (int e = tid; e < (k0 + 1 - 32 * LZ_QR) * NP; e += CR_T) {
    const int row = 32 * LZ_QR + e / NP, col = e % NP;
    vl[e] = col < n ? V[(size_t)row * n + col] : 0.0;
  }
  if (tid < NP) {
    f[tid] = tid < n ? V[(size_t)k0 * n + tid] : 0.0;
    w[tid] = 0.0;
  }
  __syncthreads();
  for (int k = k0; k < k1; ++k) {
    {
      // rows g + 32 i; rows and columns past the last: in-range values, dropped.
      // Four columns at a time: more loads in flight would spill V
      double s[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) s[i] = 0.0;
#pragma unroll 4
      for (int j = 0; j < NJ; ++j) {
        const int col = min(c16 + 16 * j, n - 1);
        const double x = f[c16 + 16 * j];
#pragma unroll
        for (int i = 0; i < NI; ++i) s[i] += A[(size_t)min(g + 32 * i, n - 1) * n + col] * x;
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const double t = sum16(s[i]);
        if (c16 == 0 && g + 32 * i < n) w[g + 32 * i] = t;
      }
    }
    __syncthreads();
    const int nq = k / 32;                  // vectors g + 32 q, q <= nq, may exist
    for (int pass = 0; pass < 2; ++pass) {
      double wr[NJ], u[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        wr[j] = w[c16 + 16 * j];
        u[j] = 0.0;
      }
#pragma unroll
      for (int q = 0; q < LZ_QR; ++q)
        if (q <= nq) {
          double t = 0.0;
#pragma unroll
          for (int j = 0; j < NJ; ++j) t += vr[q][j] * wr[j];
          t = sum16(t);                     // 0 for a vector that is not there yet
          if (pass == 0 && g + 32 * q == k && c16 == 0) alpha[k] = t;
#pragma unroll
          for (int j = 0; j < NJ; ++j) u[j] += t * vr[q][j];
        }
      for (int row = g + 32 * LZ_QR; row <= k; row += 32) {
        const double* x = vl + (row - 32 * LZ_QR) * NP + c16;
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < NJ; ++j) t += x[16 * j] * wr[j];
        t = sum16(t);
        if (pass == 0 && row == k && c16 == 0) alpha[k] = t;
#pragma unroll
        for (int j = 0; j < NJ; ++j) u[j] += t * x[16 * j];
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        u[j] += __shfl_xor(u[j], 16, 64);
        u[j] += __shfl_xor(u[j], 32, 64);
        if ((tid & 63) < 16) part[wv * NP + c16 + 16 * j] = u[j];
      }
      __syncthreads();
      if (tid < n) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) t += part[q * NP + tid];
        w[tid] -= t;
      }
      __syncthreads();
    }
    double t = tid < n ? w[tid] * w[tid] : 0.0;
    for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
    if ((tid & 63) == 0) red[wv] = t;
    __syncthreads();
    double b2 = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) b2 += red[q];
    if (tid == 0) bq[k] = b2;
    if (k + 1 >= n) break;
    const int kn = k + 1;
    if (tid < NP) {
      const double v = tid < n ? w[tid] * (b2 > 0.0 ? 1.0 / sqrt(b2) : 0.0) : 0.0;
      if (tid < n) V[(size_t)kn * n + tid] = v;
      f[tid] = v;
      if (kn >= 32 * LZ_QR) vl[(kn - 32 * LZ_QR) * NP + tid] = v;
    }
    __syncthreads();
    if (g == kn % 32) {
#pragma unroll
      for (int q = 0; q < LZ_QR; ++q)
        if (q == kn / 32)
#pragma unroll
          for (int j = 0; j < NJ; ++j) vr[q][j] = f[c16 + 16 * j];
    }
  }
}

// one wave per (m, polarisation)
__global__ void __launch_bounds__(256) k_cheb_dots(const double* __restrict__ fc, const double* __restrict__ out, int n,
                                                   int steps, double* __restrict__ S) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= 3 * steps) return;
  const int m = w / 3, p = w % 3;
  const double* x = m == 0 ? fc + (size_t)p * n : out + ((size_t)(m - 1) * 3 + p) * n;
  const double* y = out + ((size_t)m * 3 + p) * n;
  double s = 0, t = 0;
  for (int i = lane; i < n; i += 64) {
    const double v = x[i];
    s += v * v;
    t += y[i] * v;
  }
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_down(s, off, 64);
    t += __shfl_down(t, off, 64);
  }
  if (lane == 0) {
    S[(size_t)m * 6 + p] = s;
    S[(size_t)m * 6 + 3 + p] = t;
  }
}

// 64 components x 16 slices of the steps a block (slice j: m = j, j + 16, ..),
// the slices added in order
constexpr int CS_W = 8, CS_SL = 16;
__global__ void __launch_bounds__(1024) k_cheb_states(const double* __restrict__ fc, const double* __restrict__ out,
                                                      int n, int k0, int steps, const double* __restrict__ g, int N,
                                                      int n_w, double* __restrict__ F) {
  __shared__ double red[CS_SL][64];
  const int c = threadIdx.x & 63, j = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + c;
  const bool live = i < 3 * n;
  double acc[CS_W];
#pragma unroll
  for (int q = 0; q < CS_W; ++q) acc[q] = 0;
  if (live) {
#pragma unroll 4
    for (int m = j; m < steps; m += CS_SL) {
      const double v = out[(size_t)m * 3 * n + i];
#pragma unroll
      for (int q = 0; q < CS_W; ++q)
        if (q < n_w) acc[q] += g[(size_t)q * N + k0 + 1 + m] * v;
    }
  }
#pragma unroll
  for (int q = 0; q < CS_W; ++q) {
    if (q >= n_w) break;
    __syncthreads();
    red[j][c] = acc[q];
    __syncthreads();
    if (j == 0 && live) {
      double s = k0 == 0 ? g[(size_t)q * N] * fc[i] : F[(size_t)q * 3 * n + i];
#pragma unroll
      for (int k = 0; k < CS_SL; ++k) s += red[k][c];
      F[(size_t)q * 3 * n + i] = s;
    }
  }
}

int cheb_res_max() { return 1024; }

template <int NI, int NJ, bool MULTI>
static hipError_t cheb_res_go(const double* A, int n, const double* fc, const double* fp, double* out, int steps,
                              int first, double a, double b, int* err, hipStream_t st) {
  constexpr int E = NI * NJ, EL = E < cr_reg(NI) ? 0 : E - cr_reg(NI);
  const size_t lds = sizeof(double) * (2 * 16 * NJ + (size_t)EL * CR_T);
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_cheb_res<NI, NJ, MULTI>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int nwg = MULTI ? (n + 32 * NI - 1) / (32 * NI) : 1;
  hipLaunchKernelGGL((k_cheb_res<NI, NJ, MULTI>), dim3(3 * nwg), dim3(CR_T), lds, st, A, n, fc, fp, out, steps, first,
                     1.0 / a, b, nwg, err);
  return hipGetLastError();
}

hipError_t launch_cheb_res(const double* A, int n, const double* fc, const double* fp, double* out, int steps, int k0,
                           double a, double b, int* err, hipStream_t st) {
  if (n < 1 || n > cheb_res_max() || steps < 1 || steps > CHEB_SEG) return hipErrorInvalidValue;
  const int first = k0 == 0 ? 1 : 0;
  // columns in tiles of 16, rows in tiles of 32; 208 is where A outgrows the
  // registers of one workgroup (up to 256 the rest sits in LDS: 2.4 us a step
  // against 0.88 when n = 200 ran that way)
  if (n <= 64) return cheb_res_go<2, 4, false>(A, n, fc, fp, out, steps, first, a, b, err, st);
  if (n <= 128) return cheb_res_go<4, 8, false>(A, n, fc, fp, out, steps, first, a, b, err, st);
  if (n <= 208) return cheb_res_go<8, 13, false>(A, n, fc, fp, out, steps, first, a, b, err, st);
  if (n <= 256) return cheb_res_go<8, 16, false>(A, n, fc, fp, out, steps, first, a, b, err, st);
  const size_t tot = (size_t)steps * 3 * n;
  hipLaunchKernelGGL(k_cheb_empty, dim3((unsigned)std::min<size_t>((tot + 255) / 256, 4096)), dim3(256), 0, st,
                     reinterpret_cast<unsigned long long*>(out), tot);
  if (n <= 512) return cheb_res_go<4, 32, true>(A, n, fc, fp, out, steps, first, a, b, err, st);
  return cheb_res_go<2, 64, true>(A, n, fc, fp, out, steps, first, a, b, err, st);
}

__global__ void k_cheb_missed(int* err) { *err = 1; }
hipError_t launch_cheb_missed(int n, double* out, int steps, int* err, hipStream_t st) {
  const size_t tot = (size_t)steps * 3 * n;
  hipLaunchKernelGGL(k_cheb_empty, dim3((unsigned)std::min<size_t>((tot + 255) / 256, 4096)), dim3(256), 0, st,
                     reinterpret_cast<unsigned long long*>(out), tot);
  hipLaunchKernelGGL(k_cheb_missed, dim3(1), dim3(1), 0, st, err);
  return hipGetLastError();
}

template <int NJ>
static hipError_t lanczos_res_go(const double* A, int n, double* V, int k0, int k1, double* alpha, double* bq,
                                 hipStream_t st) {
  constexpr int NP = 16 * NJ, NW = CR_T / 64;
  const size_t lds = sizeof(double) * ((size_t)(2 + NW) * NP + NW + (size_t)std::max(0, n - 32 * LZ_QR) * NP);
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_lanczos_res<NJ>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_lanczos_res<NJ>, dim3(1), dim3(CR_T), lds, st, A, n, V, k0, k1, alpha, bq);
  return hipGetLastError();
}
// n = 208: V past its first 128 vectors takes 133 KB of LDS
int lanczos_res_max() { return 208; }
hipError_t launch_lanczos_res(const double* A, int n, double* V, int k0, int k1, double* alpha, double* bq,
                              hipStream_t st) {
  if (n < 1 || n > lanczos_res_max() || k0 < 0 || k1 > n || k0 >= k1) return hipErrorInvalidValue;
  if (n <= 64) return lanczos_res_go<4>(A, n, V, k0, k1, alpha, bq, st);
  if (n <= 128) return lanczos_res_go<8>(A, n, V, k0, k1, alpha, bq, st);
  return lanczos_res_go<13>(A, n, V, k0, k1, alpha, bq, st);
}

hipError_t launch_cheb_dots(const double* fc, const double* out, int n, int k0, int steps, double* S, hipStream_t st) {
  if (n < 1 || steps < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cheb_dots, dim3((3 * steps + 3) / 4), dim3(256), 0, st, fc, out, n, steps, S + (size_t)k0 * 6);
  return hipGetLastError();
}

hipError_t launch_cheb_states(const double* fc, const double* out, int n, int k0, int steps, const double* g, int N,
                              int n_w, double* F, hipStream_t st) {
  if (n < 1 || steps < 1 || n_w < 1 || n_w > CS_W) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cheb_states, dim3((3 * n + 63) / 64), dim3(1024), 0, st, fc, out, n, k0, steps, g, N, n_w, F);
  return hipGetLastError();
}

}  // namespace bse
