// Fourier-operator screening surrogate: forward, backward and Adam kernels
// for gfx950 (FP32 activations and accumulation, weights rounded to BF16).
//
// Spectral convolution on the kept modes K = {kx, ky in [-m, m), kz in
// [0, m)}: a truncated 3-D DFT that forms the kept frequencies only (planes to
// the kept (ky, kz), then x lines), a per-mode complex channel mix, and the
// adjoint path, whose last axes are part of the GEMM of the pointwise layer.
// The codelets are those of fft_lines.h.
#include <hip/hip_runtime.h>

#include "fft_lines.h"
#include "fno_kernels.h"

#include <algorithm>

namespace bse {

// the twiddle table copied into LDS (the transforms then read it through the
// LDS counter, not behind the vector-memory loads of the data)
template <int N>
__device__ __forceinline__ void fno_tw_lds(float2* t, const float2* __restrict__ tw, int tid, int nthr) {
  for (int i = tid; i < N; i += nthr) t[i] = tw[i];
}

// ---------------------------------------------------------------------------
// Truncated transforms.  Only K's frequencies are ever formed: with N = N1 N2
// (j = j1 N2 + j2, k1 = k mod N1),
//   X[k]  = sum_j2 w^(j2 k) A[k1][j2],  A[k1][j2] = DFT_N1 over j1 of x,
//   x[j]  = DFT_N1^-1 over k1 of  sum_{k = k1 mod N1} U[k] w^(-j2 k),
// so an axis costs its N1-point codelets and N2 products per kept frequency,
// and what passes between the axes is the kept part: planes P[field][x][c],
// c = (ky + m) m + kz, 2 m^2 of the N^2 values of a plane.
// ---------------------------------------------------------------------------
template <int N> struct FnoGeo {
  static constexpr int N1 = Fac<N>::N1, N2 = Fac<N>::N2;
  static constexpr int S = N + 8;                        // LDS row of y values: eight rows on distinct banks
  static constexpr int G = N * N2 < 256 ? 256 / (N * N2) : 1;   // planes a block takes at once
  static constexpr int IPT = G * N * N2 / 256;
};

// real planes -> kept (ky, kz): z rows from registers (lanes over j2, then y),
// then the y lines of the m kept kz.  A block walks `per` groups of G planes,
// the next group's loads in flight.  Bound by reading the field once and by
// its four barriers: 64^3, 256 fields, m = 8, 268 MB in 82 us (3.3 TB/s) plus
// 6 us for the x lines, against 287 + 29 us for full plane transforms that
// wrote all N^2 complex values of a plane and gathered the kept ones.
template <int N, int MM>
__global__ void __launch_bounds__(256) k_fno_plane_fwd(const float* __restrict__ in, unsigned np, int per,
                                                       const float2* __restrict__ tw, int m_,
                                                       float2* __restrict__ out) {
  using Ge = FnoGeo<N>;
  constexpr int N1 = Ge::N1, N2 = Ge::N2, S = Ge::S, G = Ge::G, IPT = Ge::IPT, ZS = N + 1;
  extern __shared__ unsigned char smem_raw[];
  const int m = MM ? MM : m_, ncol = 2 * m * m, tid = threadIdx.x;
  float2* t = reinterpret_cast<float2*>(smem_raw);
  float2* Z = t + G * N * S;
  float2* twl = Z + G * m * ZS;
  fno_tw_lds<N>(twl, tw, tid, 256);
  float a[IPT][N1];
  auto load = [&](unsigned p) {
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const int w = tid + 256 * it;
      const unsigned pp = min(p + (unsigned)(w / (N * N2)), np - 1);
      const float* src = in + (size_t)pp * (N * N) + (size_t)((w / N2) % N) * N + w % N2;
#pragma unroll
      for (int j1 = 0; j1 < N1; ++j1) a[it][j1] = src[j1 * N2];
    }
  };
  const unsigned p0 = blockIdx.x * (unsigned)(per * G);
  load(p0);
  for (int q = 0; q < per; ++q) {
    const unsigned p = p0 + q * G;
    if (p >= np) break;
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
      const int w = tid + 256 * it, g = w / (N * N2), y = (w / N2) % N, j2 = w % N2;
      float2 v[N1];
#pragma unroll
      for (int j1 = 0; j1 < N1; ++j1) v[j1] = make_float2(a[it][j1], 0.f);
      Dft<N1, -1, float2>::run(v);
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1)
        if (k1 < m) t[(g * N + k1 * N2 + j2) * S + y] = v[k1];
    }
    __syncthreads();
    if (q + 1 < per && p + G < np) load(p + G);
    for (int w = tid; w < G * m * N; w += 256) {
      const int y = w % N, k = (w / N) % m, g = w / (N * m);
      const float2* r = t + (g * N + (k % N1) * N2) * S + y;
      float2 acc = r[0];
#pragma unroll
      for (int j2 = 1; j2 < N2; ++j2) acc = cadd(acc, cmul(r[j2 * S], twl[(j2 * k) % N]));
      Z[(g * m + k) * ZS + y] = acc;
    }
    __syncthreads();
    for (int w = tid; w < G * m * N2; w += 256) {
      const int kz = w % m, j2 = (w / m) % N2, g = w / (m * N2);
      float2 v[N1];
#pragma unroll
      for (int j1 = 0; j1 < N1; ++j1) v[j1] = Z[(g * m + kz) * ZS + j1 * N2 + j2];
      Dft<N1, -1, float2>::run(v);
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) t[g * N * S + (k1 * N2 + j2) * m + kz] = v[k1];
    }
    __syncthreads();
    for (int w = tid; w < G * ncol; w += 256) {
      const int c = w % ncol, g = w / ncol, kz = c % m, k = (c / m - m + N) % N;
      const float2* r = t + g * N * S + (k % N1) * N2 * m + kz;
      float2 acc = r[0];
#pragma unroll
      for (int j2 = 1; j2 < N2; ++j2) acc = cadd(acc, cmul(r[j2 * m], twl[(j2 * k) % N]));
      if (p + g < np) out[(size_t)(p + g) * ncol + c] = acc;
    }
    __syncthreads();
  }
}

// x lines of KC kept columns, P[f][x][c] -> V[f][kx][c] (times c_k/ng if
// ck_scale); V's mode order is kx-major, then ky, then kz
constexpr int KC = 32;
template <int N>
__global__ void __launch_bounds__(256) k_fno_x_fwd(const float2* __restrict__ P, const float2* __restrict__ tw, int m,
                                                   int ck_scale, float2* __restrict__ V) {
  constexpr int N1 = Fac<N>::N1, N2 = Fac<N>::N2;
  __shared__ float2 t[N * KC];
  __shared__ float2 twl[N];
  const int f = blockIdx.y, tid = threadIdx.x, ncol = 2 * m * m, c0 = blockIdx.x * KC;
  fno_tw_lds<N>(twl, tw, tid, 256);
  for (int w = tid; w < N2 * KC; w += 256) {
    const int c = w % KC, j2 = w / KC;
    if (c0 + c >= ncol) continue;
    const float2* src = P + ((size_t)f * N + j2) * ncol + c0 + c;
    float2 v[N1];
#pragma unroll
    for (int j1 = 0; j1 < N1; ++j1) v[j1] = src[(size_t)j1 * N2 * ncol];
    Dft<N1, -1, float2>::run(v);
#pragma unroll
    for (int k1 = 0; k1 < N1; ++k1) t[(k1 * N2 + j2) * KC + c] = v[k1];
  }
  __syncthreads();
  const float inv = 1.0f / ((float)N * N * N);
  for (int w = tid; w < 2 * m * KC; w += 256) {
    const int c = w % KC, jx = w / KC, k = (jx - m + N) % N;
    if (c0 + c >= ncol) continue;
    const float2* r = t + (k % N1) * N2 * KC + c;
    float2 acc = r[0];
#pragma unroll
    for (int j2 = 1; j2 < N2; ++j2) acc = cadd(acc, cmul(r[j2 * KC], twl[(j2 * k) % N]));
    if (ck_scale) acc = cscale(acc, ((c0 + c) % m == 0 ? 1.0f : 2.0f) * inv);
    V[((size_t)f * 2 * m + jx) * ncol + c0 + c] = acc;
  }
}

// adjoint of k_fno_x_fwd: U[f][kx][c] (times c_k/ng if ck_scale) -> P[f][x][c]
template <int N>
__global__ void __launch_bounds__(256) k_fno_x_inv(const float2* __restrict__ U, const float2* __restrict__ tw, int m,
                                                   int ck_scale, float2* __restrict__ P) {
  constexpr int N1 = Fac<N>::N1, N2 = Fac<N>::N2;
  __shared__ float2 t[N * KC];
  __shared__ float2 twl[N];
  const int f = blockIdx.y, tid = threadIdx.x, ncol = 2 * m * m, c0 = blockIdx.x * KC;
  fno_tw_lds<N>(twl, tw, tid, 256);
  const float inv = 1.0f / ((float)N * N * N);
  for (int w = tid; w < 2 * m * KC; w += 256) {
    const int c = w % KC, jx = w / KC;
    float2 v = make_float2(0.f, 0.f);
    if (c0 + c < ncol) {
      v = U[((size_t)f * 2 * m + jx) * ncol + c0 + c];
      if (ck_scale) v = cscale(v, ((c0 + c) % m == 0 ? 1.0f : 2.0f) * inv);
    }
    t[jx * KC + c] = v;
  }
  __syncthreads();
  for (int w = tid; w < N2 * KC; w += 256) {
    const int c = w % KC, j2 = w / KC;
    if (c0 + c >= ncol) continue;
    float2 v[N1];
#pragma unroll
    for (int k1 = 0; k1 < N1; ++k1) {
      float2 acc = make_float2(0.f, 0.f);
      for (int k = k1; k < m; k += N1) acc = cadd(acc, cmulc(t[(k + m) * KC + c], twl[(j2 * k) % N]));
      for (int k = N - N1 + k1; k >= N - m; k -= N1)
        acc = cadd(acc, cmulc(t[(k - N + m) * KC + c], twl[(j2 * k) % N]));
      v[k1] = acc;
    }
    Dft<N1, +1, float2>::run(v);
    float2* dst = P + ((size_t)f * N + j2) * ncol + c0 + c;
#pragma unroll
    for (int j1 = 0; j1 < N1; ++j1) dst[(size_t)j1 * N2 * ncol] = v[j1];
  }
}

// ---------------------------------------------------------------------------
// spectral channel mix
// ---------------------------------------------------------------------------
// U[b][o][k] = sum_i V[b][i][k] R[k][i][o]
__global__ void k_spec_mix(const float2* __restrict__ V, const float2* __restrict__ R, int B, int C,
                           int K, float2* __restrict__ U) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t tot = (size_t)B * K * C;
  if (idx >= tot) return;
  const int o = (int)(idx % C);
  const int k = (int)((idx / C) % K);
  const int b = (int)(idx / ((size_t)C * K));
  float ax = 0.f, ay = 0.f;
  for (int i = 0; i < C; ++i) {
    const float2 v = V[((size_t)b * C + i) * K + k];
    const float2 r = R[((size_t)k * C + i) * C + o];
    ax += v.x * r.x - v.y * r.y;
    ay += v.x * r.y + v.y * r.x;
  }
  U[((size_t)b * C + o) * K + k] = make_float2(ax, ay);
}

// GV[b][i][k] = sum_o GU[b][o][k] conj(R[k][i][o])
__global__ void k_spec_mix_bwd_v(const float2* __restrict__ GU, const float2* __restrict__ R, int B,
                                 int C, int K, float2* __restrict__ GV) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t tot = (size_t)B * K * C;
  if (idx >= tot) return;
  const int i = (int)(idx % C);
  const int k = (int)((idx / C) % K);
  const int b = (int)(idx / ((size_t)C * K));
  float ax = 0.f, ay = 0.f;
  for (int o = 0; o < C; ++o) {
    const float2 g = GU[((size_t)b * C + o) * K + k];
    const float2 r = R[((size_t)k * C + i) * C + o];
    ax += g.x * r.x + g.y * r.y;
    ay += g.y * r.x - g.x * r.y;
  }
  GV[((size_t)b * C + i) * K + k] = make_float2(ax, ay);
}

// GR[k][i][o] = sum_b conj(V[b][i][k]) GU[b][o][k]
__global__ void k_spec_mix_bwd_r(const float2* __restrict__ V, const float2* __restrict__ GU, int B,
                                 int C, int K, float2* __restrict__ GR) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t tot = (size_t)K * C * C;
  if (idx >= tot) return;
  const int o = (int)(idx % C);
  const int i = (int)((idx / C) % C);
  const int k = (int)(idx / ((size_t)C * C));
  float ax = 0.f, ay = 0.f;
  for (int b = 0; b < B; ++b) {
    const float2 v = V[((size_t)b * C + i) * K + k];
    const float2 g = GU[((size_t)b * C + o) * K + k];
    ax += v.x * g.x + v.y * g.y;
    ay += v.x * g.y - v.y * g.x;
  }
  GR[idx] = make_float2(ax, ay);
}

// ---------------------------------------------------------------------------
// The same three products on the matrix cores (v_mfma_f32_16x16x4f32, FP32
// operands and accumulation), one wave per Fourier mode k, for channel
// counts up to 32 (padded with zeros to CP, a multiple of 16).  A complex
// product X Y is the real product of [Xr | Xi] with the 2 x 2 block form of
// Y, so the real and imaginary parts of an output are two column tiles of
// one real GEMM.  Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] of
// a 16 x 4 by 4 x 16 step and holds D[4 (l / 16) + j][l % 16], j < 4.
// Every output is written once (no atomics): results do not depend on
// scheduling.
// ---------------------------------------------------------------------------
typedef float mf4 __attribute__((ext_vector_type(4)));

// U_k = V_k R_k: rows b (16 per pass), columns [Ur | Ui], contraction over
// [i re | i im] with blocks [[Rr, Ri], [-Ri, Rr]]
template <int CP>
__global__ void __launch_bounds__(256) k_spec_mix_mfma(const float2* __restrict__ V,
                                                       const float2* __restrict__ R, int B, int C, int K,
                                                       float2* __restrict__ U) {
  constexpr int S = CP / 4, T = CP / 16;
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= K) return;
  const int lr = lane & 15, lk = lane >> 4;
  const float2* Rk = R + (size_t)k * C * C;
  float2 r[S][T];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int i = 4 * s + lk, o = 16 * t + lr;
      r[s][t] = (i < C && o < C) ? Rk[(size_t)i * C + o] : make_float2(0.f, 0.f);
    }
  for (int b0 = 0; b0 < B; b0 += 16) {
    const int b = b0 + lr;
    float2 v[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int i = 4 * s + lk;
      v[s] = (b < B && i < C) ? V[((size_t)b * C + i) * K + k] : make_float2(0.f, 0.f);
    }
    mf4 acc[2 * T];
#pragma unroll
    for (int t = 0; t < 2 * T; ++t) acc[t] = mf4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float a = part == 0 ? v[s].x : v[s].y;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float2 rr = r[s][t];
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, part == 0 ? rr.x : -rr.y, acc[t], 0, 0, 0);
          acc[T + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, part == 0 ? rr.y : rr.x, acc[T + t], 0, 0, 0);
        }
      }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = b0 + 4 * lk + j, o = 16 * t + lr;
        if (row < B && o < C) U[((size_t)row * C + o) * K + k] = make_float2(acc[t][j], acc[T + t][j]);
      }
  }
}

// GV_k = GU_k conj(R_k)^T: rows b, columns [GVr | GVi] over i, contraction
// over [o re | o im] with blocks [[Rr^T, -Ri^T], [Ri^T, Rr^T]]
template <int CP>
__global__ void __launch_bounds__(256) k_spec_mix_bwd_v_mfma(const float2* __restrict__ GU,
                                                             const float2* __restrict__ R, int B, int C,
                                                             int K, float2* __restrict__ GV) {
  constexpr int S = CP / 4, T = CP / 16;
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= K) return;
  const int lr = lane & 15, lk = lane >> 4;
  const float2* Rk = R + (size_t)k * C * C;
  float2 r[S][T];                       // r[s][t] = R[i = 16 t + lr][o = 4 s + lk]
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int o = 4 * s + lk, i = 16 * t + lr;
      r[s][t] = (i < C && o < C) ? Rk[(size_t)i * C + o] : make_float2(0.f, 0.f);
    }
  for (int b0 = 0; b0 < B; b0 += 16) {
    const int b = b0 + lr;
    float2 g[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int o = 4 * s + lk;
      g[s] = (b < B && o < C) ? GU[((size_t)b * C + o) * K + k] : make_float2(0.f, 0.f);
    }
    mf4 acc[2 * T];
#pragma unroll
    for (int t = 0; t < 2 * T; ++t) acc[t] = mf4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const float a = part == 0 ? g[s].x : g[s].y;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float2 rr = r[s][t];
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, part == 0 ? rr.x : rr.y, acc[t], 0, 0, 0);
          acc[T + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, part == 0 ? -rr.y : rr.x, acc[T + t], 0, 0, 0);
        }
      }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = b0 + 4 * lk + j, i = 16 * t + lr;
        if (row < B && i < C) GV[((size_t)row * C + i) * K + k] = make_float2(acc[t][j], acc[T + t][j]);
      }
  }
}

// GR_k = V_k^H GU_k: rows i, columns [GRr | GRi] over o, contraction over
// [b re | b im] (four batch entries per step) with blocks
// [[GUr, GUi], [GUi, -GUr]]
template <int CP>
__global__ void __launch_bounds__(256) k_spec_mix_bwd_r_mfma(const float2* __restrict__ V,
                                                             const float2* __restrict__ GU, int B, int C,
                                                             int K, float2* __restrict__ GR) {
  constexpr int T = CP / 16;
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= K) return;
  const int lr = lane & 15, lk = lane >> 4;
  mf4 acc[T][2 * T];
#pragma unroll
  for (int m = 0; m < T; ++m)
#pragma unroll
    for (int t = 0; t < 2 * T; ++t) acc[m][t] = mf4{0.f, 0.f, 0.f, 0.f};
  for (int b0 = 0; b0 < B; b0 += 4) {
    const int b = b0 + lk;
    float2 va[T], gb[T];
#pragma unroll
    for (int m = 0; m < T; ++m) {
      const int i = 16 * m + lr;
      va[m] = (b < B && i < C) ? V[((size_t)b * C + i) * K + k] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int o = 16 * t + lr;
      gb[t] = (b < B && o < C) ? GU[((size_t)b * C + o) * K + k] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int m = 0; m < T; ++m) {
        const float a = part == 0 ? va[m].x : va[m].y;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float2 g = gb[t];
          acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, part == 0 ? g.x : g.y, acc[m][t], 0, 0, 0);
          acc[m][T + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, part == 0 ? g.y : -g.x, acc[m][T + t], 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int m = 0; m < T; ++m)
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = 16 * m + 4 * lk + j, o = 16 * t + lr;
        if (i < C && o < C) GR[((size_t)k * C + i) * C + o] = make_float2(acc[m][t][j], acc[m][T + t][j]);
      }
}

// ---------------------------------------------------------------------------
// pointwise channel layers
// ---------------------------------------------------------------------------
__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.3989422804014327f;
}

// out[b][o][r] = sum_i Wm[o][i] in[b][i][r] + bias[o] (the lift and the
// projection).  CIN/COUT > 0: compile-time channel counts (inputs stay in
// registers).
constexpr int PW_MAXC = 64;
template <int CIN, int COUT>
__global__ void __launch_bounds__(256) k_pointwise(const float* __restrict__ in, int Cin_,
                                                   const float* __restrict__ Wm,
                                                   const float* __restrict__ bias, int Cout_, size_t ng,
                                                   float* __restrict__ out) {
  const int Cin = CIN > 0 ? CIN : Cin_;
  const int Cout = COUT > 0 ? COUT : Cout_;
  __shared__ float sw[PW_MAXC * PW_MAXC];
  __shared__ float sb[PW_MAXC];
  for (int e = threadIdx.x; e < Cin * Cout; e += 256) sw[e] = Wm[e];
  for (int e = threadIdx.x; e < Cout; e += 256) sb[e] = bias ? bias[e] : 0.f;
  __syncthreads();
  const size_t r = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int b = blockIdx.y;
  if (r >= ng) return;
  float xin[CIN > 0 ? CIN : PW_MAXC];
#pragma unroll
  for (int i = 0; i < (CIN > 0 ? CIN : PW_MAXC); ++i)
    if (i < Cin) xin[i] = in[((size_t)b * Cin + i) * ng + r];
#pragma unroll 4
  for (int o = 0; o < Cout; ++o) {
    float acc = sb[o];
#pragma unroll
    for (int i = 0; i < (CIN > 0 ? CIN : PW_MAXC); ++i)
      if (i < Cin) acc += sw[o * Cin + i] * xin[i];
    out[((size_t)b * Cout + o) * ng + r] = acc;
  }
}

// One Fourier layer behind the channel mix, on the FP32 matrix cores: for a
// row of z points (b, x, y)
//   q[o][z] = sum_i M[o][i] in[i][z] + bias[o] + Re sum_kz Y[o][kz] e^(i kz z)
// is one GEMM with contraction over [i | Re kz, Im kz], Y the inverse y
// transform of the kept plane P (rows of eight or so y lines at a time in
// LDS), so the spectral part never exists as a field.  Then
//   forward:  zout = q (kept for the backward pass when given),
//             out = gelu(q) (act) or q
//   backward: (M = W^T through trans, no bias) out = q gelu'(zg) when zg is
//             given: the gradient in front of the previous layer's gelu.
// Lane l supplies row l % 16 of M or Y and points CT (l % 16) .. of the CT
// column tiles (one 16-byte load per channel at 64 points a row) and holds
// rows 4 (l / 16) + v of those points, so rows of `out` are written whole.
// A block takes one x plane's y = j1 N2 + j2 for nj values of j2; a wave
// takes one y at a time with the next one's loads in flight.  KQ > 0: m <= 8,
// the z phases in registers.  Bound by the fields read and written and by
// erff: at 64^3, 32 channels, batch 8 (all three fields) 0.20 ms for 805 MB,
// batch 3 without zout 64 us for 201 MB, against 281 (inverse planes) + 50
// (scatter) + 71 (clearing the work array) + 259 us (pointwise) at batch 8,
// and in the backward pass 179 (pointwise) + 224 us (gelu').
template <int N, int T, int KQ>
__global__ void __launch_bounds__(256, T <= 2 ? 2 : 1)
    k_fno_layer(const float* __restrict__ in, const float* __restrict__ M, int trans, const float* __restrict__ bias,
                int W, const float2* __restrict__ P, int m, const float2* __restrict__ tw, int nj, int act,
                float* __restrict__ zout, const float* __restrict__ zg, float* __restrict__ out) {
  constexpr int N1 = Fac<N>::N1, N2 = Fac<N>::N2, CT = N / 16, WP = 16 * T;
  typedef float vec __attribute__((ext_vector_type(CT)));
  extern __shared__ unsigned char smem_raw[];
  const int ks = KQ ? KQ : (2 * m + 3) / 4, Qp = 4 * ks + 4;
  float* yc = reinterpret_cast<float*>(smem_raw);               // [row][o][2 kz, 2 kz + 1]
  float2* twl = reinterpret_cast<float2*>(yc + N1 * nj * WP * Qp);
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
  const int ngr = N2 / nj, x = blockIdx.x / ngr, j20 = (blockIdx.x % ngr) * nj, b = blockIdx.y;
  const size_t ng = (size_t)N * N * N;
  const int ncol = 2 * m * m;
  fno_tw_lds<N>(twl, tw, tid, 256);
  float am[T][4 * T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int s = 0; s < 4 * T; ++s) {
      const int o = 16 * t + lr, i = 4 * s + lk;
      am[t][s] = (o < W && i < W) ? (trans ? M[i * W + o] : M[o * W + i]) : 0.f;
    }
  float ab[T][4];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) ab[t][v] = (bias && 16 * t + 4 * lk + v < W) ? bias[16 * t + 4 * lk + v] : 0.f;
  const int nrow = N1 * nj, wv = tid >> 6;
  auto row_off = [&](int r) -> size_t {
    return (size_t)x * N * N + (size_t)((r % N1) * N2 + j20 + r / N1) * N;
  };
  // channels past the last: a copy of it times a zero of M
  vec nx[4 * T];
  auto load = [&](int r) {
    const float* src = in + (size_t)b * W * ng + row_off(r) + CT * lr;
#pragma unroll
    for (int s = 0; s < 4 * T; ++s) nx[s] = *reinterpret_cast<const vec*>(src + (size_t)min(4 * s + lk, W - 1) * ng);
  };
  if (wv < nrow) load(wv);
  __syncthreads();
  // inverse y transform of the kept plane for this block's rows
  for (int w = tid; w < W * m; w += 256) {
    const int o = w / m, kz = w % m;
    const float2* src = P + ((size_t)(b * W + o) * N + x) * ncol + kz;
    for (int jj = 0; jj < nj; ++jj) {
      const int j2 = j20 + jj;
      float2 v[N1];
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) v[k1] = make_float2(0.f, 0.f);
      // loads past the kept frequencies go to the last one and count as zero, so
      // that those of several rounds are in flight together (32^3, 16 modes, 32
      // channels, batch 4: 58 -> 35 us; 64^3, 32 modes, batch 1: 114 -> 67)
#pragma unroll 4
      for (int kb = 0; kb < m; kb += N1) {
#pragma unroll
        for (int k1 = 0; k1 < N1; ++k1) {
          const int k = kb + k1;
          float2 p = src[(min(k, m - 1) + m) * m];
          if (k >= m) p = make_float2(0.f, 0.f);
          v[k1] = cadd(v[k1], cmulc(p, twl[(j2 * k) % N]));
        }
      }
#pragma unroll 4
      for (int kb = N1; kb < m + N1; kb += N1) {
#pragma unroll
        for (int k1 = 0; k1 < N1; ++k1) {
          const int k = N - kb + k1;
          float2 p = src[(max(k, N - m) - N + m) * m];
          if (k < N - m) p = make_float2(0.f, 0.f);
          v[k1] = cadd(v[k1], cmulc(p, twl[(j2 * k) % N]));
        }
      }
      Dft<N1, +1, float2>::run(v);
#pragma unroll
      for (int j1 = 0; j1 < N1; ++j1)
        *reinterpret_cast<float2*>(yc + ((jj * N1 + j1) * WP + o) * Qp + 2 * kz) = v[j1];
    }
  }
  // contraction entries past the last frequency
  const int np = 4 * ks - 2 * m;
  for (int w = tid; w < nrow * WP * np; w += 256) yc[(w / np) * Qp + 2 * m + w % np] = 0.f;
  float tq[KQ ? KQ : 1][CT];
  auto phase = [&](int s, int c) -> float {
    const int q = 4 * s + lk, kz = q >> 1;
    const float2 e = twl[(kz * (CT * lr + c)) % N];
    return kz < m ? ((q & 1) ? e.y : e.x) : 0.f;
  };
  if (KQ) {
#pragma unroll
    for (int s = 0; s < KQ; ++s)
#pragma unroll
      for (int c = 0; c < CT; ++c) tq[s][c] = phase(s, c);
  }
  __syncthreads();
  for (int r = wv; r < nrow; r += 4) {
    vec cx[4 * T];
#pragma unroll
    for (int s = 0; s < 4 * T; ++s) cx[s] = nx[s];
    if (r + 4 < nrow) load(r + 4);
    mf4 acc[T][CT];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[t][c] = mf4{ab[t][0], ab[t][1], ab[t][2], ab[t][3]};
    const float* yr = yc + (size_t)r * WP * Qp + lr * Qp + lk;
    if (KQ) {
#pragma unroll
      for (int s = 0; s < KQ; ++s)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float ay = yr[16 * t * Qp + 4 * s];
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ay, tq[s][c], acc[t][c], 0, 0, 0);
        }
    } else {
      for (int s = 0; s < ks; ++s) {
        float e[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) e[c] = phase(s, c);
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const float ay = yr[16 * t * Qp + 4 * s];
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ay, e[c], acc[t][c], 0, 0, 0);
        }
      }
    }
    // the channels in chains of 16, added to the spectral part's: shorter
    // FP32 chains than one over everything
#pragma unroll
    for (int h = 0; h < T; ++h) {
      mf4 part[T][CT];
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) part[t][c] = mf4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 4 * h; s < 4 * h + 4; ++s)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int c = 0; c < CT; ++c)
            part[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(am[t][s], cx[s][c], part[t][c], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] += part[t][c];
    }
    const size_t off = (size_t)b * W * ng + row_off(r) + CT * lr;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int o = 16 * t + 4 * lk + v;
        if (o >= W) continue;
        const size_t oi = off + (size_t)o * ng;
        vec q;
#pragma unroll
        for (int c = 0; c < CT; ++c) q[c] = acc[t][c][v];
        if (zout) *reinterpret_cast<vec*>(zout + oi) = q;
        if (act) {
#pragma unroll
          for (int c = 0; c < CT; ++c) q[c] = gelu_f(q[c]);
        }
        if (zg) {
          const vec zv = *reinterpret_cast<const vec*>(zg + oi);
#pragma unroll
          for (int c = 0; c < CT; ++c) q[c] *= gelu_grad_f(zv[c]);
        }
        *reinterpret_cast<vec*>(out + oi) = q;
      }
  }
}

// Outer products over points, gW[o][i] = sum_{b,r} A[b][o][r] X[b][i][r] and
// gb[o] = sum_{b,r} A[b][o][r], on the FP32 matrix cores: lane l supplies
// channel l % 16 of a 16-channel tile of A and of X, four consecutive points
// 4 (l / 16) .. + 3 of a 16-point stage (one 16-byte load per tile), and
// holds D[4 (l / 16) + v][l % 16].  64 points are summed in FP32 (as before,
// a chain of 64 terms), everything above them in FP64.  A wave walks wp
// points, a block's waves are added through LDS, and part[blk] holds the
// block's FP64 sums.  X may be a caller's buffer: xal = 0 reads it four bytes
// at a time.  Bound by reading A and X once: at B = 8, 64^3, 32 channels 537
// MB in 0.138 ms (3.9 TB/s) and 8 us for the reduction, against 1.31 ms for
// vector FMA on LDS tiles (64 LDS reads per output and tile) and 0.59 ms for
// a reduction whose threads each walked all 2048 partials.
constexpr int OP_NW = 4;
template <int TA, int TX>
__global__ void __launch_bounds__(256) k_outer_mfma(const float* __restrict__ A, int Co, const float* __restrict__ X,
                                                    int Ci, size_t ng, int wp, int nblk_per_b, int xal,
                                                    double* __restrict__ part) {
  __shared__ double red[OP_NW - 1][64 * 4];
  const int b = blockIdx.x / nblk_per_b;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, lr = lane & 15, lk = lane >> 4;
  const size_t r0 = (size_t)(blockIdx.x % nblk_per_b) * (OP_NW * wp) + (size_t)w * wp;
  const size_t r1 = min(ng, r0 + wp);
  // rows past the last channel: a copy of it, never stored
  const float* pa[TA];
  const float* px[TX];
#pragma unroll
  for (int t = 0; t < TA; ++t) pa[t] = A + ((size_t)b * Co + min(16 * t + lr, Co - 1)) * ng + 4 * lk;
#pragma unroll
  for (int t = 0; t < TX; ++t) px[t] = X + ((size_t)b * Ci + min(16 * t + lr, Ci - 1)) * ng + 4 * lk;
  double sum[TA][TX][4], sa[TA];
#pragma unroll
  for (int t = 0; t < TA; ++t) {
    sa[t] = 0;
#pragma unroll
    for (int u = 0; u < TX; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) sum[t][u][v] = 0;
  }
  for (size_t r = r0; r < r1; r += 64) {
    mf4 acc[TA][TX];
    float fa[TA];
#pragma unroll
    for (int t = 0; t < TA; ++t) {
      fa[t] = 0.f;
#pragma unroll
      for (int u = 0; u < TX; ++u) acc[t][u] = mf4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int q = 0; q < 64; q += 16) {
      float4 a[TA], x[TX];
#pragma unroll
      for (int t = 0; t < TA; ++t) a[t] = *reinterpret_cast<const float4*>(pa[t] + r + q);
#pragma unroll
      for (int u = 0; u < TX; ++u) {
        const float* p = px[u] + r + q;
        x[u] = xal ? *reinterpret_cast<const float4*>(p) : make_float4(p[0], p[1], p[2], p[3]);
      }
#pragma unroll
      for (int t = 0; t < TA; ++t) {
        fa[t] += (a[t].x + a[t].y) + (a[t].z + a[t].w);
#pragma unroll
        for (int u = 0; u < TX; ++u) {
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].x, x[u].x, acc[t][u], 0, 0, 0);
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].y, x[u].y, acc[t][u], 0, 0, 0);
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].z, x[u].z, acc[t][u], 0, 0, 0);
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].w, x[u].w, acc[t][u], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < TA; ++t) {
      sa[t] += fa[t];
#pragma unroll
      for (int u = 0; u < TX; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) sum[t][u][v] += acc[t][u][v];
    }
  }
  // the waves' sums in order, one tile at a time; wave 0 stores
  double* out = part + (size_t)blockIdx.x * (Co * Ci + Co);
#pragma unroll
  for (int t = 0; t < TA; ++t) {
#pragma unroll
    for (int u = 0; u < TX; ++u) {
      __syncthreads();
      if (w > 0)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[w - 1][4 * lane + v] = sum[t][u][v];
      __syncthreads();
      if (w == 0)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double s = sum[t][u][v];
#pragma unroll
          for (int k = 0; k < OP_NW - 1; ++k) s += red[k][4 * lane + v];
          const int o = 16 * t + 4 * lk + v, i = 16 * u + lr;
          if (o < Co && i < Ci) out[o * Ci + i] = s;
        }
    }
    // sums of A: the four lane groups hold the same channel's other points
    double s = sa[t];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    __syncthreads();
    if (w > 0) red[w - 1][lane] = s;
    __syncthreads();
    if (w == 0) {
#pragma unroll
      for (int k = 0; k < OP_NW - 1; ++k) s += red[k][lane];
      if (lk == 0 && 16 * t + lr < Co) out[Co * Ci + 16 * t + lr] = s;
    }
  }
}

// out[j] = sum_k part[k][j] (j < npair to gW, the rest to gb): a block sums 8
// outputs in 32 slices of the blocks (slice q: k = q, q + 32, ...) and adds
// the slices in order
__global__ void __launch_bounds__(256) k_sum_partials(const double* __restrict__ part, int nblk, int len, int npair,
                                                      float* __restrict__ gW, float* __restrict__ gb) {
  __shared__ double red[32][8];
  const int o = threadIdx.x & 7, q = threadIdx.x >> 3;
  const int j = blockIdx.x * 8 + o;
  double s = 0;
  if (j < len)
#pragma unroll 4
    for (int k = q; k < nblk; k += 32) s += part[(size_t)k * len + j];
  red[q][o] = s;
  __syncthreads();
  if (q == 0 && j < len) {
    double t = 0;
#pragma unroll
    for (int k = 0; k < 32; ++k) t += red[k][o];
    if (j < npair) gW[j] = (float)t;
    else gb[j - npair] = (float)t;
  }
}

// gh[b][i][r] = Q[i] gy[b][r]
__global__ void k_proj_bwd(const float* __restrict__ gy, const float* __restrict__ Q, int C, size_t ng,
                           float* __restrict__ gh) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (r >= ng) return;
  const float g = gy[(size_t)b * ng + r];
  for (int i = 0; i < C; ++i) gh[((size_t)b * C + i) * ng + r] = Q[i] * g;
}

// per-sample sums: sq[b] = sum (y - t)^2, tt[b] = sum t^2 (partials per block)
__global__ void __launch_bounds__(256) k_loss_partial(const float* __restrict__ y, const float* __restrict__ t,
                                                      size_t ng, int nblk_per_b, double* __restrict__ part) {
  const int b = blockIdx.x / nblk_per_b;
  const size_t r0 = (size_t)(blockIdx.x % nblk_per_b) * 4096;
  double a = 0, c = 0;
  for (size_t r = r0 + threadIdx.x; r < r0 + 4096 && r < ng; r += 256) {
    const double d = (double)y[(size_t)b * ng + r] - (double)t[(size_t)b * ng + r];
    const double tv = t[(size_t)b * ng + r];
    a += d * d;
    c += tv * tv;
  }
  __shared__ double ra[256], rc[256];
  ra[threadIdx.x] = a;
  rc[threadIdx.x] = c;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      ra[threadIdx.x] += ra[threadIdx.x + s];
      rc[threadIdx.x] += rc[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * (size_t)blockIdx.x] = ra[0];
    part[2 * (size_t)blockIdx.x + 1] = rc[0];
  }
}

// gy = (2/B) (y - t) / tn[b]
__global__ void k_loss_grad(const float* __restrict__ y, const float* __restrict__ t,
                            const double* __restrict__ tn, int B, size_t ng, float* __restrict__ gy) {
  const size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (r >= ng) return;
  const size_t i = (size_t)b * ng + r;
  gy[i] = (float)(2.0 / B * ((double)y[i] - (double)t[i]) / tn[b]);
}

// Adam on the FP32 master copy; the compute copy holds the BF16-rounded values
__global__ void k_adam(float* __restrict__ master, float* __restrict__ compute,
                       const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       size_t n, float lr, float b1, float b2, float eps, float c1, float c2,
                       int bf16) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float p = master[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  master[i] = p;
  compute[i] = bf16 ? (float)(__bf16)p : p;
}

__global__ void k_round_copy(const float* __restrict__ src, float* __restrict__ dst, size_t n, int bf16) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = bf16 ? (float)(__bf16)src[i] : src[i];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int N>
struct FnoLaunch {
  using Ge = FnoGeo<N>;
  static size_t fwd_lds(int m) { return sizeof(float2) * ((size_t)Ge::G * N * Ge::S + (size_t)Ge::G * m * (N + 1) + N); }
  static hipError_t fwd(const float* in, int F, const float2* tw, int m, int ck, float2* P, float2* V,
                        hipStream_t st) {
    // groups a block walks: four, so that loads overlap the transforms, but
    // no fewer than about 1024 blocks (four per CU)
    const unsigned np = (unsigned)F * N, groups = (np + Ge::G - 1) / Ge::G;
    const int per = (int)std::min(4u, std::max(1u, groups / 1024));
    const dim3 g((groups + per - 1) / per);
    if (m == 8)
      hipLaunchKernelGGL((k_fno_plane_fwd<N, 8>), g, dim3(256), fwd_lds(m), st, in, np, per, tw, m, P);
    else
      hipLaunchKernelGGL((k_fno_plane_fwd<N, 0>), g, dim3(256), fwd_lds(m), st, in, np, per, tw, m, P);
    hipLaunchKernelGGL(k_fno_x_fwd<N>, dim3((2 * m * m + KC - 1) / KC, F), dim3(256), 0, st, P, tw, m, ck, V);
    return hipGetLastError();
  }
  static hipError_t x_inv(const float2* U, int F, const float2* tw, int m, int ck, float2* P, hipStream_t st) {
    hipLaunchKernelGGL(k_fno_x_inv<N>, dim3((2 * m * m + KC - 1) / KC, F), dim3(256), 0, st, U, tw, m, ck, P);
    return hipGetLastError();
  }
  static size_t layer_lds(int T, int m, int nj) {
    const int ks = m <= 8 ? 4 : (2 * m + 3) / 4;
    return sizeof(float) * (size_t)Ge::N1 * nj * 16 * T * (4 * ks + 4) + sizeof(float2) * N;
  }
  template <int T>
  static hipError_t layer_t(const FnoLayerArgs& a, hipStream_t st) {
    // 16 rows a block while three blocks fit on a CU, else fewer (one value
    // of j2 fits for every allowed width and mode count); fewer too where 16
    // would leave under four blocks per CU (64^3, batch 3: 68.5 us with 8
    // rows, 70.7 with 16)
    int nj = 16 / Ge::N1;
    while (nj > 1 && (layer_lds(T, a.m, nj) > 52 * 1024 || N * (Ge::N2 / nj) * a.B < 1024)) nj /= 2;
    const size_t lds = layer_lds(T, a.m, nj);
    const dim3 g(N * (Ge::N2 / nj), a.B);
    const void* k = a.m <= 8 ? (const void*)k_fno_layer<N, T, 4> : (const void*)k_fno_layer<N, T, 0>;
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    if (a.m <= 8)
      hipLaunchKernelGGL((k_fno_layer<N, T, 4>), g, dim3(256), lds, st, a.in, a.M, a.trans, a.bias, a.W, a.P, a.m, a.tw,
                         nj, a.act, a.zout, a.zg, a.out);
    else
      hipLaunchKernelGGL((k_fno_layer<N, T, 0>), g, dim3(256), lds, st, a.in, a.M, a.trans, a.bias, a.W, a.P, a.m, a.tw,
                         nj, a.act, a.zout, a.zg, a.out);
    return hipGetLastError();
  }
  static hipError_t layer(const FnoLayerArgs& a, hipStream_t st) {
    switch ((a.W + 15) / 16) {
      case 1: return layer_t<1>(a, st);
      case 2: return layer_t<2>(a, st);
      case 3: return layer_t<3>(a, st);
      case 4: return layer_t<4>(a, st);
      default: return hipErrorInvalidValue;
    }
  }
};

bool fno_grid_supported(int n) { return n == 16 || n == 32 || n == 64; }

#define FNO_DISPATCH(n, CALL)                 \
  switch (n) {                                \
    case 16: return FnoLaunch<16>::CALL;      \
    case 32: return FnoLaunch<32>::CALL;      \
    case 64: return FnoLaunch<64>::CALL;      \
    default: return hipErrorInvalidValue;     \
  }

hipError_t fno_fft_fwd(int n, const float* in, int F, const float2* tw, int m, int ck, float2* P,
                       float2* V, hipStream_t st) {
  FNO_DISPATCH(n, fwd(in, F, tw, m, ck, P, V, st));
}
hipError_t fno_x_inv(int n, const float2* U, int F, const float2* tw, int m, int ck, float2* P, hipStream_t st) {
  FNO_DISPATCH(n, x_inv(U, F, tw, m, ck, P, st));
}
hipError_t fno_layer(int n, const FnoLayerArgs& a, hipStream_t st) { FNO_DISPATCH(n, layer(a, st)); }

static inline unsigned nb(size_t n) { return (unsigned)((n + 255) / 256); }

// path 0: the matrix-core products for up to 32 channels (the vector-FMA
// ones above beyond); path 1: the vector-FMA products only
hipError_t fno_spec_mix(const float2* V, const float2* R, int B, int C, int K, float2* U, int path,
                        hipStream_t st) {
  const int g_spec_mix_path = path;
  const unsigned nw = (unsigned)((K + 3) / 4);
  if (g_spec_mix_path == 0 && C <= 16)
    hipLaunchKernelGGL(k_spec_mix_mfma<16>, dim3(nw), dim3(256), 0, st, V, R, B, C, K, U);
  else if (g_spec_mix_path == 0 && C <= 32)
    hipLaunchKernelGGL(k_spec_mix_mfma<32>, dim3(nw), dim3(256), 0, st, V, R, B, C, K, U);
  else
    hipLaunchKernelGGL(k_spec_mix, dim3(nb((size_t)B * K * C)), dim3(256), 0, st, V, R, B, C, K, U);
  return hipGetLastError();
}
hipError_t fno_spec_mix_bwd(const float2* V, const float2* GU, const float2* R, int B, int C, int K,
                            float2* GV, float2* GR, int path, hipStream_t st) {
  const int g_spec_mix_path = path;
  const unsigned nw = (unsigned)((K + 3) / 4);
  if (g_spec_mix_path == 0 && C <= 16) {
    hipLaunchKernelGGL(k_spec_mix_bwd_v_mfma<16>, dim3(nw), dim3(256), 0, st, GU, R, B, C, K, GV);
    hipLaunchKernelGGL(k_spec_mix_bwd_r_mfma<16>, dim3(nw), dim3(256), 0, st, V, GU, B, C, K, GR);
  } else if (g_spec_mix_path == 0 && C <= 32) {
    hipLaunchKernelGGL(k_spec_mix_bwd_v_mfma<32>, dim3(nw), dim3(256), 0, st, GU, R, B, C, K, GV);
    hipLaunchKernelGGL(k_spec_mix_bwd_r_mfma<32>, dim3(nw), dim3(256), 0, st, V, GU, B, C, K, GR);
  } else {
    hipLaunchKernelGGL(k_spec_mix_bwd_v, dim3(nb((size_t)B * K * C)), dim3(256), 0, st, GU, R, B, C, K, GV);
    hipLaunchKernelGGL(k_spec_mix_bwd_r, dim3(nb((size_t)K * C * C)), dim3(256), 0, st, V, GU, B, C, K, GR);
  }
  return hipGetLastError();
}
hipError_t fno_pointwise(const float* in, int Cin, const float* Wm, const float* bias, int Cout,
                         int B, size_t ng, float* out, hipStream_t st) {
  if (Cin > PW_MAXC || Cout > PW_MAXC) return hipErrorInvalidValue;
  const dim3 g(nb(ng), B);
  if (Cin == 3 && Cout == 32)
    hipLaunchKernelGGL((k_pointwise<3, 32>), g, dim3(256), 0, st, in, Cin, Wm, bias, Cout, ng, out);
  else if (Cin == 32 && Cout == 1)
    hipLaunchKernelGGL((k_pointwise<32, 1>), g, dim3(256), 0, st, in, Cin, Wm, bias, Cout, ng, out);
  else
    hipLaunchKernelGGL((k_pointwise<0, 0>), g, dim3(256), 0, st, in, Cin, Wm, bias, Cout, ng, out);
  return hipGetLastError();
}
// points per wave: about 2048 waves (two per SIMD), 64 to 1024 points each
static int outer_wp(int B, size_t ng) {
  const size_t w = ((size_t)B * ng / 2048 + 63) / 64 * 64;
  return (int)std::min<size_t>(1024, std::max<size_t>(64, w));
}
static size_t outer_blocks(int B, size_t ng) {
  const size_t blk = (size_t)OP_NW * outer_wp(B, ng);
  return (size_t)B * ((ng + blk - 1) / blk);
}
// for batches of up to B samples
size_t fno_outer_part_len(int Co, int Ci, int B, size_t ng) {
  size_t m = 0;
  for (int b = 1; b <= B; ++b) m = std::max(m, outer_blocks(b, ng));
  return m * (size_t)(Co * Ci + Co);
}
template <int TA>
static void outer_go(int tx, unsigned g, hipStream_t st, const float* A, int Co, const float* X, int Ci, size_t ng,
                     int wp, int nbb, int xal, double* part) {
  switch (tx) {
    case 1: hipLaunchKernelGGL((k_outer_mfma<TA, 1>), dim3(g), dim3(256), 0, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
    case 2: hipLaunchKernelGGL((k_outer_mfma<TA, 2>), dim3(g), dim3(256), 0, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
    case 3: hipLaunchKernelGGL((k_outer_mfma<TA, 3>), dim3(g), dim3(256), 0, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
    default: hipLaunchKernelGGL((k_outer_mfma<TA, 4>), dim3(g), dim3(256), 0, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
  }
}
// gW[o][i] (Co x Ci) and gb[o] = sums over points of A x X, A
hipError_t fno_outer(const float* A, int Co, const float* X, int Ci, int B, size_t ng, double* part,
                     float* gW, float* gb, hipStream_t st) {
  // 64-point chains and 16-byte loads: every grid has a multiple of 64 points
  if (Co < 1 || Ci < 1 || Co > PW_MAXC || Ci > PW_MAXC || ng % 64) return hipErrorInvalidValue;
  const int wp = outer_wp(B, ng), nblk = (int)outer_blocks(B, ng), nbb = nblk / B, tx = (Ci + 15) / 16;
  const int xal = reinterpret_cast<size_t>(X) % 16 == 0;
  switch ((Co + 15) / 16) {
    case 1: outer_go<1>(tx, nblk, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
    case 2: outer_go<2>(tx, nblk, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
    case 3: outer_go<3>(tx, nblk, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
    default: outer_go<4>(tx, nblk, st, A, Co, X, Ci, ng, wp, nbb, xal, part); break;
  }
  const int len = Co * Ci + Co;
  hipLaunchKernelGGL(k_sum_partials, dim3((len + 7) / 8), dim3(256), 0, st, part, nblk, len, Co * Ci, gW, gb);
  return hipGetLastError();
}
hipError_t fno_proj_bwd(const float* gy, const float* Q, int C, int B, size_t ng, float* gh, hipStream_t st) {
  hipLaunchKernelGGL(k_proj_bwd, dim3(nb(ng), B), dim3(256), 0, st, gy, Q, C, ng, gh);
  return hipGetLastError();
}
int fno_loss_blocks(size_t ng) { return (int)((ng + 4095) / 4096); }
hipError_t fno_loss_partial(const float* y, const float* t, int B, size_t ng, double* part, hipStream_t st) {
  const int nbb = fno_loss_blocks(ng);
  hipLaunchKernelGGL(k_loss_partial, dim3(B * nbb), dim3(256), 0, st, y, t, ng, nbb, part);
  return hipGetLastError();
}
hipError_t fno_loss_grad(const float* y, const float* t, const double* tn, int B, size_t ng, float* gy,
                         hipStream_t st) {
  hipLaunchKernelGGL(k_loss_grad, dim3(nb(ng), B), dim3(256), 0, st, y, t, tn, B, ng, gy);
  return hipGetLastError();
}
hipError_t fno_adam(float* master, float* compute, const float* g, float* m, float* v, size_t n,
                    float lr, float b1, float b2, float eps, int step, int bf16, hipStream_t st) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(nb(n)), dim3(256), 0, st, master, compute, g, m, v, n, lr, b1, b2,
                     eps, c1, c2, bf16);
  return hipGetLastError();
}
hipError_t fno_round_copy(const float* src, float* dst, size_t n, int bf16, hipStream_t st) {
  hipLaunchKernelGGL(k_round_copy, dim3(nb(n)), dim3(256), 0, st, src, dst, n, bf16);
  return hipGetLastError();
}

// training batches under the symmetries of the cube: output point (o0, o1,
// o2), after the flips o_k -> n - 1 - o_k, reads input point i with
// i[perm[k]] = o_k
__global__ void k_gather_sym(const float* __restrict__ src, const int* __restrict__ idx, int C, int n,
                             int p0, int p1, int p2, int fmask, float* __restrict__ dst) {
  const size_t ng = (size_t)n * n * n;
  const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= ng) return;
  const int c = blockIdx.y, b = blockIdx.z;
  int oc[3] = {(int)(o / ((size_t)n * n)), (int)((o / n) % n), (int)(o % n)};
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if ((fmask >> k) & 1) oc[k] = n - 1 - oc[k];
  int ic[3];
  ic[p0] = oc[0];
  ic[p1] = oc[1];
  ic[p2] = oc[2];
  const size_t i = ((size_t)ic[0] * n + ic[1]) * n + ic[2];
  dst[((size_t)b * C + c) * ng + o] = src[((size_t)idx[b] * C + c) * ng + i];
}

hipError_t fno_gather_sym(const float* src, const int* idx, int B, int C, int n, const int perm[3],
                          int flip_mask, float* dst, hipStream_t st) {
  const size_t ng = (size_t)n * n * n;
  hipLaunchKernelGGL(k_gather_sym, dim3((unsigned)((ng + 255) / 256), C, B), dim3(256), 0, st, src, idx, C, n,
                     perm[0], perm[1], perm[2], flip_mask, dst);
  return hipGetLastError();
}

}  // namespace bse
