// The two passes of a time step that apply exp(-i T dt), in FP64: the x factor
// fused with the pointwise step before it, and the y and z factors on whole
// y-z planes fused with the induced density, for gfx950.
//
// Along an axis exp(-i k^2 dt / 2) is a circulant matrix.  A transform, a
// phase and a transform back cost about 45 vector instructions per point and
// axis, seven trips through LDS per plane and a block barrier for each: the
// plane pass in FP64 moved 0.8 to 2.2 TB/s.  Here the circulant of N = R J
// points is split by its translations by J into R matrices of J x J (J = 16 or
// 12): with x_m(j) = sum_s x(j + J s) w^(-ms), w = exp(2 pi i / R),
//   y_m = M_m x_m,  M_m[j][j'] = (1/R) sum_s c(j - j' + J s) w^(-ms),
// c the kernel of the circulant.  The R-point DFTs are butterflies inside a
// lane (no twiddles), the products four real 16 x 16 matrix products, 128
// flops per point and axis at any N, and a lane holds the same elements of its
// line before and after, so the x pass needs no exchange at all and the plane
// pass one transpose.  Rounding: one FMA chain of 2 J terms and the small DFTs
// per axis, nearer to exact than the transforms (24^3, 200 steps: W within
// 1.7e-15 of 64-bit arithmetic, 1.3e-14 before).
//
// Measured (us, 10 orbitals a pair; transforms -> products):
//   plane pass  16^3 8 pairs 19 -> 6;   24^3 8 pairs 45 -> 12;  32^3 12 pairs 63 -> 34
//               48^3 12 pairs 256 -> 118; 64^3 11 pairs 414 -> 319 (2.9 TB/s)
//   x pass      16^3 8 pairs 18 -> 5;   24^3 8 pairs 22 -> 9;   32^3 12 pairs 32 -> 24
// What bounds them now: on the small grids latency; at 64^3 occupancy: a plane
// and its tables are 82944 bytes of LDS, 2 KB over half a CU, so one block of
// four waves runs on a CU, one wave a SIMD, and memory and matrix cores overlap
// little.
#include <hip/hip_ext.h>

#include "fft_lines.h"
#include "kin_mfma.h"

#include <algorithm>
#include <cmath>
#include <complex>

namespace bse {

// ------------------------------------------------------------------ tables
static int kin_j(int n) { return n == 24 ? 12 : 16; }

// Slot v < J / 4 of lane group g = lane / 16 holds block element 4 v + g, as
// operand (column of chunk v) and as result (row 4 v + g of the instruction).
void kin_table(int n, double h, double dt, std::vector<double>& out) {
  using ld = long double;
  const ld pi = 3.14159265358979323846264338327950288L;
  const int J = kin_j(n), R = n / J, VJ = J / 4;
  // the circulant's kernel c(d) = 1/n sum_k exp(-i k^2 dt / 2) exp(2 pi i k d / n)
  std::vector<std::complex<ld>> c(n);
  for (int d = 0; d < n; ++d) {
    std::complex<ld> s = 0;
    for (int m = 0; m < n; ++m) {
      const int mm = (m < (n + 1) / 2) ? m : m - n;
      const ld k = 2 * pi * mm / ((ld)n * h);
      const ld a = 2 * pi * (ld)((m * d) % n) / n - k * k * (ld)dt / 2;
      s += std::complex<ld>(std::cos(a), std::sin(a));
    }
    c[d] = s / (ld)n;
  }
  out.assign((size_t)2 * R * VJ * 64, 0.0);
  for (int m = 0; m < R; ++m) {
    for (int kc = 0; kc < VJ; ++kc)
      for (int l = 0; l < 64; ++l) {
        const int j = l % 16, jp = 4 * kc + l / 16;   // row, column
        if (j >= J) continue;
        std::complex<ld> v = 0;
        for (int s = 0; s < R; ++s) {
          const ld a = -2 * pi * (ld)((m * s) % R) / R;
          v += c[((j - jp + J * s) % n + n) % n] * std::complex<ld>(std::cos(a), std::sin(a));
        }
        const size_t o = 2 * (((size_t)m * VJ + kc) * 64 + l);
        out[o] = (double)(v.real() / R);
        out[o + 1] = (double)(v.imag() / R);
      }
  }
}

// ------------------------------------------------------------------ the step
using f64x4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;

template <int N> struct Kin {
  using C = double2;
  static constexpr int R = KinGeo<N>::R, J = KinGeo<N>::J, VJ = J / 4;
  static_assert(N == R * J && J % 4 == 0 && J <= 16, "blocks of at most 16 points");
  // slot (v, s) of lane group g is element uni(v, s) + g of its line: the
  // first part the same in every lane (a scalar offset of the access)
  static constexpr unsigned uni(int v, int s) { return 4 * v + J * s; }

  // x[v][s] = slot (v, s) of the line n = lane % 16, before and after
  template <typename Mat>
  static __device__ __forceinline__ void step(C (&x)[VJ][R], Mat& mat) {
    mat.anew();
#pragma unroll
    for (int v = 0; v < VJ; ++v) Dft<R, -1, C>::run(x[v]);
#pragma unroll
    for (int m = 0; m < R; ++m) {
      f64x4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
      // the imaginary parts first: the large diagonal terms enter last
#pragma unroll
      for (int k = 0; k < VJ; ++k) {
        const C c = mat(m, k);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(c.y, -x[k][m].y, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(c.y, x[k][m].x, im, 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < VJ; ++k) {
        const C c = mat(m, k);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(c.x, x[k][m].x, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(c.x, x[k][m].y, im, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < VJ; ++v) x[v][m] = cmk<C>(re[v], im[v]);
    }
#pragma unroll
    for (int v = 0; v < VJ; ++v) Dft<R, +1, C>::run(x[v]);
  }
};

// The matrices of an axis, staged in LDS and read at each use: in registers
// they would cost a third of the waves a SIMD can hold.
template <int N> struct KinMat {
  using C = double2;
  static constexpr int E = Kin<N>::R * Kin<N>::VJ * 64;
  const C* t;
  int l;
  // by a block of nthr threads, before its next barrier
  static __device__ __forceinline__ void stage(C* lds, const C* __restrict__ tab, int nthr) {
    for (int i = threadIdx.x; i < E; i += nthr) lds[i] = tab[i];
  }
  __device__ __forceinline__ KinMat(const C* lds, int lane) : t(lds), l(lane) {}
  __device__ __forceinline__ C operator()(int m, int k) const { return t[(m * Kin<N>::VJ + k) * 64 + l]; }
  // keeps the compiler from moving the reads out of a loop into registers
  __device__ __forceinline__ void anew() { asm volatile("" : "+v"(l)); }
};

// ---------------------------------------------------------------------------
// x pass: pre-kinetic pointwise step and the x factor
//   PX_ETA0: out = Pf * in                                  (unperturbed set)
//   PX_FULL: out = Pf * (d - i dt u_b H_l)                  (mid-step state)
//   PX_HALF: out = Ph * (d - i dt/2 u_b (Ph H_l))           (cleaned end state)
// A wave takes 16 neighbouring columns (y, z), a 256-byte row of every x, and orbitals l0, l0 + ls, ... of its pair; u_b stays in registers and the
// state of the next orbital loads during the products.
// ---------------------------------------------------------------------------
template <int N, bool ETA>
__device__ __forceinline__ void kin_x_item(const PropXArgs<double>& a, int fb, int col0, int l0, int ls, KinMat<N> mat) {
  using K = Kin<N>;
  using C = double2;
  constexpr int R = K::R, VJ = K::VJ;
  constexpr unsigned NN = N * N, ng = N * NN;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned c = (lane >> 4) * NN + (unsigned)(col0 + 16 * wv) + (lane & 15);
  if constexpr (ETA) {
    const C* in = a.din + (size_t)fb * ng;
    C* out = a.dout + (size_t)fb * ng;
    C x[VJ][R];
#pragma unroll
    for (int v = 0; v < VJ; ++v)
#pragma unroll
      for (int s = 0; s < R; ++s) x[v][s] = cmul((a.pf + K::uni(v, s) * NN)[c], (in + K::uni(v, s) * NN)[c]);
    K::step(x, mat);
#pragma unroll
    for (int v = 0; v < VJ; ++v)
#pragma unroll
      for (int s = 0; s < R; ++s) (out + K::uni(v, s) * NN)[c] = x[v][s];
  } else {
    const bool half = a.mode == PX_HALF;
    const double cu = half ? 0.5 * a.dt : a.dt;
    const C* ptab = half ? a.ph : a.pf;
    const double* __restrict__ ub = a.u + (size_t)fb * ng;
    const C* din = a.din + ((size_t)fb * a.L + l0) * ng;
    C* dout = a.dout + ((size_t)fb * a.L + l0) * ng;
    const C* __restrict__ h = a.H + (size_t)l0 * ng;
    const size_t adv = (size_t)ls * ng;
    double uu[VJ][R];
    C dn[VJ][R];
#pragma unroll
    for (int v = 0; v < VJ; ++v)
#pragma unroll
      for (int s = 0; s < R; ++s) {
        dn[v][s] = (din + K::uni(v, s) * NN)[c];
        uu[v][s] = cu * (ub + K::uni(v, s) * NN)[c];
      }
    for (int l = l0; l < a.L; l += ls) {
      // the phases come from the cache for each orbital, not from registers
      const C* p0 = ptab;
      asm volatile("" : "+s"(p0));
      C x[VJ][R];
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) {
          const C p = (p0 + K::uni(v, s) * NN)[c];
          C hh = (h + K::uni(v, s) * NN)[c];
          if (half) hh = cmul(p, hh);
          x[v][s] = cmul(p, cmk<C>(dn[v][s].x + uu[v][s] * hh.y, dn[v][s].y - uu[v][s] * hh.x));
        }
      din += adv;
      h += adv;
      if (l + ls < a.L) {
#pragma unroll
        for (int v = 0; v < VJ; ++v)
#pragma unroll
          for (int s = 0; s < R; ++s) dn[v][s] = (din + K::uni(v, s) * NN)[c];
      }
      K::step(x, mat);
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) (dout + K::uni(v, s) * NN)[c] = x[v][s];
      dout += adv;
    }
  }
}

// Lines of 48 points and more need more registers than two waves on a SIMD
// leave with the next orbital in flight (64^3, 11 pairs: 228 us, the
// transforms 216; 48^3, 12 pairs: 148 and 100): they keep the transforms.
// a workgroup of TC columns; the fields of a launch are its pairs times the
// ls groups of orbitals
template <int N, int TC, bool ETA>
__global__ void __launch_bounds__(4 * TC, 3) k_kin_x(PropXArgs<double> a) {
  __shared__ double2 tab[KinMat<N>::E];
  int f, tile;
  if (!field_tile(a.order, a.nf * a.ls, N * N / TC, f, tile)) return;
  KinMat<N>::stage(tab, a.kin, 4 * TC);
  __syncthreads();
  kin_x_item<N, ETA>(a, f / a.ls, tile * TC, f % a.ls, a.ls, KinMat<N>(tab, threadIdx.x & 63));
}

// the pairs and the ne fields of the unperturbed set, one step ahead, in one
// launch
template <int N, int TC>
__global__ void __launch_bounds__(4 * TC, 3) k_kin_x_both(PropXArgs<double> a) {
  __shared__ double2 tab[KinMat<N>::E];
  int f, tile;
  if (!field_tile(a.order, a.nf * a.ls + a.ne, N * N / TC, f, tile)) return;
  KinMat<N>::stage(tab, a.kin, 4 * TC);
  __syncthreads();
  const KinMat<N> mat(tab, threadIdx.x & 63);
  if (f < a.nf * a.ls) {
    kin_x_item<N, false>(a, f / a.ls, tile * TC, f % a.ls, a.ls, mat);
  } else {
    PropXArgs<double> e = a;
    e.din = a.ein;
    e.dout = a.eout;
    kin_x_item<N, true>(e, f - a.nf * a.ls, tile * TC, 0, 1, mat);
  }
}

// ---------------------------------------------------------------------------
// plane pass: the y and z factors on P whole y-z planes, and the induced
// density dn_b = 4 sum_l Re(conj(H_l) d_{b,l}) of the post-kinetic state
// (linearised Eq. 11 source).  A workgroup takes its planes of one orbital
// after the other, a 16-line tile per wave: y lines from memory, through LDS
// into z lines, back to memory, the next orbital's planes and this one's
// unperturbed planes in flight during the products.
// The density is summed in G groups of orbitals (g, g + G, ...) and then over
// the groups in order, whether one workgroup takes all groups (parts = 1) or,
// where the planes alone would leave the chip idle, each group has its own
// (parts = G, the partial sums to dens[g]; the Poisson loader adds them): the
// same bits either way.
// ---------------------------------------------------------------------------
template <int N> struct KinYZ {
  static constexpr int P = N == 24 ? 2 : 1;              // planes: whole 16-line tiles
  static constexpr int WP = P * N / 16;                  // waves
  static constexpr int G = kin_yz_groups(N);
  static constexpr int S = N + 1;                        // LDS row
  template <int W> static constexpr int threads() { return 64 * WP * W; }
  template <int W> static constexpr size_t lds() {
    return sizeof(double2) * ((size_t)P * W * N * S + KinMat<N>::E);
  }
  static constexpr bool TOT_MEM = N >= 48;               // the sum over groups in dens, not in registers
};

// W: 1, or 2 for twice the planes; x0: first plane; group gb only if part, else
// all groups
template <int N, int W, bool DENS>
__device__ __forceinline__ void kin_yz_item(const PropYZArgs<double>& a, int x0, int b, bool part, int gb,
                                            double2* lds, KinMat<N> mat) {
  using K = Kin<N>;
  using Y = KinYZ<N>;
  using C = double2;
  constexpr int R = K::R, VJ = K::VJ, S = Y::S, G = Y::G;
  constexpr bool TM = Y::TOT_MEM;
  constexpr unsigned ng = N * N * N;
  const int lane = threadIdx.x & 63, t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned g = lane >> 4;
  const int L = DENS ? a.L : 1;
  // y line (plane q / N, column z = q % N), z line = row q of the planes
  const int q = 16 * t + (lane & 15);
  const unsigned y0 = (unsigned)x0 * N * N + (q / N) * (N * N) + q % N + g * N;
  const unsigned z0 = (unsigned)x0 * N * N + q * N + g;
  C* py = lds + (q / N) * (N * S) + q % N + g * S;
  C* pz = lds + q * S + g;
  C* db = a.d + (size_t)b * L * ng;
  C x[VJ][R];
  double acc[VJ][R], tot[TM ? 1 : VJ][TM ? 1 : R];
  double* dn = DENS ? a.dens + ((size_t)(part ? gb : 0) * a.nf + b) * ng + z0 : nullptr;
#pragma unroll
  for (int v = 0; v < VJ; ++v)
#pragma unroll
    for (int s = 0; s < R; ++s) {
      if (gb < L) x[v][s] = (db + (size_t)gb * ng + K::uni(v, s) * N)[y0];
      if constexpr (!TM) tot[v][s] = 0;
    }
  const int ge = min(L, part ? gb + 1 : G);
  bool first = true;
  for (int grp = gb; grp < ge; ++grp) {
#pragma unroll
    for (int v = 0; v < VJ; ++v)
#pragma unroll
      for (int s = 0; s < R; ++s) acc[v][s] = 0;
    for (int l = grp; l < L; l += G) {
      K::step(x, mat);
      if (!first) __syncthreads();           // the last orbital's rows are read
      first = false;
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) py[K::uni(v, s) * S] = x[v][s];
      __syncthreads();
      // loads before the stores below: a wait for a later one would wait for
      // the stores as well
      C hh[DENS ? VJ : 1][DENS ? R : 1];
      if constexpr (DENS) {
        const C* __restrict__ h = a.H + (size_t)l * ng;
#pragma unroll
        for (int v = 0; v < VJ; ++v)
#pragma unroll
          for (int s = 0; s < R; ++s) hh[v][s] = (h + K::uni(v, s))[z0];
      }
      const int nl = l + G < L ? l + G : grp + 1 < ge ? grp + 1 : L;
      if (nl < L) {
        const C* dn = db + (size_t)nl * ng;
#pragma unroll
        for (int v = 0; v < VJ; ++v)
#pragma unroll
          for (int s = 0; s < R; ++s) x[v][s] = (dn + K::uni(v, s) * N)[y0];
      }
      C z[VJ][R];
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) z[v][s] = pz[K::uni(v, s)];
      K::step(z, mat);
      C* dc = db + (size_t)l * ng;
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) (dc + K::uni(v, s))[z0] = z[v][s];
      if constexpr (DENS) {
#pragma unroll
        for (int v = 0; v < VJ; ++v)
#pragma unroll
          for (int s = 0; s < R; ++s) acc[v][s] += hh[v][s].x * z[v][s].x + hh[v][s].y * z[v][s].y;
      }
    }
    if constexpr (DENS && TM) {
      // a partial sum stays unscaled: the loader scales the sum
      const double sc = part || grp + 1 < ge ? 1.0 : 4.0;
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) {
          if (grp > gb) acc[v][s] = dn[K::uni(v, s)] + acc[v][s];
          dn[K::uni(v, s)] = sc * acc[v][s];
        }
    } else if constexpr (DENS) {
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) tot[v][s] += acc[v][s];
    }
  }
  if constexpr (DENS) {
    if constexpr (TM) {
      if (gb >= L) {
#pragma unroll
        for (int v = 0; v < VJ; ++v)
#pragma unroll
          for (int s = 0; s < R; ++s) dn[K::uni(v, s)] = 0;
      }
      return;
    } else {
      const double sc = part ? 1.0 : 4.0;
#pragma unroll
      for (int v = 0; v < VJ; ++v)
#pragma unroll
        for (int s = 0; s < R; ++s) dn[K::uni(v, s)] = sc * tot[v][s];
    }
  }
}

// grid: (planes, fields or pairs, groups) with the plane fastest: blocks
// running together stream consecutive planes of one field
template <int N, int W, bool DENS>
__global__ void __launch_bounds__(KinYZ<N>::template threads<W>(), 2) k_kin_yz(PropYZArgs<double> a) {
  extern __shared__ unsigned char smem_raw[];
  using Y = KinYZ<N>;
  double2* lds = reinterpret_cast<double2*>(smem_raw);
  double2* tab = lds + Y::P * W * N * Y::S;
  KinMat<N>::stage(tab, a.kin, Y::template threads<W>());
  __syncthreads();
  const KinMat<N> mat(tab, threadIdx.x & 63);
  if (DENS && (int)blockIdx.y >= a.nf) {
    // a field of the unperturbed set, one step ahead, beside the pairs
    const int fe = ((int)blockIdx.y - a.nf) * a.parts + (int)blockIdx.z;
    if (fe >= a.ne) return;
    PropYZArgs<double> e = a;
    e.d = a.ed;
    kin_yz_item<N, W, false>(e, blockIdx.x * Y::P * W, fe, false, 0, lds, mat);
    return;
  }
  kin_yz_item<N, W, DENS>(a, blockIdx.x * Y::P * W, blockIdx.y, a.parts > 1, blockIdx.z, lds, mat);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// plain launch, or one that records ev's events in its own dispatch
template <typename K, typename A>
static hipError_t kin_go(K kern, dim3 grid, int block, size_t lds, hipStream_t st, const LaunchEvents* ev,
                         const A& a) {
  if (ev)
    hipExtLaunchKernelGGL(kern, grid, dim3(block), (uint32_t)lds, st, ev->start, ev->stop, 0, a);
  else
    hipLaunchKernelGGL(kern, grid, dim3(block), lds, st, a);
  return hipGetLastError();
}

template <int N, int TC>
static hipError_t kin_x_tc(const PropXArgs<double>& a, int F, hipStream_t st, const LaunchEvents* ev) {
  PropXArgs<double> b = a;
  b.nf = F;
  // a pair's orbitals go to several waves while those are fewer than eight on
  // a SIMD (24^3, 8 pairs: 20.6 us unsplit, 9 split in ten)
  b.ls = a.mode == PX_ETA0 ? 1 : std::max(1, std::min(a.L, 8192 / (F * (N * N / 16) + a.busy)));
  const dim3 grid = field_tile_grid(a.order, F * b.ls + a.ne, N * N / TC);
  if (a.mode == PX_ETA0) return kin_go(k_kin_x<N, TC, true>, grid, 4 * TC, 0, st, ev, b);
  if (a.ne > 0) return kin_go(k_kin_x_both<N, TC>, grid, 4 * TC, 0, st, ev, b);
  return kin_go(k_kin_x<N, TC, false>, grid, 4 * TC, 0, st, ev, b);
}
template <int N>
static hipError_t kin_x_n(const PropXArgs<double>& a, int F, hipStream_t st, int tc, const LaunchEvents* ev) {
  switch (tc) {
    case 16: return kin_x_tc<N, 16>(a, F, st, ev);
    case 32: return kin_x_tc<N, 32>(a, F, st, ev);
    case 0:
    case 64: return kin_x_tc<N, 64>(a, F, st, ev);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_kin_x(int n, const PropXArgs<double>& a, int F, hipStream_t st, int tc, const LaunchEvents* ev) {
  switch (n) {
    case 16: return kin_x_n<16>(a, F, st, tc, ev);
    case 24: return kin_x_n<24>(a, F, st, tc, ev);
    case 32: return kin_x_n<32>(a, F, st, tc, ev);
    default: return hipErrorInvalidValue;
  }
}

template <int N, int W>
static hipError_t kin_yz_w(const PropYZArgs<double>& a, int nb, hipStream_t st, const LaunchEvents* ev) {
  using Y = KinYZ<N>;
  PropYZArgs<double> b = a;
  b.nf = nb;
  if (!a.density) b.parts = 1;
  if (b.parts != 1 && b.parts != Y::G) return hipErrorInvalidValue;
  if (a.ne > 0 && (b.parts < 2 || !a.ed)) return hipErrorInvalidValue;
  const dim3 grid(N / (Y::P * W), nb + (a.ne + b.parts - 1) / b.parts, b.parts);
  const int nt = Y::template threads<W>();
  const size_t lds = Y::template lds<W>();
  if (a.density) return kin_go(k_kin_yz<N, W, true>, grid, nt, lds, st, ev, b);
  return kin_go(k_kin_yz<N, W, false>, grid, nt, lds, st, ev, b);
}
// nt: 0 or 256 the default shape, 512 twice the planes
template <int N>
static hipError_t kin_yz_n(const PropYZArgs<double>& a, int nb, hipStream_t st, int nt, const LaunchEvents* ev) {
  if (nt == 0 || nt == 256) return kin_yz_w<N, 1>(a, nb, st, ev);
  if (nt == 512) return kin_yz_w<N, 2>(a, nb, st, ev);
  return hipErrorInvalidValue;
}
hipError_t launch_kin_yz(int n, const PropYZArgs<double>& a, int nb, hipStream_t st, int nt, const LaunchEvents* ev) {
  switch (n) {
    case 16: return kin_yz_n<16>(a, nb, st, nt, ev);
    case 24: return kin_yz_n<24>(a, nb, st, nt, ev);
    case 32: return kin_yz_n<32>(a, nb, st, nt, ev);
    case 48: return kin_yz_n<48>(a, nb, st, nt, ev);
    case 64: return kin_yz_n<64>(a, nb, st, nt, ev);
    default: return hipErrorInvalidValue;
  }
}

// The groups apart pay while the waves of the planes alone (B n^2 / 16) leave
// the chip short: up to 32 points (five groups) below two on a SIMD (32^3, 12
// pairs: 53 us together, 34 apart), above (two groups) below six (64^3, 11
// pairs: 329 and 319; 48^3, 12 pairs: 146 and 118).
int kin_yz_parts(int n, int B, int busy) {
  return kin_yz_grid(n) && ((long long)B * n + busy) * n / 16 < (n <= 32 ? 2048 : 6144) ? kin_yz_groups(n) : 1;
}

template <int N, int W> static void kin_conf_w() {
  const int lds = (int)KinYZ<N>::template lds<W>();
  (void)hipFuncSetAttribute((const void*)k_kin_yz<N, W, true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  (void)hipFuncSetAttribute((const void*)k_kin_yz<N, W, false>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}
template <int N> static void kin_conf() {
  static_assert(KinYZ<N>::template lds<2>() <= 160 * 1024 && KinYZ<N>::template threads<2>() <= 512, "fits a CU");
  kin_conf_w<N, 1>();
  kin_conf_w<N, 2>();
}
void configure_kin(int n) {
  switch (n) {
    case 16: return kin_conf<16>();
    case 24: return kin_conf<24>();
    case 32: return kin_conf<32>();
    case 48: return kin_conf<48>();
    case 64: return kin_conf<64>();
    default: return;
  }
}

}  // namespace bse
