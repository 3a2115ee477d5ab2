// Chebyshev recursion f^{k+1} = 2 A~ f^k - f^{k-1}, A~ = (A - b)/a, of the
// three dipole start vectors with A resident on the chip (Eqs. 7-8, FP64).
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>

namespace bse {

// largest A (rows) the resident recursion takes, and the steps of one launch
int cheb_res_max();
constexpr int CHEB_SEG = 512;

// One segment: rows out[k][3][n], k < steps, become f^{k0+1} .. f^{k0+steps}
// from fc = f^{k0} and fp = f^{k0-1} ([3][n]; k0 = 0: fp unused and f^1 = A~
// f^0).  err: device word, set to 1 when a workgroup waited in vain for the
// others of its polarisation (they were never resident together); the rows
// are then not valid.  The caller clears it first and reads it at the end.
hipError_t launch_cheb_res(const double* A, int n, const double* fc, const double* fp, double* out, int steps, int k0,
                           double a, double b, int* err, hipStream_t st);

// what a segment leaves whose workgroups never met (rows still empty, err
// raised), for tests of the path behind it
hipError_t launch_cheb_missed(int n, double* out, int steps, int* err, hipStream_t st);

// S[m][0..2] = <f^m|f^m>, S[m][3..5] = <f^{m+1}|f^m> for m = k0 .. k0 + steps - 1
// (fc = f^{k0}, out as above)
hipError_t launch_cheb_dots(const double* fc, const double* out, int n, int k0, int steps, double* S, hipStream_t st);
// F[q][3][n] (k0 = 0: g[q][0] f^0 plus) += sum_{k0 < m <= k0 + steps} g[q][m] f^m, g [n_w][N]
hipError_t launch_cheb_states(const double* fc, const double* out, int n, int k0, int steps, const double* g, int N,
                              int n_w, double* F, hipStream_t st);

// Lanczos iterations k0 .. k1-1 for n <= lanczos_res_max(): basis V[n+1][n]
// (v_0 .. v_k0 set), alpha[k], bq[k] = |w_k|^2
int lanczos_res_max();
hipError_t launch_lanczos_res(const double* A, int n, double* V, int k0, int k1, double* alpha, double* bq,
                              hipStream_t st);

}  // namespace bse
