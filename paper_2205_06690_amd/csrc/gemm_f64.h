// FP64 contractions over the grid on the matrix cores: the A matrix of the
// FP64 mode (Eq. 1) and the occupied-space projection of the mixed
// representation (Eq. 6).
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>

namespace bse {

// C[m][n] = scale * sum_r A[m][r] B[n][r], K a multiple of 16, rows 16-byte
// aligned; part holds gemm_part_elems(M, N, K) doubles
size_t gemm_part_elems(int M, int N, size_t K);
hipError_t launch_gemm_f64(const double* A, int M, const double* B, int N, size_t K, double scale,
                           double* part, double* C, hipStream_t st);

// out_j -= sum_s C[j][s] phi_s for nf fields [nf][ng]
hipError_t launch_project_out(double* out, int nf, const double* phi, int S, const double* C, size_t ng,
                              hipStream_t st);

// The same on af without storing it, then the Chebyshev step of n_pol sets of
// n_o fields: fn = 2 (x - b fc)/a - fp (first: (x - b fc)/a) with x = af - sum_s
// C phi_s, and S[p] = dv <fc|fc>, S[3 + p] = dv <fn|fc> of set p (n_pol <= 3;
// entries of absent sets are 0).  part holds project_part_elems(n_pol n_o, ng);
// part and S both null: the step without the sums.
size_t project_part_elems(int nf, size_t ng);
hipError_t launch_project_cheb(const double* af, int n_o, int n_pol, const double* phi, int S, const double* C,
                               size_t ng, const double* fc, const double* fp, double* fn, double a, double b,
                               int first, double dv, double* part, double* Sk, hipStream_t st);

}  // namespace bse
