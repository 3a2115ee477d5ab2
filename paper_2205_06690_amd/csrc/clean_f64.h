// Cleaning projection of the perturbed stochastic orbitals (Eq. 15,
// linearised) in FP64 on the matrix cores.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>

namespace bse {

// mid-step to end-of-step conversion applied on the fly: d <- ph (d - i hdt u_b H_l), E_l = ph H_l
struct MidArgs64 {
  int on;
  const double* u;     // [B][ng]
  const double2* H;    // [L][ng]
  const double2* ph;   // [ng]
  double half_dt;
};

// coefficients of the F perturbed fields and, in rows F .. F + L - 1, of the
// L unperturbed ones: coef[f][s] = dv sum_r phi_s(r) d_f(r) for s < S and, for
// f < F, coef[f][S] = dv <E_l, d_f>, l = f % L.  E [L][ng] is read unless
// mid.on.  part holds coef64_part_entries(F, L, S, ng) entries; ng must be a
// multiple of 8.
hipError_t launch_coef_f64(const double2* d, int F, const double* phi, int S, const double2* E, int L, size_t ng,
                           double dv, double2* part, double2* coef, hipStream_t st, const MidArgs64& mid);
// the largest need over batches of L, 2 L, .. F fields
size_t coef64_part_entries(int F, int L, int S, size_t ng);
// d_f <- fin(d_f) - sum_s coef[f][s] phi_s - coef[f][S].x E_l, fin the end of the step when mid.on
hipError_t launch_update_f64(double2* d, int F, const double* phi, int S, const double2* E, int L, size_t ng,
                             const double2* coef, hipStream_t st, const MidArgs64& mid);

}  // namespace bse
