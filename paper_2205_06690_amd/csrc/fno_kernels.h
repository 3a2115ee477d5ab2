// Launchers of the Fourier-operator surrogate kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>

namespace bse {
bool fno_grid_supported(int n);
// V[F][K] = DFT of real fields on the kept modes (times c_k/ng if ck);
// P [F][n][2 m^2] takes the planes' kept columns on the way
hipError_t fno_fft_fwd(int n, const float* in, int F, const float2* tw, int m, int ck, float2* P,
                       float2* V, hipStream_t st);
// P[F][n][2 m^2] = unnormalised inverse DFT along x of U on the kept modes (U times c_k/ng if ck)
hipError_t fno_x_inv(int n, const float2* U, int F, const float2* tw, int m, int ck, float2* P, hipStream_t st);
// q[b][o] = sum_i M[o][i] in[b][i] + bias[o] + Re inverse (y, z) DFT of P[b][o];
// zout = q; out = gelu(q) (act) or q, times gelu'(zg) where zg is given
struct FnoLayerArgs {
  const float* in;      // [B][W][ng]
  const float* M;       // [W][W]; trans: its transpose is applied
  int trans;
  const float* bias;    // nullable [W]
  int W, B, m;
  const float2* P;      // [B W][n][2 m^2]
  const float2* tw;
  int act;
  float* zout;          // nullable [B][W][ng]
  const float* zg;      // nullable [B][W][ng]
  float* out;           // [B][W][ng]
};
hipError_t fno_layer(int n, const FnoLayerArgs& a, hipStream_t st);
// per-mode channel mix U[b][o][k] = sum_i V[b][i][k] R[k][i][o] and its two
// backward products; path 0: matrix cores (up to 32 channels), 1: vector FMA
hipError_t fno_spec_mix(const float2* V, const float2* R, int B, int C, int K, float2* U, int path,
                        hipStream_t st);
hipError_t fno_spec_mix_bwd(const float2* V, const float2* GU, const float2* R, int B, int C, int K,
                            float2* GV, float2* GR, int path, hipStream_t st);
hipError_t fno_pointwise(const float* in, int Cin, const float* Wm, const float* bias, int Cout,
                         int B, size_t ng, float* out, hipStream_t st);
size_t fno_outer_part_len(int Co, int Ci, int B, size_t ng);
hipError_t fno_outer(const float* A, int Co, const float* X, int Ci, int B, size_t ng, double* part,
                     float* gW, float* gb, hipStream_t st);
hipError_t fno_proj_bwd(const float* gy, const float* Q, int C, int B, size_t ng, float* gh, hipStream_t st);
int fno_loss_blocks(size_t ng);
hipError_t fno_loss_partial(const float* y, const float* t, int B, size_t ng, double* part, hipStream_t st);
hipError_t fno_loss_grad(const float* y, const float* t, const double* tn, int B, size_t ng, float* gy,
                         hipStream_t st);
hipError_t fno_adam(float* master, float* compute, const float* g, float* m, float* v, size_t n,
                    float lr, float b1, float b2, float eps, int step, int bf16, hipStream_t st);
hipError_t fno_round_copy(const float* src, float* dst, size_t n, int bf16, hipStream_t st);
// dst[b][c] = sample idx[b] of src[.][C][n^3] under a symmetry of the cube:
// output axis k is input axis perm[k], and the output axes in flip_mask
// (bit k) run backwards
hipError_t fno_gather_sym(const float* src, const int* idx, int B, int C, int n, const int perm[3],
                          int flip_mask, float* dst, hipStream_t st);
}  // namespace bse
