// Launchers of the constrained-reconstruction kernels (admm.hip).
#pragma once

#include "common.h"

namespace mx {

// The input of a TV prox: z, or z + *ufac u when u is given; lam, or 1 / *rho when rho is given.
struct TvInput {
  const float2 *z, *u;
  const double *ufac, *rho;
  float lam;
};
// x = prox of lam TV at the input (x must not alias it); P and P2 hold nd * N complex values
// each (the dual field, double-buffered); iters Chambolle steps from P = 0.
hipError_t tv_prox_launch(int nd, const int64_t* n, const TvInput& in, int iters, float2* P, float2* P2, float2* x,
                          hipStream_t st);
// z_j = y_j + eps_j (v_j - y_j) / max(||v_j - y_j||, eps_j) with v = w, or w + *ufac u when u is
// given; t (optional, needs u) = z - *ufac u - w.  part holds ball_part_doubles(J) doubles.
hipError_t ball_project_launch(const float2* w, const float2* u, const double* ufac, const float2* y, const float* eps,
                               int64_t M, int J, double* part, float2* z, float2* t, hipStream_t st);
int ball_part_doubles(int J);
// z0 = u0 = 0 (n0 entries), zk = uk = 0 (n1 entries), *rho = rho0, *ufac = 1
hipError_t admm_init_launch(float2* z0, float2* u0, int64_t n0, float2* zk, float2* uk, int64_t n1, double rho0,
                            double* rho, double* ufac, hipStream_t st);
// x = 0, r = d = g + z0 - *ufac u0 - p, partials of <r, r> (DOT_BLOCKS)
hipError_t admm_start_launch(const float2* g, const float2* z0, const float2* u0, const double* ufac, const float2* p,
                             int64_t n, float2* x, float2* r, float2* d, double* part, hipStream_t st);
// u = *ufac u + A p - z over both blocks, t = zk - zkp, partials of ||A p - z||^2 (DOT_BLOCKS)
hipError_t admm_dual_launch(const float2* p, const float2* z0, float2* u0, int64_t n0, const float2* Fp,
                            const float2* zk, const float2* zkp, float2* uk, float2* t, int64_t n1, const double* ufac,
                            double* part, hipStream_t st);
// partials of ||g + z0 - z0p||^2 (DOT_BLOCKS)
hipError_t admm_dres_launch(const float2* g, const float2* z0, const float2* z0p, int64_t n, double* part,
                            hipStream_t st);
// residual balancing from the two partials: hist = (rho, r, s); rho and the dual factor updated
hipError_t admm_rho_launch(const double* part_r, const double* part_s, double* rho, double* ufac, double* hist,
                           hipStream_t st);

}  // namespace mx
