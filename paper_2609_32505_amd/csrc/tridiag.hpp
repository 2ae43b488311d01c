// Symmetric eigenvectors through a tridiagonal matrix: H = Q T Q^T by
// Householder reflections, T = Z diag(lam) Z^T, V = Q Z.
#pragma once
#include "common.hpp"

// Sizes up to kTriMax take this route (k_tri_column has a thread for four
// columns); up to kTriSlab the back-transformation holds slabs of V in
// registers, above it is matrix products.
constexpr int kTriMax = 4096;
constexpr int kTriSlab = 1024;
// Up to kTriPolish every matrix gets the Newton-Schulz step, above it those with
// close eigenvalues.
constexpr int kTriPolish = 128;

struct TriWs {
  int batch, n, np;  // np: leading dimension of every square array below
  float* A;          // batch x np x np: H, symmetrised and zero padded; destroyed
  float* HV;         // batch x np x np: row j is the Householder vector of column j
  double* Z;         // batch x np x np: forward pivots, then eigenvectors of T (column k)
  double* Zb;        // batch x np x np: backward pivots
  float* V;          // batch x np x np: the result (may overlay Zb)
  double* d;         // batch x np: diagonal of T (scaled)
  double* e;         // batch x np: off-diagonal of T (scaled)
  double* zinv;      // batch x np: 1 / |column of Z|
  float* tau;        // batch x np: the reflectors' factors
  float* T;          // batch x tri_t_floats(np): compact-WY factors, one per panel
  double* lam;       // batch x np: eigenvalues of the perturbed T, ascending, up to a shift (k_tri_vectors)
  float* mx;         // batch x (np / 64)^2: max |h_ij| per setup workgroup
  float *S, *T4, *C;  // np > kTriSlab, batch x np x 128 each: Gram matrices and WY factors of 128
                     // reflectors, and 128 rows of products
  float* Y;          // np > kTriSlab, batch x np x np: T4^T V^T (may overlay Zb behind V)
  int* risk;         // batch: 1 where V gets the Newton-Schulz step: eigenvalues nearly coincide
  int* bad;          // batch: 1 where V was not orthonormal, 2 where it still is not
};

// In tridiag_kernels.hpp:
// tri_t_floats: floats of T per matrix.
// tri_eig: V (row-major, leading dimension np) and risk of the matrices of
// `mask` (null: all); their sweep counts are set to 0.  Z may overlay A and
// other memory that is free by then, V may overlay Zb.
// tri_check: bad[b] = 1 where max |G - I| > 1e-4 for the Gram matrix G of V,
// among those of risk.
// tri_polish: Gram matrix, tri_check and the Newton-Schulz step to V2, up to
// kTriPolish.
// tri_rescue: the vectors of close eigenvalues orthogonalised for the matrices of
// bad, which is 2 (and flags[b] |= EIGH_NOT_CONVERGED, unless flags is null) where
// they were too many.
