// The scoring chains of the general vector screen (device code only).  The
// C = 16 encoder runs them too, for the candidates whose rounding is on a
// knife edge: there the score jumps by percents with the last bits of the fit,
// and every screen is to take the same decision.
#pragma once

#include "awsrc_internal.h"

namespace awsrc {

// Per-element weights: the Cholesky factor of G + eps I (G: lower triangle
// with eps on the diagonal, identity rows for padded columns), the solve for
// the fit, the rounding and the score of Sec. 3.2, in fp32.
template <int PB>
__device__ __forceinline__ float chol_score32(const float (&bv)[PB], const float (&G)[PB][PB], float eps, float qmax,
                                              float inv_qmax, bool pow2, bool* edge) {
  float L[PB][PB], inv[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p)
#pragma unroll
    for (int q = 0; q <= p; ++q) {
      float acc = G[p][q];
#pragma unroll
      for (int k = 0; k < q; ++k) acc -= L[p][k] * L[q][k];
      if (p == q) {
        L[p][p] = sqrtf(fmaxf(acc, 1e-30f));
        inv[p] = 1.0f / L[p][p];
      } else {
        L[p][q] = acc * inv[q];
      }
    }
  // solve L L^T alpha = b
  float z[PB], al[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    float acc = bv[p];
#pragma unroll
    for (int k = 0; k < p; ++k) acc -= L[p][k] * z[k];
    z[p] = acc * inv[p];
  }
#pragma unroll
  for (int p = PB - 1; p >= 0; --p) {
    float acc = z[p];
#pragma unroll
    for (int k = p + 1; k < PB; ++k) acc -= L[k][p] * al[k];
    al[p] = acc * inv[p];
  }
  // quantize with one scale and score
  float m = 0.0f;
#pragma unroll
  for (int p = 0; p < PB; ++p) m = fmaxf(m, fabsf(al[p]));
  float isc;
  bool ed;
  const float sc = pow2 ? screen_scale<true>(m, inv_qmax, &isc, &ed) : screen_scale<false>(m, inv_qmax, &isc, &ed);
  float g = 0.0f;
  if (sc > 0.0f) {
    float q[PB], t1 = 0.0f, qq = 0.0f;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const float x = al[p] * isc;
      q[p] = fminf(fmaxf(rintf(x), -qmax), qmax);
      ed = ed || code_edge(x, qmax);
      t1 += q[p] * bv[p];
      qq += q[p] * q[p];
    }
    float quad = 0.0f;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
      float y = 0.0f;
#pragma unroll
      for (int i = k; i < PB; ++i) y += L[i][k] * q[i];
      quad += y * y;
    }
    quad -= eps * qq;
    g = sc * (2.0f * t1 - sc * quad);
  }
  *edge = ed;
  return g;
}

// Per-column weights: LDL^T of G + eps I (lower triangle) in fp64, stored in
// fp32 in the layout of the per-column factor table (strict lower L by rows,
// then 1/e, then e).  G is SPD: d > 0 and the columns are orthonormal.
template <int PB, typename OUT>
__device__ __forceinline__ void col_factor64(const double (&G)[PB][PB], OUT&& out) {
  double L[PB][PB], e[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p) {
#pragma unroll
    for (int q = 0; q < p; ++q) {
      double acc = G[p][q];
#pragma unroll
      for (int k = 0; k < q; ++k) acc -= L[p][k] * L[q][k] * e[k];
      L[p][q] = acc / e[q];
    }
    double acc = G[p][p];
#pragma unroll
    for (int k = 0; k < p; ++k) acc -= L[p][k] * L[p][k] * e[k];
    e[p] = fmax(acc, 1e-300);
  }
#pragma unroll
  for (int p = 0; p < PB; ++p) {
#pragma unroll
    for (int q = 0; q < p; ++q) out[ltri(p, q)] = (float)L[p][q];
    out[PB * (PB - 1) / 2 + p] = (float)(1.0 / e[p]);
    out[PB * (PB - 1) / 2 + PB + p] = (float)e[p];
  }
}

}  // namespace awsrc
