// Cholesky factor and inverse factor of one Hermitian positive definite block of
// order up to 64 by one workgroup, and what it is made of.
#pragma once
#include <float.h>

#include "common.h"

namespace mvpb {

typedef double zd4_t __attribute__((ext_vector_type(4)));

// One K = 4 complex step on the FP64 matrix cores as three real products
// (p1 = ar br, p2 = ai bi, p3 = (ar + ai)(br + bi)).  Lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] and holds D[l / 16 + 4 v][l % 16].
// D therefore has the lane layout of the B operand of a next product: register
// v is its step v.
struct Acc3 {
  zd4_t p1, p2, p3;
  MVPB_DEV void clear() { p1 = p2 = p3 = zd4_t{0.0, 0.0, 0.0, 0.0}; }
  MVPB_DEV void step(cd a, cd b) {
    p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re, b.re, p1, 0, 0, 0);
    p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.im, b.im, p2, 0, 0, 0);
    p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.re + a.im, b.re + b.im, p3, 0, 0, 0);
  }
  MVPB_DEV cd get(int v) const { return mk(p1[v] - p2[v], p3[v] - p1[v] - p2[v]); }
};

// ---------------------------------------------------------------------------
// Cholesky factor and inverse factor of a 16 x 16 Hermitian tile by one
// wavefront: lane (r = l % 16, g = l / 16) keeps columns 4 g .. 4 g + 3 of row r
// of the tile and of the inverse in registers, and step j passes column j (zero
// down to row j) and row j of the inverse through LDS once, unscaled as in
// L D L^H: the update then needs no selects, and the scalings by the square roots
// of the pivots wait until the end.  One wavefront issues an instruction every
// four to five cycles, so the instructions of a step are its time (with selects
// and scalings in the step 1016 cycles, without 660).  Reads the lower triangle
// of D; writes L and L^-1 with zero upper triangles.  Returns (uniformly) 0 or
// one more than the column of the first pivot that is not positive and finite.
// ---------------------------------------------------------------------------
struct Factor16 {
  cd col[16], row[16];
  double piv[16];
};
template <int LDD>
MVPB_DEV int factor16(cd *D, cd *I, Factor16 &sm) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  cd a[4], x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = 4 * g + u;
    const cd v = D[r * LDD + c];
    a[u] = r >= c ? v : mk(0.0, 0.0);
    x[u] = mk(r == c ? 1.0 : 0.0, 0.0);
  }
  int bad = 0;
#pragma unroll 1
  for (int jg = 0; jg < 4; ++jg)
#pragma unroll
    for (int ju = 0; ju < 4; ++ju) {
      const int j = 4 * jg + ju;
      if (g == jg) {
        sm.col[r] = r > j ? a[ju] : mk(0.0, 0.0);
        if (r == j) sm.piv[j] = a[ju].re;
      }
      if (r == j) {
#pragma unroll
        for (int u = 0; u < 4; ++u) sm.row[4 * g + u] = x[u];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
      const double piv = sm.piv[j];
      const cd cr = sm.col[r];
      cd cc[4], xr[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        cc[u] = conj(sm.col[4 * g + u]);
        xr[u] = sm.row[4 * g + u];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
      if (bad == 0 && !(piv > 0.0 && piv <= DBL_MAX)) bad = j + 1;
      const cd l = -quick_rcp(piv) * cr;   // zero for r <= j
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = cfma(l, cc[u], a[u]);
        x[u] = cfma(l, xr[u], x[u]);
      }
    }
  double t, sr;
  sqrt_rcp(sm.piv[r], t, sr);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = 4 * g + u;
    double sc;
    sqrt_rcp(sm.piv[c], t, sc);
    D[r * LDD + c] = r > c ? sc * a[u] : mk(r == c ? t : 0.0, 0.0);
    I[r * LDD + c] = r >= c ? sr * x[u] : mk(0.0, 0.0);
  }
  return bad;
}

// ---------------------------------------------------------------------------
// A block of order nb <= 64 (first entry A, leading dimension ld, lower triangle
// read) by 256 threads: L to A, X = L^-1 with a zero upper triangle to Xo.  Tiles
// of 16: the diagonal tile by one wavefront, then the tiles of L below it and of
// the inverse left of it, then the trailing ones, on the matrix cores.  Bound by
// the chain of its 64 columns.  Returns (uniformly) 0, or one more than the column
// of the first pivot that is not positive and finite.
// ---------------------------------------------------------------------------
constexpr int CHOL_B = 64;
struct Chol64 {
  cd D[CHOL_B * (CHOL_B + 1)], I[CHOL_B * (CHOL_B + 1)];
  Factor16 fs;
  int bad;
};
MVPB_DEV int chol64(cd *A, cd *X, size_t ld, int nb, Chol64 &sm) {
  constexpr int LD = CHOL_B + 1;
  cd *D = sm.D, *I = sm.I;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  {
    cd v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int e = tid + 256 * u, r = e % CHOL_B, c = e / CHOL_B;
      v[u] = gld(A, (r < nb && c < nb && r >= c) ? (size_t)c * ld + r : 0);
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int e = tid + 256 * u, r = e % CHOL_B, c = e / CHOL_B;
      D[r * LD + c] = (r < nb && c < nb && r >= c) ? v[u] : mk(r == c ? 1.0 : 0.0, 0.0);
      I[r * LD + c] = mk(0.0, 0.0);
    }
  }
  if (tid == 0) sm.bad = 0;
  __syncthreads();
#pragma unroll 1
  for (int p = 0; p < 4 && 16 * p < nb; ++p) {
    const int p0 = 16 * p;
    if (wv == 0) {
      const int first = factor16<LD>(D + p0 * LD + p0, I + p0 * LD + p0, sm.fs);
      if (first && lane == 0) sm.bad = p0 + first;
    }
    __syncthreads();
    if (sm.bad) return sm.bad;
    // wavefront w: a tile of L below the diagonal tile, or one of the inverse left of it
    const int below = 3 - p;
    if (wv < below) {
      const int i0 = 16 * (p + 1 + wv);
      Acc3 o;
      o.clear();
#pragma unroll
      for (int k = 0; k < 16; k += 4)
        o.step(D[(i0 + li) * LD + p0 + k + lk], conj(I[(p0 + li) * LD + p0 + k + lk]));
#pragma unroll
      for (int v = 0; v < 4; ++v) D[(i0 + lk + 4 * v) * LD + p0 + li] = o.get(v);
    } else if (wv - below < p) {
      const int c0 = 16 * (wv - below);
      Acc3 s, o;
      s.clear();
      o.clear();
      for (int k = c0; k < p0; k += 4) s.step(D[(p0 + li) * LD + k + lk], I[(k + lk) * LD + c0 + li]);
#pragma unroll
      for (int v = 0; v < 4; ++v) o.step(I[(p0 + li) * LD + p0 + 4 * v + lk], s.get(v));
#pragma unroll
      for (int v = 0; v < 4; ++v) I[(p0 + lk + 4 * v) * LD + c0 + li] = -o.get(v);
    }
    __syncthreads();
    // trailing tiles (i, k), p < k <= i
    const int nt = below * (below + 1) / 2;
    for (int t = wv; t < nt; t += 4) {
      int i = 0;
      while ((i + 1) * (i + 2) / 2 <= t) ++i;
      const int k0 = 16 * (p + 1 + t - i * (i + 1) / 2), i0 = 16 * (p + 1 + i);
      Acc3 u;
      u.clear();
#pragma unroll
      for (int k = 0; k < 16; k += 4)
        u.step(D[(i0 + li) * LD + p0 + k + lk], conj(D[(k0 + li) * LD + p0 + k + lk]));
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        cd *d = &D[(i0 + lk + 4 * v) * LD + k0 + li];
        *d = *d - u.get(v);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int e = tid + 256 * u, r = e % CHOL_B, c = e / CHOL_B;
    if (r >= nb || c >= nb) continue;
    if (r >= c) gst(A, (size_t)c * ld + r, D[r * LD + c]);
    gst(X, (size_t)c * ld + r, r >= c ? I[r * LD + c] : mk(0.0, 0.0));
  }
  return 0;
}

}  // namespace mvpb
