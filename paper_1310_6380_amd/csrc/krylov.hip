// Lowest eigenpairs of C(k) by shift-invert block Krylov, for FP64 solves that
// want a small part of the spectrum.
//
// With C + sigma I = L L^H, the wanted lowest eigenvalues of C are the largest,
// best separated ones of B = (C + sigma I)^-1 = L^-H L^-1.  A block Lanczos
// recurrence of HB = 16 vectors with full reorthogonalisation projects B on a
// basis of m = 16 s vectors; the projection is block tridiagonal with upper
// triangular subdiagonal blocks, i.e. Hermitian of half bandwidth exactly HB,
// which is the form the bulge chasing takes.  Its eigenpairs, by the same
// kernels as after stage 1 but of order m instead of n, give n x nb Ritz
// vectors, and the FP64 Rayleigh-Ritz step on the kept C(k) ends the solve as
// on the reduction path.
//
// Why: the reduction reads and writes the trailing matrix twice per 16 columns
// (n / 16 passes over HBM) and chases n bulges; the factorisation touches each
// entry of the matrix in tiles of 64 x 64 on the matrix cores, (4/3) (n^3 + p
// r^3) real operations with the inverse within p parts of r rows instead of
// (16/3) n^3 bandwidth-bound ones, and the chain of sequential sweeps is m long
// instead of n. Convergence per step is that of a gap of 16 eigenvalues: the
// residual of the last wanted pair falls by 10 to 30 per step on the phononic
// spectra (eigenvalue counts grow like a power of the frequency), and every item
// checks it: an item that misses the bar is solved again, with more steps or by
// the reduction.
// Measured, plan build included, against the reduction: 60 points of 2N = 882,
// 18 bands, 20.3 -> 10.4 ms; 60 points of 2N = 1922, 24 bands, 123.6 -> 44.6 ms;
// 960 points of 2N = 242 .. 1250, 10 bands, 228 -> 95.9 ms.
#include <float.h>

#include <algorithm>

#include "chol64.h"
#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace mvpb {

constexpr int KB = 64;        // block of the factorisation
constexpr int KS = HB;        // vectors of a Krylov block
constexpr int KPB = 9;        // most blocks of a part of the inverse factor
constexpr int KR = 16;        // rows of the factor per workgroup of a product
constexpr int KCH = KRY_ROWS; // rows of a block per workgroup of the orthogonalisation
// Shift as a fraction of the nb-th band of the homogeneous medium (see KryMedium;
// the (d + 1)-th where fewer are wanted: the first d vanish at Gamma).  Small enough
// not to slow the convergence, which a shift above the wanted values would stop: a
// fraction 1 / 64 of the nb-th smallest diagonal entry of C, which the stiff parts
// set, is 2.4 of the nb-th value at a stiffness ratio of 1e3 and 4 to 20 from 1e4
// on, with residuals of 3e-5 and 1e-2 after the steps that reach 1e-9 here, and 40
// points of 2N = 882, 18 bands, soft inclusions of ratio 1e4, then took two attempts
// and the reduction, 34.0 ms against 7.2 ms here and 16.5 by the reduction alone.
// Large enough that L and the blocks' factors stay well conditioned where C is
// singular (the zero modes at Gamma: orthogonality of the basis 1e-11, 1e-8 at the
// worst).
constexpr double KRY_SHIFT = 1.0 / 8.0;
constexpr double KRY_TOL_MODES = 1e-10;

// Shift of every item, added to the diagonal of the working copy, and the weights of
// the start block's rows.  (Bands of the homogeneous medium at every plane wave,
// rank counting in LDS, one workgroup per item, one value per thread and pass.)
__global__ void __launch_bounds__(1024) kry_shift(const KryItem *__restrict__ items) {
  __shared__ double dg[MAX_N + 8];
  __shared__ double sel, peak[16];
  const KryItem it = items[blockIdx.x];
  const int n = it.n, tid = threadIdx.x, d = it.d, N = n / d;
  const int m2 = 2 * it.M2 + 1, m3 = 2 * it.M3 + 1;
  for (int r = tid; r < N; r += 1024) {
    const double g[3] = {(double)(r / m3 / m2 - it.M1), (double)(r / m3 % m2 - it.M2), (double)(r % m3 - it.M3)};
    double k2 = 0.0;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const double K = it.kap[l] + (it.B[3 * l] * g[0] + it.B[3 * l + 1] * g[1] + it.B[3 * l + 2] * g[2]);
      k2 = fma(K, K, k2);
    }
    for (int l = 0; l + 1 < d; ++l) dg[d * r + l] = it.ct2 * k2;
    dg[d * r + d - 1] = it.cl2 * k2;
  }
  if (tid < 8) dg[n + tid] = INFINITY;
  if (tid == 0) {
    sel = NAN;
    gst(it.status, 0, 0);
  }
  __syncthreads();
  const int want = max(it.nb, d + 1) - 1;
  for (int r = tid; r < n; r += 1024) {
    const double v = dg[r];
    int rank = 0;
    for (int q0 = 0; q0 < n; q0 += 8) {
      double w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = dg[q0 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) rank += (w[u] < v) | ((w[u] == v) & (q0 + u < r));
    }
    if (rank == want) sel = v;
  }
  __syncthreads();
  const double lam = sel, sg = KRY_SHIFT * lam;
  for (int r = tid; r < N; r += 1024) gst(it.weight, r, dg[d * r] > lam ? lam / dg[d * r] : 1.0);
  double top = 0.0;
  for (int r = tid; r < n; r += 1024) {
    const size_t e = (size_t)r * n + r;
    const double c = gld(it.Ak, e).re;
    top = fmax(top, c);
    gst(it.A, e, mk(c + sg, 0.0));
  }
  for (int o = 32; o > 0; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
  if ((tid & 63) == 0) peak[tid >> 6] = top;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; ++w) top = fmax(top, peak[w]);
    gst(it.top, 0, top);
  }
}

// ---------------------------------------------------------------------------
// Left-looking blocked Cholesky with the inverse factor, block column j:
//   kry_chol_diag  L_jj and X_jj = L_jj^-1 of the (fully updated) diagonal
//                  block, one workgroup per item;
//   kry_chol_step  below the diagonal, L_ij = (A_ij - sum_{k<j} L_ik L_jk^H)
//                  X_jj^H, and the update A_ii -= L_ij L_ij^H that keeps the
//                  later diagonal blocks current; left of it, within the part
//                  of the inverse that block j belongs to,
//                  X_jc = -X_jj sum_{k=c}^{j-1} L_jk X_kc.
// Every tile of L and X is written once, so a step streams its operands (K =
// 64 j deep) at the arithmetic intensity of a 64 x 64 product instead of
// reading and writing the trailing matrix per 64 columns.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) kry_chol_diag(const KryItem *__restrict__ items, int jb) {
  __shared__ Chol64 sm;
  const KryItem it = items[blockIdx.x];
  const int n = it.n;
  if (jb >= n || gld(it.status, 0)) return;
  const size_t ld = (size_t)n, o = (size_t)jb * ld + jb;
  const int bad = chol64(it.A + o, it.Xi + o, ld, min(KB, n - jb), sm);
  if (bad && threadIdx.x == 0) gst(it.status, 0, 1);
}

constexpr int SK = 8;         // columns of an operand step
constexpr int SLD = KB + 1;

// One tile of block column j: PAN: row block at i0 of L and the update of its
// diagonal block; else: column block at c0 of row block j of X.
template <bool PAN>
MVPB_DEV void chol_tile(const KryItem &it, int jb, int i0, int c0, cd (&sm)[2][2][SK * SLD]) {
  const int n = it.n, rows = PAN ? KB : min(KB, n - jb);
  const int kbeg = PAN ? 0 : c0, kend = jb;
  const size_t ld = (size_t)n;
  cd *A = it.A, *X = it.Xi;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  // operands of a step: SK columns of rows of block j of L, and of rows of block i
  // of L or SK rows of columns of X; thread t takes entries t and t + 256.  PF
  // steps are in flight; the loads are unconditional (the last ones are repeated),
  // as a conditional load makes the compiler wait for it at the end of its branch.
  constexpr int PF = 2;
  static_assert(KB / SK % PF == 0, "whole rounds of the prefetch registers");
  const int e1 = tid + 256;
  const cd *pa = A + (size_t)(tid / KB) * ld + jb + min(tid % KB, rows - 1);
  const cd *pb = PAN ? A + (size_t)(tid / KB) * ld + min(i0 + tid % KB, n - 1)
                     : X + (size_t)(c0 + tid / SK) * ld + tid % SK;
  const size_t da = (256 / KB) * ld, db = PAN ? (256 / KB) * ld : (256 / SK) * ld;
  cd va[PF][2], vb[PF][2];
  auto load = [&](int k, cd *a, cd *b) {
    const int kc = min(k, kend - SK);
    const cd *qa = pa + (size_t)kc * ld, *qb = PAN ? pb + (size_t)kc * ld : pb + kc;
    a[0] = gld(qa, 0);
    a[1] = gld(qa, da);
    b[0] = gld(qb, 0);
    b[1] = gld(qb, db);
  };
  auto store = [&](cd *As, cd *Bs, const cd *a, const cd *b) {
    As[(tid / KB) * SLD + tid % KB] = PAN ? conj(a[0]) : a[0];
    As[(e1 / KB) * SLD + e1 % KB] = PAN ? conj(a[1]) : a[1];
    Bs[PAN ? (tid / KB) * SLD + tid % KB : (tid % SK) * SLD + tid / SK] = b[0];
    Bs[PAN ? (e1 / KB) * SLD + e1 % KB : (e1 % SK) * SLD + e1 / SK] = b[1];
  };
  Acc3 acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q].clear();
  if (kbeg < kend) {
#pragma unroll
    for (int f = 0; f < PF; ++f) load(kbeg + f * SK, va[f], vb[f]);
    for (int k0 = kbeg; k0 < kend; k0 += PF * SK) {
#pragma unroll
      for (int f = 0; f < PF; ++f) {
        cd *As = sm[f & 1][0], *Bs = sm[f & 1][1];
        store(As, Bs, va[f], vb[f]);
        lds_barrier();
        load(k0 + (f + PF) * SK, va[f], vb[f]);
        // every LDS read of the step is issued before its first product
        cd fa[SK / 4][4], fb[SK / 4];
#pragma unroll
        for (int kk = 0; kk < SK / 4; ++kk) {
          fb[kk] = Bs[(4 * kk + lk) * SLD + 16 * wv + li];
#pragma unroll
          for (int q = 0; q < 4; ++q) fa[kk][q] = As[(4 * kk + lk) * SLD + 16 * q + li];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < SK / 4; ++kk)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q].step(fa[kk][q], fb[kk]);
      }
    }
  }
  // PAN: t[q][v] = (A_ij - sum)(row 16 wv + li, column 16 q + lk + 4 v);
  // else the sum itself (row 16 q + lk + 4 v, column 16 wv + li)
  cd t[4][4];
  if (PAN) {
    const int r = min(i0 + 16 * wv + li, n - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        t[q][v] = gld(A, (size_t)(jb + 16 * q + lk + 4 * v) * ld + r);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) t[q][v] = t[q][v] - acc[q].get(v);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) t[q][v] = acc[q].get(v);
  }
  // times X_jj^H from the right, or X_jj from the left (lower triangular): the
  // lanes' values are already the B operand
  Acc3 up[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) up[q].clear();
  cd *Ls = sm[0][0];   // 16 columns of L_ij, all 64 rows (both operands of a buffer)
  static_assert(2 * SK >= 16, "a 16-column tile fits one LDS buffer");
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    __builtin_amdgcn_sched_barrier(0);   // one block row of X_jj in registers at a time
    Acc3 o;
    o.clear();
#pragma unroll
    for (int kb = 0; kb <= mb; ++kb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = 16 * mb + li, k = 16 * kb + 4 * v + lk;
        const bool in = m < rows && k <= m;
        cd x = gld(X, in ? (size_t)(jb + k) * ld + jb + m : (size_t)jb * ld + jb);
        x = in ? (PAN ? conj(x) : x) : mk(0.0, 0.0);
        o.step(x, t[kb][v]);
      }
    if (PAN) {
      cd ov[4];
      lds_barrier();   // the previous contents of Ls have been read
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        ov[v] = o.get(v);
        Ls[(lk + 4 * v) * SLD + 16 * wv + li] = ov[v];
        if (i0 + 16 * wv + li < n) gst(A, (size_t)(jb + 16 * mb + lk + 4 * v) * ld + i0 + 16 * wv + li, ov[v]);
      }
      lds_barrier();
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
        if (rb >= wv) {
#pragma unroll
          for (int v = 0; v < 4; ++v) up[rb].step(Ls[(4 * v + lk) * SLD + 16 * rb + li], conj(ov[v]));
        }
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * mb + lk + 4 * v;
        if (r < rows) gst(X, (size_t)(c0 + 16 * wv + li) * ld + jb + r, -o.get(v));
      }
    }
  }
  if (!PAN) return;
  // A_ii -= L_ij L_ij^H, lower triangle
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
    if (rb >= wv) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = i0 + 16 * rb + lk + 4 * v, c = i0 + 16 * wv + li;
        if (r < n && c <= r) gst(A, (size_t)c * ld + r, gld(A, (size_t)c * ld + r) - up[rb].get(v));
      }
    }
}

// Parts of the inverse factor of an operator of order n (see kry_forward) and the
// blocks of one.  By the order alone, so that a point's result does not depend on
// the points solved with it.  A part saves most of its blocks' inverse and costs
// four launches per Krylov step (about 7 us each).  At most KPB = 9 blocks (chosen), 6
// and 17, plan build included: 60 points of n = 882, 18 bands, in 2 parts of 7 blocks
// 10.5 ms, 3 of 5 10.6, whole 11.1; of n = 1922, 24 bands, in 4 of 8 44.8, 6 of 6 45.5,
// 2 of 16 46.3; 30 points of a spatial n = 1029 in 2 of 9 13.5, 3 of 6 13.6, whole 13.4;
// 960 points of n = 242 .. 1250 95.7, 94.9 and 106.9.
MVPB_HD int kry_parts(int n) { return ((n + KB - 1) / KB + KPB - 1) / KPB; }
MVPB_HD int kry_part_blocks(int n) { return ((n + KB - 1) / KB + kry_parts(n) - 1) / kry_parts(n); }

__global__ void __launch_bounds__(256, 2) kry_chol_step(const KryItem *__restrict__ items, int n_items, int S, int jb) {
  __shared__ cd sm[2][2][SK * SLD];   // [buffer][A, B][k][row or column]
  int item, slot;
  if (!xcd_slot(S, n_items, item, slot)) return;
  const KryItem it = items[item];
  const int n = it.n;
  if (jb >= n || gld(it.status, 0)) return;
  const int j = jb / KB, below = (n + KB - 1) / KB - 1 - j;
  const int pb = kry_part_blocks(n), j0 = j / pb * pb;   // first block of j's part
  if (slot >= below + j - j0) return;
  if (slot < below)
    chol_tile<true>(it, jb, jb + KB * (slot + 1), 0, sm);
  else
    chol_tile<false>(it, jb, 0, KB * (j0 + slot - below), sm);
}

// ---------------------------------------------------------------------------
// Block Lanczos.  Blocks are stored row by row (16 entries, 256 bytes per row),
// so that the operands of a 16-wide matrix-core step are contiguous.  Z holds
// the next, not yet normalised block; its Gram matrix G = Z^H Z = R^H R comes
// from the same kernel, and the normalisation Z R^-1 is applied by the next
// product.
// ---------------------------------------------------------------------------
MVPB_DEV double kry_random(unsigned a, unsigned b) {
  unsigned long long z = ((unsigned long long)a << 32 | b) * 0x9E3779B97F4A7C15ull + 0xD1B54A32D192ED03ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(long long)(z >> 11) * (1.0 / 4503599627370496.0) - 1.0;   // [-1, 1)
}

MVPB_HD int kry_chunks(int n) { return (n + KCH - 1) / KCH; }

// Entry e of G = Z^H Z: the chunks' parts, eight loads in flight, added in order.
MVPB_DEV cd kry_gram(const KryItem &it, int e) {
  const int nch = kry_chunks(it.n);
  cd g = mk(0.0, 0.0);
  for (int c0 = 0; c0 < nch; c0 += 8) {
    cd p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) p[u] = gld(it.G, (size_t)min(c0 + u, nch - 1) * 256 + e);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (c0 + u < nch) g = g + p[u];
  }
  return g;
}

// Q_j = Z R_j^-1 from the Gram matrix G = Z^H Z = R_j^H R_j, KCH rows per
// workgroup (each factors G itself: a sixteen-step chain in one wavefront).  The
// workgroup of the first rows writes -R_j below the diagonal of the projection
// (eigenvalues of -B, lowest first).
__global__ void __launch_bounds__(512, 4) kry_norm(const KryItem *__restrict__ items, int j) {
  __shared__ cd Gs[16 * 17], Ri[16 * 17];
  __shared__ Factor16 fs;
  __shared__ int bad;
  const KryItem it = items[blockIdx.y];
  const int n = it.n, r0 = KCH * blockIdx.x;
  if (r0 >= n || gld(it.status, 0)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  const size_t r = (size_t)(r0 + 16 * wv + li);
  cd z[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) z[v] = gld(it.Z, r * KS + 4 * v + lk);
  if (tid < 256) {
    Gs[(tid >> 4) * 17 + (tid & 15)] = kry_gram(it, tid);
    if (tid == 0) bad = 0;
  }
  __syncthreads();
  if (wv == 0) {
    const int first = factor16<17>(Gs, Ri, fs);
    if (first && lane == 0) bad = 1;
  }
  __syncthreads();
  if (bad) {
    if (tid == 0) gst(it.status, 0, 2);
    return;
  }
  Acc3 o;
  o.clear();
#pragma unroll
  for (int v = 0; v < 4; ++v) o.step(conj(Ri[li * 17 + 4 * v + lk]), z[v]);
  cd *Q = it.Q + (size_t)j * it.npad * KS;   // zero rows beyond n, as in Z
#pragma unroll
  for (int v = 0; v < 4; ++v) gst(Q, r * KS + lk + 4 * v, o.get(v));
  if (blockIdx.x == 0 && j > 0 && tid < 256) {
    const int tr = tid & 15, tc = tid >> 4;   // -R(tr, tc) = -conj(L(tc, tr))
    gst(it.T, (size_t)(KS * (j - 1) + tc) * it.m + KS * j + tr, tr <= tc ? -conj(Gs[tc * 17 + tr]) : mk(0.0, 0.0));
  }
}

// The two solves of B = L^-H L^-1, in kry_parts parts of the rows: L^-1 is at hand
// only within each part (a whole inverse costs as much again as the
// factorisation, one of p parts 1 / p^2 of that), so the forward solve runs
//   W_0 = X_00 Q_0;   Z_I = Q_I - L_I,<I W_<I (SUB),  W_I = X_II Z_I
// and the backward one
//   Z_p = X_pp^H W_p;   W_I -= L_>I,I^H Z_>I (SUB),   Z_I = X_II^H W_I.
// 16 rows (or columns of the factor) by 16 per workgroup, the depth dealt to its
// four wavefronts 16 at a time, the operands of the next 16 in flight during the
// products; computed transposed (D^T = V^T M^T), so that a lane's loads of the
// factor run down its columns, 256 bytes (forward) or, with two consecutive rows
// per lane, 128 bytes (backward) at a time.  Bound by reading the factor and the
// parts of its inverse once.
struct KrySum {
  cd red[4][4][64];
};
// acc += the depth [klo, khi) dealt to this wavefront; load(kg, a, b) fetches the
// 16 deep from kg: a[q] of V, b[q] of the factor.
template <typename L>
MVPB_DEV void kry_depth(int klo, int khi, const L &load, Acc3 &acc) {
  const int wv = threadIdx.x >> 6, last = klo + (khi - klo - 1) / 16 * 16;
  acc.clear();
  int kg = klo + 16 * wv;
  if (kg >= khi) return;
  cd a0[4], a1[4], b0[4], b1[4];
  load(kg, a0, b0);
  for (; kg < khi; kg += 128) {
    load(min(kg + 64, last), a1, b1);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc.step(a0[q], b0[q]);
    load(min(kg + 128, last), a0, b0);
    if (kg + 64 < khi) {
#pragma unroll
      for (int q = 0; q < 4; ++q) acc.step(a1[q], b1[q]);
    }
  }
}
// Sum over the wavefronts: wavefront w receives register w.
MVPB_DEV cd kry_sum(KrySum &sm, const Acc3 &acc) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < 4; ++v) sm.red[wv][v][lane] = acc.get(v);
  __syncthreads();
  return (sm.red[0][wv][lane] + sm.red[1][wv][lane]) + (sm.red[2][wv][lane] + sm.red[3][wv][lane]);
}

template <bool SUB>
__global__ void __launch_bounds__(256) kry_forward(const KryItem *__restrict__ items, int n_items, int S, int part,
                                                   int j) {
  __shared__ KrySum sm;
  int item, slot;
  if (!xcd_slot(S, n_items, item, slot)) return;
  const KryItem it = items[item];
  const int n = it.n, w = KB * kry_part_blocks(n), start = w * part, end = min(start + w, n);
  const int nrb = (end - start + KR - 1) / KR;   // <= 0: the item has fewer parts
  if (slot >= nrb || gld(it.status, 0)) return;
  const int r0 = start + KR * (nrb - 1 - slot);   // longest rows first
  const size_t ld = (size_t)n;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const cd *Q = it.Q + (size_t)j * it.npad * KS;
  const cd *__restrict__ M = SUB ? it.A : it.Xi;
  const cd *__restrict__ V = SUB ? it.W : (part == 0 ? Q : it.Z);
  Acc3 acc;
  const int r = r0 + li;
  kry_depth(SUB ? 0 : start, SUB ? start : min(r0 + KR, end),
            [&](int kg, cd (&a)[4], cd (&b)[4]) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int k = kg + 4 * q + lk;
                const size_t kc = (size_t)min(k, n - 1) * ld;   // V has zero rows beyond n
                a[q] = gld(V, (size_t)k * KS + li);
                b[q] = gld(M, kc + min(r, n - 1));
              }
            },
            acc);
  const cd s = kry_sum(sm, acc);
  if (r < n) {
    const size_t e = (size_t)r * KS + lk + 4 * wv;
    if (SUB)
      gst(it.Z, e, gld(Q, e) - s);
    else
      gst(it.W, e, s);
  }
}

template <bool SUB>
__global__ void __launch_bounds__(256) kry_backward(const KryItem *__restrict__ items, int n_items, int S, int part) {
  __shared__ KrySum sm;
  int item, slot;
  if (!xcd_slot(S, n_items, item, slot)) return;
  const KryItem it = items[item];
  const int n = it.n, w = KB * kry_part_blocks(n), start = w * part, end = min(start + w, n);
  const int r0 = start + KR * slot;
  if (r0 >= end || (SUB && end >= n) || gld(it.status, 0)) return;
  const size_t ld = (size_t)n;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const cd *__restrict__ M = SUB ? it.A : it.Xi;
  const cd *__restrict__ V = SUB ? it.Z : it.W;
  Acc3 acc;
  const int r = r0 + li;
  kry_depth(SUB ? end : r0, SUB ? n : end,
            [&](int kg, cd (&a)[4], cd (&b)[4]) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int k = kg + 8 * (q >> 1) + 2 * lk + (q & 1), kc = min(k, n - 1);   // V: zero rows beyond n
                a[q] = gld(V, (size_t)k * KS + li);
                b[q] = conj(gld(M, (size_t)min(r, n - 1) * ld + kc));
              }
            },
            acc);
  const cd s = kry_sum(sm, acc);
  if (r < n) {
    const size_t e = (size_t)r * KS + lk + 4 * wv;
    if (SUB)
      gst(it.W, e, gld(it.W, e) - s);
    else
      gst(it.Z, e, s);
  }
}

// P_i = Q_i^H Z of one basis block i <= j: one workgroup per (block, item), the
// rows over its eight wavefronts; the workgroups of an item on one XCD, so that Z
// is fetched into one L2 (it is read once per basis block).  Bound by reading the
// basis.
__global__ void __launch_bounds__(512) kry_project(const KryItem *__restrict__ items, int n_items, int j) {
  __shared__ cd red[8][4][64];
  int item, i;
  if (!xcd_slot(j + 1, n_items, item, i)) return;
  const KryItem it = items[item];
  if (gld(it.status, 0)) return;
  const int n = it.n;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  const cd *__restrict__ Q = it.Q + (size_t)i * it.npad * KS;
  const cd *__restrict__ Z = it.Z;
  Acc3 acc;
  acc.clear();
  for (int kg = 16 * wv; kg < n; kg += 128) {
    cd a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = kg + 4 * q + lk;
      a[q] = gld(Q, (size_t)min(k, n - 1) * KS + li);
      b[q] = gld(Z, (size_t)k * KS + li);   // zero rows beyond n
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) acc.step(conj(a[q]), b[q]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wv][v][lane] = acc.get(v);
  __syncthreads();
  if (tid < 256) {
    const int v = tid >> 6;
    cd s = red[0][v][lane];
#pragma unroll
    for (int w = 1; w < 8; ++w) s = s + red[w][v][lane];
    gst(it.P, (size_t)i * 256 + (lk + 4 * v) * KS + li, s);
  }
}

// Z -= sum_{i <= j} Q_i P_i and the chunk's part of G = Z^H Z; 128 rows per
// workgroup, 16 per wavefront.  START: Z = pseudo-random instead (and zero
// rows beyond n in Z and W), the rows of a plane wave scaled by min(1, lambda / its
// lowest band of the homogeneous medium), lambda the wanted one: the low modes lie on
// the long waves, which saves a step.  The workgroup of chunk 0 writes the diagonal
// block of the projection, -(P_j + P_j^H) / 2.
template <bool START>
__global__ void __launch_bounds__(512) kry_update(const KryItem *__restrict__ items, int j) {
  extern __shared__ __align__(16) unsigned char kry_raw[];
  cd *Ps = (cd *)kry_raw;   // [j + 1][16][16], then the wavefronts' Gram parts [8][4][64]
  const KryItem it = items[blockIdx.y];
  const int n = it.n, r0 = KCH * blockIdx.x;
  if (r0 >= n || (!START && gld(it.status, 0))) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int rw = r0 + 16 * wv;
  cd z[4];
  if (START) {
    const int N = n / it.d;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = rw + lk + 4 * v;
      const double w = gld(it.weight, min(r, n - 1) % N);
      z[v] = r < n ? mk(w * kry_random(r, 2 * li), w * kry_random(r, 2 * li + 1)) : mk(0.0, 0.0);
      gst(it.Z, (size_t)r * KS + li, z[v]);
      if (r >= n) gst(it.W, (size_t)r * KS + li, mk(0.0, 0.0));
    }
  } else {
    for (int e = tid; e < (j + 1) * 256; e += 512) Ps[e] = gld(it.P, e);
#pragma unroll
    for (int v = 0; v < 4; ++v) z[v] = gld(it.Z, (size_t)(rw + lk + 4 * v) * KS + li);
    __syncthreads();
    Acc3 acc;
    acc.clear();
    const cd *q0 = it.Q + (size_t)min(rw + li, n - 1) * KS;
    for (int i = 0; i <= j; ++i) {
      cd a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = gld(q0, (size_t)i * it.npad * KS + 4 * q + lk);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc.step(a[q], Ps[i * 256 + (4 * q + lk) * KS + li]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = rw + lk + 4 * v;
      z[v] = r < n ? z[v] - acc.get(v) : mk(0.0, 0.0);
      if (r < n) gst(it.Z, (size_t)r * KS + li, z[v]);
    }
    if (blockIdx.x == 0 && tid < 256) {
      const int tr = tid & 15, tc = tid >> 4;
      const cd p = Ps[j * 256 + tr * KS + tc], q = Ps[j * 256 + tc * KS + tr];
      gst(it.T, (size_t)(KS * j + tc) * it.m + KS * j + tr, mk(-0.5 * (p.re + q.re), -0.5 * (p.im - q.im)));
    }
    __syncthreads();
  }
  Acc3 g;
  g.clear();
#pragma unroll
  for (int v = 0; v < 4; ++v) g.step(conj(z[v]), z[v]);
#pragma unroll
  for (int v = 0; v < 4; ++v) Ps[(wv * 4 + v) * 64 + lane] = g.get(v);
  __syncthreads();
  if (tid < 256) {
    const int v = tid >> 6;
    cd s = Ps[v * 64 + lane];
#pragma unroll
    for (int w = 1; w < 8; ++w) s = s + Ps[(w * 4 + v) * 64 + lane];
    gst(it.G, (size_t)blockIdx.x * 256 + (lk + 4 * v) * KS + li, s);
  }
}

// Ritz vectors, once more by B: with Z the next block, B [Q_0 .. Q_{s-1}] y =
// theta [Q_0 .. Q_{s-1}] y + Z y_last (y_last: the last 16 entries of y), so Y =
// [Q_0 .. Q_{s-1}] y + Z y_last / theta is a step of inverse iteration at the price
// of one more block here.  It takes a vector's error along an eigenvector of value
// lambda' down by (lambda + sigma) / (lambda' + sigma): the residual in C of modes at
// their bar from 1e3 times a dense solver's to a few times.  128 rows and 16 bands per
// workgroup.
__global__ void __launch_bounds__(512) kry_ritz(const KryItem *__restrict__ items) {
  extern __shared__ __align__(16) unsigned char kry_raw[];
  cd *Yl = (cd *)kry_raw;   // [m + 16][16]
  const KryItem it = items[blockIdx.z];
  const int n = it.n, nb = it.nb, m = it.m, r0 = KCH * blockIdx.x, b0 = 16 * blockIdx.y;
  if (r0 >= n || b0 >= nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, li = lane & 15, lk = lane >> 4;
  for (int e = tid; e < 16 * m; e += 512) {
    const int k = e % m, b = e / m;
    const cd y = b0 + b < nb ? gld(it.Ys, (size_t)(b0 + b) * m + k) : mk(0.0, 0.0);
    Yl[k * 16 + b] = y;
    if (k >= m - KS) Yl[(k + KS) * 16 + b] = b0 + b < nb ? (-1.0 / gld(it.lam_s, b0 + b)) * y : mk(0.0, 0.0);
  }
  __syncthreads();
  const int r = r0 + 16 * wv + li;
  const cd *q0 = it.Q + (size_t)min(r, n - 1) * KS;
  Acc3 acc;
  acc.clear();
  const cd *z0 = it.Z + (size_t)min(r, n - 1) * KS;
  for (int i = 0; i <= m / KS; ++i) {
    const cd *p = i < m / KS ? q0 + (size_t)i * it.npad * KS : z0;
    cd b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = gld(p, 4 * q + lk);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc.step(Yl[(KS * i + 4 * q + lk) * 16 + li], b[q]);
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int b = b0 + lk + 4 * v;
    if (r < n && b < nb) gst(it.Y, (size_t)b * n + r, acc.get(v));
  }
}

// Whether an item's pairs stand: for each, the residual |B y - theta y| =
// |R_s y_last| (y_last: the last 16 entries of the projection's eigenvector)
// is at most tol theta (with modes, or as much as eps |C| moves the value in a
// dense solver, up to KRY_TOL_MODES theta), and no run of nearly equal values is so long that the
// block of 16 could have missed copies (a block Krylov space holds at most 16
// vectors of one eigenvalue).  Failing items are flagged: their frequencies
// come out NaN and the host solves them again by the reduction.
__global__ void __launch_bounds__(64) kry_check(const KryItem *__restrict__ items, double tol) {
  __shared__ cd Gs[256];
  const KryItem it = items[blockIdx.x];
  const int lane = threadIdx.x, nb = it.nb, m = it.m;
  const double top = gld(it.top, 0);
  int bad = gld(it.status, 0) | gld(it.flag_s, 0);
  for (int e = lane; e < 256; e += 64) {
    Gs[e] = kry_gram(it, e);
  }
  __syncthreads();
  if (!bad)
    for (int b = lane; b < nb; b += 64) {
      const cd *y = it.Ys + (size_t)b * m + m - KS;
      double s = 0.0;
      for (int r = 0; r < KS; ++r) {
        cd t = mk(0.0, 0.0);
        for (int c = 0; c < KS; ++c) t = cfma(Gs[r * 16 + c], gld(y, c), t);
        const cd yr = gld(y, r);
        s += yr.re * t.re + yr.im * t.im;
      }
      const double th = -gld(it.lam_s, b);
      const double bar = fmax(tol, fmin(DBL_EPSILON * top * th, KRY_TOL_MODES));
      if (!(th > 0.0) || !(s <= bar * bar * th * th)) bad = 1;
      // a run of KS - 1 neighbouring values within 1e-4
      if (b + KS - 2 < nb && !(gld(it.lam_s, b + KS - 2) - gld(it.lam_s, b) > 1e-4 * th)) bad = 1;
    }
  for (int o = 32; o > 0; o >>= 1) bad |= __shfl_xor(bad, o, 64);
  if (lane == 0) gst(it.flag, 0, bad ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Launches
// ---------------------------------------------------------------------------

// Krylov steps for nb wanted pairs: the residual of the last pair reaches 1e-9 of its
// value in the median and 1e-7 at the worst (nb = 5 and 8, at stiffness ratios beyond
// 1e3) or, with modes wanted, 1e-13 and 3e-12; with few modes the rounding of the first
// formula is felt, and spatial spectra, which are denser, take two steps more.  Measured on
// planar cells of 2N = 162 .. 1922 and ratios 1e-5 .. 1e5 and on spatial ones of 3N = 375
// and 1029; points of high symmetry, where 16 values past the last wanted one are
// hardly larger, miss the bar.
int krylov_steps(int nb, int dim, bool modes) {
  const int s = 6 + (9 * nb + 24) / 25 + (dim == 3 ? 1 : 0);
  if (!modes) return s;
  const int m = s + 2 + nb / 12, more = nb < 12 ? (dim == 3 ? 2 : (9 * nb + 24) % 25 >= 12) : (dim == 3 ? 1 : 0);
  return std::max(m, std::min(m + more, KRY_MAX_STEPS - KRY_RETRY_STEPS));
}

hipError_t launch_krylov(const KryItem *items, int n_items, int n_max, int s, hipStream_t st) {
  const int nblk = (n_max + KB - 1) / KB, parts = kry_parts(n_max);
  {
    ProfScope ps(K_FACTOR, st);
    hipLaunchKernelGGL(kry_shift, dim3(n_items), dim3(1024), 0, st, items);
    for (int j = 0; j < nblk; ++j) {
      hipLaunchKernelGGL(kry_chol_diag, dim3(n_items), dim3(256), 0, st, items, j * KB);
      if (nblk > 1)
        hipLaunchKernelGGL(kry_chol_step, dim3(xcd_grid(nblk - 1, n_items)), dim3(256), 0, st, items, n_items,
                           nblk - 1, j * KB);
    }
  }
  ProfScope ps(K_KRYLOV, st);
  const int nch = kry_chunks(n_max), nrb = KB / KR * std::min(nblk, KPB);
  const size_t red = sizeof(cd) * 8 * 256;
  const dim3 g(xcd_grid(nrb, n_items)), b(256);
  hipLaunchKernelGGL(kry_update<true>, dim3(nch, n_items), dim3(512), red, st, items, 0);
  for (int j = 0; j < s; ++j) {
    hipLaunchKernelGGL(kry_norm, dim3(nch, n_items), dim3(512), 0, st, items, j);
    for (int p = 0; p < parts; ++p) {
      if (p > 0) hipLaunchKernelGGL(kry_forward<true>, g, b, 0, st, items, n_items, nrb, p, j);
      hipLaunchKernelGGL(kry_forward<false>, g, b, 0, st, items, n_items, nrb, p, j);
    }
    for (int p = parts - 1; p >= 0; --p) {
      if (p < parts - 1) hipLaunchKernelGGL(kry_backward<true>, g, b, 0, st, items, n_items, nrb, p);
      hipLaunchKernelGGL(kry_backward<false>, g, b, 0, st, items, n_items, nrb, p);
    }
    hipLaunchKernelGGL(kry_project, dim3(xcd_grid(j + 1, n_items)), dim3(512), 0, st, items, n_items, j);
    hipLaunchKernelGGL(kry_update<false>, dim3(nch, n_items), dim3(512),
                       std::max(red, sizeof(cd) * 256 * (size_t)(j + 1)), st, items, j);
  }
  return hipGetLastError();
}

hipError_t launch_krylov_ritz(const KryItem *items, int n_items, int n_max, int nb, int s, double tol,
                              hipStream_t st) {
  ProfScope ps(K_KRYLOV, st);
  hipLaunchKernelGGL(kry_ritz, dim3(kry_chunks(n_max), (nb + 15) / 16, n_items), dim3(512),
                     sizeof(cd) * 16 * KS * (size_t)(s + 1), st, items);
  hipLaunchKernelGGL(kry_check, dim3(n_items), dim3(64), 0, st, items, tol);
  return hipGetLastError();
}

hipError_t init_krylov_attributes() {
  const int most = (int)(sizeof(cd) * 256 * (KRY_MAX_STEPS + 1));
  hipError_t e = hipFuncSetAttribute((const void *)kry_update<false>, hipFuncAttributeMaxDynamicSharedMemorySize, most);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void *)kry_ritz, hipFuncAttributeMaxDynamicSharedMemorySize, most);
  return e;
}

}  // namespace mvpb
