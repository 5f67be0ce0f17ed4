// Small operators (order <= SMALL_MAX_N): C(k) reduced to tridiagonal form in
// one workgroup per item, and the matching back-transform.
//
// The two-stage reduction pays one launch chain of ~60 us per 16 columns and
// about 4 us per bulge-chasing sweep, whatever the order; below 128 rows the
// whole matrix fits the registers of one CU (128 x 128 complex FP64 = 256 KB of
// 512 KB), and a Householder column costs three barriers instead.  Measured at
// n = 98, 30 points: stage 1, bulge chasing and back-transforms 870 -> 245 us.
#include <algorithm>
#include <utility>

#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace mvpb {

// Householder tridiagonalisation A = Q T Q^H, T real, lower convention: column k
// is annihilated below its subdiagonal by H_k = I - tau v v^H (v_{k+1} = 1),
// H_k^H x = beta e_1 with beta real, A <- H_k^H A H_k.  With x = tau A v and
// a' = -(tau / 2)(x^H v) = -(|tau|^2 / 2) v^H A v, a real number, that is the
// update A - v x^H - (x + 2 a' v) v^H.
// Thread (r = t % ROWS, q = t / ROWS) keeps the entries of row r in the columns
// c = kb + 4 i + q in registers (both triangles, so that a product needs no sums
// across rows).  Every four columns the registers move down by one and kb up by
// four: the current column is always entry 0, every register index is static,
// and the loop body stays small.  (Unrolled stages instead of the moves: 100 KB
// of code, fetched once per launch, 230 us at n = 98; eight threads per row: the
// same 195 us, and 128 rows spill.)
// Three barriers per column:
//   1 the column and its norm are in LDS: all wavefronts multiply A by it as it
//     is, the first ROWS threads also form beta, tau and the scale of v;
//   2 the partial products are in LDS: the first ROWS threads form v, and
//     x = tau scale (sum - beta A e_{k+1}), as A v = scale (A col - beta A e_{k+1});
//   3 v, x and a' are in LDS: update, and the owners of the next column publish
//     it with its norm.
// Bound by the chain of a column: about 1500 cycles to the partial products, 900
// for x and its product with v, 1500 for the update (timestamps at column 40 of
// n = 98), of which the FP64 issue of 12 FMAs per entry is the smaller part.
constexpr int SQ = 4;   // threads per row

template <int ROWS>
__global__ void __launch_bounds__(SQ * ROWS) small_tridiag(const EigItem *__restrict__ items) {
  constexpr int NE = ROWS / SQ, RW = ROWS / 64;
  // column, v, x (each with zeros for the columns that a group of four entries
  // reaches past the last), next column, then the partial products [SQ]
  constexpr int PAD = 4 * SQ, VB = ROWS + PAD, XB = 2 * VB, NXT = 3 * VB, PART = NXT + ROWS;
  __shared__ cd sm[PART + SQ * ROWS];
  __shared__ double ap[RW], nrm[RW];
  const EigItem it = items[blockIdx.x];
  const int n = it.n;
  if (n > ROWS || (ROWS > 64 && n <= 64)) return;   // the other instance's item
  const int t = threadIdx.x, r = t % ROWS, q = t / ROWS, lane = t & 63;
  cd *const sr = sm + r, *const sq = sm + q;   // entries of this row; of the columns 4 i + q
  cd a[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int c = SQ * i + q;
    const bool in = r < n && c < n;
    const cd v = gld(it.Ak, in ? (size_t)c * n + r : 0);
    a[i] = in ? v : mk(0.0, 0.0);
  }
  if (t < PAD) sm[ROWS + t] = sm[VB + ROWS + t] = sm[XB + ROWS + t] = mk(0.0, 0.0);
  if (t == 0) gst(it.flag, 0, 0);
  cd *V = (cd *)it.A, *tau_out = (cd *)it.tau2;
  // column k from its owners (rows below k; row k is d_k) and its norm^2 below row k + 1
  auto publish = [&](int k, cd e) {
    sr[0] = r > k ? e : mk(0.0, 0.0);
    if (r == k) gst(it.d, k, e.re);
    const double s = wave_sum(r > k + 1 ? abs2(e) : 0.0);
    if (lane == 0) nrm[(t >> 6) % RW] = s;
  };
  if (q == 0) publish(0, a[0]);
#pragma unroll 1
  for (int kb = 0; kb < n; kb += SQ) {
    const int cnt = (n - kb + SQ - 1) / SQ;   // entries still in range
#pragma unroll 1
    for (int kk = 0; kk < SQ; ++kk) {
      const int k = kb + kk;
      if (k >= n - 1) break;
      const bool last = kk == SQ - 1, next = q == (last ? 0 : kk + 1);   // next: owns column k + 1
      __syncthreads();
      if (next) {
        const cd e0 = a[0], e1 = a[1];
        sr[NXT] = mk(last ? e1.re : e0.re, last ? e1.im : e0.im);
      }
      cd p = mk(0.0, 0.0);
#pragma unroll
      for (int i0 = 0; i0 < NE; i0 += 4)
        if (i0 < cnt) {
#pragma unroll
          for (int i = i0; i < min(i0 + 4, NE); ++i) p = cfma(a[i], sq[kb + SQ * i], p);
        }
      sr[PART + ROWS * q] = p;
      double beta = 0.0;
      cd tau = mk(0.0, 0.0), scale = mk(0.0, 0.0);
      if (q == 0) {
        const cd alpha = sm[k + 1];
        double x2 = nrm[0];
#pragma unroll
        for (int h = 1; h < RW; ++h) x2 += nrm[h];
        beta = alpha.re;
        if (x2 != 0.0 || alpha.im != 0.0) {
          double rb;
          sqrt_rcp(abs2(alpha) + x2, beta, rb);
          beta = -copysign(beta, alpha.re);
          rb = -copysign(rb, alpha.re);
          const double dr = alpha.re - beta, den = quick_rcp(dr * dr + alpha.im * alpha.im);
          tau = mk(-dr * rb, -alpha.im * rb);
          scale = mk(dr * den, -alpha.im * den);
        }
        if (t == 0) {
          gst(it.e, k, beta);
          gst(tau_out, k, tau);
        }
      }
      __syncthreads();
      if (q == 0) {
        cd s = mk(0.0, 0.0);
#pragma unroll
        for (int w = 0; w < SQ; w += 4) {
          s = s + ((sr[PART + ROWS * w] + sr[PART + ROWS * (w + 1)]) +
                   (sr[PART + ROWS * (w + 2)] + sr[PART + ROWS * (w + 3)]));
          __builtin_amdgcn_sched_barrier(0);
        }
        // with a zero column (tau = 0) v = e_{k+1}, x = 0
        const cd v = r == k + 1 ? mk(1.0, 0.0) : scale * sr[0];
        const cd x = r > k ? (tau * scale) * (s - beta * sr[NXT]) : mk(0.0, 0.0);
        sr[VB] = v;
        sr[XB] = x;
        // Re(tau conj(x) v)
        const cd xv = mk(x.re * v.re + x.im * v.im, x.re * v.im - x.im * v.re);
        const double sa = wave_sum(tau.re * xv.re - tau.im * xv.im);
        if (lane == 0) ap[t >> 6] = sa;
        if (r > k && r < n) gst(V, (size_t)k * n + r, v);
      }
      __syncthreads();
      double a2 = ap[0];   // -2 a'
#pragma unroll
      for (int h = 1; h < RW; ++h) a2 += ap[h];
      const cd v = sr[VB], z = sr[XB] - a2 * v;
#pragma unroll
      for (int i0 = 0; i0 < NE; i0 += 4)
        if (i0 < cnt) {
#pragma unroll
          for (int i = i0; i < min(i0 + 4, NE); ++i) {
            const cd vc = sq[VB + kb + SQ * i], xc = sq[XB + kb + SQ * i];
            a[i] = cfma(-v, conj(xc), a[i]);
            a[i] = cfma(-z, conj(vc), a[i]);
          }
        }
      if (next) {
        const cd e0 = a[0], e1 = a[1];
        publish(k + 1, mk(last ? e1.re : e0.re, last ? e1.im : e0.im));
      }
    }
#pragma unroll
    for (int i = 0; i + 1 < NE; ++i) a[i] = a[i + 1];
    a[NE - 1] = mk(0.0, 0.0);
  }
}

// Sum of a complex number over the wavefront (every lane receives it): the
// first halving step trades the real and imaginary parts between the half-
// wavefronts, so that the other steps carry one value instead of two.
MVPB_DEV cd wave_sum_c(cd v) {
  double x = swap_add<0>(v.re, v.im);
  x += xchg<1>(x);
  x += xchg<2>(x);
  x += xchg<3>(x);
  x += xchg<4>(x);
  x += xchg<5>(x);
  const double y = xchg<0>(x);
  const bool up = (__lane_id() & 32) != 0;
  return mk(up ? y : x, up ? x : y);
}

// Y = H_0 H_1 .. H_{n-2} X, one wavefront per column of X, lane l holding rows
// l and l + 64; the reflectors of four steps are loaded ahead.  Bound by the
// instructions and latency of one wavefront sum per reflector.
constexpr int SMALL_COLS = 4;   // columns (wavefronts) per workgroup
__global__ void __launch_bounds__(64 * SMALL_COLS) small_back(const EigItem *__restrict__ items) {
  const EigItem it = items[blockIdx.y];
  const int n = it.n, nb = it.nb, lane = threadIdx.x & 63, b = blockIdx.x * SMALL_COLS + (threadIdx.x >> 6);
  if (b >= nb) return;
  const cd *V = (const cd *)it.A, *tau = (const cd *)it.tau2;
  const int r0 = lane, r1 = lane + 64, q0 = min(r0, n - 1), q1 = min(r1, n - 1);
  cd y0 = mk(r0 < n ? gld(it.X, (size_t)q0 * nb + b) : 0.0, 0.0);
  cd y1 = mk(r1 < n ? gld(it.X, (size_t)q1 * nb + b) : 0.0, 0.0);
  constexpr int U = 4;
  cd v0[U], v1[U], ts[U];
  auto fetch = [&](int k, cd &a0, cd &a1, cd &tt) {
    const int kc = max(k, 0);
    const cd x0 = gld(V, (size_t)(kc * n + q0)), x1 = gld(V, (size_t)(kc * n + q1));
    tt = gld(tau, kc);
    a0 = (k >= 0 && r0 > kc && r0 < n) ? x0 : mk(0.0, 0.0);
    a1 = (k >= 0 && r1 > kc && r1 < n) ? x1 : mk(0.0, 0.0);
  };
#pragma unroll
  for (int u = 0; u < U; ++u) fetch(n - 2 - u, v0[u], v1[u], ts[u]);
  for (int k = n - 2; k >= 0; k -= U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const cd a0 = v0[u], a1 = v1[u], tt = ts[u];   // zero beyond the last reflector
      fetch(k - u - U, v0[u], v1[u], ts[u]);
      const cd s = tt * wave_sum_c(cfma_cj(a1, y1, cfma_cj(a0, y0, mk(0.0, 0.0))));
      y0 = cfma(-a0, s, y0);
      y1 = cfma(-a1, s, y1);
    }
  }
  if (r0 < n) gst(it.Y, (size_t)b * n + r0, y0);
  if (r1 < n) gst(it.Y, (size_t)b * n + r1, y1);
}

hipError_t launch_small_tridiag(const EigItem *items, int n_items, int n_min, int n_max, hipStream_t st) {
  ProfScope ps(K_SMALL, st);
  if (n_min <= 64) hipLaunchKernelGGL(small_tridiag<64>, dim3(n_items), dim3(SQ * 64), 0, st, items);
  if (n_max > 64) hipLaunchKernelGGL(small_tridiag<128>, dim3(n_items), dim3(SQ * 128), 0, st, items);
  return hipGetLastError();
}

hipError_t launch_small_back(const EigItem *items, int n_items, int nb, hipStream_t st) {
  ProfScope ps(K_BACKTRANSFORM, st);
  hipLaunchKernelGGL(small_back, dim3((nb + SMALL_COLS - 1) / SMALL_COLS, n_items), dim3(64 * SMALL_COLS), 0, st, items);
  return hipGetLastError();
}

}  // namespace mvpb
