// Learned screening surrogate: a small periodic CNN that maps a binary
// 32 x 32 pixel cell to its lowest 10 bands at 40 k-points (normalised
// frequencies), trained on bands computed by the method itself.
//
//   conv1 3x3  1->32 s1, conv2..4 3x3 32->32 s2 (circular padding, ReLU)
//   flatten 4x4x32 = 512 -> fc1 256 (ReLU) -> fc2 400, mean squared error.
//
// Activations are NHWC FP32.  With FP32 products a convolution is one GEMM of FMA
// tiles whose A operand is the implicit im2col of its input (the tile loads gather
// the taps straight from the activations, circular padding, power-of-two grids),
// also for the weight gradients; the backward data pass is a GEMM into a column
// buffer and a gather col2im (every input pixel collects its taps, so no atomics
// and bitwise-reproducible results).  With BF16 products and FP32 accumulation
// (v_mfma_f32_16x16x32_bf16) the four convolutions of a cell run in one workgroup
// (conv_chain), the data pass gathers its taps directly (conv_dx), the gradients of
// all four layers share a launch (conv_grads), and the fully connected layers are
// GEMMs.  Bias and ReLU are applied in the epilogues, long reductions split over
// workgroups; master weights and Adam moments stay FP32.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../include/mvpb.h"
#include "common.h"
#include "kernels.h"

namespace mvpb {

// ---------------------------------------------------------------------------
// GEMM, row-major: C[M x N] = act(alpha op(A) op(B) + beta C + bias).
// op(A) = A (A[i*lda+k]) or A^T (A[k*lda+i]); op(B) = B (B[k*ldb+j]) or B^T (B[j*ldb+k]).
// Long reductions (the weight gradients of the convolutions sum over every
// output pixel of the batch) are split over blockIdx.z: split z sums its K
// range into its own slice of a partial buffer, and gemm_reduce adds the
// slices in a fixed order (reproducible), applying alpha, beta and bias.
// ---------------------------------------------------------------------------
constexpr int GBM = 64, GBN = 64;

// Implicit im2col operand: column matrix col[p][k], p = (b, oy, ox) an output
// pixel, k = (ky 3 + kx) C + c, col[p][k] = in[b][(s oy + ky - 1) mod H]
// [(s ox + kx - 1) mod W][c] with H, W, C and the output grid Ho = H / s,
// Wo = W / s powers of two (given as log2).
struct ConvA {
  const float *in = nullptr;   // NHWC input; nullptr: A is an ordinary matrix
  int lH = 0, lW = 0, lC = 0, lHo = 0, lWo = 0, s = 1;
};
MVPB_DEV size_t conv_index(const ConvA &cv, int p, int k) {   // of col[p][k] in the input
  const int c = k & ((1 << cv.lC) - 1), tap = k >> cv.lC;
  const int ky = tap / 3, kx = tap - 3 * ky;
  const int ox = p & ((1 << cv.lWo) - 1), t = p >> cv.lWo;
  const int oy = t & ((1 << cv.lHo) - 1), b = t >> cv.lHo;
  const int y = (cv.s * oy + ky - 1) & ((1 << cv.lH) - 1), x = (cv.s * ox + kx - 1) & ((1 << cv.lW) - 1);
  return (((((size_t)b << cv.lH) + y) << cv.lW) + x) << cv.lC | (size_t)c;
}

struct GemmArgs {
  int M, N, K;
  float alpha, beta;
  const float *A;   // unused when conv.in is set (op(A) is then the implicit column matrix)
  int lda;
  const float *B;
  int ldb;
  float *C;          // output, or the partial buffer [splits][M][N] when kchunk < K
  int ldc;
  int kchunk;        // K range of one split
  const float *bias; // per column, nullable (applied when not split)
  int relu;
  ConvA conv;
};

// Every load of a thread is issued, from element 0 where masked, before its
// first LDS store, so that all of them are in flight together.
template <int TA, int TB, int BK>
MVPB_DEV void load_tiles(const GemmArgs &g, int m0, int n0, int k0, int k1, float (&As)[BK][GBM + 4],
                         float (&Bs)[BK][GBN + 4]) {
  constexpr int PA = GBM * BK / 256, PB = BK * GBN / 256;
  static_assert(PA * 256 == GBM * BK && PB * 256 == BK * GBN, "tile entries per thread");
  const int tid = threadIdx.x;
  float va[PA], vb[PB];
  bool oa[PA], ob[PB];
#pragma unroll
  for (int u = 0; u < PA; ++u) {
    const int e = tid + 256 * u;
    const int i = TA == 0 ? e / BK : e % GBM, k = TA == 0 ? e % BK : e / GBM;
    const int gi = m0 + i, gk = k0 + k;
    oa[u] = gi < g.M && gk < k1;
    if (g.conv.in) {   // op(A)[gi][gk] = col[gi][gk] (TA = 0) or col[gk][gi] (TA = 1)
      const size_t x = TA == 0 ? conv_index(g.conv, gi, gk) : conv_index(g.conv, gk, gi);
      va[u] = gld(g.conv.in, oa[u] ? x : 0);
    } else {
      const size_t x = TA == 0 ? (size_t)gi * g.lda + gk : (size_t)gk * g.lda + gi;
      va[u] = gld(g.A, oa[u] ? x : 0);
    }
  }
#pragma unroll
  for (int u = 0; u < PB; ++u) {
    const int e = tid + 256 * u;
    const int k = TB == 0 ? e / GBN : e % BK, j = TB == 0 ? e % GBN : e / BK;
    const int gk = k0 + k, gj = n0 + j;
    ob[u] = gk < k1 && gj < g.N;
    vb[u] = gld(g.B, ob[u] ? (TB == 0 ? (size_t)gk * g.ldb + gj : (size_t)gj * g.ldb + gk) : 0);
  }
#pragma unroll
  for (int u = 0; u < PA; ++u) {
    const int e = tid + 256 * u;
    const int i = TA == 0 ? e / BK : e % GBM, k = TA == 0 ? e % BK : e / GBM;
    As[k][i] = oa[u] ? va[u] : 0.f;
  }
#pragma unroll
  for (int u = 0; u < PB; ++u) {
    const int e = tid + 256 * u;
    const int k = TB == 0 ? e / GBN : e % BK, j = TB == 0 ? e % GBN : e / BK;
    Bs[k][j] = ob[u] ? vb[u] : 0.f;
  }
}

// Store one result: straight (with alpha, beta, the column's bias bj, ReLU)
// or into the split's partial slice.
MVPB_DEV void gemm_store(const GemmArgs &g, int z, int i, int j, float acc, float bj) {
  if (i >= g.M || j >= g.N) return;
  if (g.kchunk < g.K) {
    g.C[((size_t)z * g.M + i) * g.N + j] = acc;
    return;
  }
  float *c = g.C + (size_t)i * g.ldc + j;
  float v = g.alpha * acc + (g.beta != 0.f ? g.beta * *c : 0.f) + bj;
  *c = g.relu ? fmaxf(v, 0.f) : v;
}
// Bias of column j (zero without bias or for a split), loaded from an
// in-range address so that a thread's loads are in flight together.
MVPB_DEV float gemm_bias(const GemmArgs &g, int j) {
  if (!g.bias || g.kchunk < g.K) return 0.f;   // uniform
  const float b = gld(g.bias, j < g.N ? (size_t)j : 0);
  return j < g.N ? b : 0.f;
}

template <int TA, int TB>
__global__ void __launch_bounds__(256) sgemm_f32(GemmArgs g) {
  constexpr int BK = 16;
  __shared__ float As[BK][GBM + 4];
  __shared__ float Bs[BK][GBN + 4];
  const int m0 = blockIdx.y * GBM, n0 = blockIdx.x * GBN;
  const int kb = blockIdx.z * g.kchunk, ke = min(g.K, kb + g.kchunk);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4] = {};
  for (int k0 = kb; k0 < ke; k0 += BK) {
    load_tiles<TA, TB, BK>(g, m0, n0, k0, ke, As, Bs);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = As[kk][ty + 16 * q];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = Bs[kk][tx + 16 * q];
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[p][q] = fmaf(a[p], b[q], acc[p][q]);
    }
    __syncthreads();
  }
  float bj[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) bj[q] = gemm_bias(g, n0 + tx + 16 * q);
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) gemm_store(g, blockIdx.z, m0 + ty + 16 * p, n0 + tx + 16 * q, acc[p][q], bj[q]);
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

MVPB_DEV f4v gld4(const float *p, size_t i) { return *((const MVPB_GAS f4v *)(p + i)); }
MVPB_DEV void gst4(float *p, size_t i, f4v v) { *((MVPB_GAS f4v *)(p + i)) = v; }
MVPB_DEV bf8v to_bf16(const float (&v)[8]) {
  bf8v r;
#pragma unroll
  for (int u = 0; u < 8; ++u) r[u] = (__bf16)v[u];
  return r;
}

// Eight consecutive k (from gk) of one row of op(A) or column of op(B), zero
// outside.  KC: k contiguous in memory, read as two vectors (base, leading
// dimension and K allow it, see gemm: all eight or none exist); else one load per
// k, consecutive threads on consecutive rows.  No branches: a load under one is
// waited for where the paths meet.
template <bool KC>
MVPB_DEV void load_k8(const float *__restrict__ p, int ld, int row, int rows, int gk, int k1, float (&v)[8]) {
  const bool in = row < rows;
  if constexpr (KC) {
    const bool ok = in && gk < k1;
    const size_t x = ok ? (size_t)row * ld + gk : 0;
    const f4v a = gld4(p, x), b = gld4(p, ok ? x + 4 : 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[u] = ok ? a[u] : 0.f;
      v[4 + u] = ok ? b[u] : 0.f;
    }
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool ok = in && gk + u < k1;
      const float x = gld(p, ok ? (size_t)(gk + u) * ld + row : 0);
      v[u] = ok ? x : 0.f;
    }
  }
}
// The same of a transposed column matrix, col[gk + u][gi]: tap and channel belong
// to the thread (dy, dx: its input pixel's offset), the output pixels gk + u to
// the wavefront.
MVPB_DEV void load_col8(const ConvA &cv, int dy, int dx, int c, bool in, int gk, int k1, float (&v)[8]) {
  const int mH = (1 << cv.lH) - 1, mW = (1 << cv.lW) - 1;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int p = min(gk + u, k1 - 1), ox = p & ((1 << cv.lWo) - 1), t = p >> cv.lWo;
    const int oy = t & ((1 << cv.lHo) - 1), b = t >> cv.lHo;
    const int y = (cv.s * oy + dy) & mH, x = (cv.s * ox + dx) & mW;
    const unsigned off = (unsigned)(((y << cv.lW) + x) << cv.lC) + (unsigned)c;
    const float z = gld(cv.in + ((size_t)b << (cv.lH + cv.lW + cv.lC)), off);
    v[u] = in && gk + u < k1 ? z : 0.f;
  }
}

// Matrix-core GEMM: 64 x 64 block tile, 4 wavefronts of 32 x 32 (2 x 2
// v_mfma_f32_16x16x32_bf16 tiles, 32-deep K steps).  Lane l feeds
// A[row = l%16][k = 8(l/16)+v] and B[k = 8(l/16)+v][col = l%16], v < 8, and
// receives D[4(l/16)+v][l%16], v < 4.  Inputs are rounded to BF16 (nearest even)
// on their way into LDS, where a lane's operand is 16 contiguous bytes;
// accumulation is FP32.  Bound by the chain of K steps (one workgroup per CU at
// most, and the convolutions' weight gradients 64 steps deep): two LDS buffers,
// the loads of the next four steps in flight, one barrier a step.
// The weight gradient of the second convolution at 256 cells 53 -> 41 us (inputs
// held as FP32 in LDS and one step's loads in flight before), fc1 of 4096 cells
// 30 -> 15 us.
struct GemmLds {
  __attribute__((aligned(16))) __bf16 A[2][GBM * 40], B[2][GBN * 40];
};
// Tile (bx, by) of split bz.
template <int TA, int TB, bool CONV>
MVPB_DEV void gemm_bf16_tile(const GemmArgs &g, int bx, int by, int bz, GemmLds &sm) {
  static_assert(!CONV || TA == 1, "the column matrix is only read transposed");
  constexpr int BK = 32, LD = BK + 8;
  const int m0 = by * GBM, n0 = bx * GBN;
  const int kb = bz * g.kchunk, ke = min(g.K, kb + g.kchunk);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = (w >> 1) * 32, wc = (w & 1) * 32;
  // this thread's entries of a step: row (column) ia (ib), eight k from ka (kb8)
  constexpr bool KA = TA == 0, KBC = TB == 1;
  const int ia = KA ? tid >> 2 : lane, ka = KA ? (tid & 3) * 8 : w * 8;
  const int ib = KBC ? tid >> 2 : lane, kq = KBC ? (tid & 3) * 8 : w * 8;
  const int gt = CONV ? min(m0 + ia, g.M - 1) : 0, tap = gt >> g.conv.lC, ci = gt & ((1 << g.conv.lC) - 1);
  const int dy = tap / 3 - 1, dx = tap % 3 - 1;   // CONV: row m0 + ia of op(A)
  constexpr int PF = 4;   // steps whose loads are in flight
  float va[PF][8], vb[PF][8];
  auto load_step = [&](int k0, float (&va)[8], float (&vb)[8]) {
    if constexpr (CONV)
      load_col8(g.conv, dy, dx, ci, m0 + ia < g.M, k0 + ka, ke, va);
    else
      load_k8<KA>(g.A, g.lda, m0 + ia, g.M, k0 + ka, ke, va);
    load_k8<KBC>(g.B, g.ldb, n0 + ib, g.N, k0 + kq, ke, vb);
  };
  f4v acc[2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[p][q] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < PF; ++u) load_step(kb + BK * u, va[u], vb[u]);   // beyond ke: element 0, unused
  for (int k0 = kb; k0 < ke; k0 += PF * BK) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      if (k0 + BK * u >= ke) break;
      __bf16 *Au = sm.A[u & 1], *Bu = sm.B[u & 1];
      *(bf8v *)&Au[ia * LD + ka] = to_bf16(va[u]);
      *(bf8v *)&Bu[ib * LD + kq] = to_bf16(vb[u]);
      lds_barrier();
      load_step(k0 + BK * (u + PF), va[u], vb[u]);
      bf8v af[2], bf[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        af[p] = *(const bf8v *)&Au[(wr + 16 * p + (lane & 15)) * LD + 8 * (lane >> 4)];
        bf[p] = *(const bf8v *)&Bu[(wc + 16 * p + (lane & 15)) * LD + 8 * (lane >> 4)];
      }
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          acc[p][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[p], bf[q], acc[p][q], 0, 0, 0);
    }
  }
  float bj[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) bj[q] = gemm_bias(g, n0 + wc + 16 * q + (lane & 15));
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        gemm_store(g, bz, m0 + wr + 16 * p + 4 * (lane >> 4) + v, n0 + wc + 16 * q + (lane & 15), acc[p][q][v], bj[q]);
}

template <int TA, int TB>
__global__ void __launch_bounds__(256) sgemm_bf16(GemmArgs g) {
  __shared__ GemmLds sm;
  gemm_bf16_tile<TA, TB, false>(g, blockIdx.x, blockIdx.y, blockIdx.z, sm);
}

// C = act(alpha sum_z P[z] + beta C + bias), slices added in order z = 0, 1, ...
MVPB_DEV float slice_sum(const float *__restrict__ P, int splits, size_t MN, int e) {
  // eight slices' loads in flight at a time, added in slice order
  constexpr int U = 8;
  float acc = 0.f;
  int z = 0;
  for (; z + U <= splits; z += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = gld(P, (size_t)(z + u) * MN + e);
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u];
  }
  for (; z < splits; ++z) acc += P[(size_t)z * MN + e];
  return acc;
}
__global__ void __launch_bounds__(256) gemm_reduce(const float *__restrict__ P, int splits, int M, int N, float alpha,
                                                   float beta, float *__restrict__ C, int ldc,
                                                   const float *__restrict__ bias, int relu) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= M * N) return;
  const int i = e / N, j = e % N;
  const float acc = slice_sum(P, splits, (size_t)M * N, e);
  float *c = C + (size_t)i * ldc + j;
  float v = alpha * acc + (beta != 0.f ? beta * *c : 0.f) + (bias ? bias[j] : 0.f);
  *c = relu ? fmaxf(v, 0.f) : v;
}

// Split K so that every output tile gets enough workgroups: long reductions
// (K >= 4096) are cut into chunks of at least 1024, at most 128 chunks, and
// only while the output tiles alone leave the chip idle.
static int gemm_splits(int M, int N, int K) {
  const long tiles = (long)((M + GBM - 1) / GBM) * ((N + GBN - 1) / GBN);
  if (K < 4096 || tiles >= 256) return 1;
  int sp = (int)std::min<long>(128, (512 + tiles - 1) / tiles);
  sp = std::min(sp, std::max(1, K / 1024));
  return sp;
}

// Chunk of K of one split and the number of splits (align: the K step).
static int gemm_chunk(int M, int N, int K, int align, size_t split_cap, int *splits) {
  int sp = gemm_splits(M, N, K);
  if ((size_t)sp * M * N > split_cap) sp = 1;
  const int kchunk = sp == 1 ? K : ((K + sp - 1) / sp + align - 1) / align * align;
  *splits = (K + kchunk - 1) / kchunk;
  return kchunk;
}

static hipError_t gemm(bool bf16, int ta, int tb, int M, int N, int K, float alpha, const float *A, int lda,
                       const float *B, int ldb, float beta, float *C, int ldc, hipStream_t st,
                       const float *bias = nullptr, int relu = 0, float *split_buf = nullptr,
                       size_t split_cap = 0, const ConvA &conv = ConvA()) {
  int sp = 1;
  const int kchunk = gemm_chunk(M, N, K, bf16 ? 32 : 16, split_buf ? split_cap : 0, &sp);
  GemmArgs g{M, N, K, alpha, beta, A, lda, B, ldb, sp == 1 ? C : split_buf, ldc, kchunk, bias, relu, conv};
  dim3 grid((N + GBN - 1) / GBN, (M + GBM - 1) / GBM, sp);
  if (bf16) {
    // 16-byte reads along k of the operands that have it contiguous (splits are
    // multiples of 32); the convolutions have kernels of their own
    auto ok = [&](bool along, const float *p, int ld) {
      return !along || (ld % 4 == 0 && K % 8 == 0 && (uintptr_t)p % 16 == 0);
    };
    if (conv.in || !ok(ta == 0, A, lda) || !ok(tb == 1, B, ldb)) return hipErrorInvalidValue;
#define MVPB_GEMM_CASE(TA, TB) \
  if (ta == TA && tb == TB) hipLaunchKernelGGL((sgemm_bf16<TA, TB>), grid, dim3(256), 0, st, g);
    MVPB_GEMM_CASE(0, 0)
    MVPB_GEMM_CASE(0, 1)
    MVPB_GEMM_CASE(1, 0)
#undef MVPB_GEMM_CASE
  } else {
#define MVPB_GEMM_CASE(TA, TB) \
  if (ta == TA && tb == TB) hipLaunchKernelGGL((sgemm_f32<TA, TB>), grid, dim3(256), 0, st, g);
    MVPB_GEMM_CASE(0, 0)
    MVPB_GEMM_CASE(0, 1)
    MVPB_GEMM_CASE(1, 0)
#undef MVPB_GEMM_CASE
  }
  if (sp > 1)
    hipLaunchKernelGGL(gemm_reduce, dim3((M * N + 255) / 256), dim3(256), 0, st, split_buf, sp, M, N, alpha, beta, C,
                       ldc, bias, relu);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The four convolutions of one cell in one workgroup (BF16 products).  Their
// activations are 4 bytes x 32 x (1024 + 256 + 64) per cell, written and read
// back through HBM when each layer is a launch of its own; here a layer's output
// goes to LDS, rounded to BF16 as the next product rounds it anyway (FP32 to
// memory too where the backward pass wants it).  Products are transposed, D =
// W^T col^T, so that a lane holds four consecutive channels of one pixel; the
// weights stay in registers over all cells of the workgroup.  Wavefront w: output
// channels 16 (w & 1) .., a quarter w >> 1 of each layer's pixels.  A pixel of 32
// channels takes 80 bytes of LDS (40-byte steps would break the 16-byte reads,
// 64 would put every second pixel on the same banks).  Bound by instruction issue:
// 4096 cells in 97 us, the four launches 870 us before.
// ---------------------------------------------------------------------------
constexpr int CPX = 40;   // BF16 entries per pixel in LDS
struct ConvChain {
  const uint8_t *cells;
  const float *W[4], *b[4];
  float *out[4];   // NHWC activations; the first three only with KEEP
  int B;
};
// One 3 x 3 stride-2 layer: 16 output pixels from `first` (row-major in a grid of
// 2^lw columns) over the input `in` (a grid of twice the columns), taps in order.
MVPB_DEV f4v conv_s2_tile(const __bf16 *in, int first, int lw, const bf8v (&wf)[9]) {
  const int lane = threadIdx.x & 63, p = first + (lane & 15), ox = p & ((1 << lw) - 1), oy = p >> lw;
  const int m = (2 << lw) - 1;
  f4v acc = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ky = 0; ky < 3; ++ky)
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      const int y = (2 * oy + ky - 1) & m, x = (2 * ox + kx - 1) & m;
      const bf8v col = *(const bf8v *)&in[((y << (lw + 1)) + x) * CPX + 8 * (lane >> 4)];
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[3 * ky + kx], col, acc, 0, 0, 0);
    }
  return acc;
}
template <bool KEEP>
__global__ void __launch_bounds__(512) conv_chain(ConvChain c) {
  __shared__ __attribute__((aligned(16))) __bf16 a1[1024 * CPX];
  __shared__ __attribute__((aligned(16))) __bf16 a2[256 * CPX];
  __shared__ __attribute__((aligned(16))) __bf16 a3[64 * CPX];
  __shared__ unsigned bits[32];   // rows of the cell
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), quarter = w >> 1, ch = 16 * (w & 1);
  // weights: row = channel ch + li, k = 8 lk + v of each tap; biases of channels ch + 4 lk + v
  bf8v w1, wf[3][9];
  f4v bias[4];
  {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = 8 * lk + u;
      v[u] = gld(c.W[0], (size_t)(k < 9 ? k : 0) * 32 + ch + li);
      if (k >= 9) v[u] = 0.f;
    }
    w1 = to_bf16(v);
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
      for (int t = 0; t < 9; ++t) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = gld(c.W[l + 1], (size_t)(32 * t + 8 * lk + u) * 32 + ch + li);
        wf[l][t] = to_bf16(v);
      }
#pragma unroll
    for (int l = 0; l < 4; ++l)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) bias[l][v4] = gld(c.b[l], (size_t)(ch + 4 * lk + v4));
  }
  // bias and ReLU; pixel p of layer l to LDS (dst) and memory
  auto put = [&](int l, f4v acc, int p, __bf16 *dst, size_t cell_pixels, size_t cell) {
    f4v v;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = fmaxf(acc[u] + bias[l][u], 0.f);
    if (dst) {
      typedef __bf16 bf4v __attribute__((ext_vector_type(4)));
      bf4v h;
#pragma unroll
      for (int u = 0; u < 4; ++u) h[u] = (__bf16)v[u];
      *(bf4v *)&dst[p * CPX + ch + 4 * lk] = h;
    }
    if (KEEP || l == 3) gst4(c.out[l], (cell * cell_pixels + p) * 32 + ch + 4 * lk, v);
  };
  // 64 pixels of a ballot are two rows
  auto fetch = [&](int cell, uint8_t &x0, uint8_t &x1) {
    const MVPB_GAS uint8_t *q = (const MVPB_GAS uint8_t *)(c.cells + (size_t)cell * 1024);
    x0 = q[tid];
    x1 = q[tid + 512];
  };
  uint8_t x0 = 0, x1 = 0;
  fetch(blockIdx.x, x0, x1);
  for (int cell = blockIdx.x; cell < c.B; cell += gridDim.x) {
    const unsigned long long r0 = __ballot(x0 != 0), r1 = __ballot(x1 != 0);
    if (lane < 2) {
      bits[2 * w + lane] = (unsigned)(r0 >> (32 * lane));
      bits[16 + 2 * w + lane] = (unsigned)(r1 >> (32 * lane));
    }
    lds_barrier();
    if (cell + (int)gridDim.x < c.B) fetch(cell + gridDim.x, x0, x1);
#pragma unroll 2
    for (int t = 0; t < 16; ++t) {
      const int first = 256 * quarter + 16 * t, y = first >> 5, x = (first & 31) + li;
      unsigned pat = 0;   // the nine taps' bits
#pragma unroll
      for (int ky = 0; ky < 3; ++ky) {
        const unsigned r = bits[(y + ky - 1) & 31];
        pat |= (__builtin_amdgcn_alignbit(r, r, (x - 1) & 31) & 7u) << (3 * ky);
      }
      pat = lk < 2 ? pat >> (8 * lk) : 0u;   // k = 8 lk + v
      union {
        unsigned u[4];
        bf8v v;
      } col;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        col.u[q] = ((pat >> (2 * q)) & 1u) * 0x3F80u | ((pat >> (2 * q + 1)) & 1u) * 0x3F800000u;
      const f4v acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, col.v, f4v{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      put(0, acc, first + li, a1, 1024, cell);
    }
    lds_barrier();
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
      const int first = 64 * quarter + 16 * t;
      put(1, conv_s2_tile(a1, first, 4, wf[0]), first + li, a2, 256, cell);
    }
    lds_barrier();
    put(2, conv_s2_tile(a2, 16 * quarter, 3, wf[1]), 16 * quarter + li, a3, 64, cell);
    lds_barrier();
    if (quarter == 0) put(3, conv_s2_tile(a3, 0, 2, wf[2]), li, nullptr, 16, cell);
  }
}

// Backward data pass of a stride-2 3 x 3 layer (32 channels each way, BF16
// products): da[y][x][.] = sum over the taps (ky, kx) that read pixel (y, x) of
// W_tap dz[oy][ox], each tap's product rounded to FP32 before the sum, taps in
// order, and zero where the activation is not positive (the ReLU of the layer
// below).  One wavefront per 16 output pixels: the pixel's own and its right, lower
// and diagonal neighbours' dz serve the four input pixels of its 2 x 2 cell, one,
// two, two and four taps.  Bound by writing da.  256 cells,
// grid 32: 23 us, before (product to a column buffer, gather, mask) 140 us.
struct ConvDx {
  const float *dz, *W, *act;
  float *da;
  int tiles, lH;   // 16-pixel tiles over the batch, input grid 2^lH square
};
__global__ void __launch_bounds__(256) conv_dx(ConvDx c) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int lo = c.lH - 1, mo = (1 << lo) - 1;
  const int stride = gridDim.x * 4;
  bf8v wf[9][2];   // row = input channel 16 h + li, k = output channel 8 lk + v
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const size_t x = (size_t)(32 * t + 16 * h + li) * 32 + 8 * lk;
      const f4v p = gld4(c.W, x), q = gld4(c.W, x + 4);
      const float v[8] = {p[0], p[1], p[2], p[3], q[0], q[1], q[2], q[3]};
      wf[t][h] = to_bf16(v);
    }
  for (int t = blockIdx.x * 4 + (threadIdx.x >> 6); t < c.tiles; t += stride) {
    const int pix = 16 * t + li, ox = pix & mo, oy = (pix >> lo) & mo, b = pix >> (2 * lo);
    bf8v z[2][2];   // dz at (oy + i, ox + j)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const size_t x = (((((size_t)b << lo) + ((oy + i) & mo)) << lo) + ((ox + j) & mo)) * 32 + 8 * lk;
        const f4v p = gld4(c.dz, x), q = gld4(c.dz, x + 4);
        const float v[8] = {p[0], p[1], p[2], p[3], q[0], q[1], q[2], q[3]};
        z[i][j] = to_bf16(v);
      }
    f4v a[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int y = 2 * oy + (q >> 1), x = 2 * ox + (q & 1);
        a[q][h] = gld4(c.act, (((((size_t)b << c.lH) + y) << c.lH) + x) * 32 + 16 * h + 4 * lk);
      }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int py = q >> 1, px = q & 1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f4v s = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
          for (int kx = 0; kx < 3; ++kx) {
            // the output row reads input row 2 oy' + ky - 1: oy' = (y - ky + 1) / 2
            if ((py - ky + 1) & 1 || (px - kx + 1) & 1) continue;
            const int i = (py - ky + 1) / 2, j = (px - kx + 1) / 2;
            s += __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[3 * ky + kx][h], z[i][j], f4v{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (!(a[q][h][u] > 0.f)) s[u] = 0.f;
        const int y = 2 * oy + py, x = 2 * ox + px;
        gst4(c.da, (((((size_t)b << c.lH) + y) << c.lH) + x) * 32 + 16 * h + 4 * lk, s);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Elementwise and reduction kernels
// ---------------------------------------------------------------------------
__global__ void cells_to_float(const uint8_t *__restrict__ cells, float *__restrict__ x, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = cells[i] ? 1.f : 0.f;
}

// Gather form of col2im: da[b][y][x][c] = sum over taps of dcol at the output
// pixel that reads (y, x) through that tap (if any).
__global__ void col2im(const float *__restrict__ dcol, float *__restrict__ da, int B, int H, int W, int C, int s) {
  const int Ho = H / s, Wo = W / s, K = 9 * C;
  const size_t total = (size_t)B * H * W * C;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % C);
    const size_t pix = e / C;
    const int x = (int)(pix % W), y = (int)((pix / W) % H), b = (int)(pix / ((size_t)W * H));
    float acc = 0.f;
    for (int ky = 0; ky < 3; ++ky) {
      const int ty = (y - ky + 1 + H) % H;
      if (ty % s) continue;
      const int oy = ty / s;
      for (int kx = 0; kx < 3; ++kx) {
        const int tx = (x - kx + 1 + W) % W;
        if (tx % s) continue;
        const int ox = tx / s;
        const size_t p = ((size_t)b * Ho + oy) * Wo + ox;
        acc += dcol[p * K + (ky * 3 + kx) * C + c];
      }
    }
    da[e] = acc;
  }
}

__global__ void relu_mask(float *__restrict__ d, const float *__restrict__ a, size_t n) {
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
    if (!(a[e] > 0.f)) d[e] = 0.f;
}

// Partial column sums: block (x, y) sums rows y, y + gridDim.y, ... of the
// 64-column slab x into part[y][c]; column_sums_fin adds the parts in order.
MVPB_DEV void column_part(const float *__restrict__ d, size_t rows, int C, float *__restrict__ part, int slab, int y,
                          int parts) {
  __shared__ float red[4][64];
  const int c = slab * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6;
  float acc = 0.f;
  if (c < C) {
    // eight rows' loads in flight at a time, added in row order
    constexpr int U = 8;
    const size_t r0 = (size_t)y * 4 + g, step = (size_t)parts * 4;
    size_t r = r0;
    for (; r + (U - 1) * step < rows; r += U * step) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = gld(d, (r + u * step) * C + c);
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v[u];
    }
    for (; r < rows; r += step) acc += d[r * C + c];
  }
  red[g][threadIdx.x & 63] = acc;
  __syncthreads();
  if (g == 0 && c < C) part[(size_t)y * C + c] = red[0][threadIdx.x] + red[1][threadIdx.x] +
                                                 red[2][threadIdx.x] + red[3][threadIdx.x];
}
__global__ void __launch_bounds__(256) column_sums(const float *__restrict__ d, size_t rows, int C,
                                                   float *__restrict__ part) {
  column_part(d, rows, C, part, blockIdx.x, blockIdx.y, gridDim.y);
}

MVPB_DEV float part_sum(const float *__restrict__ part, int parts, int C, int c) {
  // eight parts' loads in flight at a time, added in part order
  constexpr int U = 8;
  float acc = 0.f;
  int p = 0;
  for (; p + U <= parts; p += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = gld(part, (size_t)(p + u) * C + c);
#pragma unroll
    for (int u = 0; u < U; ++u) acc += v[u];
  }
  for (; p < parts; ++p) acc += part[(size_t)p * C + c];
  return acc;
}
__global__ void column_sums_fin(const float *__restrict__ part, int parts, int C, float *__restrict__ db) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < C) db[c] = part_sum(part, parts, C, c);
}

// The weight and bias gradients of the four convolutions, BF16 products: with dz of
// every layer at hand, one launch for all partial sums and one for their sums in
// order, instead of four launches per layer of which no weight gradient but one
// fills the chip (256 cells: 20, 80, 320 and 128 workgroups of 33 to 61 us each).
// Workgroups of the first launch: the tiles and splits of each layer's product, then
// the row blocks of each layer's bias gradient.  At 256 cells 71 + 14 us
// against 245 us of the sixteen.
struct ConvGrads {
  GemmArgs g[4];         // C: the layer's partial slices, or dW itself when not split
  int splits[4], tiles[4];
  const float *dz[4];
  float *part[4];        // partial column sums
  int rows[4], parts[4];
  float *dW[4], *db[4];
  int end[8];            // of each layer's workgroups, products then row blocks
};
__global__ void __launch_bounds__(256) conv_grads(ConvGrads c) {
  __shared__ GemmLds sm;
  int q = 0;
  while ((int)blockIdx.x >= c.end[q]) ++q;   // the grid is c.end[7]
  const int l = q & 3, r = blockIdx.x - (q > 0 ? c.end[q - 1] : 0);
  if (q < 4)
    gemm_bf16_tile<1, 0, true>(c.g[l], 0, r % c.tiles[l], r / c.tiles[l], sm);
  else
    column_part(c.dz[l], (size_t)c.rows[l], 32, c.part[l], 0, r, c.parts[l]);
}
__global__ void __launch_bounds__(256) conv_grads_fin(ConvGrads c) {
  const int l = blockIdx.y, e = blockIdx.x * 256 + threadIdx.x, mn = c.g[l].M * 32;
  if (e < mn && c.splits[l] > 1) c.dW[l][e] = slice_sum(c.g[l].C, c.splits[l], (size_t)mn, e);
  if (blockIdx.x == 0 && threadIdx.x < 32) c.db[l][threadIdx.x] = part_sum(c.part[l], c.parts[l], 32, threadIdx.x);
}

// dout = 2 (out - y) / n and per-block partial sums of (out - y)^2
__global__ void __launch_bounds__(256) mse_grad(const float *__restrict__ out, const float *__restrict__ y, int n,
                                                float *__restrict__ dout, float *__restrict__ partial) {
  __shared__ float red[256];
  float acc = 0.f;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
    const float r = out[e] - y[e];
    dout[e] = 2.f * r / (float)n;
    acc += r * r;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void adam_step(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                          int n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void init_uniform(float *__restrict__ p, int n, float lim, unsigned long long seed, unsigned long long offset) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  // counter-based hash (splitmix64 finaliser) -> uniform in [-lim, lim)
  unsigned long long z = seed + 0x9E3779B97F4A7C15ull * (offset + i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  const float u = (float)((z >> 40) * (1.0 / 16777216.0));
  p[i] = (2.f * u - 1.f) * lim;
}

}  // namespace mvpb

using namespace mvpb;

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
namespace {

struct Layer {
  int ci, co, s, H, W;  // input H, W
};
const Layer kConv[4] = {{1, 32, 1, 32, 32}, {32, 32, 2, 32, 32}, {32, 32, 2, 16, 16}, {32, 32, 2, 8, 8}};
constexpr int kFcIn = 512, kFcHid = 256, kOut = 400, kPix = 32 * 32;
constexpr size_t kSplitCap = (size_t)3 << 20;   // floats of split-K partial slices (of the convolutions together 2.9 M at most)
constexpr int kColParts = 256;                  // row blocks of the bias-gradient sums

int param_offsets(int *off) {  // 12 tensors
  int o = 0, t = 0;
  for (int l = 0; l < 4; ++l) {
    off[t++] = o;
    o += 9 * kConv[l].ci * kConv[l].co;
    off[t++] = o;
    o += kConv[l].co;
  }
  off[t++] = o;
  o += kFcIn * kFcHid;
  off[t++] = o;
  o += kFcHid;
  off[t++] = o;
  o += kFcHid * kOut;
  off[t++] = o;
  o += kOut;
  return o;
}

template <typename T>
struct Buf {
  T *p = nullptr;
  size_t n = 0;
  ~Buf() {
    if (p) (void)hipFree(p);
  }
  hipError_t alloc(size_t count) {
    n = count;
    return hipMalloc(&p, sizeof(T) * count);
  }
};

}  // namespace

struct mvpb_sur_s {
  mvpb_ctx ctx = nullptr;
  hipStream_t st = nullptr;
  int max_batch = 0;
  bool bf16 = true;
  int n_params = 0;
  int off[12];
  long long step = 0;
  uint64_t seed = 0;
  Buf<float> params, grads, m, v;
  Buf<float> act[5];        // act[0] input [B,32,32,1]; act[l+1] output of conv l (NHWC)
  Buf<float> dcol, dact, dact2;
  Buf<float> h, out, dout, dh, dflat, partial;
  Buf<float> split;     // partial slices of split-K GEMMs
  Buf<float> colpart;   // partial column sums (bias gradients)
  Buf<uint8_t> cells;
  Buf<float> target;
  float *loss_host = nullptr;         // pinned
  hipEvent_t loss_ready = nullptr;    // loss_host holds the last batch's partial sums
  ~mvpb_sur_s() {
    if (loss_host) (void)hipHostFree(loss_host);
    if (loss_ready) (void)hipEventDestroy(loss_ready);
  }
};

extern "C" int mvpb_sur_destroy(mvpb_sur net);

// GEMM with the network's precision and split-K scratch.
static hipError_t net_gemm(mvpb_sur net, int ta, int tb, int M, int N, int K, const float *A, int lda, const float *B,
                           int ldb, float *C, int ldc, const float *bias = nullptr, int relu = 0,
                           const ConvA &conv = ConvA()) {
  return gemm(net->bf16, ta, tb, M, N, K, 1.f, A, lda, B, ldb, 0.f, C, ldc, net->st, bias, relu, net->split.p,
              net->split.n, conv);
}

static int ilog2_exact(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

// The implicit column matrix of conv layer L over the activations `in`.
static ConvA conv_operand(const Layer &L, const float *in) {
  ConvA cv;
  cv.in = in;
  cv.lH = ilog2_exact(L.H);
  cv.lW = ilog2_exact(L.W);
  cv.lC = ilog2_exact(L.ci);
  cv.lHo = ilog2_exact(L.H / L.s);
  cv.lWo = ilog2_exact(L.W / L.s);
  cv.s = L.s;
  return cv;
}

// db[c] = sum over rows of d[r][c] (blocks of rows, then the blocks in order).
static int col_parts(size_t rows) { return (int)std::min<size_t>(kColParts, (rows + 511) / 512); }
static void col_sums(mvpb_sur net, const float *d, size_t rows, int C, float *db) {
  const int parts = col_parts(rows);
  hipLaunchKernelGGL(column_sums, dim3((C + 63) / 64, parts), dim3(256), 0, net->st, d, rows, C, net->colpart.p);
  hipLaunchKernelGGL(column_sums_fin, dim3((C + 255) / 256), dim3(256), 0, net->st, net->colpart.p, parts, C, db);
}

// keep: leave every layer's activations in net->act for a backward pass.
static int sur_forward(mvpb_sur net, int B, const uint8_t *cells, bool keep) {
  hipStream_t st = net->st;
  float *P = net->params.p;
  hipError_t e = hipSuccess;
  if (net->bf16) {
    ConvChain c{};
    c.cells = cells;
    c.B = B;
    for (int l = 0; l < 4; ++l) {
      c.W[l] = P + net->off[2 * l];
      c.b[l] = P + net->off[2 * l + 1];
      c.out[l] = net->act[l + 1].p;
    }
    const dim3 grid(std::min(B, 256));   // one workgroup per CU, each over its share of the cells
    if (keep)
      hipLaunchKernelGGL(conv_chain<true>, grid, dim3(512), 0, st, c);
    else
      hipLaunchKernelGGL(conv_chain<false>, grid, dim3(512), 0, st, c);
    e = hipGetLastError();
  }
  for (int l = 0; l < 4 && !net->bf16 && e == hipSuccess; ++l) {
    const Layer &L = kConv[l];
    const int Ho = L.H / L.s, Wo = L.W / L.s;
    const size_t rows = (size_t)B * Ho * Wo;
    const int K = 9 * L.ci;
    // convolution as one GEMM over the implicit column matrix, bias and ReLU in its epilogue
    e = net_gemm(net, 0, 0, (int)rows, L.co, K, nullptr, K, P + net->off[2 * l], L.co, net->act[l + 1].p, L.co,
                 P + net->off[2 * l + 1], 1, conv_operand(L, net->act[l].p));
  }
  // fc1 (ReLU), fc2
  if (e == hipSuccess)
    e = net_gemm(net, 0, 0, B, kFcHid, kFcIn, net->act[4].p, kFcIn, P + net->off[8], kFcHid, net->h.p, kFcHid,
                 P + net->off[9], 1);
  if (e == hipSuccess)
    e = net_gemm(net, 0, 0, B, kOut, kFcHid, net->h.p, kFcHid, P + net->off[10], kOut, net->out.p, kOut,
                 P + net->off[11], 0);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "surrogate forward: %s", hipGetErrorString(e));
  return MVPB_OK;
}

// Backward from net->dout; gradients into net->grads.
static int sur_backward(mvpb_sur net, int B) {
  hipStream_t st = net->st;
  float *P = net->params.p, *G = net->grads.p;
  hipError_t e = net_gemm(net, 1, 0, kFcHid, kOut, B, net->h.p, kFcHid, net->dout.p, kOut, G + net->off[10], kOut);
  col_sums(net, net->dout.p, (size_t)B, kOut, G + net->off[11]);
  if (e == hipSuccess) e = net_gemm(net, 0, 1, B, kFcHid, kOut, net->dout.p, kOut, P + net->off[10], kOut, net->dh.p, kFcHid);
  hipLaunchKernelGGL(relu_mask, dim3((B * kFcHid + 255) / 256), dim3(256), 0, st, net->dh.p, net->h.p, (size_t)B * kFcHid);
  if (e == hipSuccess)
    e = net_gemm(net, 1, 0, kFcIn, kFcHid, B, net->act[4].p, kFcIn, net->dh.p, kFcHid, G + net->off[8], kFcHid);
  col_sums(net, net->dh.p, (size_t)B, kFcHid, G + net->off[9]);
  // BF16: dz of the first layer in dact, of the others in dact2; else the two in turn
  float *dz[4] = {net->dact.p, net->dact2.p, net->dact2.p + (size_t)B * 8192, net->dact2.p + (size_t)B * 10240};
  if (e == hipSuccess)
    e = net_gemm(net, 0, 1, B, kFcIn, kFcHid, net->dh.p, kFcHid, P + net->off[8], kFcHid,
                 net->bf16 ? dz[3] : net->dact.p, kFcIn);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "surrogate backward: %s", hipGetErrorString(e));
  if (net->bf16) {
    hipLaunchKernelGGL(relu_mask, dim3((B * kFcIn + 255) / 256), dim3(256), 0, st, dz[3], net->act[4].p,
                       (size_t)B * kFcIn);
    ConvGrads c{};
    size_t slices = 0;
    for (int l = 3; l >= 0; --l) {
      const Layer &L = kConv[l];
      const int rows = B * (L.H / L.s) * (L.W / L.s), K = 9 * L.ci;
      if (l > 0) {
        ConvDx x{dz[l], P + net->off[2 * l], net->act[l].p, dz[l - 1], rows / 16, ilog2_exact(L.H)};
        hipLaunchKernelGGL(conv_dx, dim3(std::min((x.tiles + 3) / 4, 512)), dim3(256), 0, st, x);
      }
      int sp = 1;
      const int kchunk = gemm_chunk(K, L.co, rows, 32, net->split.n, &sp);
      c.dW[l] = G + net->off[2 * l];
      c.db[l] = G + net->off[2 * l + 1];
      c.g[l] = GemmArgs{K, L.co, rows, 1.f, 0.f, nullptr, K, dz[l], L.co, sp > 1 ? net->split.p + slices : c.dW[l], L.co,
                        kchunk, nullptr, 0, conv_operand(L, net->act[l].p)};
      if (sp > 1) slices += (size_t)sp * K * L.co;
      c.splits[l] = sp;
      c.tiles[l] = (K + GBM - 1) / GBM;
      c.dz[l] = dz[l];
      c.part[l] = net->colpart.p + (size_t)l * kColParts * L.co;
      c.rows[l] = rows;
      c.parts[l] = col_parts(rows);
    }
    if (slices > net->split.n) return set_error(MVPB_E_DEVICE, "internal: %zu floats of partial sums", slices);
    int end = 0;
    for (int l = 0; l < 4; ++l) c.end[l] = end += c.splits[l] * c.tiles[l];
    for (int l = 0; l < 4; ++l) c.end[4 + l] = end += c.parts[l];
    hipLaunchKernelGGL(conv_grads, dim3(end), dim3(256), 0, st, c);
    hipLaunchKernelGGL(conv_grads_fin, dim3((9 * 32 * 32 + 255) / 256, 4), dim3(256), 0, st, c);
    e = hipGetLastError();
    if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "surrogate backward: %s", hipGetErrorString(e));
    return MVPB_OK;
  }
  float *da = net->dact.p, *da_next = net->dact2.p;
  for (int l = 3; l >= 0; --l) {
    const Layer &L = kConv[l];
    const int Ho = L.H / L.s, Wo = L.W / L.s;
    const size_t rows = (size_t)B * Ho * Wo;
    const int K = 9 * L.ci;
    // dz = da * relu'(act[l+1])
    hipLaunchKernelGGL(relu_mask, dim3((unsigned)std::min<size_t>((rows * L.co + 255) / 256, 65535)), dim3(256), 0, st,
                       da, net->act[l + 1].p, rows * L.co);
    // dW = col^T dz over the implicit column matrix (split over the output pixels), db = column sums of dz
    e = net_gemm(net, 1, 0, K, L.co, (int)rows, nullptr, K, da, L.co, G + net->off[2 * l], L.co, nullptr, 0,
                 conv_operand(L, net->act[l].p));
    col_sums(net, da, rows, L.co, G + net->off[2 * l + 1]);
    if (l > 0 && e == hipSuccess) {
      // dcol = dz W^T, then gather back onto the input pixels
      e = net_gemm(net, 0, 1, (int)rows, K, L.co, da, L.co, P + net->off[2 * l], L.co, net->dcol.p, K);
      const size_t tin = (size_t)B * L.H * L.W * L.ci;
      hipLaunchKernelGGL(col2im, dim3((unsigned)std::min<size_t>((tin + 255) / 256, 65535)), dim3(256), 0, st,
                         net->dcol.p, da_next, B, L.H, L.W, L.ci, L.s);
      std::swap(da, da_next);
    }
    if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "surrogate backward: %s", hipGetErrorString(e));
  }
  e = hipGetLastError();
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "surrogate backward: %s", hipGetErrorString(e));
  return MVPB_OK;
}

// Cells (and targets) on the device: *cells_dev, *tgt_dev.  x: also as the floats
// of act[0] (of the FP32 products and the weight gradients).
static int stage_inputs(mvpb_sur net, int B, const uint8_t *cells, const float *target, unsigned flags, bool x,
                        const uint8_t **cells_dev, const float **tgt_dev) {
  const bool dev = flags & MVPB_F_DEVICE_PTRS;
  const uint8_t *c = cells;
  if (!dev) {
    hipError_t e = hipMemcpyAsync(net->cells.p, cells, (size_t)B * kPix, hipMemcpyHostToDevice, net->st);
    if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "upload: %s", hipGetErrorString(e));
    c = net->cells.p;
  }
  *cells_dev = c;
  if (x)
    hipLaunchKernelGGL(cells_to_float, dim3((B * kPix + 255) / 256), dim3(256), 0, net->st, c, net->act[0].p, B * kPix);
  if (target) {
    if (!dev) {
      hipError_t e = hipMemcpyAsync(net->target.p, target, sizeof(float) * B * kOut, hipMemcpyHostToDevice, net->st);
      if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "upload: %s", hipGetErrorString(e));
      *tgt_dev = net->target.p;
    } else {
      *tgt_dev = target;
    }
  }
  return MVPB_OK;
}

// dout and the loss's partial sums, on their way to the host; loss_read waits for
// them only (the backward pass is in the queue by then: reading them at once left
// the GPU idle for 45 us of a 414 us training step).
constexpr int kLossBlocks = 64;
static int loss_and_grad_out(mvpb_sur net, int B, const float *tgt) {
  hipLaunchKernelGGL(mse_grad, dim3(kLossBlocks), dim3(256), 0, net->st, net->out.p, tgt, B * kOut, net->dout.p,
                     net->partial.p);
  hipError_t e = hipMemcpyAsync(net->loss_host, net->partial.p, sizeof(float) * kLossBlocks, hipMemcpyDeviceToHost,
                                net->st);
  if (e == hipSuccess) e = hipEventRecord(net->loss_ready, net->st);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "loss: %s", hipGetErrorString(e));
  return MVPB_OK;
}
static int loss_read(mvpb_sur net, int B, float *loss) {
  const hipError_t e = hipEventSynchronize(net->loss_ready);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "loss: %s", hipGetErrorString(e));
  double s = 0.0;
  for (int i = 0; i < kLossBlocks; ++i) s += net->loss_host[i];
  if (loss) *loss = (float)(s / (B * kOut));
  return MVPB_OK;
}

extern "C" int mvpb_sur_create(mvpb_ctx ctx, int max_batch, int precision, uint64_t seed, mvpb_sur *out) {
  if (!ctx || !out) return set_error(MVPB_E_INVALID, "NULL argument");
  if (ctx_closing(ctx)) return set_error(MVPB_E_INVALID, "context has been destroyed");
  if (max_batch < 1 || max_batch > 65536) return set_error(MVPB_E_INVALID, "max_batch out of range");
  if (precision != 0 && precision != 1) return set_error(MVPB_E_INVALID, "precision must be 0 (FP32) or 1 (BF16)");
  (void)hipSetDevice(ctx_device(ctx));
  mvpb_sur net = new mvpb_sur_s();
  net->ctx = ctx;
  net->st = ctx_stream(ctx);
  net->max_batch = max_batch;
  net->bf16 = precision == 1;
  net->seed = seed;
  net->n_params = param_offsets(net->off);
  const size_t B = max_batch;
  size_t colmax = 0, actmax = 0;
  for (int l = 0; l < 4; ++l) {
    const Layer &L = kConv[l];
    colmax = std::max(colmax, B * (L.H / L.s) * (L.W / L.s) * 9 * L.ci);
    actmax = std::max(actmax, B * L.H * L.W * L.ci);
    actmax = std::max(actmax, B * (L.H / L.s) * (L.W / L.s) * L.co);
  }
  hipError_t e = hipSuccess;
  auto A = [&](Buf<float> &b, size_t n) {
    if (e == hipSuccess) e = b.alloc(n);
  };
  A(net->params, net->n_params);
  A(net->grads, net->n_params);
  A(net->m, net->n_params);
  A(net->v, net->n_params);
  A(net->act[0], B * kPix);
  for (int l = 0; l < 4; ++l) A(net->act[l + 1], B * (kConv[l].H / kConv[l].s) * (kConv[l].W / kConv[l].s) * kConv[l].co);
  if (!net->bf16) A(net->dcol, colmax);   // the BF16 backward pass has no column buffer
  A(net->dact, actmax);
  A(net->dact2, actmax);
  A(net->h, B * kFcHid);
  A(net->dh, B * kFcHid);
  A(net->out, B * kOut);
  A(net->dout, B * kOut);
  A(net->partial, kLossBlocks);
  A(net->target, B * kOut);
  A(net->split, kSplitCap);
  A(net->colpart, (size_t)kColParts * kOut);
  if (e == hipSuccess) e = net->cells.alloc(B * kPix);
  if (e == hipSuccess) e = hipHostMalloc((void **)&net->loss_host, sizeof(float) * kLossBlocks, hipHostMallocDefault);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&net->loss_ready, hipEventDisableTiming);
  if (e != hipSuccess) {
    delete net;
    return set_error(MVPB_E_NOMEM, "surrogate buffers: %s", hipGetErrorString(e));
  }
  // He-uniform weights (counter-based generator), zero biases and moments
  for (int t = 0; t < 12; ++t) {
    const int n = (t + 1 < 12 ? net->off[t + 1] : net->n_params) - net->off[t];
    if (t % 2 == 1) {
      e = hipMemsetAsync(net->params.p + net->off[t], 0, sizeof(float) * n, net->st);
    } else {
      const int fan_in = t < 8 ? 9 * kConv[t / 2].ci : (t == 8 ? kFcIn : kFcHid);
      hipLaunchKernelGGL(init_uniform, dim3((n + 255) / 256), dim3(256), 0, net->st, net->params.p + net->off[t], n,
                         sqrtf(6.f / fan_in), (unsigned long long)seed, (unsigned long long)net->off[t]);
    }
  }
  if (e == hipSuccess) e = hipMemsetAsync(net->m.p, 0, sizeof(float) * net->n_params, net->st);
  if (e == hipSuccess) e = hipMemsetAsync(net->v.p, 0, sizeof(float) * net->n_params, net->st);
  if (e == hipSuccess) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) {
    delete net;
    return set_error(MVPB_E_DEVICE, "surrogate init: %s", hipGetErrorString(e));
  }
  ctx_retain(ctx);
  *out = net;
  return MVPB_OK;
}

extern "C" int mvpb_sur_destroy(mvpb_sur net) {
  if (!net) return MVPB_OK;
  mvpb_ctx ctx = net->ctx;
  (void)hipSetDevice(ctx_device(ctx));
  (void)hipStreamSynchronize(net->st);
  delete net;
  ctx_release_child(ctx);
  return MVPB_OK;
}

extern "C" int mvpb_sur_n_params(mvpb_sur net, int *n) {
  if (!net || !n) return set_error(MVPB_E_INVALID, "NULL argument");
  *n = net->n_params;
  return MVPB_OK;
}

extern "C" int mvpb_sur_get_params(mvpb_sur net, float *host) {
  if (!net || !host) return set_error(MVPB_E_INVALID, "NULL argument");
  (void)hipSetDevice(ctx_device(net->ctx));
  hipError_t e = hipMemcpyAsync(host, net->params.p, sizeof(float) * net->n_params, hipMemcpyDeviceToHost, net->st);
  if (e == hipSuccess) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "get params: %s", hipGetErrorString(e));
  return MVPB_OK;
}

extern "C" int mvpb_sur_set_params(mvpb_sur net, const float *host) {
  if (!net || !host) return set_error(MVPB_E_INVALID, "NULL argument");
  for (int i = 0; i < net->n_params; ++i)
    if (!isfinite(host[i])) return set_error(MVPB_E_INVALID, "non-finite parameter %d", i);
  (void)hipSetDevice(ctx_device(net->ctx));
  hipError_t e = hipMemcpyAsync(net->params.p, host, sizeof(float) * net->n_params, hipMemcpyHostToDevice, net->st);
  if (e == hipSuccess) e = hipMemsetAsync(net->m.p, 0, sizeof(float) * net->n_params, net->st);
  if (e == hipSuccess) e = hipMemsetAsync(net->v.p, 0, sizeof(float) * net->n_params, net->st);
  if (e == hipSuccess) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "set params: %s", hipGetErrorString(e));
  net->step = 0;
  return MVPB_OK;
}

static int check_batch(mvpb_sur net, int B, const void *cells) {
  if (!net || !cells) return set_error(MVPB_E_INVALID, "NULL argument");
  if (B < 1 || B > net->max_batch) return set_error(MVPB_E_INVALID, "batch %d outside [1, %d]", B, net->max_batch);
  return MVPB_OK;
}

extern "C" int mvpb_sur_infer(mvpb_sur net, int batch, const uint8_t *cells, float *out, unsigned flags) {
  int rc = check_batch(net, batch, cells);
  if (rc) return rc;
  if (!out) return set_error(MVPB_E_INVALID, "NULL output");
  (void)hipSetDevice(ctx_device(net->ctx));
  const uint8_t *cells_dev = nullptr;
  rc = stage_inputs(net, batch, cells, nullptr, flags, !net->bf16, &cells_dev, nullptr);
  if (!rc) rc = sur_forward(net, batch, cells_dev, false);
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(out, net->out.p, sizeof(float) * batch * kOut,
                                (flags & MVPB_F_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, net->st);
  if (e == hipSuccess && !(flags & MVPB_F_ASYNC)) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "infer: %s", hipGetErrorString(e));
  return MVPB_OK;
}

extern "C" int mvpb_sur_gradients(mvpb_sur net, int batch, const uint8_t *cells, const float *target, float *loss,
                                  float *grads, unsigned flags) {
  int rc = check_batch(net, batch, cells);
  if (rc) return rc;
  if (!target || !grads) return set_error(MVPB_E_INVALID, "NULL argument");
  (void)hipSetDevice(ctx_device(net->ctx));
  const float *tgt = nullptr;
  const uint8_t *cells_dev = nullptr;
  rc = stage_inputs(net, batch, cells, target, flags, true, &cells_dev, &tgt);
  if (!rc) rc = sur_forward(net, batch, cells_dev, true);
  if (!rc) rc = loss_and_grad_out(net, batch, tgt);
  if (!rc) rc = sur_backward(net, batch);
  if (!rc) rc = loss_read(net, batch, loss);
  if (rc) return rc;
  hipError_t e = hipMemcpyAsync(grads, net->grads.p, sizeof(float) * net->n_params,
                                (flags & MVPB_F_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, net->st);
  if (e == hipSuccess) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "gradients: %s", hipGetErrorString(e));
  return MVPB_OK;
}

extern "C" int mvpb_sur_train_step(mvpb_sur net, int batch, const uint8_t *cells, const float *target, float lr,
                                   float *loss, unsigned flags) {
  int rc = check_batch(net, batch, cells);
  if (rc) return rc;
  if (!target) return set_error(MVPB_E_INVALID, "NULL target");
  if (!(lr > 0.f) || !isfinite(lr)) return set_error(MVPB_E_INVALID, "learning rate must be positive");
  (void)hipSetDevice(ctx_device(net->ctx));
  const float *tgt = nullptr;
  const uint8_t *cells_dev = nullptr;
  rc = stage_inputs(net, batch, cells, target, flags, true, &cells_dev, &tgt);
  if (!rc) rc = sur_forward(net, batch, cells_dev, true);
  if (!rc) rc = loss_and_grad_out(net, batch, tgt);
  if (!rc) rc = sur_backward(net, batch);
  if (rc) return rc;
  net->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, (float)net->step), c2 = 1.f - powf(b2, (float)net->step);
  hipLaunchKernelGGL(adam_step, dim3((net->n_params + 255) / 256), dim3(256), 0, net->st, net->params.p, net->grads.p,
                     net->m.p, net->v.p, net->n_params, lr, b1, b2, 1e-8f, c1, c2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "adam: %s", hipGetErrorString(e));
  return loss_read(net, batch, loss);
}

// ---------------------------------------------------------------------------
// Checkpoints: header, then the parameters and both Adam moments (FP32,
// little-endian as in memory).
// ---------------------------------------------------------------------------
namespace {
struct SurHeader {
  char magic[8];          // "MVPBSUR1"
  int32_t version;        // 1
  int32_t n_params;
  int32_t precision;      // 0 FP32, 1 BF16 products
  int32_t reserved;
  int64_t step;           // Adam steps taken (bias-correction counter)
  uint64_t seed;          // initialisation seed of the network
};
const char kSurMagic[8] = {'M', 'V', 'P', 'B', 'S', 'U', 'R', '1'};
}  // namespace

extern "C" int mvpb_sur_save(mvpb_sur net, const char *path) {
  if (!net || !path) return set_error(MVPB_E_INVALID, "NULL argument");
  (void)hipSetDevice(ctx_device(net->ctx));
  const size_t n = (size_t)net->n_params;
  std::vector<float> buf(3 * n);
  hipError_t e = hipMemcpyAsync(buf.data(), net->params.p, sizeof(float) * n, hipMemcpyDeviceToHost, net->st);
  if (e == hipSuccess) e = hipMemcpyAsync(buf.data() + n, net->m.p, sizeof(float) * n, hipMemcpyDeviceToHost, net->st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(buf.data() + 2 * n, net->v.p, sizeof(float) * n, hipMemcpyDeviceToHost, net->st);
  if (e == hipSuccess) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) return set_error(MVPB_E_DEVICE, "save: %s", hipGetErrorString(e));
  SurHeader h{};
  memcpy(h.magic, kSurMagic, 8);
  h.version = 1;
  h.n_params = net->n_params;
  h.precision = net->bf16 ? 1 : 0;
  h.step = net->step;
  h.seed = net->seed;
  FILE *f = fopen(path, "wb");
  if (!f) return set_error(MVPB_E_INVALID, "cannot open %s for writing", path);
  const bool ok = fwrite(&h, sizeof h, 1, f) == 1 && fwrite(buf.data(), sizeof(float), 3 * n, f) == 3 * n;
  const bool closed = fclose(f) == 0;
  if (!ok || !closed) return set_error(MVPB_E_INVALID, "write to %s failed", path);
  return MVPB_OK;
}

extern "C" int mvpb_sur_load(mvpb_ctx ctx, const char *path, int max_batch, mvpb_sur *out) {
  if (!ctx || !path || !out) return set_error(MVPB_E_INVALID, "NULL argument");
  FILE *f = fopen(path, "rb");
  if (!f) return set_error(MVPB_E_INVALID, "cannot open %s", path);
  SurHeader h{};
  std::vector<float> buf;
  bool ok = fread(&h, sizeof h, 1, f) == 1 && memcmp(h.magic, kSurMagic, 8) == 0 && h.version == 1 &&
            (h.precision == 0 || h.precision == 1) && h.step >= 0;
  int off[12];
  ok = ok && h.n_params == param_offsets(off);
  if (ok) {
    buf.resize(3 * (size_t)h.n_params);
    ok = fread(buf.data(), sizeof(float), buf.size(), f) == buf.size();
    char extra;
    ok = ok && fread(&extra, 1, 1, f) == 0;   // nothing after the moments
  }
  fclose(f);
  if (!ok) return set_error(MVPB_E_INVALID, "%s is not a surrogate checkpoint of this network", path);
  for (float x : buf)
    if (!isfinite(x)) return set_error(MVPB_E_INVALID, "%s holds non-finite values", path);
  mvpb_sur net = nullptr;
  int rc = mvpb_sur_create(ctx, max_batch, h.precision, h.seed, &net);
  if (rc) return rc;
  const size_t n = (size_t)h.n_params;
  hipError_t e = hipMemcpyAsync(net->params.p, buf.data(), sizeof(float) * n, hipMemcpyHostToDevice, net->st);
  if (e == hipSuccess) e = hipMemcpyAsync(net->m.p, buf.data() + n, sizeof(float) * n, hipMemcpyHostToDevice, net->st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(net->v.p, buf.data() + 2 * n, sizeof(float) * n, hipMemcpyHostToDevice, net->st);
  if (e == hipSuccess) e = hipStreamSynchronize(net->st);
  if (e != hipSuccess) {
    mvpb_sur_destroy(net);
    return set_error(MVPB_E_DEVICE, "load: %s", hipGetErrorString(e));
  }
  net->step = h.step;
  *out = net;
  return MVPB_OK;
}
