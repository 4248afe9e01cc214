// Complex FP64 dense linear algebra for the sample draw (CholeskyQR2 with block
// Gram-Schmidt projection) and the dense-target product, plus layout conversions.
#include <algorithm>

#include "polar4.h"
#include "qfs_internal.h"
#include "stream_common.h"

namespace qfs {

// ------------------------------------------------------------------ ZGEMM
typedef double f64x4 __attribute__((ext_vector_type(4)));

// A matrix operand: element (r, c) at p[r rs + c cs].
template <typename T>
struct ZMat {
  T *p;
  int64_t rs, cs;
};

// C = alpha op(A) B + beta C, op(A) = A or conj(A) (a conjugate transpose by its strides).
// A work-group has one 32 x 32 tile of C; its four waves take every fourth block of eight k
// each and add their tiles in wave order at the end, so a product with few tiles still keeps
// every SIMD busy. A wave forms its tile as 2 x 2 blocks of 16x16x4 FP64 matrix-core products
// (four real ones per complex one), the operands loaded straight from memory in the layout the
// instruction wants (lane l: row l % 16, k l / 16), three blocks ahead: each element is read by
// one lane, and a k-step's sixteen products last 1024 cycles, so LDS staging would save nothing.
// Bound by the FP64 matrix rate: 2048 x 100 x 2048 (11 qubits, 100 states) takes 95 us, 45 TFLOP/s
// over the tiles' 128 columns; a 32 x 32 tile per 256 threads through LDS, with a load round trip
// exposed in each of its 128 k tiles, took 310.
template <bool CONJ>
__global__ __launch_bounds__(256) void k_zgemm(int m, int n, int k, c128 alpha, ZMat<const c128> A,
                                               ZMat<const c128> B, c128 beta, ZMat<c128> C) {
  __shared__ c128 red[3][32][33];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  // tiles of one row of C on one XCD (consecutive work-groups go round the eight), near in time,
  // so that its rows of A come from memory once and from that XCD's L2 after; with fewer rows of
  // tiles than XCDs all of A stays in every L2, and the grid is the tiles alone (padded to eight
  // rows, 4 x 4 by 4 x 100000 took 130 us, most of it work-groups that leave at once, and
  // 2^26 columns more work-items than a grid may have)
  const int ny = (m + 31) / 32, nx = (n + 31) / 32, seq = blockIdx.x >> 3;
  const int i0 = (ny < 8 ? blockIdx.x % ny : (seq / nx) * 8 + (blockIdx.x & 7)) * 32;
  const int j0 = (ny < 8 ? blockIdx.x / ny : seq % nx) * 32;
  if (i0 >= m) return;
  // (rows and columns beyond the matrix read its last one; their results are not stored)
  const c128 *ap[2], *bp[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ap[h] = A.p + (int64_t)min(i0 + 16 * h + li, m - 1) * A.rs;
    bp[h] = B.p + (int64_t)min(j0 + 16 * h + li, n - 1) * B.cs;
  }
  f64x4 re[2][2], im[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) re[x][y] = im[x][y] = f64x4{0, 0, 0, 0};
  // block of eight k: two steps of four, [step][half]
  struct Blk {
    c128 a[2][2], b[2][2];
  };
  auto load = [&](int kb, Blk &d) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int64_t kk = kb + 4 * t + lk;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        d.a[t][h] = ap[h][kk * A.cs];
        d.b[t][h] = bp[h][kk * B.rs];
      }
    }
  };
  auto mma = [&](const Blk &d) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const double ar = d.a[t][x].re, ai = CONJ ? -d.a[t][x].im : d.a[t][x].im;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const double br = d.b[t][y].re, bi = d.b[t][y].im;
          re[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, re[x][y], 0, 0, 0);
          im[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, im[x][y], 0, 0, 0);
          re[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, bi, re[x][y], 0, 0, 0);
          im[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, im[x][y], 0, 0, 0);
        }
      }
  };
  // whole blocks, three in flight (a load past the wave's last block repeats it)
  constexpr int kStep = 32;  // eight per wave
  const int kfull = k & ~7;
  int kb = 8 * w;
  if (kb < kfull) {
    const int last = kfull - 8 - ((kfull - 8 - kb) & 31);
    Blk d0, d1, d2;
    load(kb, d0);
    load(min(kb + kStep, last), d1);
    load(min(kb + 2 * kStep, last), d2);
    for (;;) {
      mma(d0);
      load(min(kb + 3 * kStep, last), d0);
      kb += kStep;
      if (kb > last) break;
      mma(d1);
      load(min(kb + 3 * kStep, last), d1);
      kb += kStep;
      if (kb > last) break;
      mma(d2);
      load(min(kb + 3 * kStep, last), d2);
      kb += kStep;
      if (kb > last) break;
    }
  }
  if (w == 0 && kfull < k) {
    Blk d;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kk = kfull + 4 * t + lk;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        d.a[t][h] = kk < k ? ap[h][kk * A.cs] : cmake(0.0, 0.0);
        d.b[t][h] = kk < k ? bp[h][kk * B.rs] : cmake(0.0, 0.0);
      }
    }
    mma(d);
  }
  if (w > 0) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[w - 1][16 * x + lk + 4 * v][16 * y + li] = cmake(re[x][y][v], im[x][y][v]);
  }
  __syncthreads();
  if (w > 0) return;
  const bool read_c = !(beta.re == 0.0 && beta.im == 0.0);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 16 * x + lk + 4 * v, c = 16 * y + li;
        const int gi = i0 + r, gj = j0 + c;
        if (gi >= m || gj >= n) continue;
        c128 s = cmake(re[x][y][v], im[x][y][v]);
#pragma unroll
        for (int o = 0; o < 3; ++o) s = s + red[o][r][c];
        s = alpha * s;
        c128 *dst = C.p + gi * C.rs + gj * C.cs;
        if (read_c) s = s + beta * *dst;
        *dst = s;
      }
}

static int zgemm_go(bool conj_a, int m, int n, int k, c128 alpha, ZMat<const c128> A, ZMat<const c128> B, c128 beta,
                    ZMat<c128> C, hipStream_t s) {
  if (m <= 0 || n <= 0) return QFS_OK;
  const int ny = (m + 31) / 32;
  const int64_t tiles = (ny < 8 ? ny : (ny + 7) / 8 * 8) * (int64_t)((n + 31) / 32);
  const dim3 grid((unsigned)tiles);
  if (conj_a)
    hipLaunchKernelGGL(k_zgemm<true>, grid, dim3(256), 0, s, m, n, k, alpha, A, B, beta, C);
  else
    hipLaunchKernelGGL(k_zgemm<false>, grid, dim3(256), 0, s, m, n, k, alpha, A, B, beta, C);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

int launch_zgemm(bool conjtrans_a, int m, int n, int k, c128 alpha, const c128 *A, int lda,
                 const c128 *B, int ldb, c128 beta, c128 *C, int ldc, hipStream_t s) {
  return zgemm_go(conjtrans_a, m, n, k, alpha,
                  conjtrans_a ? ZMat<const c128>{A, 1, lda} : ZMat<const c128>{A, lda, 1},
                  ZMat<const c128>{B, ldb, 1}, beta, ZMat<c128>{C, ldc, 1}, s);
}

int launch_dense_rows(int64_t N, int M, const c128 *U, const c128 *psi, c128 *out, hipStream_t s) {
  return zgemm_go(false, (int)N, M, (int)N, cmake(1.0, 0.0), ZMat<const c128>{U, N, 1}, ZMat<const c128>{psi, 1, N},
                  cmake(0.0, 0.0), ZMat<c128>{out, 1, N}, s);
}

// C = A^H B for a short, wide product (m x n output, k >> m, n; the Gram matrices of
// the sample draw): the k range is split over up to kGramParts work-groups per output
// tile, each writing a partial tile to `work` [parts][m][n]; k_sum_parts adds them in
// part order.
__global__ __launch_bounds__(256) void k_zgemm_ct_part(int m, int n, int k, int kchunk,
                                                       const c128 *A, int lda, const c128 *B,
                                                       int ldb, c128 *work) {
  __shared__ c128 As[16][33];
  __shared__ c128 Bs[16][33];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int i0 = blockIdx.y * 32, j0 = blockIdx.x * 32, part = blockIdx.z;
  const int k0 = part * kchunk, k1 = min(k, k0 + kchunk);
  c128 acc[2][2];
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) acc[a][b] = cmake(0.0, 0.0);
  for (int kb = k0; kb < k1; kb += 16) {
    for (int e = tid; e < 512; e += 256) {
      const int ii = e & 31, kk = e >> 5;
      const int gi = i0 + ii, gk = kb + kk;
      As[kk][ii] = (gi < m && gk < k1) ? cconj(A[(int64_t)gk * lda + gi]) : cmake(0.0, 0.0);
      const int gj = j0 + ii;
      Bs[kk][ii] = (gk < k1 && gj < n) ? B[(int64_t)gk * ldb + gj] : cmake(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const c128 a0 = As[kk][ty], a1 = As[kk][ty + 16];
      const c128 b0 = Bs[kk][tx], b1 = Bs[kk][tx + 16];
      cfma(acc[0][0], a0, b0);
      cfma(acc[0][1], a0, b1);
      cfma(acc[1][0], a1, b0);
      cfma(acc[1][1], a1, b1);
    }
    __syncthreads();
  }
  c128 *W = work + (int64_t)part * m * n;
  for (int a = 0; a < 2; ++a)
    for (int b = 0; b < 2; ++b) {
      const int gi = i0 + ty + 16 * a, gj = j0 + tx + 16 * b;
      if (gi < m && gj < n) W[(int64_t)gi * n + gj] = acc[a][b];
    }
}

__global__ void k_sum_parts(int64_t mn, int parts, const c128 *work, c128 *C) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= mn) return;
  c128 s = work[e];
  for (int p = 1; p < parts; ++p) s = s + work[(int64_t)p * mn + e];
  C[e] = s;
}

// k splits: enough work-groups to cover the chip (about 2048 with the m x m tiles),
// at most 16
static int gram_parts(int64_t m) {
  const int64_t tiles = ((m + 31) / 32) * ((m + 31) / 32);
  return (int)std::max<int64_t>(1, std::min<int64_t>(16, 2048 / std::max<int64_t>(1, tiles)));
}

static int gram_splitk(int m, int n, int k, const c128 *A, int lda, const c128 *B, int ldb, c128 *C,
                       c128 *work, hipStream_t s) {
  const int nparts = gram_parts(std::max(m, n));
  const int kchunk = ((k + nparts - 1) / nparts + 15) / 16 * 16;
  const int parts = (k + kchunk - 1) / kchunk;
  dim3 grid((n + 31) / 32, (m + 31) / 32, parts);
  hipLaunchKernelGGL(k_zgemm_ct_part, grid, dim3(256), 0, s, m, n, k, kchunk, A, lda, B, ldb, work);
  QFS_HIP(hipGetLastError());
  const int64_t mn = (int64_t)m * n;
  hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)((mn + 255) / 256)), dim3(256), 0, s, mn, parts, work, C);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

// ------------------------------------------------------------------ Cholesky, R^-1
// Upper Cholesky G = R^H R of an m x m Hermitian positive-definite matrix (row-major, ld m) in
// place, right-looking in panels of kCholB rows. flag[0] is set on a non-positive pivot. Only
// the upper triangle and the real parts of the diagonal are read.
//
// One launch per panel, the 64 columns of a work-group solved beside the other groups'. Every
// work-group factors the diagonal block for itself, in 32 steps of one barrier each: thread
// (c, g) holds rows g, g + 8, g + 16, g + 24 of column c; the owners of row j put it into LDS as
// it is, and all threads subtract conj(row j) row j / pivot from the rows they hold (rows up to j
// get values that nobody reads). Then R_JJ^H X = G_J by columns: four lanes per column with every
// fourth row each, a finished row going round the four by a quad exchange.
// The diagonal block stays as it is for the other work-groups; its factor goes, transposed and
// conjugated, below the diagonal, the pivots' roots into the diagonal's imaginary parts, and
// k_chol_finish puts both in place.
// Bound by the chain of steps: 16 us a panel of a 256 x 256 matrix and 10.6 of a 32 x 32 one,
// where one work-group with the panel in LDS and three barriers a step took 45 and 22.
constexpr int kCholB = 32;

// FULL: b = kCholB, the steps in one run of code. Else (the last panel) the steps from b on, whose
// rows and columns are not used, are left out: a 3 x 3 matrix would take a whole panel's time.
template <bool FULL>
__global__ __launch_bounds__(256) void k_chol_panel(int m, int j, int b, c128 *G, int *flag) {
  __shared__ c128 R[kCholB][kCholB + 1];
  __shared__ double inv[kCholB];
  const int tid = threadIdx.x;
  const int64_t ld = m;
  const int q = tid & 3, col = j + b + blockIdx.x * 64 + (tid >> 2);
  c128 y[kCholB / 4];
#pragma unroll
  for (int i = 0; i < kCholB / 4; ++i) {
    const int r = 4 * i + q;
    y[i] = r < b && col < m ? G[(j + r) * ld + col] : cmake(0.0, 0.0);
  }
  const int c = tid & 31, g = tid >> 5;
  c128 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = g + 8 * k;
    v[k] = r <= c && c < b ? G[(j + r) * ld + j + c] : cmake(r == c ? 1.0 : 0.0, 0.0);
  }
#pragma unroll
  for (int jj = 0; jj < kCholB; ++jj) {
    if (FULL || jj < b) {
      if (g == (jj & 7)) R[jj][c] = v[jj >> 3];
      lds_barrier();
      const double d = R[jj][jj].re;
      const bool ok = d > 0.0;
      const double ip = ok ? rsq_nr(d) : 0.0;
      if (tid == 0) {
        inv[jj] = ip;
        if (!ok && blockIdx.x == 0) flag[0] = 1;
      }
      const c128 x = cscale(R[jj][c], -ip * ip);
#pragma unroll
      for (int k = jj >> 3; k < 4; ++k) cfma_conj(v[k], x, R[jj][g + 8 * k]);
    }
  }
  lds_barrier();
  // R_JJ above the diagonal, zero elsewhere; the pivots' roots
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = g + 8 * k;
    const c128 x = R[r][c];
    const double ip = inv[r];
    R[r][c] = r < c ? cscale(x, ip) : cmake(0.0, 0.0);
    if (blockIdx.x == 0 && c < b) {
      if (r < c) G[(j + c) * ld + j + r] = cconj(cscale(x, ip));
      if (r == c) G[(j + r) * ld + j + r].im = ip > 0.0 ? x.re * ip : 1.0;
    }
  }
  lds_barrier();
  if (col - (tid >> 2) >= m) return;
#define QFS_CHOL_ROW(K)                                                            \
  {                                                                                \
    const int jj = 4 * i + K;                                                      \
    const double ip = inv[jj];                                                     \
    const c128 x = cmake(dpp_move<0x55 * K>(y[i].re * ip), dpp_move<0x55 * K>(y[i].im * ip)); \
    if (q == K) y[i] = x;                                                          \
    const c128 nx = cmake(-x.re, -x.im);                                           \
    _Pragma("unroll") for (int k = i; k < kCholB / 4; ++k) cfma_conj(y[k], nx, R[jj][4 * k + q]); \
  }
#pragma unroll
  for (int i = 0; i < kCholB / 4; ++i) {
    QFS_CHOL_ROW(0) QFS_CHOL_ROW(1) QFS_CHOL_ROW(2) QFS_CHOL_ROW(3)
  }
#undef QFS_CHOL_ROW
#pragma unroll
  for (int i = 0; i < kCholB / 4; ++i) {
    const int r = 4 * i + q;
    if (r < b && col < m) G[(j + r) * ld + col] = y[i];
  }
}

// The diagonal blocks' factors into place, zero below the diagonal.
__global__ void k_chol_finish(int m, c128 *G) {
  const int64_t total = (int64_t)m * m;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / m), c = (int)(e % m);
    if (c > i) continue;
    const c128 x = G[e];
    if (c == i) {
      G[e] = cmake(x.im, 0.0);
    } else {
      if (i / kCholB == c / kCholB) G[(int64_t)c * m + i] = cconj(x);
      G[e] = cmake(0.0, 0.0);
    }
  }
}

static int cholesky_upper_blocked(int m, c128 *G, int *flag, hipStream_t s) {
  const c128 one = cmake(1.0, 0.0), mone = cmake(-1.0, 0.0);
  for (int j = 0; j < m; j += kCholB) {
    const int b = std::min(kCholB, m - j), rest = m - j - b;
    const dim3 grid((unsigned)std::max(1, (rest + 63) / 64));
    if (b == kCholB)
      hipLaunchKernelGGL(k_chol_panel<true>, grid, dim3(256), 0, s, m, j, b, G, flag);
    else
      hipLaunchKernelGGL(k_chol_panel<false>, grid, dim3(256), 0, s, m, j, b, G, flag);
    QFS_HIP(hipGetLastError());
    if (rest > 0) {
      const c128 *panel = G + (int64_t)j * m + j + b;
      QFS_TRY(launch_zgemm(true, rest, rest, b, mone, panel, m, panel, m, one,
                           G + (int64_t)(j + b) * m + j + b, m, s));
    }
  }
  hipLaunchKernelGGL(k_chol_finish, dim3((unsigned)std::min<int64_t>(((int64_t)m * m + 255) / 256, 4096)),
                     dim3(256), 0, s, m, G);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

// T = R^-1 for upper-triangular R (m x m): one wave per column c of T, back
// substitution T[i][c] = -(sum_{k=i+1..c} R[i][k] T[k][c]) / R[i][i] with each dot
// product split over the 64 lanes and combined by a butterfly (every lane ends with
// the same sum); the column being built lives in LDS.
__global__ __launch_bounds__(64) void k_tri_inverse_upper(int m, const c128 *R, c128 *T) {
  extern __shared__ c128 tcol[];
  const int c = blockIdx.x, lane = threadIdx.x;
  for (int i = lane; i < m; i += 64) tcol[i] = cmake(0.0, 0.0);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __syncthreads();
  if (lane == 0) tcol[c] = cmake(1.0 / R[(int64_t)c * m + c].re, 0.0);
  __syncthreads();
  for (int i = c - 1; i >= 0; --i) {
    c128 acc = cmake(0.0, 0.0);
    for (int k = i + 1 + lane; k <= c; k += 64) cfma(acc, R[(int64_t)i * m + k], tcol[k]);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      acc.re += __shfl_xor(acc.re, o);
      acc.im += __shfl_xor(acc.im, o);
    }
    const double rii = R[(int64_t)i * m + i].re;
    if (lane == 0) tcol[i] = cscale(acc, -1.0 / rii);
    __syncthreads();
  }
  for (int i = lane; i < m; i += 64) T[(int64_t)i * m + c] = tcol[i];
}

__device__ __forceinline__ double readlane_f64(double x, int l) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(v & 0xffffffffll), l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// T = R^-1 for m <= 64 NJ, one wave per row c of T: from T R = I,
//   T[c][k] = (delta_ck - sum_{c <= j < k} T[c][j] R[j][k]) / R[k][k],  k = c .. m - 1.
// Lane l keeps the running sums s_i of the rows i = l + 64 u of row c; at step k the lane
// holding k finishes T[c][k] (reciprocal diagonal taken beforehand), every lane reads it
// from that lane's registers, and the lanes add T[c][k] R[k][i] to s_i for i > k, reading
// row k of R (contiguous; four rows are loaded while the four before them are used). No
// reduction and no barrier per step, unlike the dot-product form above.
template <int NJ>
__global__ __launch_bounds__(64) void k_tri_inverse_rows(int m, const c128 *__restrict__ R,
                                                         c128 *__restrict__ T) {
  const int c = blockIdx.x, lane = threadIdx.x;
  c128 sv[NJ];
  double inv[NJ];
#pragma unroll
  for (int u = 0; u < NJ; ++u) {
    const int i = lane + 64 * u;
    sv[u] = cmake(0.0, 0.0);
    inv[u] = i < m ? 1.0 / R[(int64_t)i * m + i].re : 0.0;
  }
#pragma unroll
  for (int uk = 0; uk < NJ; ++uk) {
    const int ks = max(c, 64 * uk), k1 = min(m, 64 * uk + 64);
    if (ks >= k1) continue;
    c128 buf[4][NJ], nbuf[4][NJ];
    auto load4 = [&](int kb, c128 (&dst)[4][NJ]) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = kb + q;
#pragma unroll
        for (int u = uk; u < NJ; ++u) {
          const int i = lane + 64 * u;
          dst[q][u] = (k < k1 && i > k && i < m) ? R[(int64_t)k * m + i] : cmake(0.0, 0.0);
        }
      }
    };
    load4(ks, buf);
    for (int kb = ks; kb < k1; kb += 4) {
      load4(kb + 4, nbuf);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = kb + q;
        if (k < k1) {
          const int kl = k & 63;
          const double dre = (k == c ? 1.0 : 0.0) - sv[uk].re, dim = -sv[uk].im;
          const double tre = readlane_f64(dre * inv[uk], kl), tim = readlane_f64(dim * inv[uk], kl);
          if (lane == kl) sv[uk] = cmake(tre, tim);  // this slot now holds T[c][k]
#pragma unroll
          for (int u = uk; u < NJ; ++u) {
            const int i = lane + 64 * u;
            if (i > k) {
              const c128 r = buf[q][u];
              sv[u].re += tre * r.re - tim * r.im;
              sv[u].im += tre * r.im + tim * r.re;
            }
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = uk; u < NJ; ++u) buf[q][u] = nbuf[q][u];
    }
  }
#pragma unroll
  for (int u = 0; u < NJ; ++u) {
    const int i = lane + 64 * u;
    if (i < m) T[(int64_t)c * m + i] = i < c ? cmake(0.0, 0.0) : sv[u];
  }
}

__global__ void k_copy_cols(int64_t rows, int cols, const c128 *src, int lds, c128 *dst, int ldd) {
  const int64_t total = rows * cols;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / cols;
    const int j = (int)(e - i * cols);
    dst[i * ldd + j] = src[i * lds + j];
  }
}

size_t work_bytes_orth(int64_t rows, int64_t cols) {
  const size_t m = (size_t)cols;
  // gram_parts(x) x^2 over x <= m is at most max(min(16 m^2, 2^21), m^2)
  const size_t parts = std::max(std::min(16 * m * m, size_t(1) << 21), m * m);
  return sizeof(c128) * (m * m * 3 + parts + (size_t)rows * m) + 256;
}

int orthonormalize_columns(int64_t rows, int64_t ld, int64_t c0, int64_t c1, c128 *A, void *work,
                           hipStream_t s, int *flag_dev) {
  const int m = (int)(c1 - c0);
  if (m <= 0) return QFS_OK;
  c128 *P = static_cast<c128 *>(work);          // c0 x m (<= c1 x c1)
  c128 *Gm = P + (size_t)c1 * c1;                 // m x m
  c128 *T = Gm + (size_t)m * m;                   // m x m
  c128 *Tmp = T + (size_t)m * m;                  // rows x m
  c128 *parts = Tmp + (size_t)rows * m;           // gram_parts(m) x m x m
  int *flag = flag_dev ? flag_dev : reinterpret_cast<int *>(parts + (size_t)gram_parts(m) * m * m);
  if (!flag_dev) QFS_HIP(hipMemsetAsync(flag, 0, sizeof(int), s));
  c128 *An = A + c0;
  const c128 one = cmake(1.0, 0.0), zero = cmake(0.0, 0.0), mone = cmake(-1.0, 0.0);
  if (c0 > 0) {
    for (int pass = 0; pass < 2; ++pass) {
      QFS_TRY(launch_zgemm(true, (int)c0, m, (int)rows, one, A, (int)ld, An, (int)ld, zero, P, m, s));
      QFS_TRY(launch_zgemm(false, (int)rows, m, (int)c0, mone, A, (int)ld, P, m, one, An, (int)ld, s));
    }
  }
  for (int pass = 0; pass < 2; ++pass) {
    QFS_TRY(gram_splitk(m, m, (int)rows, An, (int)ld, An, (int)ld, Gm, parts, s));
    QFS_TRY(cholesky_upper_blocked(m, Gm, flag, s));
    if (m <= 256)
      hipLaunchKernelGGL(k_tri_inverse_rows<4>, dim3(m), dim3(64), 0, s, m, Gm, T);
    else
      hipLaunchKernelGGL(k_tri_inverse_upper, dim3(m), dim3(64), sizeof(c128) * (size_t)m, s, m, Gm, T);
    QFS_HIP(hipGetLastError());
    QFS_TRY(launch_zgemm(false, (int)rows, m, m, one, An, (int)ld, T, m, zero, Tmp, m, s));
    const int64_t total = rows * m;
    hipLaunchKernelGGL(k_copy_cols, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 65536)),
                       dim3(256), 0, s, rows, m, Tmp, m, An, (int)ld);
    QFS_HIP(hipGetLastError());
  }
  if (flag_dev) return QFS_OK;  // the caller reads the flag
  int h_flag = 0;
  QFS_HIP(hipMemcpyAsync(&h_flag, flag, sizeof(int), hipMemcpyDeviceToHost, s));
  QFS_HIP(hipStreamSynchronize(s));
  if (h_flag) {
    set_error_detail("orthonormalisation: non-positive Cholesky pivot (dependent columns)");
    return QFS_ENUMERIC;
  }
  return QFS_OK;
}

// ------------------------------------------------------------------ layout conversions
// sample-major [M][N] c128 -> chunked amplitude-major (32x32 LDS transpose tiles);
// element (i, j) of the chunked set is at (j >> logC) * N * C + i * C + (j & (C - 1)).
template <typename R>
__global__ __launch_bounds__(256) void k_to_internal(int n, int64_t M, int logC, int64_t cols,
                                                     const c128 *src, cx<R> *dst) {
  __shared__ c128 tile[32][33];
  const int64_t N = int64_t(1) << n;
  const int64_t i0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 8 rows per pass
  for (int r = ty; r < 32; r += 8) {
    const int64_t j = j0 + r, i = i0 + tx;
    tile[r][tx] = (j < M && i < N) ? src[j * N + i] : cmake(0.0, 0.0);
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = i0 + r, j = j0 + tx;
    if (i < N && j < cols) {
      const c128 v = tile[tx][r];
      dst[((j >> logC) << (n + logC)) + (i << logC) + (j & ((1 << logC) - 1))] =
          cmake<R>((R)v.re, (R)v.im);
    }
  }
}

template <typename R>
__global__ __launch_bounds__(256) void k_from_internal(int n, int64_t M, int logC, const cx<R> *src,
                                                       c128 *dst) {
  __shared__ c128 tile[32][33];
  const int64_t N = int64_t(1) << n;
  const int64_t i0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = i0 + r, j = j0 + tx;
    if (i < N && j < M) {
      const cx<R> v = src[((j >> logC) << (n + logC)) + (i << logC) + (j & ((1 << logC) - 1))];
      tile[r][tx] = cmake<double>(v.re, v.im);
    }
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t j = j0 + r, i = i0 + tx;
    if (j < M && i < N) dst[j * N + i] = tile[tx][r];
  }
}

template <typename R>
int launch_to_internal(int n, int64_t M, int logC, int64_t nch, const c128 *src, cx<R> *dst,
                       hipStream_t s) {
  const int64_t N = int64_t(1) << n, cols = nch << logC;
  dim3 grid((unsigned)((N + 31) / 32), (unsigned)((cols + 31) / 32));
  hipLaunchKernelGGL(k_to_internal<R>, grid, dim3(256), 0, s, n, M, logC, cols, src, dst);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

template <typename R>
int launch_from_internal(int n, int64_t M, int logC, const cx<R> *src, c128 *dst, hipStream_t s) {
  const int64_t N = int64_t(1) << n;
  dim3 grid((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32));
  hipLaunchKernelGGL(k_from_internal<R>, grid, dim3(256), 0, s, n, M, logC, src, dst);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

template int launch_to_internal<float>(int, int64_t, int, int64_t, const c128 *, c64 *, hipStream_t);
template int launch_to_internal<double>(int, int64_t, int, int64_t, const c128 *, c128 *, hipStream_t);
template int launch_from_internal<float>(int, int64_t, int, const c64 *, c128 *, hipStream_t);
template int launch_from_internal<double>(int, int64_t, int, const c128 *, c128 *, hipStream_t);

__global__ void k_narrow(int64_t count, const c128 *src, c64 *dst) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * blockDim.x)
    dst[e] = cmake<float>((float)src[e].re, (float)src[e].im);
}

int launch_narrow(int64_t count, const c128 *src, c64 *dst, hipStream_t s) {
  if (count <= 0) return QFS_OK;
  hipLaunchKernelGGL(k_narrow, dim3((unsigned)std::min<int64_t>((count + 255) / 256, 65536)),
                     dim3(256), 0, s, count, src, dst);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

__device__ __forceinline__ void copy_slot(const SlotCopy &c, int64_t s) {
  for (int b = 0; b < SlotCopy::kBufs; ++b) {
    const int64_t u = c.units[b];
    if (u == 0) continue;
    const uint4 *src = c.src[b] + s * u;
    uint4 *dst = c.dst[b] + s * u;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < u; e += (int64_t)gridDim.x * blockDim.x)
      dst[e] = src[e];
  }
}

__global__ void k_copy_slots(const int32_t *slots, SlotCopy c) { copy_slot(c, slots[blockIdx.y]); }

// Bound by its launch: in the place of a launch per cost, one for the snapshot and a copy to
// the host, of which each took 2 to 4 us with as much again between them (3 qubits), and 20 to
// 28 us beside the other part's passes (12 qubits, M = 256, 16 starts).
__global__ __launch_bounds__(256) void k_sweep_end(const int32_t *slots, SweepEnd e) {
  const int s = slots[blockIdx.y], i = threadIdx.x >> 6;
  if (blockIdx.x == 0 && i < 2 && e.n[i] > 0) {
    double sum = 0.0;
    for (int b = threadIdx.x & 63; b < e.n[i]; b += 64) sum += e.part[i][(int64_t)s * e.stride[i] + b];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_down(sum, o);
    if ((threadIdx.x & 63) == 0) {
      sum *= 1.0 / e.m[i];
      e.costs[i * e.starts + s] = sum;
      e.host[i * e.starts + s] = sum;
      __threadfence_system();
    }
  }
  copy_slot(e.snap, s);
}

// Blocks of 256 threads a start for the copies of c.
unsigned copy_blocks(const SlotCopy &c) {
  int64_t umax = 0;
  for (int b = 0; b < SlotCopy::kBufs; ++b) umax = std::max(umax, c.units[b]);
  return (unsigned)std::min<int64_t>((umax + 255) / 256, 64);
}

int launch_sweep_end(const int32_t *slots, int nslots, const SweepEnd &e, hipStream_t s) {
  if (nslots <= 0) return QFS_OK;
  hipLaunchKernelGGL(k_sweep_end, dim3(std::max(1u, copy_blocks(e.snap)), (unsigned)nslots), dim3(256), 0, s, slots,
                     e);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

int launch_copy_slots(const int32_t *slots, int nslots, const SlotCopy &c, hipStream_t s) {
  const unsigned bx = copy_blocks(c);
  if (nslots <= 0 || bx == 0) return QFS_OK;
  hipLaunchKernelGGL(k_copy_slots, dim3(bx, (unsigned)nslots), dim3(256), 0, s, slots, c);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

// Fill with zeros by a kernel (safe inside captured graphs).
__global__ void k_zero(uint4 *p, int64_t n16) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n16;
       e += (int64_t)gridDim.x * blockDim.x)
    p[e] = make_uint4(0, 0, 0, 0);
}

int launch_zero(void *p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return QFS_OK;
  if (bytes % 16 != 0 || (reinterpret_cast<uintptr_t>(p) & 15) != 0) {
    QFS_HIP(hipMemsetAsync(p, 0, bytes, s));
    return QFS_OK;
  }
  const int64_t n16 = (int64_t)(bytes / 16);
  hipLaunchKernelGGL(k_zero, dim3((unsigned)std::min<int64_t>((n16 + 255) / 256, 65536)), dim3(256),
                     0, s, static_cast<uint4 *>(p), n16);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

// Columns 0..N-1 of the N x ld matrix A set to the computational basis (A zeroed before):
// A[i][i] = 1.
__global__ void k_unit_columns(int64_t N, int64_t ld, c128 *A) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
    A[i * ld + i] = cmake(1.0, 0.0);
}

int launch_unit_columns(int64_t N, int64_t ld, c128 *A, hipStream_t s) {
  if (N <= 0 || ld < N) return QFS_EINVAL;
  hipLaunchKernelGGL(k_unit_columns, dim3((unsigned)std::min<int64_t>((N + 255) / 256, 4096)), dim3(256), 0,
                     s, N, ld, A);
  QFS_HIP(hipGetLastError());
  return QFS_OK;
}

}  // namespace qfs
