// P_C by an explicit inverse for small meshes.  K is constant over the DD
// iterations (Section 2: the paper factorises it once); for up to kDenseMaxDof
// DOFs its inverse is formed once on the GPU and kept per (mesh, Dirichlet
// pattern) on the dataset, and every P_C is then one product of K^-1 with the
// two right-hand sides (E and S of eqs. "KuE", "KeS") -- a stream of n^2
// doubles instead of hundreds of CG iterations.
//
// Inversion.  The nodes are numbered plane by plane and an element joins two
// neighbouring planes, so K is block tridiagonal in groups of planes (diagonal
// blocks A_k, subdiagonal blocks B_k) and symmetric positive definite (with
// identity rows and columns at Dirichlet DOFs).  With the Schur complements
// S_0 = A_0, S_{k+1} = A_{k+1} - L_k B_k^T, L_k = B_k S_k^-1, the inverse X
// follows from its last block upwards:
//   X_{P P} = S_P^-1,  X_{k j} = -L_k^T X_{k+1 j} (j > k),
//   X_{k k} = S_k^-1 - X_{k k+1} L_k,  X_{j k} = X_{k j}^T,
// in place (S_k^-1 and L_k stand where X_{k k} and X_{k+1 k} come to stand).
// That is n^2 b operations with blocks of b DOFs instead of the 2 n^3 of an
// elimination that does not see the band (16^3 elements: n = 14739, b = 867).
// The products are FP64 MFMA tiles; the diagonal blocks are inverted by blocked
// Gauss-Jordan without pivoting on a copy padded to a multiple of 64 with
// identity.  For each 64-block k of it:
//   A_kk <- A_kk^-1;  A_ik <- -A_ik A_kk (i != k);  A_ij <- A_ij + A_ik A_kj
//   (i, j != k);  A_kj <- A_kk A_kj (j != k).
// Measured, 16^3 elements, whole formation: 27 ms (430 ms by Gauss-Jordan over
// the whole matrix on the vector FP64 units, the trailing updates 375 of them,
// and the matrix assembled on the host).  What is left is the chain of 238
// diagonal 64-blocks, each waiting for the one before.
#include <algorithm>
#include <cstring>
#include <list>
#include <memory>
#include <mutex>
#include <vector>

#include "solve.h"

namespace dd {

namespace {

constexpr int kB = 64;   // block size of the Gauss-Jordan sweep

struct MeshDims {
  int nx, ny, nz;
};

// Rows of one block of K (DOFs row0 .. row0 + rows - 1) from the element
// stiffness Ke: the columns of the same block to W (leading dimension ldw) and
// those of the block before (DOFs prev0 ..) to B (ldb).  One thread per (row,
// neighbouring node); W and B start at zero.  An entry sums the elements that
// share both nodes in element order.  Dirichlet rows and columns are those of
// the identity.
__global__ __launch_bounds__(256) void assemble_block_kernel(
    MeshDims d, const double* __restrict__ Ke, const uint8_t* __restrict__ mask, int64_t row0,
    int64_t rows, int64_t prev0, double* __restrict__ W, int64_t ldw, double* __restrict__ B,
    int64_t ldb) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= 27 * rows) return;
  const int64_t lr = id / 27, row = row0 + lr;
  const int nb = (int)(id - 27 * lr);
  const int comp = (int)(row % 3);
  const int64_t nd = row / 3;
  const int sx = d.nx + 1, sy = d.ny + 1;
  const int i = (int)(nd % sx), j = (int)((nd / sx) % sy), k = (int)(nd / ((int64_t)sx * sy));
  const int ii = i + nb % 3 - 1, jj = j + (nb / 3) % 3 - 1, kk = k + nb / 9 - 1;
  if (ii < 0 || jj < 0 || kk < 0 || ii > d.nx || jj > d.ny || kk > d.nz) return;
  if (mask[row]) {
    if (nb == 13) W[lr * ldw + lr] = 1.0;
    return;
  }
  const int64_t col0 = 3 * (ii + (int64_t)sx * (jj + (int64_t)sy * kk));
  double s[3] = {0.0, 0.0, 0.0};
  for (int ez = max(k, kk) - 1; ez <= min(k, kk); ++ez)
    for (int ey = max(j, jj) - 1; ey <= min(j, jj); ++ey)
      for (int ex = max(i, ii) - 1; ex <= min(i, ii); ++ex) {
        if (ex < 0 || ey < 0 || ez < 0 || ex >= d.nx || ey >= d.ny || ez >= d.nz) continue;
        const int a = (i - ex) + 2 * (j - ey) + 4 * (k - ez);
        const int b = (ii - ex) + 2 * (jj - ey) + 4 * (kk - ez);
        for (int c = 0; c < 3; ++c) s[c] += Ke[24 * (3 * a + comp) + 3 * b + c];
      }
  for (int c = 0; c < 3; ++c) {
    const int64_t col = col0 + c;
    if (mask[col] || col >= row0 + rows) continue;   // the next block's columns are its own
    if (col >= row0)
      W[lr * ldw + (col - row0)] = s[c];
    else
      B[lr * ldb + (col - prev0)] = s[c];
  }
}

__global__ void identity_kernel(double* __restrict__ B, int64_t b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < b * b) B[i] = i / b == i % b ? 1.0 : 0.0;
}

__global__ void pad_identity_kernel(double* __restrict__ W, int64_t n, int64_t n_pad) {
  const int64_t r = n + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n_pad) W[r * n_pad + r] = 1.0;
}

// ---------------------------------------------------------------------------
// C = beta C + alpha op(A) op(B) in FP64 MFMA (v_mfma_f64_16x16x4: A lane
// supplies row lane % 16, k = lane / 16; B the same of its column; D register i
// holds row lane / 16 + 4 i of column lane % 16).  Row-major, any sizes; a
// workgroup computes a 64 x 64 tile, a wavefront 32 x 32 of it, in steps of 16
// along K staged through LDS as [k][row] and [k][column], the next step's
// operands loaded while the current one is multiplied.
// ---------------------------------------------------------------------------
constexpr int kGT = 64, kGK = 16, kGLd = kGT + 2;

template <bool TA, bool TB>
__global__ __launch_bounds__(256) void gemm64_kernel(int64_t m, int64_t n, int64_t kdim, double alpha,
                                                     const double* __restrict__ A, int64_t lda,
                                                     const double* __restrict__ B, int64_t ldb,
                                                     double beta, double* __restrict__ C, int64_t ldc) {
  __shared__ double as[2][kGK][kGLd], bs[2][kGK][kGLd];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * kGT, j0 = (int64_t)blockIdx.y * kGT;
  double ra[4], rb[4];
  // element v of the step's 64 x 16 operand: along K where K is contiguous
  // (op(A) = A, op(B) = B^T), else along the rows or columns
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = t + 256 * v;
      const int ka = TA ? e / kGT : e % kGK, ia = TA ? e % kGT : e / kGK;
      const bool in_a = i0 + ia < m && k0 + ka < kdim;
      ra[v] = in_a ? (TA ? A[(k0 + ka) * lda + i0 + ia] : A[(i0 + ia) * lda + k0 + ka]) : 0.0;
      const int kb = TB ? e % kGK : e / kGT, jb = TB ? e / kGK : e % kGT;
      const bool in_b = j0 + jb < n && k0 + kb < kdim;
      rb[v] = in_b ? (TB ? B[(j0 + jb) * ldb + k0 + kb] : B[(k0 + kb) * ldb + j0 + jb]) : 0.0;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = t + 256 * v;
      as[buf][TA ? e / kGT : e % kGK][TA ? e % kGT : e / kGK] = ra[v];
      bs[buf][TB ? e % kGK : e / kGT][TB ? e / kGK : e % kGT] = rb[v];
    }
  };
  f64x4_t acc[2][2] = {};
  const int wi = 32 * (wave >> 1), wj = 32 * (wave & 1), c = lane & 15, q = lane >> 4;
  load(0);
  store(0);
  __syncthreads();
  int cur = 0;
  for (int64_t k0 = 0; k0 < kdim; k0 += kGK) {
    const bool more = k0 + kGK < kdim;
    if (more) load(k0 + kGK);
#pragma unroll
    for (int s = 0; s < kGK / 4; ++s) {
      double a[2], b[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        a[u] = as[cur][4 * s + q][wi + 16 * u + c];
        b[u] = bs[cur][4 * s + q][wj + 16 * u + c];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
          acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
    }
    if (more) store(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + wi + 16 * u + q + 4 * r, j = j0 + wj + 16 * v + c;
        if (i >= m || j >= n) continue;
        double* p = C + i * ldc + j;
        *p = beta == 0.0 ? alpha * acc[u][v][r] : fma(alpha, acc[u][v][r], beta * *p);
      }
}

template <bool TA, bool TB>
void gemm64(int64_t m, int64_t n, int64_t k, double alpha, const double* A, int64_t lda,
            const double* B, int64_t ldb, double beta, double* C, int64_t ldc, hipStream_t st) {
  if (m <= 0 || n <= 0) return;
  hipLaunchKernelGGL((gemm64_kernel<TA, TB>),
                     dim3((unsigned)((m + kGT - 1) / kGT), (unsigned)((n + kGT - 1) / kGT)), dim3(256),
                     0, st, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc);
}

// dst[j][i] = src[i][j] for i < rows, j < cols (32 x 32 tiles through LDS).
__global__ __launch_bounds__(256) void transpose_kernel(const double* __restrict__ src, int64_t lds_,
                                                        int64_t rows, int64_t cols,
                                                        double* __restrict__ dst, int64_t ldd) {
  __shared__ double s[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t i0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
  for (int r = ty; r < 32; r += 8)
    if (i0 + r < rows && j0 + tx < cols) s[r][tx] = src[(i0 + r) * lds_ + j0 + tx];
  __syncthreads();
  for (int r = ty; r < 32; r += 8)
    if (j0 + r < cols && i0 + tx < rows) dst[(j0 + r) * ldd + i0 + tx] = s[tx][r];
}

// Inverts the diagonal block [k0, k0+64)^2 in place (and copies it to Akk).
// Four lanes hold a row in registers (16 columns each); at each pivot its row
// goes to the others through LDS and its column through the lanes of a row, so
// a pivot is one barrier and 16 fused multiply-adds (all in LDS, with two
// barriers and 16 read-modify-writes per thread, a block took 152 us; this 28,
// and the division is not what it waits for).
__global__ __launch_bounds__(256) void gj_diag_kernel(double* __restrict__ A, int64_t n_pad,
                                                      int64_t k0, double* __restrict__ Akk) {
  __shared__ double rowp[2][kB];
  const int t = threadIdx.x, r = t >> 2, q = t & 3;   // row r, columns 16 q .. 16 q + 15
  double s[16];
  double* src = A + (k0 + r) * n_pad + k0 + 16 * q;
#pragma unroll
  for (int c = 0; c < 16; ++c) s[c] = src[c];
  for (int pq = 0; pq < 4; ++pq) {
#pragma unroll
    for (int pc = 0; pc < 16; ++pc) {
      const int p = 16 * pq + pc, buf = pc & 1;
      const double colv = __shfl(s[pc], (int)(threadIdx.x & 60) + pq);   // A[r][p]
      if (r == p) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          rowp[buf][16 * q + c] = s[c];
          s[c] = 0.0;   // the pivot row becomes d times itself
        }
      }
      __syncthreads();
      const double d = 1.0 / rowp[buf][p];
      const double f = r == p ? d : -colv * d;
#pragma unroll
      for (int c = 0; c < 16; ++c) s[c] = fma(f, rowp[buf][16 * q + c], s[c]);
      if (q == pq) s[pc] = f;   // the pivot column: d at the pivot, -A[r][p] d elsewhere
    }
  }
  double* out = Akk + r * kB + 16 * q;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    src[c] = s[c];
    out[c] = s[c];
  }
}

// Column panel: rows i outside the block, A[i, k] <- -A[i, k] Akk.  4 rows per block.
__global__ __launch_bounds__(256) void gj_col_kernel(double* __restrict__ A, int64_t n_pad,
                                                     int64_t k0, const double* __restrict__ Akk) {
  __shared__ double inv[kB][kB + 1];
  __shared__ double row[4][kB];
  const int t = threadIdx.x;
  for (int e = t; e < kB * kB; e += 256) inv[e / kB][e % kB] = Akk[e];
  const int ri = t / kB, c = t % kB;
  int64_t i = (int64_t)blockIdx.x * 4 + ri;      // index among rows outside the block
  if (i >= k0) i += kB;
  const bool v = i < n_pad;
  row[ri][c] = v ? A[i * n_pad + k0 + c] : 0.0;
  __syncthreads();
  if (!v) return;
  double acc = 0.0;
#pragma unroll 8
  for (int q = 0; q < kB; ++q) acc = fma(row[ri][q], inv[q][c], acc);
  A[i * n_pad + k0 + c] = -acc;
}

// Trailing update of one 64x64 tile outside block row/column k:
// A[I, J] += A[I, k] A[k, J], a wavefront 32 x 32 of it in FP64 MFMA.
__global__ __launch_bounds__(256) void gj_update_kernel(double* __restrict__ A, int64_t n_pad,
                                                        int64_t k0) {
  __shared__ double a[kB][kB + 2];   // [k][row] of A[I, k]
  __shared__ double b[kB][kB + 2];   // A[k, J]
  const int64_t nb = n_pad / kB;
  int64_t bi = blockIdx.x % (nb - 1), bj = blockIdx.x / (nb - 1);
  const int64_t kb = k0 / kB;
  if (bi >= kb) ++bi;
  if (bj >= kb) ++bj;
  const int64_t I0 = bi * kB, J0 = bj * kB;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int e = t; e < kB * kB; e += 256) {
    const int r = e / kB, c = e % kB;
    a[c][r] = A[(I0 + r) * n_pad + k0 + c];
    b[r][c] = A[(k0 + r) * n_pad + J0 + c];
  }
  const int wi = 32 * (wave >> 1), wj = 32 * (wave & 1), c = lane & 15, q = lane >> 4;
  f64x4_t acc[2][2];
  double* tile = A + (I0 + wi + q) * n_pad + J0 + wj + c;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[u][v][r] = tile[(16 * u + 4 * r) * n_pad + 16 * v];
  __syncthreads();
#pragma unroll 4
  for (int s = 0; s < kB / 4; ++s) {
    double av[2], bv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      av[u] = a[4 * s + q][wi + 16 * u + c];
      bv[u] = b[4 * s + q][wj + 16 * u + c];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
        acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[v], acc[u][v], 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) tile[(16 * u + 4 * r) * n_pad + 16 * v] = acc[u][v][r];
}

// Row panel: columns j outside the block, A[k, j] <- Akk A[k, j].  4 columns per block.
__global__ __launch_bounds__(256) void gj_row_kernel(double* __restrict__ A, int64_t n_pad,
                                                     int64_t k0, const double* __restrict__ Akk) {
  __shared__ double inv[kB][kB + 1];
  __shared__ double colv[4][kB];
  const int t = threadIdx.x;
  for (int e = t; e < kB * kB; e += 256) inv[e / kB][e % kB] = Akk[e];
  const int cj = t / kB, r = t % kB;
  int64_t j = (int64_t)blockIdx.x * 4 + cj;
  if (j >= k0) j += kB;
  const bool v = j < n_pad;
  colv[cj][r] = v ? A[(k0 + r) * n_pad + j] : 0.0;
  __syncthreads();
  if (!v) return;
  double acc = 0.0;
#pragma unroll 8
  for (int q = 0; q < kB; ++q) acc = fma(inv[r][q], colv[cj][q], acc);
  A[(k0 + r) * n_pad + j] = acc;
}

// x_s = K^-1 b_s for the two systems; one wavefront per row, fixed reduction order.
__global__ __launch_bounds__(256) void dense_apply_kernel(const double* __restrict__ inv,
                                                          int64_t n_pad, int64_t n,
                                                          const double* __restrict__ b,
                                                          double* __restrict__ x) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= n) return;
  const double* row = inv + r * n_pad;
  double a0 = 0.0, a1 = 0.0;
  // unrolled so that several iterations' loads are in flight; the FMA chain
  // keeps its order
#pragma unroll 8
  for (int64_t j = lane; j < n; j += 64) {
    const double k = row[j];
    a0 = fma(k, b[j], a0);
    a1 = fma(k, b[n + j], a1);
  }
  for (int off = 32; off > 0; off >>= 1) {
    a0 += __shfl_xor(a0, off);
    a1 += __shfl_xor(a1, off);
  }
  if (lane == 0) {
    x[r] = a0;
    x[n + r] = a1;
  }
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// In-place inverse of W (n x n, n a multiple of 64).
static void gauss_jordan(double* W, int64_t n, double* akk, hipStream_t st) {
  const int64_t nb = n / kB;
  for (int64_t k0 = 0; k0 < n; k0 += kB) {
    hipLaunchKernelGGL(gj_diag_kernel, dim3(1), dim3(256), 0, st, W, n, k0, akk);
    if (nb == 1) return;
    hipLaunchKernelGGL(gj_col_kernel, dim3(blocks_for(n - kB, 4)), dim3(256), 0, st, W, n, k0, akk);
    hipLaunchKernelGGL(gj_update_kernel, dim3((unsigned)((nb - 1) * (nb - 1))), dim3(256), 0, st, W, n,
                       k0);
    hipLaunchKernelGGL(gj_row_kernel, dim3(blocks_for(n - kB, 4)), dim3(256), 0, st, W, n, k0, akk);
  }
}

// Smallest block of planes: below it a block's launches cost more than the
// elimination saves.
constexpr int64_t kMinBlock = 256;

// Forms K^-1 (row-major, leading dimension n_pad) on st.
static dd_status form_inverse(const FEMesh& M, const double* Ke, const uint8_t* mask, DenseInverse& D,
                              hipStream_t st) {
  const int64_t n = M.n_dof, n_pad = (n + kB - 1) / kB * kB;
  D.n = n;
  D.n_pad = n_pad;
  DD_TRY(D.inv.alloc(sizeof(double) * (size_t)(n_pad * n_pad)));
  // blocks of whole planes
  const int64_t plane = 3 * (int64_t)(M.nx + 1) * (M.ny + 1);
  const int64_t per = std::max<int64_t>(1, (kMinBlock + plane - 1) / plane);
  std::vector<int64_t> off;
  for (int64_t k = 0; k <= M.nz; k += per) off.push_back(k * plane);
  if (off.size() > 1 && n - off.back() < per * plane) off.pop_back();   // a short last group joins
  int64_t P = (int64_t)off.size();
  off.push_back(n);
  int64_t bmax = 0;
  for (int64_t k = 0; k < P; ++k) bmax = std::max(bmax, off[k + 1] - off[k]);
  const int64_t wmax = (bmax + kB - 1) / kB * kB;
  // one block, or few so large that their three work blocks would take more than
  // half of the inverse's memory beside it: the whole matrix in place
  if (6 * wmax * wmax > n_pad * n_pad) P = 1;
  DevBuf wbuf, sbuf, bbuf, akk, dke, dmask;
  if (P > 1) {
    DD_TRY(wbuf.alloc(sizeof(double) * (size_t)(wmax * wmax)));
    DD_TRY(sbuf.alloc(sizeof(double) * (size_t)(wmax * wmax)));
    DD_TRY(bbuf.alloc(sizeof(double) * (size_t)(bmax * bmax)));
  }
  DD_TRY(akk.alloc(sizeof(double) * kB * kB));
  DD_TRY(dke.alloc(sizeof(double) * 24 * 24));
  DD_TRY(dmask.alloc((size_t)n));
  DD_HIP(hipMemcpyAsync(dke.p, Ke, sizeof(double) * 24 * 24, hipMemcpyHostToDevice, st));
  DD_HIP(hipMemcpyAsync(dmask.p, mask, (size_t)n, hipMemcpyHostToDevice, st));
  double *X = D.inv.as<double>(), *W = wbuf.as<double>(), *S = sbuf.as<double>(),
         *B = bbuf.as<double>();
  const MeshDims dims{M.nx, M.ny, M.nz};
  if (P == 1) {
    DD_HIP(hipMemsetAsync(X, 0, D.inv.bytes, st));
    hipLaunchKernelGGL(assemble_block_kernel, dim3(blocks_for(27 * n, 256)), dim3(256), 0, st, dims,
                       dke.as<double>(), dmask.as<uint8_t>(), (int64_t)0, n, (int64_t)0, X, n_pad,
                       (double*)nullptr, (int64_t)0);
    hipLaunchKernelGGL(pad_identity_kernel, dim3(1), dim3(64), 0, st, X, n, n_pad);
    gauss_jordan(X, n_pad, akk.as<double>(), st);
    DD_HIP(hipGetLastError());
    DD_HIP(hipStreamSynchronize(st));
    return DD_OK;
  }
  for (int64_t k = 0; k < P; ++k) {
    const int64_t o = off[k], b = off[k + 1] - o, w = (b + kB - 1) / kB * kB;
    const int64_t po = k ? off[k - 1] : 0, pb = k ? o - po : 0;
    DD_HIP(hipMemsetAsync(W, 0, sizeof(double) * (size_t)(w * w), st));
    if (k) DD_HIP(hipMemsetAsync(B, 0, sizeof(double) * (size_t)(b * pb), st));
    hipLaunchKernelGGL(assemble_block_kernel, dim3(blocks_for(27 * b, 256)), dim3(256), 0, st, dims,
                       dke.as<double>(), dmask.as<uint8_t>(), o, b, po, W, w, B, pb);
    if (w > b)
      hipLaunchKernelGGL(pad_identity_kernel, dim3(1), dim3(64), 0, st, W, b, w);
    if (k) {
      double* L = X + o * n_pad + po;   // L_{k-1}, where X_{k k-1} comes to stand
      gemm64<false, false>(b, pb, pb, 1.0, B, pb, X + po * n_pad + po, n_pad, 0.0, L, n_pad, st);
      gemm64<false, true>(b, b, pb, -1.0, L, n_pad, B, pb, 1.0, W, w, st);
    }
    DD_HIP(hipMemcpyAsync(S, W, sizeof(double) * (size_t)(w * w), hipMemcpyDeviceToDevice, st));
    gauss_jordan(W, w, akk.as<double>(), st);
    DD_HIP(hipMemcpy2DAsync(X + o * n_pad + o, sizeof(double) * n_pad, W, sizeof(double) * w,
                            sizeof(double) * b, (size_t)b, hipMemcpyDeviceToDevice, st));
    // one Newton step, X += X (I - S X), the residual in B: without it the errors
    // of the blocks add up along the planes (u of a 16^3 solve 5.7e-14 off the
    // 64-bit solution, 3.1e-14 with it, 2.8e-14 by Gauss-Jordan over the whole)
    hipLaunchKernelGGL(identity_kernel, dim3(blocks_for(b * b, 256)), dim3(256), 0, st, B, b);
    gemm64<false, false>(b, b, b, -1.0, S, w, X + o * n_pad + o, n_pad, 1.0, B, b, st);
    gemm64<false, false>(b, b, b, 1.0, W, w, B, b, 1.0, X + o * n_pad + o, n_pad, st);
    DD_HIP(hipGetLastError());
  }
  for (int64_t k = P - 2; k >= 0; --k) {
    const int64_t o = off[k], b = off[k + 1] - o, no = off[k + 1], nb = off[k + 2] - no;
    const double* L = X + no * n_pad + o;
    gemm64<true, false>(b, n - no, nb, -1.0, L, n_pad, X + no * n_pad + no, n_pad, 0.0,
                        X + o * n_pad + no, n_pad, st);
    gemm64<false, false>(b, b, nb, -1.0, X + o * n_pad + no, n_pad, L, n_pad, 1.0, X + o * n_pad + o,
                         n_pad, st);
    // the rows above are done: their transpose takes the place of L
    hipLaunchKernelGGL(transpose_kernel, dim3(blocks_for(b, 32), blocks_for(n - no, 32)), dim3(256), 0,
                       st, X + o * n_pad + no, n_pad, b, n - no, X + no * n_pad + o, n_pad);
    DD_HIP(hipGetLastError());
  }
  DD_HIP(hipStreamSynchronize(st));
  return DD_OK;
}

std::shared_ptr<DenseInverse> dense_inverse_cached(const Dataset& ds, const FEMesh& M,
                                                   const uint8_t* mask) {
  const int64_t n = M.n_dof;
  auto same = [&](const DenseInverse& d) {
    return d.nx == M.nx && d.ny == M.ny && d.nz == M.nz && d.hx == M.hx && d.hy == M.hy &&
           d.hz == M.hz && (int64_t)d.mask.size() == n &&
           std::memcmp(d.mask.data(), mask, (size_t)n) == 0;
  };
  std::lock_guard<std::mutex> lk(ds.cache_mu);
  for (auto it = ds.pc_cache.begin(); it != ds.pc_cache.end(); ++it) {
    if (same(**it)) {
      ds.pc_cache.splice(ds.pc_cache.begin(), ds.pc_cache, it);   // most recently used first
      return ds.pc_cache.front();
    }
  }
  return nullptr;
}

dd_status dense_inverse_for(const Dataset& ds, const FEMesh& M, const uint8_t* mask,
                            std::shared_ptr<DenseInverse>& out, hipStream_t st) {
  const int64_t n = M.n_dof;
  out = dense_inverse_cached(ds, M, mask);
  if (out) return DD_OK;
  auto d = std::make_shared<DenseInverse>();
  d->nx = M.nx;
  d->ny = M.ny;
  d->nz = M.nz;
  d->hx = M.hx;
  d->hy = M.hy;
  d->hz = M.hz;
  d->mask.assign(mask, mask + n);
  double Ke[24 * 24];
  element_stiffness(M, ds.C, Ke);
  DD_TRY(form_inverse(M, Ke, mask, *d, st));
  std::lock_guard<std::mutex> lk(ds.cache_mu);
  ds.pc_cache.push_front(d);
  int64_t bytes = 0;
  for (auto it = ds.pc_cache.begin(); it != ds.pc_cache.end();) {
    bytes += (int64_t)(*it)->inv.bytes;
    if (bytes > kDenseCacheBytes && it != ds.pc_cache.begin())
      it = ds.pc_cache.erase(it);   // solvers still using it hold their own reference
    else
      ++it;
  }
  out = d;
  return DD_OK;
}

dd_status dense_apply(const DenseInverse& D, const double* b, double* x, hipStream_t st) {
  hipLaunchKernelGGL(dense_apply_kernel, dim3(blocks_for(D.n, 4)), dim3(256), 0, st,
                     D.inv.as<double>(), D.n_pad, D.n, b, x);
  DD_HIP(hipGetLastError());
  return DD_OK;
}

}  // namespace dd
