// P_C by operators formed once.  K is constant over the DD iterations (Section 2:
// the paper factorises it once): for small meshes its inverse is formed on the
// GPU and kept per (mesh, Dirichlet pattern) on the dataset, and every P_C is then
// one product of K^-1 with the two right-hand sides (E and S of eqs. "KuE",
// "KeS") -- a stream of n^2 doubles instead of hundreds of CG iterations.  Larger
// meshes keep the block elimination of their node planes instead (below).
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
//   A_kk <- A_kk^-1;  A_kj <- A_kk A_kj (j != k);  A_ij <- A_ij - A_ik A_kj
//   (i, j != k);  A_ik <- -A_ik A_kk (i != k).
// Measured, 16^3 elements, whole formation (before the planes took that size): 27
// ms; 430 ms by Gauss-Jordan over the whole matrix on the vector FP64 units, the
// trailing updates 375 of them, and the matrix assembled on the host.  What is
// left is the chain of diagonal 64-blocks, each waiting for the one before; 11^3
// elements now take 8.1 ms (9.2 with four launches a block).
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
// those of the block before (DOFs prev0 ..) to B (ldb; null: left out).  One
// thread per (row, neighbouring node); W and B start at zero.  An entry sums the elements that
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
    else if (B)
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

struct Gemm {
  int64_t m, n, k;
  const double* A;
  int64_t lda;
  const double* B;
  int64_t ldb;
  double* C;
  int64_t ldc;
};
struct GemmPair {
  Gemm g[2];   // blockIdx.z
};

template <bool TA, bool TB>
__global__ __launch_bounds__(256) void gemm64_kernel(GemmPair G, double alpha, double beta) {
  const Gemm& g = G.g[blockIdx.z];
  const int64_t m = g.m, n = g.n, kdim = g.k, lda = g.lda, ldb = g.ldb, ldc = g.ldc;
  const double* __restrict__ A = g.A;
  const double* __restrict__ B = g.B;
  double* __restrict__ C = g.C;
  if ((int64_t)blockIdx.x * kGT >= m || (int64_t)blockIdx.y * kGT >= n) return;
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
  const GemmPair G = {{{m, n, k, A, lda, B, ldb, C, ldc}, {}}};
  hipLaunchKernelGGL((gemm64_kernel<TA, TB>),
                     dim3((unsigned)((m + kGT - 1) / kGT), (unsigned)((n + kGT - 1) / kGT)), dim3(256),
                     0, st, G, alpha, beta);
}

// C_s = beta C_s + alpha A_s B_s for the first `count` of the pair
void gemm64_pair(const GemmPair& G, int count, double alpha, double beta, hipStream_t st) {
  int64_t m = 0, n = 0;
  for (int s = 0; s < count; ++s) {
    m = std::max(m, G.g[s].m);
    n = std::max(n, G.g[s].n);
  }
  hipLaunchKernelGGL((gemm64_kernel<false, false>),
                     dim3((unsigned)((m + kGT - 1) / kGT), (unsigned)((n + kGT - 1) / kGT),
                          (unsigned)count),
                     dim3(256), 0, st, G, alpha, beta);
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

// The matrices (n x n, n a multiple of 64) that one Gauss-Jordan sweep inverts
// side by side, the inverse of each one's current diagonal block and the negated
// transpose [64][n] of the column of blocks that the step eliminates.
struct SweepPair {
  double* A[2];
  int64_t n[2];
  double* Akk[2];
  double* col[2];
};

// FP64 value of lane `from` (the same in every lane)
__device__ inline double lane_d(double v, int from) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, from);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), from);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// FP64 value of lane L of each row of 16 lanes
template <int L>
__device__ inline double row_d(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x150 + L, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x150 + L, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1 / x to rounding: the hardware's estimate and two Newton steps, shorter than
// the division in the chain of pivots
__device__ inline double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// Gauss-Jordan on a 16 x 16 block: lane 16 g + r holds columns 4 g .. 4 g + 3 of row r.
template <int P>
__device__ inline void pivot16(double (&v)[4], int r, int g) {
  if constexpr (P < 16) {
    constexpr int pg = P / 4, pe = P % 4;
    const double colv = __shfl(v[pe], 16 * pg + r);
    const double d = recip(lane_d(v[pe], 16 * pg + P));
    const double f = r == P ? d : -colv * d;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fma(f, row_d<P>(v[e]), r == P ? 0.0 : v[e]);
    if (g == pg) v[pe] = f;   // the pivot column: d at the pivot, -A[r][p] d elsewhere
    pivot16<P + 1>(v, r, g);
  }
}

// m <- m^-1, 64 x 64 in LDS, by a workgroup of 256.  Gauss-Jordan by blocks of 16:
// a wavefront inverts the diagonal block in registers (the pivot goes through
// scalar registers, its row along the lanes of 16), and the rest of a block step is
// FP64 MFMA, three barriers in all.  With a barrier and
// an LDS round trip for every pivot the 64 pivots took 28 us, 15 now.
constexpr int kMLd = kB + 2;
__device__ inline void invert64(double (*m)[kMLd]) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, c = lane & 15, q = lane >> 4;
  for (int s = 0; s < 4; ++s) {
    const int o = 16 * s, b = 16 * w;
    if (w == 0) {
      double v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = m[o + c][o + 4 * q + e];
      pivot16<0>(v, c, q);
#pragma unroll
      for (int e = 0; e < 4; ++e) m[o + c][o + 4 * q + e] = v[e];
    }
    __syncthreads();
    f64x4_t col = {}, row = {};
    double neg[4];   // - the old column block, as the update's left operand
    if (w != s) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double dl = m[o + c][o + 4 * k + q], dr = m[o + 4 * k + q][o + c];
        neg[k] = -m[b + c][o + 4 * k + q];
        row = __builtin_amdgcn_mfma_f64_16x16x4f64(dl, m[o + 4 * k + q][b + c], row, 0, 0, 0);
        col = __builtin_amdgcn_mfma_f64_16x16x4f64(neg[k], dr, col, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {   // only this wavefront reads these two blocks before the barrier
        m[o + q + 4 * r][b + c] = row[r];
        m[b + q + 4 * r][o + c] = col[r];
      }
    }
    __syncthreads();
    if (w != s) {
      f64x4_t acc[3];
      int at[3];   // the other three column blocks
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        at[u] = 16 * (u + (u >= s ? 1 : 0)) + c;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[u][r] = m[b + q + 4 * r][at[u]];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int u = 0; u < 3; ++u)
          acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(neg[k], m[o + 4 * k + q][at[u]], acc[u], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) m[b + q + 4 * r][at[u]] = acc[u][r];
    }
    __syncthreads();
  }
}

__device__ inline void store_akk(const double (*m)[kMLd], double* __restrict__ Akk) {
  for (int e = threadIdx.x; e < kB * kB; e += 256) Akk[e] = m[e / kB][e % kB];
}

// Akk <- inverse of the first diagonal block (the later ones come with the update
// of the step before).
__global__ __launch_bounds__(256) void gj_first_kernel(SweepPair S) {
  __shared__ double m[kB][kMLd];
  const double* __restrict__ A = S.A[blockIdx.x];
  const int64_t n = S.n[blockIdx.x];
  for (int e = threadIdx.x; e < kB * kB; e += 256) m[e / kB][e % kB] = A[(e / kB) * n + e % kB];
  __syncthreads();
  invert64(m);
  store_akk(m, S.Akk[blockIdx.x]);
}

// The panels of step k, a workgroup per 16 rows of the column or 16 columns of the
// row, a wavefront 16 of its 64 outputs, in FP64 MFMA: col <- -A_ik^T, A_ik <- -A_ik
// Akk, A_kj <- Akk A_kj (i, j != k); the last workgroup stores A_kk <- Akk.
__global__ __launch_bounds__(256) void gj_panel_kernel(SweepPair S, int64_t k0) {
  double* __restrict__ A = S.A[blockIdx.y];
  const double* __restrict__ Akk = S.Akk[blockIdx.y];
  double* __restrict__ col = S.col[blockIdx.y];
  const int64_t n = S.n[blockIdx.y], strips = (n - kB) / 16, id = blockIdx.x;
  if (k0 >= n || id > 2 * strips) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15, q = lane >> 4;
  if (id == 2 * strips) {
    for (int r = w; r < kB; r += 4) A[(k0 + r) * n + k0 + lane] = Akk[r * kB + lane];
    return;
  }
  const bool is_row = id >= strips;
  int64_t x0 = 16 * (is_row ? id - strips : id);   // first row of the column, column of the row
  if (x0 >= k0) x0 += kB;
  double a[16], d[16];
#pragma unroll
  for (int s = 0; s < 16; ++s) {
    a[s] = is_row ? A[(k0 + 4 * s + q) * n + x0 + c] : -A[(x0 + c) * n + k0 + 4 * s + q];
    d[s] = is_row ? Akk[(16 * w + c) * kB + 4 * s + q] : Akk[(4 * s + q) * kB + 16 * w + c];
  }
  f64x4_t acc = {};
#pragma unroll
  for (int s = 0; s < 16; ++s)
    acc = is_row ? __builtin_amdgcn_mfma_f64_16x16x4f64(d[s], a[s], acc, 0, 0, 0)
                 : __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], d[s], acc, 0, 0, 0);
  __syncthreads();   // every wavefront has read the strip that all of them overwrite
  if (!is_row)
#pragma unroll
    for (int s = 0; s < 16; ++s)
      if (s / 4 == w) col[(4 * s + q) * n + x0 + c] = a[s];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    A[is_row ? (k0 + 16 * w + q + 4 * r) * n + x0 + c : (x0 + q + 4 * r) * n + k0 + 16 * w + c] = acc[r];
}

// Trailing update of step k, a workgroup per 64x64 tile outside block row and
// column k: A[I, J] += col[I]^T A[k, J], a wavefront 32 x 32 of it in FP64 MFMA, both
// operands straight from L2 (rows of 16 doubles), all loads in flight at once.
// The first workgroup has the next diagonal block and goes on to invert it while
// the others run, so that a step waits for two launches instead of four: 1344^2,
// two matrices, 36 us a step (71 with the panels, the update through LDS and the
// diagonal block in launches of their own).
__global__ __launch_bounds__(256) void gj_update_kernel(SweepPair S, int64_t k0) {
  __shared__ double m[kB][kMLd];
  double* __restrict__ A = S.A[blockIdx.y];
  const double* __restrict__ col = S.col[blockIdx.y];
  const int64_t n = S.n[blockIdx.y];
  const int64_t nb = n / kB, kb = k0 / kB;
  if (k0 >= n || blockIdx.x >= (nb - 1) * (nb - 1)) return;
  int64_t tile = blockIdx.x;
  const bool next = kb + 1 < nb && tile == 0;
  if (kb + 1 < nb) {   // the next diagonal block's tile first
    const int64_t diag = kb * (nb - 1) + kb;
    tile = tile == 0 ? diag : tile <= diag ? tile - 1 : tile;
  }
  int64_t bi = tile % (nb - 1), bj = tile / (nb - 1);
  if (bi >= kb) ++bi;
  if (bj >= kb) ++bj;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wi = 32 * (wave >> 1), wj = 32 * (wave & 1), c = lane & 15, q = lane >> 4;
  const int64_t i0 = bi * kB + wi, j0 = bj * kB + wj;
  double av[16][2], bv[16][2];
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      av[s][u] = col[(4 * s + q) * n + i0 + 16 * u + c];
      bv[s][u] = A[(k0 + 4 * s + q) * n + j0 + 16 * u + c];
    }
  f64x4_t acc[2][2];
  double* out = A + (i0 + q) * n + j0 + c;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[u][v][r] = out[(16 * u + 4 * r) * n + 16 * v];
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
        acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s][u], bv[s][v], acc[u][v], 0, 0, 0);
  if (!next) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(16 * u + 4 * r) * n + 16 * v] = acc[u][v][r];
    return;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) m[wi + 16 * u + q + 4 * r][wj + 16 * v + c] = acc[u][v][r];
  __syncthreads();
  invert64(m);
  store_akk(m, S.Akk[blockIdx.y]);   // its place in A is the next panels' to fill
}

// out[r] = (BACK: out[r] -) sum_j row[j] v[j] for both systems (v and out: the
// second n further on), a wavefront per row, fixed reduction order; unrolled so
// that several iterations' loads are in flight (the FMA chain keeps its order).
template <bool BACK>
__device__ inline void row_product(const double* __restrict__ row, const double* v, int64_t n,
                                   int64_t len, double* out, int lane) {
  double a0 = 0.0, a1 = 0.0;
#pragma unroll 8
  for (int64_t j = lane; j < len; j += 64) {
    const double k = row[j];
    a0 = fma(k, v[j], a0);
    a1 = fma(k, v[n + j], a1);
  }
  for (int off = 32; off > 0; off >>= 1) {
    a0 += __shfl_xor(a0, off);
    a1 += __shfl_xor(a1, off);
  }
  if (lane == 0) {
    out[0] = BACK ? out[0] - a0 : a0;
    out[n] = BACK ? out[n] - a1 : a1;
  }
}

// x_s = K^-1 b_s for the two systems.
__global__ __launch_bounds__(256) void dense_apply_kernel(const double* __restrict__ inv,
                                                          int64_t n_pad, int64_t n,
                                                          const double* __restrict__ b,
                                                          double* __restrict__ x) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r < n) row_product<false>(inv + r * n_pad, b, n, n, x + r, threadIdx.x & 63);
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// Doubles of one matrix's part of a sweep's workspace (Akk, col).
static int64_t sweep_len(int64_t n) { return kB * kB + kB * n; }

static SweepPair sweep_of(double* A, int64_t n, double* work) {
  return {{A}, {n}, {work}, {work + kB * kB}};
}

// In-place inverses of the first `count` matrices of the pair.
static void gauss_jordan(const SweepPair& S, int count, hipStream_t st) {
  const int64_t n = count > 1 ? std::max(S.n[0], S.n[1]) : S.n[0], nb = n / kB;
  hipLaunchKernelGGL(gj_first_kernel, dim3(count), dim3(256), 0, st, S);
  for (int64_t k0 = 0; k0 < n; k0 += kB) {
    hipLaunchKernelGGL(gj_panel_kernel, dim3((unsigned)(2 * (n - kB) / 16 + 1), count), dim3(256), 0, st,
                       S, k0);
    if (nb > 1)
      hipLaunchKernelGGL(gj_update_kernel, dim3((unsigned)((nb - 1) * (nb - 1)), count), dim3(256), 0,
                         st, S, k0);
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
  DD_TRY(akk.alloc(sizeof(double) * (size_t)sweep_len(P > 1 ? wmax : n_pad)));
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
    gauss_jordan(sweep_of(X, n_pad, akk.as<double>()), 1, st);
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
    gauss_jordan(sweep_of(W, w, akk.as<double>()), 1, st);
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

// ---------------------------------------------------------------------------
// P_C by block elimination of node planes, for meshes whose inverse would be
// read for longer than the elimination's chain of small launches takes.
//
// With the blocks of planes above, both ends of the chain are eliminated at the
// same time towards the middle block: block k couples to one next block only,
//   S_next = A_next - C_k^T H_k,  H_k = S_k^-1 C_k,  C_k = K(k, next),
// and the middle block takes both sides.  Kept are S_k^-1 and H_k (C_k is zero
// but for the plane next to the other block: H_k has that plane's columns).
// Then K x = b is
//   y_next = b_next - H_k^T y_k      (ends to middle, both sides in a launch),
//   z_k = S_k^-1 y_k                 (all blocks in one launch),
//   x_k = z_k - H_k x_next           (middle to ends),
// about 3 n b entries read instead of the inverse's n^2, in P launches.
// ---------------------------------------------------------------------------
struct PlaneBlocks {   // P blocks of whole planes: b DOFs each, the last bl
  int64_t P = 0, b = 0, bl = 0, face = 0;
  int64_t mid() const { return P / 2; }
  int64_t off(int64_t k) const { return k * b; }
  int64_t size(int64_t k) const { return k == P - 1 ? bl : b; }
};

static __host__ __device__ inline int64_t ld8(int64_t n) { return (n + 7) / 8 * 8; }   // 64-byte rows

static PlaneBlocks plane_blocks(int64_t nx, int64_t ny, int64_t nz) {
  PlaneBlocks B;
  B.face = 3 * (nx + 1) * (ny + 1);
  const int64_t per = std::max<int64_t>(1, (kMinBlock + B.face - 1) / B.face);
  B.P = std::max<int64_t>(1, (nz + 1) / per);
  B.b = per * B.face;
  B.bl = (nz + 1) * B.face - (B.P - 1) * B.b;   // a short last group joins the one before
  return B;
}

// Bytes that K^-1 must be larger by, per block, for the chain's launches to pay.
// Measured per DD iteration, cubes of n elements a side, FP64 scan of 2000 points,
// inverse / planes: n = 8 0.128 / 0.146 ms, 11 0.198 / 0.209 (15 MB a block), 12
// 0.254 / 0.224 (23 MB), 14 0.397 / 0.310, 16 0.693 / 0.392; beyond the inverse's
// sizes CG / planes: 18 6.2 / 0.51, 20 7.8 / 0.73, 24 12.9 / 1.29, 27 16.9 / 2.06.
constexpr int64_t kPlaneStepBytes = (int64_t)18 << 20;

// doubles of S_k^-1 of all blocks, and of H_k
static int64_t plane_inv_len(const PlaneBlocks& B) {
  return (B.P - 1) * B.b * ld8(B.b) + B.bl * ld8(B.bl);
}
static int64_t plane_h_len(const PlaneBlocks& B) {
  return ((B.P - 1) * B.b + B.bl) * ld8(B.face);
}

// Up to kDenseMaxDof DOFs K^-1 or the planes, whichever is applied sooner; beyond
// it the planes as long as the dataset's cache holds them (cubes of up to 27
// elements a side), else CG.  Formation, first solve of one iteration with it:
// n = 16 9.7 ms (K^-1 27 when it still took that size), 20 21 (CG 28), 24 45 (CG 55),
// 27 78 (CG 85).
PCKind pc_kind(int64_t nx, int64_t ny, int64_t nz) {
  const PlaneBlocks B = plane_blocks(nx, ny, nz);
  const int64_t n = (nz + 1) * B.face;
  const int64_t bytes = 8 * (plane_inv_len(B) + plane_h_len(B));
  const bool fits = B.P >= 3 && bytes <= kDenseCacheBytes;
  if (n > kDenseMaxDof) return fits ? PCKind::kPlanes : PCKind::kCG;
  return fits && 8 * n * n - bytes > B.P * kPlaneStepBytes ? PCKind::kPlanes : PCKind::kInverse;
}

int64_t pc_bytes(int64_t nx, int64_t ny, int64_t nz) {
  const PlaneBlocks B = plane_blocks(nx, ny, nz);
  const int64_t n_pad = ((nz + 1) * B.face + kB - 1) / kB * kB;
  switch (pc_kind(nx, ny, nz)) {
    case PCKind::kPlanes: return 8 * (plane_inv_len(B) + plane_h_len(B));
    case PCKind::kInverse: return 8 * n_pad * n_pad;
    default: return 0;
  }
}

namespace {

struct PlaneArgs {
  int64_t n, P, b, bl, face, mid;
  const double* inv;   // S_k^-1 at k b ld8(b), leading dimension ld8 of the block's size
  const double* h;     // H_k at k b ld8(face)
};

// Couplings of the DOFs c of one plane (`to`) with the plane beside it (`from`):
// val[27][face], entry 9 comp + (3 (dj + 1) + di + 1) the coupling with component
// comp of the neighbour node (i + di, j + dj).
__global__ __launch_bounds__(256) void plane_coupling_kernel(MeshDims d, const double* __restrict__ Ke,
                                                             const uint8_t* __restrict__ mask,
                                                             int64_t face, int64_t from, int64_t to,
                                                             double* __restrict__ val) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= 9 * face) return;
  const int64_t c = id % face;
  const int nb = (int)(id / face);
  const int sx = d.nx + 1, comp = (int)(c % 3), i = (int)((c / 3) % sx), j = (int)(c / 3 / sx);
  const int ii = i + nb % 3 - 1, jj = j + nb / 3 - 1;
  double s[3] = {0.0, 0.0, 0.0};
  if (ii >= 0 && jj >= 0 && ii <= d.nx && jj <= d.ny && !mask[to * face + c]) {
    const int k = (int)to, kk = (int)from, ez = min(k, kk);
    for (int ey = max(j, jj) - 1; ey <= min(j, jj); ++ey)
      for (int ex = max(i, ii) - 1; ex <= min(i, ii); ++ex) {
        if (ex < 0 || ey < 0 || ex >= d.nx || ey >= d.ny) continue;
        const int a = (i - ex) + 2 * (j - ey) + 4 * (k - ez);
        const int b = (ii - ex) + 2 * (jj - ey) + 4 * (kk - ez);
        for (int q = 0; q < 3; ++q) s[q] += Ke[24 * (3 * a + comp) + 3 * b + q];
      }
    const int64_t col0 = from * face + 3 * (ii + (int64_t)sx * jj);
    for (int q = 0; q < 3; ++q)
      if (mask[col0 + q]) s[q] = 0.0;
  }
  for (int q = 0; q < 3; ++q) val[(9 * q + nb) * face + c] = s[q];
}

// H[r][c] = sum_j X[r][row0 + j] C[j][c] over the 27 neighbours j of c (X: rows x rows, ldx)
constexpr int kHRows = 8;
__global__ __launch_bounds__(256) void plane_h_kernel(int sx, int sy, int64_t rows,
                                                      const double* __restrict__ X, int64_t ldx,
                                                      int64_t row0, const double* __restrict__ val,
                                                      double* __restrict__ H, int64_t ldh) {
  const int64_t face = 3 * (int64_t)sx * sy, c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= face) return;
  const int i = (int)((c / 3) % sx), j = (int)(c / 3 / sx);
  double v[27];
  int at[9];
#pragma unroll
  for (int nb = 0; nb < 9; ++nb) {
    const int ii = i + nb % 3 - 1, jj = j + nb / 3 - 1;
    at[nb] = ii >= 0 && jj >= 0 && ii < sx && jj < sy ? 3 * (ii + sx * jj) : 0;   // 0: coefficient 0
#pragma unroll
    for (int q = 0; q < 3; ++q) v[9 * q + nb] = val[(9 * q + nb) * face + c];
  }
  const int64_t r1 = min(rows, ((int64_t)blockIdx.y + 1) * kHRows);
  for (int64_t r = (int64_t)blockIdx.y * kHRows; r < r1; ++r) {
    const double* x = X + r * ldx + row0;
    double s = 0.0;
#pragma unroll
    for (int nb = 0; nb < 9; ++nb)
#pragma unroll
      for (int q = 0; q < 3; ++q) s = fma(x[at[nb] + q], v[9 * q + nb], s);
    H[r * ldh + c] = s;
  }
}

// S[r][c] -= sum_j C[j][r] H[j][c] over the 27 neighbours j of r: one row r per blockIdx.y
__global__ __launch_bounds__(256) void plane_schur_kernel(int sx, int sy, const double* __restrict__ val,
                                                          const double* __restrict__ H, int64_t ldh,
                                                          double* __restrict__ S, int64_t lds_) {
  const int64_t face = 3 * (int64_t)sx * sy, c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= face) return;
  const int64_t r = blockIdx.y;
  const int i = (int)((r / 3) % sx), j = (int)(r / 3 / sx);
  double s = 0.0;
#pragma unroll
  for (int nb = 0; nb < 9; ++nb) {
    const int ii = i + nb % 3 - 1, jj = j + nb / 3 - 1;
    const int64_t at = ii >= 0 && jj >= 0 && ii < sx && jj < sy ? 3 * (ii + (int64_t)sx * jj) : 0;
#pragma unroll
    for (int q = 0; q < 3; ++q) s = fma(val[(9 * q + nb) * face + r], H[(at + q) * ldh + c], s);
  }
  S[r * lds_ + c] -= s;
}

// y_next -= H_k^T y_k for step t of both sides (blockIdx.y; the middle block
// takes both sides' terms in one workgroup).  A workgroup holds 16 columns, 64
// groups of its threads every 64th row: a row of 16 doubles is a 128-byte line,
// and 1024 threads put 64 of them in flight each pass.
constexpr int kFwdCols = 16, kFwdThreads = 1024, kFwdGroups = kFwdThreads / kFwdCols;
__global__ __launch_bounds__(kFwdThreads) void plane_forward_kernel(PlaneArgs A, int64_t t, double* y) {
  __shared__ double part[2][kFwdThreads / 64][kFwdCols];
  const int side = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t kl = t, kr = A.P - 1 - t;
  const bool left = kl < A.mid, right = kr > A.mid;
  const bool both = left && right && kl + 1 == A.mid && kr - 1 == A.mid;
  if (side == 0 ? !left : (!right || both)) return;
  const int64_t ldh = ld8(A.face);
  const int64_t c = (int64_t)blockIdx.x * kFwdCols + (threadIdx.x & (kFwdCols - 1));
  const int g = threadIdx.x / kFwdCols;
  for (int s = side; s <= (both ? 1 : side); ++s) {
    const int64_t k = s == 0 ? kl : kr;
    const int64_t rows = k == A.P - 1 ? A.bl : A.b, o = k * A.b;
    const int64_t dst = s == 0 ? o + rows : o - A.face;
    const double* H = A.h + o * ldh;
    double a0 = 0.0, a1 = 0.0;
    if (c < A.face) {
#pragma unroll 8
      for (int64_t r = g; r < rows; r += kFwdGroups) {
        const double h = H[r * ldh + c];
        a0 = fma(h, y[o + r], a0);
        a1 = fma(h, y[A.n + o + r], a1);
      }
    }
    a0 += __shfl_xor(a0, 16);
    a1 += __shfl_xor(a1, 16);
    a0 += __shfl_xor(a0, 32);
    a1 += __shfl_xor(a1, 32);
    if (lane < kFwdCols) {
      part[0][wave][lane] = a0;
      part[1][wave][lane] = a1;
    }
    __syncthreads();
    if (threadIdx.x < 2 * kFwdCols) {
      const int sys = threadIdx.x / kFwdCols;
      if (c < A.face) {
        double sum = 0.0;
        for (int w = 0; w < kFwdThreads / 64; ++w) sum += part[sys][w][threadIdx.x & (kFwdCols - 1)];
        y[sys * A.n + dst + c] -= sum;
      }
    }
    __syncthreads();
  }
}

// z = S_k^-1 y_k, every block
__global__ __launch_bounds__(256) void plane_blocks_kernel(PlaneArgs A, const double* __restrict__ y,
                                                           double* __restrict__ x) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= A.n) return;
  const int64_t k = min(r / A.b, A.P - 1), len = k == A.P - 1 ? A.bl : A.b, o = k * A.b;
  row_product<false>(A.inv + o * ld8(A.b) + (r - o) * ld8(len), y + o, A.n, len, x + r, threadIdx.x & 63);
}

// x_k -= H_k x_next at step t of both sides (blockIdx.y)
__global__ __launch_bounds__(256) void plane_backward_kernel(PlaneArgs A, int64_t t, double* x) {
  const bool left = blockIdx.y == 0;
  const int64_t k = left ? t : A.P - 1 - t;
  if (left ? k >= A.mid : k <= A.mid) return;
  const int64_t rows = k == A.P - 1 ? A.bl : A.b, o = k * A.b;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  row_product<true>(A.h + (o + r) * ld8(A.face), x + (left ? o + rows : o - A.face), A.n, A.face, x + o + r,
                  threadIdx.x & 63);
}

PlaneArgs plane_args(const DenseInverse& D) {
  const PlaneBlocks B = plane_blocks(D.nx, D.ny, D.nz);
  const double* p = D.inv.as<double>();
  return {D.n, B.P, B.b, B.bl, B.face, B.mid(), p, p + plane_inv_len(B)};
}

}  // namespace

// Forms S_k^-1 and H_k on st.
static dd_status form_planes(const FEMesh& M, const double* Ke, const uint8_t* mask, DenseInverse& D,
                             hipStream_t st) {
  const PlaneBlocks B = plane_blocks(M.nx, M.ny, M.nz);
  const int64_t n = M.n_dof, inv_len = plane_inv_len(B);
  D.n = n;
  D.planes = true;
  DD_TRY(D.inv.alloc(sizeof(double) * (size_t)(inv_len + plane_h_len(B))));
  const int64_t bmax = std::max(B.b, B.bl), wmax = (bmax + kB - 1) / kB * kB;
  DevBuf work, val, akk, dke, dmask;
  DD_TRY(work.alloc(sizeof(double) * (size_t)(6 * wmax * wmax)));
  DD_TRY(val.alloc(sizeof(double) * (size_t)(2 * 27 * B.face)));
  DD_TRY(akk.alloc(sizeof(double) * (size_t)(2 * sweep_len(wmax))));
  DD_TRY(dke.alloc(sizeof(double) * 24 * 24));
  DD_TRY(dmask.alloc((size_t)n));
  DD_HIP(hipMemcpyAsync(dke.p, Ke, sizeof(double) * 24 * 24, hipMemcpyHostToDevice, st));
  DD_HIP(hipMemcpyAsync(dmask.p, mask, (size_t)n, hipMemcpyHostToDevice, st));
  const MeshDims dims{M.nx, M.ny, M.nz};
  const int sx = M.nx + 1, sy = M.ny + 1;
  const int64_t mid = B.mid(), ldh = ld8(B.face);
  double* inv = D.inv.as<double>();
  double* h = inv + inv_len;
  auto side_val = [&](int s) { return val.as<double>() + s * 27 * B.face; };
  // the blocks of a step (one of each side, the middle one alone at the end)
  for (int64_t t = 0; t <= mid; ++t) {
    int64_t blk[2];
    int count = 0;
    if (t < mid) blk[count++] = t;
    if (t < mid && B.P - 1 - t > mid) blk[count++] = B.P - 1 - t;
    if (t == mid) blk[count++] = mid;
    SweepPair S = {};
    GemmPair res = {}, add = {};
    for (int q = 0; q < count; ++q) {
      const int64_t k = blk[q], b = B.size(k), w = (b + kB - 1) / kB * kB, ld = ld8(b);
      double* W = work.as<double>() + 3 * q * wmax * wmax;
      double *S0 = W + wmax * wmax, *R = S0 + wmax * wmax, *X = inv + B.off(k) * ld8(B.b);
      DD_HIP(hipMemsetAsync(W, 0, sizeof(double) * (size_t)(w * w), st));
      hipLaunchKernelGGL(assemble_block_kernel, dim3(blocks_for(27 * b, 256)), dim3(256), 0, st, dims,
                         dke.as<double>(), dmask.as<uint8_t>(), B.off(k), b, (int64_t)0, W, w,
                         (double*)nullptr, (int64_t)0);
      if (w > b) hipLaunchKernelGGL(pad_identity_kernel, dim3(1), dim3(64), 0, st, W, b, w);
      for (int s = 0; s < 2; ++s) {   // the Schur terms of the block(s) before
        const int64_t from = s == 0 ? k - 1 : k + 1;
        const bool has = s == 0 ? from >= 0 && from < mid : from < B.P && from > mid;
        if (!has) continue;
        const double* H = h + (B.off(from) + (s == 0 ? B.size(from) - B.face : 0)) * ldh;
        double* at = W + (s == 0 ? 0 : (b - B.face) * (w + 1));
        hipLaunchKernelGGL(plane_schur_kernel, dim3(blocks_for(B.face, 256), (unsigned)B.face), dim3(256),
                           0, st, sx, sy, side_val(s), H, ldh, at, w);
      }
      DD_HIP(hipMemcpyAsync(S0, W, sizeof(double) * (size_t)(w * w), hipMemcpyDeviceToDevice, st));
      hipLaunchKernelGGL(identity_kernel, dim3(blocks_for(b * b, 256)), dim3(256), 0, st, R, b);
      S.A[q] = W;
      S.n[q] = w;
      S.Akk[q] = akk.as<double>() + q * sweep_len(wmax);
      S.col[q] = S.Akk[q] + kB * kB;
      res.g[q] = {b, b, b, S0, w, W, w, R, b};
      add.g[q] = {b, b, b, W, w, R, b, X, ld};
    }
    gauss_jordan(S, count, st);
    for (int q = 0; q < count; ++q) {
      const int64_t k = blk[q], b = B.size(k), w = S.n[q];
      DD_HIP(hipMemcpy2DAsync(add.g[q].C, sizeof(double) * ld8(b), S.A[q], sizeof(double) * w,
                              sizeof(double) * b, (size_t)b, hipMemcpyDeviceToDevice, st));
    }
    // one Newton step, X += X (I - S X): without it the blocks' errors add up
    // along the planes
    gemm64_pair(res, count, -1.0, 1.0, st);
    gemm64_pair(add, count, 1.0, 1.0, st);
    if (t == mid) break;
    for (int q = 0; q < count; ++q) {
      const int64_t k = blk[q], b = B.size(k), o = B.off(k);
      const int s = k < mid ? 0 : 1;
      // planes on both sides of the boundary
      const int64_t from = s == 0 ? (o + b) / B.face - 1 : o / B.face, to = s == 0 ? from + 1 : from - 1;
      hipLaunchKernelGGL(plane_coupling_kernel, dim3(blocks_for(9 * B.face, 256)), dim3(256), 0, st, dims,
                         dke.as<double>(), dmask.as<uint8_t>(), B.face, from, to, side_val(s));
      hipLaunchKernelGGL(plane_h_kernel, dim3(blocks_for(B.face, 256), blocks_for(b, kHRows)), dim3(256),
                         0, st, sx, sy, b, add.g[q].C, ld8(b), s == 0 ? b - B.face : (int64_t)0,
                         side_val(s), h + o * ldh, ldh);
    }
    DD_HIP(hipGetLastError());
  }
  DD_HIP(hipGetLastError());
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
  if (pc_kind(M.nx, M.ny, M.nz) == PCKind::kPlanes)
    DD_TRY(form_planes(M, Ke, mask, *d, st));
  else
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

dd_status dense_apply(const DenseInverse& D, double* b, double* x, hipStream_t st) {
  if (!D.planes) {
    hipLaunchKernelGGL(dense_apply_kernel, dim3(blocks_for(D.n, 4)), dim3(256), 0, st,
                       D.inv.as<double>(), D.n_pad, D.n, b, x);
    DD_HIP(hipGetLastError());
    return DD_OK;
  }
  const PlaneArgs A = plane_args(D);
  const dim3 fwd(blocks_for(A.face, kFwdCols), 2), bwd(blocks_for(std::max(A.b, A.bl), 4), 2);
  for (int64_t t = 0; t < A.mid; ++t)
    hipLaunchKernelGGL(plane_forward_kernel, fwd, dim3(kFwdThreads), 0, st, A, t, b);
  hipLaunchKernelGGL(plane_blocks_kernel, dim3(blocks_for(A.n, 4)), dim3(256), 0, st, A, b, x);
  for (int64_t t = A.mid - 1; t >= 0; --t)
    hipLaunchKernelGGL(plane_backward_kernel, bwd, dim3(256), 0, st, A, t, x);
  DD_HIP(hipGetLastError());
  return DD_OK;
}

}  // namespace dd
