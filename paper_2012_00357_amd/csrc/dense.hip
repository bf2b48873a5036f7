// P_C by operators formed once.  K is constant over the DD iterations (Section 2:
// the paper factorises it once): for small meshes its inverse is formed on the
// GPU and kept per (mesh, Dirichlet pattern) on the dataset, and every P_C is then
// one product of K^-1 with the two right-hand sides (E and S of eqs. "KuE",
// "KeS") -- a stream of n^2 doubles instead of hundreds of CG iterations.  Larger
// meshes keep the block elimination of their node planes instead (below).
//
// Inversion: blocked Gauss-Jordan without pivoting (K is symmetric positive
// definite, with identity rows and columns at Dirichlet DOFs), in place on a copy
// padded to a multiple of 64 with identity.  For each 64-block k:
//   A_kk <- A_kk^-1;  A_kj <- A_kk A_kj (j != k);  A_ij <- A_ij - A_ik A_kj
//   (i, j != k);  A_ik <- -A_ik A_kk (i != k).
// 8^3 elements (n = 2187), first solve of one iteration with it: 3.4 ms with the matrix
// assembled on the device, 12 with the updates on the vector FP64 units and the
// matrix from the host.  u is as near the 64-bit solution as before (8^3 8e-15,
// 10^3 1.4e-14): an update's 64 products are summed before they meet the entry
// they change, without which it is twice as far.
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

// Rows of one block of K (DOFs row0 .. row0 + rows - 1), in the columns of the same
// block, from the element stiffness Ke to W (leading dimension ldw).  One thread
// per (row, neighbouring node); W starts at zero.  An entry sums the elements that
// share both nodes in element order.  Dirichlet rows and columns are those of the
// identity.
__global__ __launch_bounds__(256) void assemble_block_kernel(
    MeshDims d, const double* __restrict__ Ke, const uint8_t* __restrict__ mask, int64_t row0,
    int64_t rows, double* __restrict__ W, int64_t ldw) {
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
    if (!mask[col] && col >= row0 && col < row0 + rows) W[lr * ldw + (col - row0)] = s[c];
  }
}

__global__ void pad_identity_kernel(double* __restrict__ W, int64_t n, int64_t n_pad) {
  const int64_t r = n + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n_pad) W[r * n_pad + r] = 1.0;
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

// Gauss-Jordan on a 16 x 16 block: lane 16 g + r holds columns 4 g .. 4 g + 3 of row r.
template <int P>
__device__ inline void pivot16(double (&v)[4], int r, int g) {
  if constexpr (P < 16) {
    constexpr int pg = P / 4, pe = P % 4;
    const double colv = __shfl(v[pe], 16 * pg + r);
    const double d = 1.0 / lane_d(v[pe], 16 * pg + P);
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
      f64x4_t acc[3] = {};
      int at[3];   // the other three column blocks
#pragma unroll
      for (int u = 0; u < 3; ++u) at[u] = 16 * (u + (u >= s ? 1 : 0)) + c;
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int u = 0; u < 3; ++u)
          acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(neg[k], m[o + 4 * k + q][at[u]], acc[u], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) m[b + q + 4 * r][at[u]] += acc[u][r];
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
  f64x4_t acc[2][2] = {}, old[2][2];   // the 64 products are summed before they meet the entry
  double* out = A + (i0 + q) * n + j0 + c;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) old[u][v][r] = out[(16 * u + 4 * r) * n + 16 * v];
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
        for (int r = 0; r < 4; ++r) out[(16 * u + 4 * r) * n + 16 * v] = old[u][v][r] + acc[u][v][r];
    return;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        m[wi + 16 * u + q + 4 * r][wj + 16 * v + c] = old[u][v][r] + acc[u][v][r];
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

// Forms K^-1 (row-major, leading dimension n_pad) on st.
static dd_status form_inverse(const FEMesh& M, const double* Ke, const uint8_t* mask, DenseInverse& D,
                              hipStream_t st) {
  const int64_t n = M.n_dof, n_pad = (n + kB - 1) / kB * kB;
  D.n = n;
  D.n_pad = n_pad;
  DD_TRY(D.inv.alloc(sizeof(double) * (size_t)(n_pad * n_pad)));
  DevBuf work, dke, dmask;
  DD_TRY(work.alloc(sizeof(double) * (size_t)sweep_len(n_pad)));
  DD_TRY(dke.alloc(sizeof(double) * 24 * 24));
  DD_TRY(dmask.alloc((size_t)n));
  DD_HIP(hipMemcpyAsync(dke.p, Ke, sizeof(double) * 24 * 24, hipMemcpyHostToDevice, st));
  DD_HIP(hipMemcpyAsync(dmask.p, mask, (size_t)n, hipMemcpyHostToDevice, st));
  double* X = D.inv.as<double>();
  DD_HIP(hipMemsetAsync(X, 0, D.inv.bytes, st));
  hipLaunchKernelGGL(assemble_block_kernel, dim3(blocks_for(27 * n, 256)), dim3(256), 0, st,
                     MeshDims{M.nx, M.ny, M.nz}, dke.as<double>(), dmask.as<uint8_t>(), (int64_t)0, n, X,
                     n_pad);
  if (n_pad > n) hipLaunchKernelGGL(pad_identity_kernel, dim3(1), dim3(64), 0, st, X, n, n_pad);
  gauss_jordan(sweep_of(X, n_pad, work.as<double>()), 1, st);
  DD_HIP(hipGetLastError());
  DD_HIP(hipStreamSynchronize(st));
  return DD_OK;
}

// Smallest block of planes: below it a block's launches cost more than the
// elimination saves.
constexpr int64_t kMinBlock = 256;

// ---------------------------------------------------------------------------
// P_C by block elimination of node planes, for meshes whose inverse would be
// read for longer than the elimination's chain of small launches takes.
//
// The nodes are numbered plane by plane and an element joins two neighbouring
// planes, so K is block tridiagonal in groups of planes (diagonal blocks A_k).  Both
// ends of that chain are eliminated at the same time towards the middle block:
// with the Schur complements S_k (S = A at the ends), block k couples to one next
// block only,
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
// inverse / planes: n = 8 0.127 / 0.149 ms, 11 0.190 / 0.208 (15 MB a block), 12
// 0.253 / 0.246 (23 MB), 14 0.396 / 0.272, 16 0.693 / 0.365; beyond the inverse's
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
// n = 16 8.3 ms, 20 15 (CG 28), 24 28 (CG 55).
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

// Padded size of the blocks that form_planes inverts.
static int64_t plane_pad(const PlaneBlocks& B) {
  return (std::max(B.b, B.bl) + kB - 1) / kB * kB;
}

int64_t pc_work_bytes(int64_t nx, int64_t ny, int64_t nz) {
  const PlaneBlocks B = plane_blocks(nx, ny, nz);
  const int64_t n = (nz + 1) * B.face, w = plane_pad(B);
  const int64_t in = 8 * 24 * 24 + n;   // element stiffness and mask
  switch (pc_kind(nx, ny, nz)) {
    case PCKind::kPlanes: return in + 8 * (2 * w * w + 2 * 27 * B.face + 2 * sweep_len(w));
    case PCKind::kInverse: return in + 8 * sweep_len((n + kB - 1) / kB * kB);
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
  const int64_t wmax = plane_pad(B);
  DevBuf work, val, akk, dke, dmask;
  DD_TRY(work.alloc(sizeof(double) * (size_t)(2 * wmax * wmax)));
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
    for (int q = 0; q < count; ++q) {
      const int64_t k = blk[q], b = B.size(k), w = (b + kB - 1) / kB * kB;
      double* W = work.as<double>() + q * wmax * wmax;
      DD_HIP(hipMemsetAsync(W, 0, sizeof(double) * (size_t)(w * w), st));
      hipLaunchKernelGGL(assemble_block_kernel, dim3(blocks_for(27 * b, 256)), dim3(256), 0, st, dims,
                         dke.as<double>(), dmask.as<uint8_t>(), B.off(k), b, W, w);
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
      S.A[q] = W;
      S.n[q] = w;
      S.Akk[q] = akk.as<double>() + q * sweep_len(wmax);
      S.col[q] = S.Akk[q] + kB * kB;
    }
    gauss_jordan(S, count, st);
    double* X[2];
    for (int q = 0; q < count; ++q) {
      const int64_t k = blk[q], b = B.size(k), w = S.n[q];
      X[q] = inv + B.off(k) * ld8(B.b);
      DD_HIP(hipMemcpy2DAsync(X[q], sizeof(double) * ld8(b), S.A[q], sizeof(double) * w,
                              sizeof(double) * b, (size_t)b, hipMemcpyDeviceToDevice, st));
    }
    if (t == mid) break;
    for (int q = 0; q < count; ++q) {
      const int64_t k = blk[q], b = B.size(k), o = B.off(k);
      const int s = k < mid ? 0 : 1;
      // planes on both sides of the boundary
      const int64_t from = s == 0 ? (o + b) / B.face - 1 : o / B.face, to = s == 0 ? from + 1 : from - 1;
      hipLaunchKernelGGL(plane_coupling_kernel, dim3(blocks_for(9 * B.face, 256)), dim3(256), 0, st, dims,
                         dke.as<double>(), dmask.as<uint8_t>(), B.face, from, to, side_val(s));
      hipLaunchKernelGGL(plane_h_kernel, dim3(blocks_for(B.face, 256), blocks_for(b, kHRows)), dim3(256),
                         0, st, sx, sy, b, X[q], ld8(b), s == 0 ? b - B.face : (int64_t)0,
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
