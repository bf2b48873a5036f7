// Culling for the exact scans of P_D (Section 2): which tiles of the data set
// can hold the nearest point of which queries.
//
// A scan need not form the distances of a query to a tile whose points all lie
// farther away than a point already known.  Every tile's points are bounded by
// a box in principal-axis coordinates y = V^T x (a rotation of the whitened
// space, so box distances are lower bounds of whitened distances); the boxes
// are made with the data set.  Per call:
//   order   the queries are sorted by their cell on the principal axes (a
//           counting sort), so that neighbours in the order need the same tiles;
//   seed    each query takes the FP64 distance of its nearest point of one near
//           tile as its bound;
//   cull    per tile a mask with one bit per group of 16 or 32 queries: set when
//           some query of the group has a box distance within its bound;
//   plan    the tiles with a bit set, as a list of work entries.
// The culled scans then take the listed tiles one by one through LDS and form
// the scores of the groups whose bit is set.  The bound is the distance of a
// data point, rounded up; a box distance is rounded down (slack and shrink
// below), so the tile of every exact minimiser, ties included, keeps its bit
// and the results are those of the scan over all tiles.
//
// Cost: a test of one box for 64 queries is about 90 vector instructions; the
// boxes are tested first against the bounding box of the wavefront's queries,
// 64 boxes at a time.
#include <algorithm>
#include <cmath>

#include "pack16.h"
#include "scan.h"

namespace dd {

namespace {

// Reads at an address that is the same in every lane, through the constant
// address space (scalar loads); the boxes are not written while a scan runs.
template <class T>
__device__ inline const __attribute__((address_space(4))) T* uniform_ptr(const T* p) {
  return (const __attribute__((address_space(4))) T*)p;
}

constexpr float kEps22 = 2.384185791015625e-07f;           // 2^-22
constexpr float kLbShrink = 1.0f - 1.9073486328125e-06f;   // 1 - 2^-19

unsigned grid1(int64_t n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

template <int C>
__device__ inline float dpp_f(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), C, 0xF, 0xF, false));
}
__device__ inline float lane_f(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
// Minimum / maximum over each row of 16 lanes, then over the wavefront (every
// lane active; the latter uniform).
__device__ inline float row_min(float v) {
  v = fminf(v, dpp_f<0xB1>(v));
  v = fminf(v, dpp_f<0x4E>(v));
  v = fminf(v, dpp_f<0x141>(v));
  return fminf(v, dpp_f<0x140>(v));
}
__device__ inline float row_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));
  v = fmaxf(v, dpp_f<0x4E>(v));
  v = fmaxf(v, dpp_f<0x141>(v));
  return fmaxf(v, dpp_f<0x140>(v));
}
__device__ inline float wave_min(float v) {
  v = row_min(v);
  return fminf(fminf(lane_f(v, 0), lane_f(v, 16)), fminf(lane_f(v, 32), lane_f(v, 48)));
}
__device__ inline float wave_max(float v) {
  v = row_max(v);
  return fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
}

}  // namespace

// ---------------------------------------------------------------------------
// Tile boxes
// ---------------------------------------------------------------------------
// Box of ROWS consecutive rows of the sorted FP64 pack, a row per lane: FP64
// coordinates on the principal axes, rounded outward to FP32 before the
// minimum and maximum (rounding is monotone, so the result is the outward
// rounding of the FP64 extremes).  Writes the rows' |x|^2 on the way.
template <int ROWS>
__global__ __launch_bounds__(ROWS) void tile_box_kernel(const double* __restrict__ w64, int64_t N,
                                                        const double* __restrict__ V,
                                                        double* __restrict__ n64,
                                                        float* __restrict__ box) {
  __shared__ float part[ROWS / 64][24];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t i = (int64_t)blockIdx.x * ROWS + t;
  const double* x = w64 + 12 * (i < N ? i : N - 1);   // row N - 1 lies in the last tile
  double v[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) v[k] = x[k];
  double n2 = 0.0;
#pragma unroll
  for (int k = 0; k < 12; ++k) n2 = fma(v[k], v[k], n2);
  if (i < N) n64[i] = n2;
#pragma unroll
  for (int a = 0; a < 12; ++a) {
    double y = 0.0;
#pragma unroll
    for (int k = 0; k < 12; ++k) y = fma(V[12 * k + a], v[k], y);
    const float lo = wave_min(__double2float_rd(y)), hi = wave_max(__double2float_ru(y));
    if (lane == 0) {
      part[wave][a] = lo;
      part[wave][12 + a] = hi;
    }
  }
  __syncthreads();
  if (t < 24) {
    float b = part[0][t];
    for (int w = 1; w < ROWS / 64; ++w) b = t < 12 ? fminf(b, part[w][t]) : fmaxf(b, part[w][t]);
    box[24 * (int64_t)blockIdx.x + t] = b;
  }
}

// Box of `fan` consecutive child boxes; one thread per node and component.
__global__ void union_box_kernel(const float* __restrict__ child, int64_t n_child, int fan,
                                 int64_t n_node, float* __restrict__ box) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 24 * n_node) return;
  const int64_t node = i / 24;
  const int c = (int)(i - 24 * node);
  const int64_t first = node * fan, last = min(first + (int64_t)fan, n_child);
  float b = child[24 * first + c];
  for (int64_t j = first + 1; j < last; ++j) {
    const float v = child[24 * j + c];
    b = c < 12 ? fminf(b, v) : fmaxf(b, v);
  }
  box[i] = b;
}

// Box of all chunks (one workgroup).
__global__ __launch_bounds__(256) void root_box_kernel(const float* __restrict__ chunk, int64_t nc,
                                                       float* __restrict__ root) {
  __shared__ float part[4][24];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  float lo[12], hi[12];
#pragma unroll
  for (int a = 0; a < 12; ++a) {
    lo[a] = INFINITY;
    hi[a] = -INFINITY;
  }
  for (int64_t c = t; c < nc; c += 256) {
#pragma unroll
    for (int a = 0; a < 12; ++a) {
      lo[a] = fminf(lo[a], chunk[24 * c + a]);
      hi[a] = fmaxf(hi[a], chunk[24 * c + 12 + a]);
    }
  }
#pragma unroll
  for (int a = 0; a < 12; ++a) {
    const float l = wave_min(lo[a]), h = wave_max(hi[a]);
    if (lane == 0) {
      part[wave][a] = l;
      part[wave][12 + a] = h;
    }
  }
  __syncthreads();
  if (t < 24) {
    float b = part[0][t];
    for (int w = 1; w < 4; ++w) b = t < 12 ? fminf(b, part[w][t]) : fmaxf(b, part[w][t]);
    root[t] = b;
  }
}

dd_status build_tile_boxes(const Dataset& D, int rows, const TileBoxes* from, TileBoxes& B,
                           hipStream_t st) {
  const int64_t n = (D.N + rows - 1) / rows, nc = cull_chunks(n);
  DD_TRY(B.tile.alloc(sizeof(float) * 24 * (size_t)n));
  DD_TRY(B.chunk.alloc(sizeof(float) * 24 * (size_t)nc));
  if (from && from->n_tiles > 0 && rows % from->rows == 0) {
    hipLaunchKernelGGL(union_box_kernel, dim3(grid1(24 * n)), dim3(256), 0, st,
                       from->tile.as<float>(), from->n_tiles, rows / from->rows, n,
                       B.tile.as<float>());
  } else if (rows == 256) {
    hipLaunchKernelGGL(tile_box_kernel<256>, dim3((unsigned)n), dim3(256), 0, st,
                       D.w64.as<double>(), D.N, D.vrot.as<double>(), D.n64.as<double>(),
                       B.tile.as<float>());
  } else if (rows == 128) {
    hipLaunchKernelGGL(tile_box_kernel<128>, dim3((unsigned)n), dim3(128), 0, st,
                       D.w64.as<double>(), D.N, D.vrot.as<double>(), D.n64.as<double>(),
                       B.tile.as<float>());
  } else {
    return set_error(DD_ERR_ARG, "tile boxes: rows");
  }
  DD_HIP(hipGetLastError());
  hipLaunchKernelGGL(union_box_kernel, dim3(grid1(24 * nc)), dim3(256), 0, st, B.tile.as<float>(), n,
                     64, nc, B.chunk.as<float>());
  DD_HIP(hipGetLastError());
  DD_TRY(B.root.alloc(sizeof(float) * 24));
  hipLaunchKernelGGL(root_box_kernel, dim3(1), dim3(256), 0, st, B.chunk.as<float>(), nc,
                     B.root.as<float>());
  DD_HIP(hipGetLastError());
  B.rows = rows;
  B.n_tiles = n;
  return DD_OK;
}

// Cells of the grouping order: each key bit halves the cell's longest edge, so
// that the queries of a cell lie within a compact box whatever the spread of
// the principal axes.
void choose_group_cells(Dataset& D) {
  GroupCells& g = D.cells;
  double edge[kKeyAxes];
  for (int a = 0; a < kKeyAxes; ++a) {
    edge[a] = D.hi[a] - D.lo[a];
    g.bits[a] = 0;
  }
  int axis_of[kGroupKeyBits];
  for (int i = 0; i < kGroupKeyBits; ++i) {
    int best = 0;
    for (int a = 1; a < kKeyAxes; ++a)
      if (edge[a] > edge[best]) best = a;
    axis_of[i] = best;
    edge[best] *= 0.5;
    ++g.bits[best];
  }
  int left[kKeyAxes];
  for (int a = 0; a < kKeyAxes; ++a) {
    left[a] = g.bits[a];
    g.target[a] = 0;
    double off = 0.0;   // the walk's coordinates are V^T x; D.lo is about the mean
    for (int k = 0; k < kDim; ++k) off += D.V[kDim * k + a] * D.mean[k];
    g.lo[a] = (float)(D.lo[a] + off);
    g.scale[a] = (float)((double)(1 << g.bits[a]) / std::max(D.hi[a] - D.lo[a], 1e-300));
  }
  for (int i = 0; i < kGroupKeyBits; ++i) {   // bit i of the key, from the top
    const int a = axis_of[i];
    const int b = --left[a];                  // bit b of the cell index of axis a
    g.target[a] |= (uint64_t)(kGroupKeyBits - 1 - i) << (4 * b);
  }
}

// ---------------------------------------------------------------------------
// Order: exclusive scan of the key histogram (one workgroup), then a scatter.
// Lanes with equal keys share one atomic, so that a batch whose states all
// fall into one cell does not queue on one address.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void order_scan_kernel(unsigned* __restrict__ hist, int n) {
  __shared__ unsigned wsum[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // n is a power of two, at least 256: n / 1024 cells per thread, four at a time
  const int quads = n >= 4096 ? n / 4096 : 1;
  constexpr int kMaxQuads = (1 << kGroupKeyBits) / 4096;
  uint4* h = reinterpret_cast<uint4*>(hist) + (int64_t)t * quads;
  const bool on = 4 * t * quads < n;
  uint4 v[kMaxQuads];
  unsigned s = 0;
#pragma unroll
  for (int i = 0; i < kMaxQuads; ++i)
    if (on && i < quads) {
      v[i] = h[i];
      s += v[i].x + v[i].y + v[i].z + v[i].w;
    }
  unsigned incl = s;
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  unsigned base = incl - s;
  for (int w = 0; w < wave; ++w) base += wsum[w];
#pragma unroll
  for (int i = 0; i < kMaxQuads; ++i)
    if (on && i < quads) {
      const uint4 c = v[i];
      h[i] = make_uint4(base, base + c.x, base + c.x + c.y, base + c.x + c.y + c.z);
      base += c.x + c.y + c.z + c.w;
    }
}

// Position of every query in the order, and the copies of its data there.
__global__ __launch_bounds__(256) void order_scatter_kernel(QueryPrep Q, int64_t m, Scale16 sc,
                                                            QueryPrep R, int* __restrict__ order) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool v = i < m;
  const unsigned p = cell_add(Q.hist, v ? (int)Q.key[i] : -1);
  if (!v) return;
  order[p] = (int)i;
  const double2* q = reinterpret_cast<const double2*>(Q.qw + 12 * i);
  double2* r = reinterpret_cast<double2*>(R.qw + 12 * (int64_t)p);
  double2 x[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    x[c] = q[c];
    r[c] = x[c];
  }
  const float4* y = reinterpret_cast<const float4*>(Q.yq + 12 * i);
  float4* z = reinterpret_cast<float4*>(R.yq + 12 * (int64_t)p);
#pragma unroll
  for (int c = 0; c < 3; ++c) z[c] = y[c];
  const double n2 = Q.qn2[i];
  const int bad = Q.invalid[i];
  R.qn2[p] = n2;
  R.u64[p] = Q.u64[i];
  R.u32[p] = Q.u32[i];
  R.invalid[p] = bad;
  if (!R.q16) return;
  float f[16], a = 0.0f;   // as load_query_column and near16 of the scan
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    f[c] = (float)((c & 1 ? x[c / 2].y : x[c / 2].x) * (double)sc.s);
    const float t = f[c] - sc.mean[c];
    a = fmaf(t, t, a);
  }
  f[12] = (float)(sqrt(n2) * (double)sc.s);
  f[13] = !bad && sc.far > 0.0f && a < sc.far * sc.far ? 1.0f : 0.0f;
  f[14] = f[15] = 0.0f;
  float4* w = reinterpret_cast<float4*>(R.q16 + 16 * (int64_t)p);
#pragma unroll
  for (int c = 0; c < 4; ++c) w[c] = make_float4(f[4 * c], f[4 * c + 1], f[4 * c + 2], f[4 * c + 3]);
}

// The queries of a list, copied in its order.
__global__ __launch_bounds__(256) void gather_queries_kernel(QueryPrep Q, QueryList L, int64_t m,
                                                             float u32_scale, QueryPrep R,
                                                             int* __restrict__ order) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= m) return;
  const int64_t i = list_query(L, p);
  order[p] = (int)i;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    R.qw[12 * p + c] = Q.qw[12 * i + c];
    R.yq[12 * p + c] = Q.yq[12 * i + c];
  }
  R.qn2[p] = Q.qn2[i];
  R.u64[p] = Q.u64[i];
  R.u32[p] = Q.u32[i] * u32_scale;
  R.invalid[p] = Q.invalid[i];
}

dd_status launch_gather(const QueryPrep& Q, QueryList L, int64_t m, float u32_scale,
                        const QueryPrep& sorted, int* order, hipStream_t st) {
  hipLaunchKernelGGL(gather_queries_kernel, dim3(grid1(m)), dim3(256), 0, st, Q, L, m, u32_scale,
                     sorted, order);
  DD_HIP(hipGetLastError());
  return DD_OK;
}

dd_status launch_order(const QueryPrep& Q, int64_t m, const Scale16& sc, const QueryPrep& sorted,
                       int* order, hipStream_t st) {
  hipLaunchKernelGGL(order_scan_kernel, dim3(1), dim3(1024), 0, st, Q.hist, 1 << Q.key_bits);
  hipLaunchKernelGGL(order_scatter_kernel, dim3(grid1(m, 64)), dim3(64), 0, st, Q, m, sc, sorted, order);
  DD_HIP(hipGetLastError());
  return DD_OK;
}

// ---------------------------------------------------------------------------
// Seed: a bound for every query from the points of one near tile, the tile
// that holds the query's own cell of the data's sort keys.  One wavefront per
// query: a 64-way search over the tiles' first keys, then the FP64 direct
// distances of the tile's rows.  (A greedy descent of the boxes from the top
// found far worse tiles: a bound that left 47 % of the (query, point) pairs at
// N = 2^24 where this one leaves 1 %, as boxes of many tiles overlap.)
// ---------------------------------------------------------------------------
__global__ void tile_key_kernel(const uint32_t* __restrict__ keys, int64_t n_tiles, int rows,
                                uint32_t* __restrict__ tkey) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_tiles) tkey[t] = keys[t * rows];
}

dd_status build_tile_keys(const uint32_t* sorted_keys, int64_t N, int rows, DevBuf& tkey,
                          hipStream_t st) {
  const int64_t n = (N + rows - 1) / rows;
  DD_TRY(tkey.alloc(sizeof(uint32_t) * (size_t)n));
  hipLaunchKernelGGL(tile_key_kernel, dim3(grid1(n)), dim3(256), 0, st, sorted_keys, n, rows,
                     tkey.as<uint32_t>());
  DD_HIP(hipGetLastError());
  return DD_OK;
}

struct SortCells {          // the sort keys' grid, in the coordinates V^T x
  float lo[kKeyAxes], scale[kKeyAxes];
};

__global__ __launch_bounds__(256) void seed_kernel(const uint32_t* __restrict__ tkey,
                                                   int64_t n_tiles, int rows, SortCells G,
                                                   const double* __restrict__ w64, int64_t N,
                                                   int64_t m, const double* __restrict__ qw,
                                                   const float* __restrict__ yq,
                                                   const int* __restrict__ invalid, double u32_scale,
                                                   double* __restrict__ u64,
                                                   float* __restrict__ u32) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t q = (int64_t)blockIdx.x * 4 + wave;
  if (q >= m || invalid[q]) return;
  uint32_t key = 0;
#pragma unroll
  for (int a = 0; a < kKeyAxes; ++a) {
    const float c = floorf((yq[12 * q + a] - G.lo[a]) * G.scale[a]);
    const float top = (float)((1 << kKeyBits) - 1);
    const int cell = c > 0.0f ? (c < top ? (int)c : (1 << kKeyBits) - 1) : 0;
#pragma unroll
    for (int b = 0; b < kKeyBits; ++b) key |= (uint32_t)((cell >> b) & 1) << (b * kKeyAxes + a);
  }
  int64_t at = 0, n = n_tiles;   // the last tile of [at, at + n) whose first key is <= key
  while (n > 1) {
    const int64_t step = (n + 63) / 64, i = at + lane * step;
    const uint64_t le = __ballot(lane * step < n && tkey[lane * step < n ? i : at] <= key);
    const int64_t skip = le ? (int64_t)(__popcll(le) - 1) * step : 0;
    at += skip;
    n = min(step, n - skip);
  }
  double x[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) x[k] = qw[12 * q + k];
  double best = INFINITY;
  const int64_t end = min((at + 1) * rows, N);
  for (int64_t i = at * rows + lane; i < end; i += 64) {
    double d = 0.0;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double t = x[k] - w64[12 * i + k];
      d = fma(t, t, d);
    }
    best = fmin(best, d);
  }
  for (int off = 32; off > 0; off >>= 1) best = fmin(best, __shfl_xor(best, off));
  if (lane == 0) {
    // as the warm start's bound: the FP64 sum carries at most ~13 ulp
    const double ub = best * (1.0 + 0x1p-40) + 1e-300;
    if (ub < u64[q]) u64[q] = ub;
    const float u = __double2float_ru(sqrt(ub) * (1.0 + 0x1p-40) * u32_scale);
    if (u < u32[q]) u32[q] = u;
  }
}

dd_status launch_seed(const Dataset& D, const QueryPrep& Q, int64_t m, double u32_scale,
                      hipStream_t st) {
  if (m <= 0) return DD_OK;
  if (!D.tkey.p || !Q.yq) return set_error(DD_ERR_ARG, "seed: no tile keys");
  SortCells G;
  for (int a = 0; a < kKeyAxes; ++a) {
    double off = 0.0;   // y = V^T x; the grid's origin D.lo is relative to the mean
    for (int k = 0; k < kDim; ++k) off += D.V[kDim * k + a] * D.mean[k];
    G.lo[a] = (float)(D.lo[a] + off);
    G.scale[a] = (float)((double)(1 << kKeyBits) / (D.hi[a] - D.lo[a]));
  }
  hipLaunchKernelGGL(seed_kernel, dim3(grid1(m, 4)), dim3(256), 0, st, D.tkey.as<uint32_t>(),
                     D.boxes.n_tiles, D.boxes.rows, G, D.w64.as<double>(), D.N, m, Q.qw, Q.yq,
                     Q.invalid, u32_scale, Q.u64, Q.u32);
  DD_HIP(hipGetLastError());
  return DD_OK;
}

// ---------------------------------------------------------------------------
// Cull: masks of the tiles to scan.  A mask word has 32 bits, one per
// SUB queries.  A wavefront takes 64 queries and `cw` units of 2^unit_log2 tiles
// (a chunk of 64, or less where there would be few wavefronts).  It tests the
// units' chunk boxes, then the tile boxes of the units left (one per lane),
// against its queries as a group; the tiles left are tested one by one with a
// query per lane, and the lanes' votes are folded to a bit per SUB queries.
//
// The group test takes 16 queries at a time (64 have so wide a bounding box that
// 11.5 thousand of 65536 tiles passed where 1.4 thousand were wanted) and uses
// the first six axes only: data lie near a surface of six dimensions (a stress
// for each strain), so a tile's extent is in those, while every tile has nearly
// the data set's whole extent on the others.  A query's distance e to that
// extent is owed to every tile, so the six-axis gap of a tile that matters is
// at most sqrt(U^2 - e^2), maximal over the group.
// ---------------------------------------------------------------------------
constexpr int kMaxCw = 8;
constexpr int kGroupAxes = 6;

template <int SUB>
__global__ __launch_bounds__(256) void cull_kernel(
    const float* __restrict__ box, int64_t n_tiles, const float* __restrict__ cbox,
    int unit_log2, int64_t n_units, const float* __restrict__ root, int cw, int64_t m, int groups,
    int words, const float* __restrict__ yq, const double* __restrict__ qn2,
    const float* __restrict__ u32, float u_scale, const int* __restrict__ invalid, float xmax,
    uint32_t* __restrict__ mask) {
  constexpr int BITS = 64 / SUB;   // mask bits of a wavefront
  const int lane = threadIdx.x & 63;
  const unsigned wave = blockIdx.x * 4 + (unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = (int)(wave % (unsigned)groups);
  const int64_t u_first = (int64_t)(wave / (unsigned)groups) * cw;
  if (u_first >= n_units) return;
  const int64_t p = (int64_t)group * 64 + lane;
  const bool v = p < m && !invalid[p < m ? p : 0];
  float y[12], U = -INFINITY, slack = 0.0f, r2 = -INFINITY;
  // squares past the FP32 range say nothing: such a query keeps every tile, with
  // coordinates that leave no inf - inf in the tests (a NaN there drops the tile)
  const float reach = v ? (float)sqrt(qn2[p]) + xmax : 0.0f;
  const bool all = !(reach < 0x1p60f);
#pragma unroll
  for (int a = 0; a < 12; ++a) y[a] = v && !all ? yq[12 * p + a] : 0.0f;
  if (v) {
    if (!all) {
      slack = kEps22 * reach + 1e-30f;
      U = u32[p] * u_scale;
      float e2 = 0.0f;
#pragma unroll
      for (int a = kGroupAxes; a < 12; ++a) {
        const float g = fmaxf(fmaxf(root[a] - y[a], y[a] - root[12 + a]), 0.0f);
        e2 = fmaf(g, g, e2);
      }
      // the tile test below is sqrt(s) shrink - slack <= U
      const float t = (U + slack) * (1.0f + 0x1p-18f);
      r2 = t * t * (1.0f + 0x1p-16f) - e2 * (1.0f - 0x1p-16f) + 1e-37f;
    } else {
      U = r2 = INFINITY;
    }
  }
  if (!__any(r2 != -INFINITY)) return;   // no query here
  // bounds of each row of 16 queries, uniform
  float glo[4][kGroupAxes], ghi[4][kGroupAxes], gr2[4];
#pragma unroll
  for (int a = 0; a < kGroupAxes; ++a) {
    const float l = row_min(v ? y[a] : INFINITY), h = row_max(v ? y[a] : -INFINITY);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      glo[r][a] = lane_f(l, 16 * r);
      ghi[r][a] = lane_f(h, 16 * r);
    }
  }
  {
    const float r = row_max(r2);
#pragma unroll
    for (int i = 0; i < 4; ++i) gr2[i] = lane_f(r, 16 * i);
  }
  // lane's box b of B may hold a near point of the group
  auto near_group = [&](const float* B, int64_t b) __attribute__((always_inline)) {
    float lo[8], hi[8];
    const float4* r = reinterpret_cast<const float4*>(B + 24 * b);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float4 l = r[i], h = r[3 + i];
      lo[4 * i] = l.x, lo[4 * i + 1] = l.y, lo[4 * i + 2] = l.z, lo[4 * i + 3] = l.w;
      hi[4 * i] = h.x, hi[4 * i + 1] = h.y, hi[4 * i + 2] = h.z, hi[4 * i + 3] = h.w;
    }
    bool near = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float s = 0.0f;
#pragma unroll
      for (int a = 0; a < kGroupAxes; ++a) {
        const float g = fmaxf(fmaxf(lo[a] - ghi[k][a], glo[k][a] - hi[a]), 0.0f);
        s = fmaf(g, g, s);
      }
      near = near || s <= gr2[k];
    }
    return near;
  };
  const int n_here = (int)min((int64_t)cw, n_units - u_first);
  uint64_t units = __ballot(lane < n_here &&
                            near_group(cbox, (u_first + (lane < n_here ? lane : 0)) >> (6 - unit_log2)));
  const int word = group * BITS / 32, shift = group * BITS % 32;
  while (units) {
    const int64_t t0 = (u_first + __builtin_ctzll(units)) << unit_log2, t = t0 + lane;
    units &= units - 1;
    const bool in = (lane >> unit_log2) == 0 && t < n_tiles;
    uint64_t todo = __ballot(near_group(box, in ? t : t0) && in);
    unsigned mine = 0;
    while (todo) {
      const int j = __builtin_ctzll(todo);
      todo &= todo - 1;
      // the box by scalar loads; three of four tests end after six axes
      const auto* b = uniform_ptr(box + 24 * (t0 + j));
      float s = 0.0f;
#pragma unroll
      for (int a = 0; a < kGroupAxes; ++a) {
        const float g = fmaxf(fmaxf(b[a] - y[a], y[a] - b[12 + a]), 0.0f);
        s = fmaf(g, g, s);
      }
      if (!__any(s <= r2)) continue;
#pragma unroll
      for (int a = kGroupAxes; a < 12; ++a) {
        const float g = fmaxf(fmaxf(b[a] - y[a], y[a] - b[12 + a]), 0.0f);
        s = fmaf(g, g, s);
      }
      const uint64_t hit = __ballot(__builtin_amdgcn_sqrtf(s) * kLbShrink - slack <= U);
      unsigned f = 0;
#pragma unroll
      for (int i = 0; i < BITS; ++i)
        f |= ((hit >> (SUB * i)) & ((1ull << SUB) - 1ull)) ? 1u << i : 0u;
      if (lane == j) mine = f;
    }
    if (mine) atomicOr(&mask[t * words + word], mine << shift);   // the masks start at zero
  }
}

// Plan: the tiles with a bit set, cut into work entries of about equal numbers
// of groups, as a few tiles (those whose rows straddle distant cells) are
// wanted by nearly every group: without the cut, their workgroups end long after
// the others (385 us against 209 us for the FP64 scan at N = 10^6, m = 4096).
// One lane per tile; entry = (tile, part | parts << 16).  (Listing the tiles in
// the cull, with a flag word per chunk, queued on those words: 50 us against 31
// us at N = 10^6, m = 4096.)
__global__ __launch_bounds__(256) void plan_kernel(const uint32_t* __restrict__ mask, int words,
                                                   int64_t n_tiles, int part,
                                                   uint2* __restrict__ entry,
                                                   unsigned* __restrict__ n_entry) {
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * 4;
  for (int64_t k0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64; k0 < n_tiles; k0 += waves * 64) {
    const int64_t t = k0 + lane;
    int c = 0;
    if (t < n_tiles) {
      const uint32_t* row = mask + t * words;
      if ((words & 3) == 0) {
        for (int w = 0; w < words; w += 4) {
          const uint4 q = *reinterpret_cast<const uint4*>(row + w);
          c += __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
        }
      } else {
        for (int w = 0; w < words; ++w) c += __popc(row[w]);
      }
    }
    const int parts = min((c + part - 1) / part, kMaskParts);
    int incl = parts;
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    unsigned at = 0;   // one atomic per wavefront: they queue on one address
    if (lane == 63 && incl) at = atomicAdd(n_entry, (unsigned)incl);
    at = (unsigned)__shfl((int)at, 63) + (unsigned)(incl - parts);
    for (int i = 0; i < parts; ++i)
      entry[at + i] = make_uint2((uint32_t)t, (unsigned)i | ((unsigned)parts << 16));
  }
}

dd_status launch_plan(const TileMasks& M, int64_t n_tiles, bool left, hipStream_t st) {
  // groups per entry: at least 32, at most kMaskParts entries per tile
  const int part = std::max(32, 32 * M.words / kMaskParts);
  const unsigned blocks = (unsigned)std::min<int64_t>((n_tiles + 255) / 256, 2048);
  hipLaunchKernelGGL(plan_kernel, dim3(blocks), dim3(256), 0, st, left ? M.left : M.mask, M.words,
                     n_tiles, part, M.entry, M.n_entry + (left ? 1 : 0));
  DD_HIP(hipGetLastError());
  return DD_OK;
}

// Masks and entry counters to zero.
__global__ void clear_kernel(uint4* __restrict__ p, int64_t n4) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n4) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

dd_status launch_cull(const Dataset& D, const TileBoxes& B, const QueryPrep& Q, int64_t m,
                      float u_scale, const TileMasks& M, hipStream_t st) {
  if (m <= 0) return DD_OK;
  if (B.n_tiles < 1 || !Q.yq) return set_error(DD_ERR_ARG, "cull: no tile boxes");
  const int64_t n_tiles = B.n_tiles, n_chunks = cull_chunks(n_tiles);
  if (M.words != mask_words(m, M.sub)) return set_error(DD_ERR_ARG, "cull: mask words");
  const int64_t n4 = (int64_t)(M.zero_bytes / 16);
  hipLaunchKernelGGL(clear_kernel, dim3(grid1(n4)), dim3(256), 0, st,
                     reinterpret_cast<uint4*>(M.zero), n4);
  const float xmax = __builtin_nextafterf((float)D.xmax, INFINITY);
  // units per wavefront: as many as leave about 16384 wavefronts; smaller units
  // where single chunks leave fewer than 4096
  const int groups = (int)((m + 63) / 64);
  const int cw = (int)std::max<int64_t>(1, std::min<int64_t>(kMaxCw, groups * n_chunks / 16384));
  int unit_log2 = 6;
  while (unit_log2 > 2 && cw == 1 && (groups * n_chunks << (6 - unit_log2)) < 4096) --unit_log2;
  const int64_t n_units = (n_tiles + (1 << unit_log2) - 1) >> unit_log2;
  const dim3 grid((unsigned)((groups * ((n_units + cw - 1) / cw) + 3) / 4));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, B.tile.as<float>(), n_tiles,
                       B.chunk.as<float>(), unit_log2, n_units, B.root.as<float>(), cw, m, groups,
                       M.words, Q.yq, Q.qn2, Q.u32, u_scale, Q.invalid, xmax, M.mask);
  };
  if (M.sub == 16) go(cull_kernel<16>);
  else if (M.sub == 32) go(cull_kernel<32>);
  else return set_error(DD_ERR_ARG, "cull: mask shape");
  DD_HIP(hipGetLastError());
  return DD_OK;
}

}  // namespace dd
