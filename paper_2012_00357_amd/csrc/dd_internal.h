// Internal declarations shared by the libdd translation units (host side).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <list>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/dd.h"
#include "pack16.h"

namespace dd {

// ---------------------------------------------------------------------------
// Error handling
// ---------------------------------------------------------------------------
dd_status set_error(dd_status st, const std::string& msg);

#define DD_HIP(call)                                                                      \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return ::dd::set_error(e_ == hipErrorOutOfMemory ? DD_ERR_OOM : DD_ERR_DEVICE,      \
                             std::string(#call) + ": " + hipGetErrorString(e_));          \
  } while (0)

#define DD_TRY(expr)                  \
  do {                                \
    dd_status s_ = (expr);            \
    if (s_ != DD_OK) return s_;       \
  } while (0)

// Device memory of the host objects below.  A released block of 1 MiB and more that
// was allocated in a KeepScope is kept for the next such allocation of its size:
// memory given to the driver is cleared by it before it is given out again, at about
// 40 GB/s, and once a process (or those before it) has been through the device's
// memory, every creation waits for that (2^25 points with BF16 pack and box tree, 6.5
// GB: 157 to 173 ms where the driver has no clean memory left, 20 where it has, 16
// from here).
// At most kPoolBytes are kept per device, each block for at most kPoolSeconds after
// its release (a thread of the library frees it then, whether the program calls the
// library or not); an allocation that fails frees them all and is tried again, and so
// does dd_dataset_destroy(NULL).  A block is kept only once the device has
// finished with it, so that any stream may have it next.  The scopes are the calls that
// create a data set, project or solve; what a server allocates goes back to the
// driver at once, as its budget says.
constexpr size_t kPoolBytes = (size_t)8 << 30;
constexpr int kPoolSeconds = 5;
class KeepScope {   // of the thread's allocations
 public:
  KeepScope();
  ~KeepScope();
  KeepScope(const KeepScope&) = delete;
  KeepScope& operator=(const KeepScope&) = delete;

 private:
  bool before;
};
hipError_t device_alloc(void** p, size_t n);
void device_free(void* p);
void device_pool_trim();   // frees every kept block
// Returns to the driver what the library holds on the device without using it: the
// idle temporaries of the creation that runs on this thread, and every kept block.
void device_give_back();
// An allocation (a function that returns its hipError_t), tried again after that if
// there was no memory for it; leaves no error behind.
template <class F>
hipError_t alloc_or_give_back(F alloc) {
  hipError_t e = alloc();
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    device_give_back();
    e = alloc();
  }
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

// Device buffer owned by a host object; released in the destructor.
struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  bool owned = true;   // false: a view into memory another DevBuf owns
  DevBuf() = default;
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
  ~DevBuf() { release(); }
  dd_status alloc(size_t n);
  void view(void* ptr, size_t n) {
    release();
    p = ptr;
    bytes = n;
    owned = false;
  }
  void release();
  template <class T> T* as() const { return static_cast<T*>(p); }
};

// Device blocks of one creation's temporaries, all of whose work is on one stream:
// a TempBuf that ends hands its block back for the next one without waiting (the
// stream orders the uses), where a hipFree waits for the device and costs with its
// hipMalloc about 30 us.  Blocks of kLeast are cut from slabs of kKeep; blocks above
// kKeep are freed at once; the rest goes with the pool, at the end of the creation,
// or when an allocation on its thread finds no memory (device_give_back).
class TempPool {
 public:
  TempPool();
  TempPool(const TempPool&) = delete;
  TempPool& operator=(const TempPool&) = delete;
  ~TempPool();
  dd_status take(size_t n, void** p, size_t* cap);
  void put(void* p, size_t cap);
  void trim();   // frees the idle blocks, and the slabs if none of their blocks is in use

 private:
  static constexpr size_t kLeast = (size_t)1 << 20, kKeep = (size_t)16 << 20;
  TempPool* before;   // the thread's pool until this one ends
  std::vector<std::pair<size_t, void*>> idle;   // (size, block)
  std::vector<void*> slabs;
};

struct TempBuf {
  TempPool& pool;
  void* p = nullptr;
  size_t bytes = 0, cap = 0;
  explicit TempBuf(TempPool& t) : pool(t) {}
  TempBuf(const TempBuf&) = delete;
  TempBuf& operator=(const TempBuf&) = delete;
  ~TempBuf() { release(); }
  dd_status alloc(size_t n) {
    release();
    if (n == 0) return DD_OK;
    const dd_status rc = pool.take(n, &p, &cap);
    if (rc == DD_OK) bytes = n;
    return rc;
  }
  void release() {
    if (p) pool.put(p, cap);
    p = nullptr;
    bytes = cap = 0;
  }
  void swap(TempBuf& o) {
    std::swap(p, o.p);
    std::swap(bytes, o.bytes);
    std::swap(cap, o.cap);
  }
  template <class T> T* as() const { return static_cast<T*>(p); }
};

// ---------------------------------------------------------------------------
// Small dense linear algebra on the host (6x6 / 12x12)
// ---------------------------------------------------------------------------
// Cholesky C = L L^T (row-major, lower); returns false if not SPD.
bool cholesky6(const double* C, double* L);
// Inverse of a lower-triangular 6x6 matrix (row-major).
void lower_inverse6(const double* L, double* Linv);
// Symmetric eigen-decomposition (cyclic Jacobi); eigenvalues descending,
// eigenvectors as columns of V (row-major n x n).
void sym_eigen(int n, const double* A, double* evals, double* V);

// ---------------------------------------------------------------------------
// Dataset
// ---------------------------------------------------------------------------
constexpr int kDim = 12;           // phase-space dimension 2M (M = 6 Voigt components)
constexpr int kKeyAxes = 6;        // principal axes used for the spatial order
constexpr int kKeyBits = 5;        // bits per axis of its sort keys
constexpr int kAnnLeaf = 64;       // points per ANN leaf (one wavefront)
constexpr int kAnnFan = 64;        // children per ANN tree node (one wavefront)
constexpr int kCounterSlots = 32;  // ANN walk statistics: slots, each on its own 128-byte line
constexpr int kCounterStride = 16; // u64 per slot (8 used)
constexpr int kKmtRecord = 20;     // floats per k-means tree child record (80 B)

// projection modes that walk a tree (warm starts, budgets, skipping)
inline bool walk_mode(int mode) { return mode == DD_ANN || mode == DD_KMEANS; }
// Sizes of the data sets with a tree that also hold a 16-bit pack (32 bytes a
// point) for exact searches by scan (scan_for_walk).
constexpr int64_t kTreeScanMin = (int64_t)1 << 13, kTreeScanMax = (int64_t)1 << 24;
constexpr int kAnnMaxLevels = 6;   // 64^6 leaves exceed any N <= 2^31 - 1

// The operator of P_C kept for one mesh and Dirichlet pattern: K^-1, padded to n_pad
// rows and columns, row-major, or the block elimination of its node planes.
struct DenseInverse {
  int nx = 0, ny = 0, nz = 0;
  double hx = 0, hy = 0, hz = 0;
  std::vector<uint8_t> mask;
  int64_t n = 0, n_pad = 0;
  bool planes = false;   // inv holds the elimination (dense.hip)
  DevBuf inv;
};
constexpr int64_t kDenseMaxDof = 16384;               // meshes up to here always keep one
constexpr int64_t kDenseCacheBytes = (int64_t)4 << 30;  // operators kept per dataset

// Device scratch of the projection, reused from call to call.  A call takes an
// idle arena (or makes one), carves its buffers out of the arena's block and
// hands the arena back when it returns, recording `done` on its stream; the
// next call that takes the arena makes its own stream wait for `done`, so the
// reuse is stream-ordered on any stream.  Requests beyond the block are
// allocated stream-ordered and freed on return, and the block then grows (up
// to kArenaKeepBytes) so that a call of the same size fits next time.
struct ScratchArena {
  void* block = nullptr;
  size_t bytes = 0;
  hipEvent_t done = nullptr;   // recorded on the last user's stream
  uint32_t* pinned = nullptr;  // kArenaPinnedWords of pinned host memory (small readbacks)
  ScratchArena() = default;
  ScratchArena(const ScratchArena&) = delete;
  ScratchArena& operator=(const ScratchArena&) = delete;
  ~ScratchArena();
};
constexpr size_t kArenaKeepBytes = (size_t)1 << 30;  // largest block an arena keeps
constexpr int kArenaKeep = 8;                         // idle arenas kept per dataset
constexpr int kArenaPinnedWords = 64;

// Boxes of the scans' tiles (csrc/cull.hip): per tile of `rows` consecutive rows
// of the sorted packs and per chunk of 64 tiles, float lo[12], hi[12] in
// principal-axis coordinates y = V^T x, rounded outward.
struct TileBoxes {
  DevBuf tile, chunk, root;   // root: the box of all points
  int64_t n_tiles = 0;
  int rows = 0;
  size_t bytes() const { return tile.bytes + chunk.bytes + root.bytes; }
};

// Cells by which a batch's queries are grouped: bit b of the cell index on axis
// a goes to bit (target[a] >> 4 b) & 15 of the key.
constexpr int kGroupKeyBits = 15;
struct GroupCells {
  float lo[kKeyAxes];
  float scale[kKeyAxes];    // cells per unit length
  int bits[kKeyAxes];
  uint64_t target[kKeyAxes];
};

struct Dataset {
  int device = 0;
  int64_t N = 0;
  uint32_t packs = 0;
  double C[36];
  double F[36];    // strain whitening F = L^T  (F^T F = C)
  double G[36];    // stress whitening G = L^-1 (G^T G = C^-1)
  // spatial order
  DevBuf perm;     // uint32 [N]: sorted position -> original index
  DevBuf iperm;    // uint32 [N]: original index -> sorted position
  // FP64 pack (sorted order), padded to n_pad64 rows
  int64_t n_pad64 = 0;
  DevBuf w64;      // double [n_pad64][12]
  DevBuf n64;      // double [n_pad64]  |x|^2 (padding rows: +inf)
  double xmax = 0; // max_j |x_j|
  // FP32 pack
  int64_t n_pad32 = 0;
  DevBuf w32;      // float [n_pad32][12]
  DevBuf n32;      // float [n_pad32] |x|^2 of the FP32 values (padding: +inf)
  double xmax32 = 0;
  // 16-bit packs (tile-centred), in coordinates scaled by sc16.s (a power of two)
  int tile = 256;
  int64_t n_tiles = 0;
  DevBuf centre;   // float [n_tiles][12] scaled tile centres
  DevBuf radius;   // float [n_tiles]  upper bound of |s x_j - c_T| over the tile
  Scale16 sc16{1.0f, 0.0f, {0}};   // scale and scaled data mean (far set per format)
  double span16 = 0.0;             // max_T |c_T - scaled mean|
  DevBuf wbf16;    // uint16 [n_tiles*tile][16]
  DevBuf wfp16;    // uint16 [n_tiles*tile][16]
  // principal axes of the whitened data (sample estimate): V[12*k + a] is
  // component k of axis a, axes by decreasing variance
  double V[kDim * kDim];
  DevBuf vrot;     // double [144]: V on the device (the walks rotate their queries with it)
  double mean[kDim];
  double lo[kKeyAxes], hi[kKeyAxes];
  GroupCells cells{};
  TileBoxes boxes;     // tiles of the FP64 and FP32 scans (kTile64 rows)
  TileBoxes boxes16;   // tiles of the 16-bit scans (tile rows)
  DevBuf tkey;         // uint32 [boxes.n_tiles]: sort key of each tile's first row
  // ANN box tree over the sorted order: level 0 boxes bound leaves of kAnnLeaf
  // consecutive points, level k+1 boxes bound kAnnFan boxes of level k; boxes
  // are float lo[12], hi[12] in principal-axis coordinates y = V^T x, rounded
  // outward.  The top stored level has at most kAnnFan boxes.
  DevBuf ann_box[kAnnMaxLevels];
  int64_t ann_n[kAnnMaxLevels] = {0};
  int ann_levels = 0;
  // compact leaves read by the walk, in principal-axis coordinates y = V^T x:
  // per leaf the FP32 centre c (mean of its points), radius r (max |y - c|,
  // rounded up, at least 2^-20) and its box quantised to 8 bits inside its
  // parent's box (rounded outward); per point the FP16 scaled offset (y - c) / r
  // (round to nearest)
  DevBuf ann_meta;   // float [n_leaf][16]: c[12], r, 1/r, 0, 0
  DevBuf ann_q0;     // uint8 [n_leaf][24]: lo[12], hi[12] in 1/255 of the parent box
  DevBuf ann_h16;    // uint16 [n_leaf*64][12]
  // k-means tree (DD_PACK_KMEANS): recursive 4-means, stored as a 64-ary cut,
  // each stored node with up to 64 child records (ball of the child's points:
  // FP32 centre c, radius >= max |x - c|; their box in principal-axis
  // coordinates, quantised to bytes inside the node's own box; code
  // (1 << 28 | node) or leaf); leaves of at most 64 points in padded 64-slot
  // blocks, compact as above
  int64_t kmt_nodes = 0, kmt_leaves = 0, kmt_records = 0;
  int kmt_rounds = 0;
  DevBuf kmt_node;   // int2 [nodes]: first child record, end of its records (node 0: root)
  DevBuf kmt_nbox;   // float [nodes][24]: box lo[12], hi[12] of the node's points (rounded outward)
  DevBuf kmt_child;  // float [records][kKmtRecord]: c[12], r, code (bits), box lo[12], hi[12] as
                     // bytes inside the owner node's box (lo rounded down, hi up)
  DevBuf kmt_meta;   // float [leaves][16]: c[12], r, 1/r, count (bits), 0
  DevBuf kmt_h16;    // uint16 [leaves*64][12]; empty slots +inf
  DevBuf kmt_pos;    // uint32 [leaves*64]: sorted position of each slot (empty: 0xFFFFFFFF)
  DevBuf kmt_slot;   // uint32 [N]: slot of each sorted position

  // operators of dd_solve, most recently used first (see DenseInverse)
  mutable std::mutex cache_mu;
  mutable std::list<std::shared_ptr<DenseInverse>> pc_cache;
  // idle projection scratch arenas (see ScratchArena); arena_bytes counts the
  // blocks of idle and busy arenas
  mutable std::mutex arena_mu;
  mutable std::vector<std::unique_ptr<ScratchArena>> arenas;
  mutable int64_t arena_bytes = 0;

  int64_t device_bytes() const;
};

// Boxes of tiles of `rows` rows, as unions of the boxes of `from` where its rows
// divide them, else from the FP64 pack.
dd_status build_tile_boxes(const Dataset& D, int rows, const TileBoxes* from, TileBoxes& B,
                           hipStream_t st);
// Sort key of the first row of every tile of `rows` rows.
dd_status build_tile_keys(const uint32_t* sorted_keys, int64_t N, int rows, DevBuf& tkey,
                          hipStream_t st);
// D.cells from the extent of the data on the principal axes.
void choose_group_cells(Dataset& D);

// Builds the k-means tree of DD_PACK_KMEANS over D's sorted FP64 pack.
dd_status build_kmeans_tree(Dataset& D, TempPool& pool, hipStream_t st);

}  // namespace dd

struct dd_dataset {
  dd::Dataset d;
};
