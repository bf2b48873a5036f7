// Projection kernels: launch interfaces (host side).
#pragma once
#include "dd_internal.h"

namespace dd {

// Whitened queries and per-query search state, produced by prepare_queries.
struct QueryPrep {
  double* qw = nullptr;     // [m][12] whitened queries (zero rows for invalid states)
  double* qn2 = nullptr;    // [m] |q|^2
  double* u64 = nullptr;    // [m] FP64-path initial bound on min d (warm start) or +inf
  float* u32 = nullptr;     // [m] sqrt-space initial bound (warm start) or +inf, in the
                            // scaled coordinates of the 16-bit scans in those modes
  int* invalid = nullptr;   // [m] 1 for non-finite states
  float* yq = nullptr;      // [m][12] queries on the principal axes of the dataset's boxes
                            // and trees, or nullptr (not wanted)
  float* q16 = nullptr;     // [m][16] 16-bit culled scans: scaled coordinates, scaled |q|, 1 or 0
                            // (0: the scan leaves the query to the fallback)
  // grouping order (culled scans; nullptr elsewhere): the cell of each query
  // and the number of queries per cell (zero before the preparation)
  uint16_t* key = nullptr;  // [m]
  unsigned* hist = nullptr; // [1 << key_bits]
  int key_bits = 0;
};

// Candidate lists written by the scans: slot = (list position * S + split) * P + part.
struct CandBuf {
  float* lb = nullptr;      // [slots][K] lower bound of the candidate (scan's own units)
  uint32_t* j = nullptr;    // [slots][K] sorted data position
  int* count = nullptr;     // [slots] number of entries; bit 30 set = overflowed
  float* U = nullptr;       // [positions][S] upper bound of the minimum (scan's units), or
                            // nullptr: every entry is within the final bound
  int K = 0, S = 0, P = 0;
};
constexpr int kOverflowBit = 1 << 30;

// Query list: the identity over [0, m) (list == nullptr), list[0..*count), or
// list[0..m) (count == nullptr).
struct QueryList {
  const int* list = nullptr;
  const int* count = nullptr;   // device counter
  int64_t m = 0;                // capacity, or the length without a counter
};

// Tiles a culled scan takes (csrc/cull.hip), for up to kMaskQueries queries:
// per tile `words` mask words of 32 bits, one bit per `sub` queries, and the
// work entries of the tiles with a bit set.  `zero` spans what starts a call at
// zero (masks and entry counters).
constexpr int64_t kMaskQueries = 65536;
constexpr int kMaskParts = 8;   // work entries per tile at most
struct TileMasks {
  void* zero = nullptr;
  size_t zero_bytes = 0;
  uint32_t* mask = nullptr;      // [tiles][words]
  uint32_t* left = nullptr;      // [tiles][words] groups the scan leaves for its extraction
  uint2* entry = nullptr;        // [min(words, kMaskParts) * tiles] (launch_plan)
  unsigned* n_entry = nullptr;   // entries under mask, entries under left
  int words = 0, sub = 0;
  // statistics, or nullptr: (query, point) pairs of the scan, (group, tile) items
  // of its extraction
  unsigned long long* pairs = nullptr;
  unsigned* items = nullptr;
};
inline int64_t cull_chunks(int64_t n_tiles) { return (n_tiles + 63) / 64; }
inline int mask_words(int64_t m, int sub) { return (int)((m + 32 * sub - 1) / (32 * sub)); }

struct Outputs {
  int64_t* idx = nullptr;       // [m] original index
  double* dist = nullptr;       // [m] 1/2 d^2 or nullptr
};

// Whiten m states (or take them as already whitened), |q|^2, coordinates on the
// principal axes (with Q.yq), grouping cells (with Q.key), warm-start bounds
// (the sqrt-space one multiplied by u32_scale: the 16-bit scans' scale, else 1).
dd_status prepare_queries(const Dataset& D, const double* states, bool whitened, int64_t m,
                          const int64_t* warm, double u32_scale, QueryPrep& Q, hipStream_t st);

// order[] = the m queries sorted by cell (Q.hist becomes the cells' ends), and
// their data in that order in `sorted`.
// With sorted.q16 also that, for the scale and reach of sc.
dd_status launch_order(const QueryPrep& Q, int64_t m, const Scale16& sc, const QueryPrep& sorted,
                       int* order, hipStream_t st);
// The same for the m queries of a list, in its order (no cells needed); u32
// times u32_scale.
dd_status launch_gather(const QueryPrep& Q, QueryList L, int64_t m, float u32_scale,
                        const QueryPrep& sorted, int* order, hipStream_t st);
// Lower Q.u64 and Q.u32 (the latter times u32_scale) of the m queries to the
// distance of the nearest point of one near tile.
dd_status launch_seed(const Dataset& D, const QueryPrep& Q, int64_t m, double u32_scale,
                      hipStream_t st);
// Masks of the tiles of B that may hold a point within a query's bound
// Q.u32 u_scale, for m <= kMaskQueries queries.
dd_status launch_cull(const Dataset& D, const TileBoxes& B, const QueryPrep& Q, int64_t m,
                      float u_scale, const TileMasks& M, hipStream_t st);

// Work entries of the tiles with a bit set in M.mask (their number: M.n_entry[0])
// or in M.left (M.n_entry[1]).
dd_status launch_plan(const TileMasks& M, int64_t n_tiles, bool left, hipStream_t st);

// FP64 MFMA scan (expanded form) over the list; fills cb (P = 4, d-space bounds).
dd_status launch_scan64(const Dataset& D, const QueryPrep& Q, QueryList L, int64_t list_len,
                        const CandBuf& cb, hipStream_t st);
// The culled FP64 scan of m sorted queries: the tiles of M (sub = 16) lower
// Q.u64 to the final bounds, then every point within its query's bound is
// appended to cb (S = 1, P = 1, counts claimed atomically, from zero).
dd_status launch_scan64_culled(const Dataset& D, const QueryPrep& Q, int64_t m, const TileMasks& M,
                               const CandBuf& cb, hipStream_t st);
// The same in FP32 (sub = 32; Q.u64 falls to FP32 bounds) and in 16 bits (sub =
// 32, the tiles of D.boxes16, Q.u32 the scaled square-root bound).
dd_status launch_scan32_culled(const Dataset& D, const QueryPrep& Q, int64_t m, const TileMasks& M,
                               const CandBuf& cb, hipStream_t st);
// The 16-bit scans' scale and the radius around the data's mean they take
// queries from.
Scale16 scan16_reach(const Dataset& D, bool fp16);
dd_status launch_scan16_culled(const Dataset& D, bool fp16, const QueryPrep& Q, int64_t m,
                               const TileMasks& M, const CandBuf& cb, hipStream_t st);
// FP32 MFMA scan (expanded form, stored norms as the accumulator input) over the
// list; fills cb (P = 2, d-space bounds), like the FP64 scan.
dd_status launch_scan32(const Dataset& D, const QueryPrep& Q, QueryList L, int64_t list_len,
                        const CandBuf& cb, hipStream_t st);
// 16-bit MFMA scan over tile-centred data (sqrt-space bounds), in phases:
//   kBound    streaming pass: U_out[p][S] = split bounds (tiles visited with stride)
//   kMark     the same, also logging work items (query group, tile) that may hold
//             candidates under the running bound
//   kExtract  recompute the logged items and append every point whose lower bound
//             is <= the query's final bound Q->u32 to cb (slot p*2 + half, counts
//             claimed atomically; cb.count must start at zero)
struct WorkItem {
  uint32_t group;   // list position of the group's first query / 32
  uint32_t tile;
};
struct Scan16Call {
  enum Phase { kBound = 0, kMark = 1, kExtract = 2 };
  int phase = kBound;
  const QueryPrep* Q = nullptr;
  QueryList L;
  int64_t list_len_max = 0;
  int S = 1;
  int stride = 1;
  float* U_out = nullptr;
  WorkItem* items = nullptr;
  unsigned* n_items = nullptr;
  unsigned item_cap = 0;
  CandBuf cb;
};
dd_status launch_scan16(const Dataset& D, bool fp16, const Scan16Call& call, hipStream_t st);
// Merge candidate lists, rerank in FP64 direct form, write outputs; queries that
// overflowed (or found no candidate) are appended to fb_list / fb_count.  The
// bound is Uq[q] when given, else the minimum of cb.U over the splits.
dd_status launch_merge_rerank(const Dataset& D, const QueryPrep& Q, QueryList L,
                              int64_t list_len, const CandBuf& cb, const float* Uq, Outputs out,
                              int* fb_list, int* fb_count, unsigned long long* n_cand,
                              hipStream_t st);
// Plain FP64 direct-form scan with lexicographic (dist, original index) minimum,
// split over the data, followed by its merge.  The per-split partial results
// (list_len x splits, splits = choose_splits(list blocks, tiles, S)) go to
// part_d / part_o.
dd_status run_direct(const Dataset& D, const QueryPrep& Q, QueryList L, int64_t list_len, int S,
                     Outputs out, hipStream_t st, double* part_d, uint32_t* part_o);

// Splits of a scan over the data (FP64 and direct scans): `requested` if > 0;
// with fewer than 64 query blocks one round of workgroups (512), otherwise
// about 2048; multiples of 8 give a grid that the scans can deal to the eight
// XCDs split by split.
int choose_splits(int64_t n_query_blocks, int64_t n_tiles, int requested);
// The splits run_direct takes for a list of list_len queries when S = 0.
int direct_splits(const Dataset& D, int64_t list_len);

// Queries per workgroup of the 16-bit pass (sixteen waves of two 32-query groups).
constexpr int kScan16Queries = 1024;

// Splits of the 16-bit pass: with fewer than 64 query blocks, one round of
// workgroups (256: one per CU), so that no second round waits on a short
// first one; otherwise about 1024 workgroups.  Multiples of 8 keep a split's
// workgroups on one XCD.
int choose_splits16(int64_t n_query_blocks, int64_t n_tiles, int requested);

// DD_ANN walk over the dataset's box tree (kmt: DD_KMEANS walk over its
// k-means tree with radius factor fd) for the queries of L (one wavefront
// each): writes outputs, appends overflowed queries to fb_list / fb_count, adds
// (points visited, boxes tested, leaves visited, candidates reranked, leaf
// boxes tested, nodes expanded) to slot blockIdx % kCounterSlots of counters
// (kCounterStride u64 per slot).
// budget = max leaves per query, 0 = exact.
// With dist2 (exact walk only) the walk certifies the two nearest points and
// writes the second distance (1/2 d^2; -1 when the query went to the fallback).
// fd_q / budget_q (device, indexed by query, optional): per-query radius factor
// (k-means walk) and leaf budget in place of fd and budget.
dd_status launch_ann_walk(const Dataset& D, const QueryPrep& Q, QueryList L, int64_t len_max,
                          const int64_t* warm, int budget, Outputs out, int* fb_list, int* fb_count,
                          unsigned long long* counters, double* dist2, hipStream_t st,
                          bool kmt = false, double fd = 1.0, const float* fd_q = nullptr,
                          const int* budget_q = nullptr);

// u32[q] = min(u32[q], min over the S split bounds U[p][S]).
dd_status launch_reduce_bounds(QueryList L, int64_t list_len_max, const float* U, int S, float* u32,
                               hipStream_t st);

// ---------------------------------------------------------------------------
// Device helpers shared by the scan translation units
// ---------------------------------------------------------------------------
constexpr float kRelUp = 1.0f + 9.5367431640625e-07f;   // 1 + 2^-20
constexpr float kRelDn = 1.0f - 9.5367431640625e-07f;   // 1 - 2^-20

// Candidate list append; a full list is compacted to the entries whose lower
// bound is still <= U before it is declared overflowed.
__device__ inline void cand_append(const CandBuf& cb, int64_t slot, int& cnt, bool& ovf, float lb,
                                   uint32_t j, float U) {
  if (ovf) return;
  float* L = cb.lb + slot * cb.K;
  uint32_t* J = cb.j + slot * cb.K;
  if (cnt == cb.K) {
    int k = 0;
    for (int c = 0; c < cb.K; ++c) {
      float v = L[c];
      if (v <= U) {
        uint32_t jj = J[c];
        L[k] = v;
        J[k] = jj;
        ++k;
      }
    }
    cnt = k;
    if (cnt == cb.K) {
      ovf = true;
      return;
    }
  }
  L[cnt] = lb;
  J[cnt] = j;
  ++cnt;
}

// atomicAdd(&counter[cell], 1) of every lane with cell >= 0 (every lane active),
// returning the value before this lane's add.  Lanes with equal cells share an
// atomic for the first kCellRounds cells of the wavefront (a batch whose states
// fall into few cells does not queue on their addresses); the lanes left, of
// many different cells, add on their own.
constexpr int kCellRounds = 4;
__device__ inline unsigned cell_add(unsigned* counter, int cell) {
  const int lane = (int)(threadIdx.x & 63);
  uint64_t todo = __ballot(cell >= 0);
  int lead = -1, rank = 0;
  unsigned at = 0;
#pragma unroll 1
  for (int r = 0; r < kCellRounds && todo; ++r) {
    const int l = __builtin_ctzll(todo);
    const uint64_t same = __ballot(cell == __builtin_amdgcn_readlane(cell, l));
    if ((same >> lane) & 1ull) {
      lead = l;
      rank = __popcll(same & ((1ull << lane) - 1ull));
      if (lane == l) at = (unsigned)__popcll(same);
    }
    todo &= ~same;
  }
  const bool alone = (todo >> lane) & 1ull;
  if (alone || lane == lead) at = atomicAdd(&counter[cell], alone ? 1u : at);
  const unsigned first = (unsigned)__shfl((int)at, lead < 0 ? lane : lead);
  return first + (unsigned)rank;
}

__device__ inline int64_t list_len(const QueryList& L) {
  return L.list && L.count ? (int64_t)*L.count : L.m;
}
__device__ inline int64_t list_query(const QueryList& L, int64_t p) { return L.list ? (int64_t)L.list[p] : p; }


}  // namespace dd
