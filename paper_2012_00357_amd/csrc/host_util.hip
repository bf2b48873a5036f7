// Host utilities: error reporting, device buffers, small dense linear algebra.
#include <unistd.h>

#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <list>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <unordered_map>

#include "dd_internal.h"

namespace dd {

static thread_local std::string g_last_error;

dd_status set_error(dd_status st, const std::string& msg) {
  g_last_error = msg;
  return st;
}

namespace {

using PoolClock = std::chrono::steady_clock;
struct PoolBlock {
  void* p;
  size_t size;
  int device;
  PoolClock::time_point since;
};
struct Pool {
  std::mutex mu;
  std::unordered_map<void*, std::pair<size_t, int>> out;   // blocks in use: size, device
  std::list<PoolBlock> idle;                               // oldest first
  std::condition_variable cv;                              // for the reaper: a first block, or stop
  std::thread reaper;
  pid_t pid = 0;                                           // the process it runs in
  bool stop = false;
};
constexpr size_t kPoolLeast = (size_t)1 << 20;
// Never destroyed: objects released at exit may still come here.
Pool& pool() {
  static Pool* p = new Pool;
  return *p;
}

// Frees blocks whose time is over, with no call of the library needed for it.
void reap() {
  Pool& P = pool();
  // hipFree here must not end a capture that some other thread of the program has open
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  std::unique_lock<std::mutex> lk(P.mu);
  while (!P.stop) {
    if (P.idle.empty()) {
      P.cv.wait(lk);
      continue;
    }
    const auto due = P.idle.front().since + std::chrono::seconds(kPoolSeconds);
    if (PoolClock::now() < due) {
      P.cv.wait_until(lk, due);
      continue;
    }
    void* p = P.idle.front().p;
    P.idle.pop_front();
    lk.unlock();
    (void)hipFree(p);
    lk.lock();
  }
}

// Ends the reaper before the HIP runtime's own end.  (A child made by fork has no such
// thread, only its record.)
void stop_reaper() {
  Pool& P = pool();
  if (P.pid != getpid()) return;
  {
    std::lock_guard<std::mutex> lk(P.mu);
    P.stop = true;
  }
  P.cv.notify_one();
  if (P.reaper.joinable()) P.reaper.join();
}

// Whether a block may be kept: the reaper runs in this process (P.mu held).
bool reaper_runs(Pool& P) {
  if (P.pid == 0) {
    P.pid = getpid();
    try {
      if (std::atexit(stop_reaper) == 0) P.reaper = std::thread(reap);
    } catch (const std::system_error&) {
    }
  }
  return P.reaper.joinable() && !P.stop && P.pid == getpid();
}

}  // namespace

void device_pool_trim() {
  std::list<PoolBlock> gone;
  {
    Pool& P = pool();
    std::lock_guard<std::mutex> lk(P.mu);
    gone.swap(P.idle);
  }
  for (const PoolBlock& b : gone) (void)hipFree(b.p);
}

static thread_local TempPool* t_temps = nullptr;

void device_give_back() {
  if (t_temps) t_temps->trim();
  device_pool_trim();
}

static thread_local bool t_keep = false;
KeepScope::KeepScope() : before(t_keep) { t_keep = true; }
KeepScope::~KeepScope() { t_keep = before; }

hipError_t device_alloc(void** p, size_t n) {
  if (n < kPoolLeast || !t_keep) return alloc_or_give_back([&] { return hipMalloc(p, n); });
  Pool& P = pool();
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  {
    std::lock_guard<std::mutex> lk(P.mu);
    for (auto it = P.idle.begin(); it != P.idle.end(); ++it) {
      if (it->device != dev || it->size != n) continue;
      *p = it->p;
      try {
        P.out[it->p] = {n, dev};
      } catch (const std::bad_alloc&) {
      }
      P.idle.erase(it);
      return hipSuccess;
    }
  }
  e = alloc_or_give_back([&] { return hipMalloc(p, n); });
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lk(P.mu);
    try {
      P.out[*p] = {n, dev};
    } catch (const std::bad_alloc&) {   // not known: not kept
    }
  }
  return e;
}

void device_free(void* p) {
  Pool& P = pool();
  PoolBlock b{p, 0, 0, {}};
  {
    std::lock_guard<std::mutex> lk(P.mu);
    auto it = P.out.find(p);
    if (it != P.out.end()) {
      b.size = it->second.first;
      b.device = it->second.second;
      P.out.erase(it);
    }
  }
  int dev = 0;
  // as hipFree does: whatever still runs on the device may use the block
  if (b.size == 0 || b.size > kPoolBytes || hipGetDevice(&dev) != hipSuccess || dev != b.device ||
      hipDeviceSynchronize() != hipSuccess) {
    (void)hipFree(p);
    return;
  }
  std::list<PoolBlock> gone;
  try {
    gone.push_back(b);
  } catch (const std::bad_alloc&) {
    (void)hipFree(p);
    return;
  }
  {
    std::lock_guard<std::mutex> lk(P.mu);
    gone.front().since = PoolClock::now();
    if (reaper_runs(P)) {
      if (P.idle.empty()) P.cv.notify_one();
      P.idle.splice(P.idle.end(), gone);
      size_t total = 0;
      for (const PoolBlock& k : P.idle)
        if (k.device == dev) total += k.size;
      for (auto it = P.idle.begin(); total > kPoolBytes;) {   // the oldest go
        const auto next = std::next(it);
        if (it->device == dev) {
          total -= it->size;
          gone.splice(gone.end(), P.idle, it);
        }
        it = next;
      }
    }
  }
  for (const PoolBlock& g : gone) (void)hipFree(g.p);
}

dd_status DevBuf::alloc(size_t n) {
  release();
  owned = true;
  if (n == 0) return DD_OK;
  hipError_t e = device_alloc(&p, n);
  if (e != hipSuccess) {
    p = nullptr;
    return set_error(e == hipErrorOutOfMemory ? DD_ERR_OOM : DD_ERR_DEVICE,
                     std::string("hipMalloc(") + std::to_string(n) + "): " + hipGetErrorString(e));
  }
  bytes = n;
  return DD_OK;
}

void DevBuf::release() {
  if (p && owned) device_free(p);
  p = nullptr;
  bytes = 0;
  owned = true;
}

dd_status TempPool::take(size_t n, void** p, size_t* cap) {
  auto best = idle.end();
  for (auto it = idle.begin(); it != idle.end(); ++it)
    if (it->first >= n && (best == idle.end() || it->first < best->first)) best = it;
  if (best != idle.end()) {
    *cap = best->first;
    *p = best->second;
    idle.erase(best);
    return DD_OK;
  }
  if (n <= kLeast) {
    void* slab = nullptr;
    if (device_alloc(&slab, kKeep) == hipSuccess) {
      slabs.push_back(slab);
      for (size_t o = kLeast; o < kKeep; o += kLeast)
        idle.emplace_back(kLeast, static_cast<char*>(slab) + o);
      *p = slab;
      *cap = kLeast;
      return DD_OK;
    }
  }
  size_t size = n;
  if (n <= kKeep)
    for (size = 2 * kLeast; size < n;) size *= 2;
  hipError_t e = device_alloc(p, size);
  if (e != hipSuccess && size > n) {   // no more than was asked for
    size = n == kLeast ? n + 1 : n;    // kLeast marks a slab's blocks
    e = device_alloc(p, size);
  }
  if (e != hipSuccess) {
    *p = nullptr;
    return set_error(e == hipErrorOutOfMemory ? DD_ERR_OOM : DD_ERR_DEVICE,
                     std::string("hipMalloc(") + std::to_string(n) + "): " + hipGetErrorString(e));
  }
  *cap = size;
  return DD_OK;
}

void TempPool::put(void* p, size_t cap) {
  if (cap > kKeep)
    device_free(p);
  else
    idle.emplace_back(cap, p);
}

void TempPool::trim() {
  size_t kept = 0;
  for (auto& b : idle) {
    if (b.first == kLeast)
      idle[kept++] = b;
    else
      device_free(b.second);
  }
  idle.resize(kept);
  if (kept * kLeast == slabs.size() * kKeep) {
    for (void* s : slabs) device_free(s);
    slabs.clear();
    idle.clear();
  }
}

TempPool::TempPool() : before(t_temps) { t_temps = this; }

TempPool::~TempPool() {
  trim();
  for (void* s : slabs) device_free(s);
  t_temps = before;
}

ScratchArena::~ScratchArena() {
  // the last user's work on the block must end before the block is freed
  if (done) (void)hipEventSynchronize(done);
  if (block) device_free(block);
  if (pinned) (void)hipHostFree(pinned);
  if (done) (void)hipEventDestroy(done);
}

bool cholesky6(const double* C, double* L) {
  std::memset(L, 0, 36 * sizeof(double));
  for (int j = 0; j < 6; ++j) {
    double s = C[6 * j + j];
    for (int k = 0; k < j; ++k) s -= L[6 * j + k] * L[6 * j + k];
    if (!(s > 0.0) || !std::isfinite(s)) return false;
    double d = std::sqrt(s);
    L[6 * j + j] = d;
    for (int i = j + 1; i < 6; ++i) {
      double t = C[6 * i + j];
      for (int k = 0; k < j; ++k) t -= L[6 * i + k] * L[6 * j + k];
      L[6 * i + j] = t / d;
    }
  }
  return true;
}

void lower_inverse6(const double* L, double* X) {
  // Forward substitution column by column: L X = I.
  std::memset(X, 0, 36 * sizeof(double));
  for (int c = 0; c < 6; ++c) {
    for (int i = 0; i < 6; ++i) {
      double s = (i == c) ? 1.0 : 0.0;
      for (int k = 0; k < i; ++k) s -= L[6 * i + k] * X[6 * k + c];
      X[6 * i + c] = s / L[6 * i + i];
    }
  }
}

void sym_eigen(int n, const double* A_in, double* evals, double* V) {
  // Cyclic Jacobi rotations on a copy of A (n <= 16).
  double A[256];
  for (int i = 0; i < n * n; ++i) A[i] = A_in[i];
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) V[n * i + j] = (i == j) ? 1.0 : 0.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) (i == j ? diag : off) += A[n * i + j] * A[n * i + j];
    if (off <= 1e-30 * diag) break;
    for (int p = 0; p < n; ++p) {
      for (int q = p + 1; q < n; ++q) {
        double apq = A[n * p + q];
        if (std::fabs(apq) < 1e-300) continue;
        double app = A[n * p + p], aqq = A[n * q + q];
        double theta = (aqq - app) / (2.0 * apq);
        double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
        for (int k = 0; k < n; ++k) {
          double akp = A[n * k + p], akq = A[n * k + q];
          A[n * k + p] = c * akp - s * akq;
          A[n * k + q] = s * akp + c * akq;
        }
        for (int k = 0; k < n; ++k) {
          double apk = A[n * p + k], aqk = A[n * q + k];
          A[n * p + k] = c * apk - s * aqk;
          A[n * q + k] = s * apk + c * aqk;
        }
        for (int k = 0; k < n; ++k) {
          double vkp = V[n * k + p], vkq = V[n * k + q];
          V[n * k + p] = c * vkp - s * vkq;
          V[n * k + q] = s * vkp + c * vkq;
        }
      }
    }
  }
  // sort descending (selection sort on eigenvalues, permuting columns)
  for (int i = 0; i < n; ++i) evals[i] = A[n * i + i];
  for (int i = 0; i < n; ++i) {
    int best = i;
    for (int j = i + 1; j < n; ++j)
      if (evals[j] > evals[best]) best = j;
    if (best != i) {
      double t = evals[i];
      evals[i] = evals[best];
      evals[best] = t;
      for (int k = 0; k < n; ++k) {
        double v = V[n * k + i];
        V[n * k + i] = V[n * k + best];
        V[n * k + best] = v;
      }
    }
  }
}

int64_t Dataset::device_bytes() const {
  int64_t b = (int64_t)(perm.bytes + iperm.bytes + w64.bytes + n64.bytes + w32.bytes + n32.bytes +
                        centre.bytes + radius.bytes + wbf16.bytes + wfp16.bytes);
  for (int l = 0; l < kAnnMaxLevels; ++l) b += (int64_t)ann_box[l].bytes;
  b += (int64_t)(boxes.bytes() + boxes16.bytes() + tkey.bytes);
  b += (int64_t)(ann_meta.bytes + ann_q0.bytes + ann_h16.bytes);
  b += (int64_t)(kmt_node.bytes + kmt_nbox.bytes + kmt_child.bytes + kmt_meta.bytes + kmt_h16.bytes +
                 kmt_pos.bytes + kmt_slot.bytes);
  std::lock_guard<std::mutex> lk(arena_mu);
  return b + arena_bytes;
}

}  // namespace dd

extern "C" const char* dd_last_error(void) { return dd::g_last_error.c_str(); }
extern "C" const char* dd_version(void) { return "libdd 0.1 (gfx950)"; }
