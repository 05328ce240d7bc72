// C ABI of libt2vattn: argument validation, the device work-list cache, and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <list>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/t2vattn.h"
#include "t2v_host.h"
#include "t2v_kernels.h"

// The no-allocation backward's scratch (see attn_bwd_noalloc_impl): one per GPU, held until
// the process ends. Host code must not use this name as a device address.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace t2v {
namespace {

int hip_fail(hipError_t e, const char* what) {
  return set_error(T2V_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// The scheduler order: longest clip first unless T2V_ORDER=natural (for ablations).
int order_from_env() {
  const char* s = std::getenv("T2V_ORDER");
  if (s != nullptr && std::strcmp(s, "natural") == 0) return T2V_ORDER_NATURAL;
  return T2V_ORDER_LONGEST_FIRST;
}

// Forward / dQ tile shape: narrow (4 waves, 128 queries) or wide (8 waves, 256 queries).
// Narrow tiles fit two workgroups per CU at D = 128 and three at D = 64, so one workgroup's
// Q loads and output stores overlap another's MFMA work; wide tiles stage each K/V tile
// once per 256 queries. Measured on MI355X (uniform packs): at D = 64 narrow is faster at
// every length (8-19% forward, 4-12% dQ); at D = 128 the forward crosses over near 1,536
// keys and dQ near 8,192-16,384, beyond which narrow tiles cost about 4% (forward) and 1%
// (dQ) more per unit of work. choose_tile_rows compares the work-weighted key length with
// those crossovers and, above them, the list-scheduling makespans of both work lists with
// that penalty: a pack of few tiles per CU (one GPU's share of a long clip under head
// sharding) loses more to a part-empty last round of wide tiles. T2V_QTILE=wide or narrow
// forces one (ablations and tests).
struct TileRule {
  int kind = 0;  // 0: dK/dV, 1: forward, 2: dQ, 3: one-pass backward of short key segments
  int wide = 0, narrow = 0;
  bool narrow_always = false;
  double max_loop = 0.0, penalty = 1.0;
  TileForm forms[2] = {};  // dK/dV: the wide and the narrow form
  int forced = 0;  // 0: chosen by the rule, 1: wide, 2: narrow
  bool same(const TileRule& o) const {
    return kind == o.kind && wide == o.wide && narrow == o.narrow && narrow_always == o.narrow_always &&
           forced == o.forced;
  }
};

int forced_tiles() {
  const char* s = std::getenv("T2V_QTILE");
  if (s != nullptr && std::strcmp(s, "wide") == 0) return 1;
  if (s != nullptr && std::strcmp(s, "narrow") == 0) return 2;
  return 0;
}

TileRule fwd_rule(int head_dim) {
  TileRule r;
  r.kind = 1;
  r.wide = fwd_tile_rows(head_dim, false);
  r.narrow = fwd_tile_rows(head_dim, true);
  r.narrow_always = head_dim == 64;
  r.max_loop = 1536.0;
  r.penalty = 1.04;
  r.forced = forced_tiles();
  return r;
}

TileRule dq_rule(int head_dim) {
  TileRule r;
  r.kind = 2;
  r.wide = dq_tile_rows(head_dim, false);
  r.narrow = dq_tile_rows(head_dim, true);
  r.narrow_always = head_dim == 64;
  r.max_loop = 8192.0;
  r.penalty = 1.01;
  r.forced = forced_tiles();
  return r;
}

// dK/dV at D = 128: 64 keys per wave (256-key tiles) or 32 (128-key tiles, two of which take
// about one wide tile's time). Item times measured on MI355X with uniform packs of 256 to 65,536
// tokens at 24 heads; the fixed part is operand loads and output stores with nothing beside them
// on the CU. Wide is 10-15% faster per unit of work (1,272 against 1,150 TFLOP/s on long clips);
// narrow wins where wide tiles are half empty (128 keys: 559 against 717 us) or leave CUs idle
// (8 x 1,024 tokens at 12 heads, 1.5 rounds of wide tiles: 108 against 118 us; 6,912 at 3 heads:
// 174 against 277 us). Between them the gain follows the rounds: 75,600 tokens at 3 heads, 3.5 rounds of
// wide tiles, 14.7 against 15.1 ms; at 6 heads, 6.9 rounds, 26.7 against 30.4 ms. Split loops and the persistent grid are in the narrow kernel only,
// and head_dim 64 has one form. T2V_KVTILE=wide or narrow forces one (ablations and tests).
TileRule dkdv_rule(int head_dim, int chunk, bool persistent) {
  TileRule r;
  r.narrow = dkdv_tile_rows(head_dim);
  r.wide = head_dim == 128 ? dkdv_wide_rows() : r.narrow;
  r.forms[0] = {r.wide, 1, 12500.0, 52.8};
  r.forms[1] = {r.narrow, 1, 8000.0, 29.2};
  const char* s = std::getenv("T2V_KVTILE");
  if (chunk > 0 || persistent || (s != nullptr && std::strcmp(s, "narrow") == 0))
    r.forced = 2;
  else if (s != nullptr && std::strcmp(s, "wide") == 0)
    r.forced = 1;
  return r;
}

// The tile rows of a work list: forced, or chosen from the offsets. `items` receives the list
// when the choice built it.
int rows_of(const TileRule& r, const int32_t* cu, const int32_t* cu_loop, int nseq, int heads, int order, int ncu,
            std::vector<Item>* items) {
  if (r.forced == 1) return r.wide;
  if (r.forced == 2 || r.wide == r.narrow) return r.narrow;
  if (r.kind == 0) return r.forms[choose_form(cu, cu_loop, nseq, heads, r.forms, 2, order, ncu, items)].rows;
  return choose_tile_rows(cu, cu_loop, nseq, heads, r.wide, r.narrow, r.narrow_always, r.max_loop, r.penalty, order,
                          ncu, items);
}

// T2V_PERSISTENT=1 launches the forward and dK/dV kernels on a persistent grid (as many
// workgroups as the GPU holds at once, each looping over the work list with a stride of the
// grid); the default is one workgroup per work item. Results are bitwise equal either way.
// (The dQ kernel always runs one workgroup per item: its looping form would spill.)
bool persistent_enabled() {
  const char* s = std::getenv("T2V_PERSISTENT");
  return s != nullptr && std::strcmp(s, "1") == 0;
}

// One-pass backward (t2v_bwd_short.hip) for cross-attention to short key segments: every segment
// fits a workgroup (256 keys), and the queries fill the CUs 2.5 times with pieces of at least
// kShortMinPiece rows. A piece costs about 28 us besides its queries (K and V in, fp32 dK and dV
// out and in again for the sum), so short pieces lose what the one pass saves. Measured on 116,904
// queries x 12 heads against 32-256 keys: general path 818-839 us; one pass with pieces of 512
// rows 680, 1,024 583-604, 1,536 543-550, 2,048 533-538, 4,096 573 (too few to balance).
// Where the pieces are short because the sequences are, an item's fixed part outweighs what one pass
// saves: with equal sequences at 12 and 24 heads against 16 to 256 keys, 1 query each took 0.89 to 1.21
// of the general path's time, 33 queries 0.88 to 1.21, 65 queries 0.86 to 1.05, 90 queries 0.79 to
// 0.96, 130 queries 0.69 to 0.81. So the pieces must have kShortMinMean queries in the mean, between
// the last size that lost and the first that always won.
// Above kShortMaxPieces pieces (eight per CU, which balance as well as more) the pieces grow instead:
// cutting a segment into equal pieces at most doubles their number, so a call's partial sums stay
// under 1 GiB (the caller's workspace).
// Returns the piece length, or 0 for the general path. T2V_SHORT=off selects that (ablations and
// tests). Self-attention takes the general path, which t2v_attn_bwd_noalloc shares.
constexpr int kShortMinPiece = 512, kShortMaxPiece = 2048, kShortMaxPieces = 2048, kShortMinMean = 80;
int short_piece(const int32_t* cu_q, const int32_t* cu_k, int nseq, int heads, int head_dim, int ncu) {
  const char* s = std::getenv("T2V_SHORT");
  if (head_dim != 128 || ncu < 1 || (s != nullptr && std::strcmp(s, "off") == 0)) return 0;
  if (cu_q == cu_k || std::memcmp(cu_q, cu_k, sizeof(int32_t) * (nseq + 1)) == 0) return 0;
  for (int i = 0; i < nseq; ++i)
    if (cu_k[i + 1] - cu_k[i] > short_keys()) return 0;
  const int64_t share = 2 * static_cast<int64_t>(heads) * cu_q[nseq] / (5 * ncu);
  if (share < kShortMinPiece) return 0;
  const int64_t least = (static_cast<int64_t>(heads) * cu_q[nseq] / kShortMaxPieces + 63) / 64 * 64;
  const int piece = static_cast<int>(
      std::min<int64_t>(std::max(std::min<int64_t>(share / 64 * 64, kShortMaxPiece), least), 1 << 30));
  int64_t pieces = 0;
  for (int i = 0; i < nseq; ++i) {
    int n = 1, step = 0;
    loop_pieces(cu_q[i + 1] - cu_q[i], piece, &n, &step);
    pieces += cu_q[i + 1] > cu_q[i] ? n : 0;
  }
  return cu_q[nseq] >= kShortMinMean * pieces ? piece : 0;
}

// A step of a one-pass item takes about 1.6 times as long with 129 to 256 keys as with fewer.
double short_weight(int32_t keys) { return keys > short_keys() / 2 ? 1.6 : 1.0; }

TileRule short_rule() {
  TileRule r;
  r.kind = 3;
  r.wide = r.narrow = short_keys();
  return r;
}

// T2V_SPLIT=off disables the dK/dV loop split (for ablations).
bool split_enabled() {
  const char* s = std::getenv("T2V_SPLIT");
  return s == nullptr || std::strcmp(s, "off") != 0;
}

int cu_count() {
  int device = 0, n = 0;
  if (hipGetDevice(&device) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return n;
}

// T2V_LOG=1: one line on stderr per new work list (items, predicted makespan, bound).
bool log_enabled() {
  const char* s = std::getenv("T2V_LOG");
  return s != nullptr && std::strcmp(s, "1") == 0;
}

// T2V_TEST_FAIL_ALLOC=1 makes the work-list allocation fail, so callers can exercise the
// T2V_ERR_OOM path (nothing is launched and the cache is unchanged).
bool fail_alloc_for_test() {
  const char* s = std::getenv("T2V_TEST_FAIL_ALLOC");
  return s != nullptr && std::strcmp(s, "1") == 0;
}

bool is_capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return false;
}

// While it lives (and `on`), this thread's calls that no graph records are allowed during a capture.
class RelaxedCapture {
 public:
  explicit RelaxedCapture(bool on) : on_(on) {
    if (on_) (void)hipThreadExchangeStreamCaptureMode(&mode_);
  }
  ~RelaxedCapture() {
    if (on_) (void)hipThreadExchangeStreamCaptureMode(&mode_);
  }
  RelaxedCapture(const RelaxedCapture&) = delete;
  RelaxedCapture& operator=(const RelaxedCapture&) = delete;

 private:
  bool on_;
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

// A copy to the device on a stream of its own, finished on return.
hipError_t upload_now(void* dst, const void* src, size_t bytes) {
  hipStream_t s = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
  const hipError_t done = hipStreamSynchronize(s);
  (void)hipStreamDestroy(s);
  return e != hipSuccess ? e : done;
}

// cu_seqlens must be host memory: the scheduler reads it on the host.
int check_host_pointer(const int32_t* cu) {
  hipPointerAttribute_t attr;
  std::memset(&attr, 0, sizeof(attr));
  const hipError_t e = hipPointerGetAttributes(&attr, cu);
  if (e != hipSuccess) {
    (void)hipGetLastError();  // plain pageable host memory is not known to HIP
    return T2V_OK;
  }
  if (attr.type == hipMemoryTypeDevice)
    return set_error(T2V_ERR_INVALID_ARG, "cu_seqlens must be a host pointer, got device memory");
  return T2V_OK;
}

// Both offset arrays are read on the host (validation, scheduling), so they are checked to
// be host memory before anything dereferences them, including the T = 0 early return.
int check_offsets_on_host(const int32_t* cu_q, const int32_t* cu_k) {
  if (cu_q == nullptr) return set_error(T2V_ERR_INVALID_ARG, "cu_seqlens is NULL");
  if (int st = check_host_pointer(cu_q)) return st;
  if (cu_k != cu_q) {
    if (cu_k == nullptr) return set_error(T2V_ERR_INVALID_ARG, "cu_seqlens_k is NULL");
    if (int st = check_host_pointer(cu_k)) return st;
  }
  return T2V_OK;
}

// Memory for work lists, per device: device chunks hold the lists the kernels read, pinned
// host chunks stage their uploads. Lists are carved out of the chunks by RangeAllocator, so a
// new list costs no hipMalloc / hipHostMalloc once the chunks are large enough (a chunk is
// added, at twice the size of the last, only when none has room). A range is handed back
// only after every event recorded behind its readers has completed: the upload's event for
// a staging range, and the last launch on each stream that read a device range. Nothing
// here waits for the device.
class ListPool {
 public:
  struct Block {
    int chunk = -1;
    uint64_t off = 0, bytes = 0;
    void* ptr = nullptr;
  };
  explicit ListPool(bool pinned) : pinned_(pinned) {}

  // Caller holds mu(). Returns T2V_OK and a block of `bytes`, or T2V_ERR_OOM.
  int alloc(uint64_t bytes, Block* out) {
    if (fail_alloc_for_test()) return set_error(T2V_ERR_OOM, "allocation of work-list memory failed (forced)");
    if (try_alloc(bytes, out)) return T2V_OK;
    reclaim();
    if (try_alloc(bytes, out)) return T2V_OK;
    uint64_t size = last_size_ == 0 ? (pinned_ ? kFirstPinned : kFirstDevice) : 2 * last_size_;
    while (size < RangeAllocator::rounded(bytes)) size *= 2;
    void* base = nullptr;
    const hipError_t e = pinned_ ? hipHostMalloc(&base, size, hipHostMallocDefault) : hipMalloc(&base, size);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return set_error(T2V_ERR_OOM, pinned_ ? "hipHostMalloc of work-list staging failed"
                                            : "hipMalloc of work-list memory failed");
    }
    chunks_.push_back({base, RangeAllocator(size)});
    last_size_ = size;
    return try_alloc(bytes, out) ? T2V_OK : set_error(T2V_ERR_OOM, "work-list pool");
  }

  // Caller holds mu(). The block returns to its chunk once `events` (taken over) complete.
  void release_after(const Block& b, std::vector<hipEvent_t> events) {
    if (b.chunk < 0) {
      recycle_events(events);
      return;
    }
    pending_.push_back({b, std::move(events)});
  }

  // Caller holds mu(). A captured graph may read the block at any time: it is kept until the next
  // trim_after_sync().
  void keep(const Block& b) {
    if (b.chunk >= 0) kept_.push_back(b);
  }

  // Caller holds mu(). An event from the pool (or a new one), for recording.
  hipError_t take_event(hipEvent_t* ev) {
    if (!events_.empty()) {
      *ev = events_.back();
      events_.pop_back();
      return hipSuccess;
    }
    return hipEventCreateWithFlags(ev, hipEventDisableTiming);
  }
  void recycle_events(std::vector<hipEvent_t>& evs) {
    for (hipEvent_t e : evs) events_.push_back(e);
    evs.clear();
  }

  // Caller holds the lock and has synchronised the device: returns every pending block and
  // frees each chunk that no live block uses (a list still held by a call in progress keeps
  // its chunk), and the idle events.
  void trim_after_sync() {
    reclaim();
    for (const Block& b : kept_) (void)chunks_[b.chunk].alloc.release(b.off, b.bytes);
    kept_.clear();
    for (auto& c : chunks_) {
      if (c.base == nullptr || c.alloc.free_bytes() != c.alloc.size()) continue;
      if (pinned_)
        (void)hipHostFree(c.base);
      else
        (void)hipFree(c.base);
      c.base = nullptr;
      c.alloc = RangeAllocator(0);  // an empty slot: indices of live blocks stay valid
    }
    // The next chunk follows the size of those that are left, not of those that were freed.
    last_size_ = 0;
    for (auto& c : chunks_) last_size_ = std::max(last_size_, c.alloc.size());
    if (last_size_ == 0) chunks_.clear();
    for (hipEvent_t e : events_) (void)hipEventDestroy(e);
    events_.clear();
  }

 private:
  static constexpr uint64_t kFirstDevice = 4u << 20, kFirstPinned = 2u << 20;
  struct Chunk {
    void* base;
    RangeAllocator alloc;
  };
  struct Pending {
    Block block;
    std::vector<hipEvent_t> events;
  };
  bool try_alloc(uint64_t bytes, Block* out) {
    for (int c = static_cast<int>(chunks_.size()) - 1; c >= 0; --c) {  // newest (largest) chunk first
      const int64_t off = chunks_[c].alloc.alloc(bytes);
      if (off < 0) continue;
      *out = {c, static_cast<uint64_t>(off), bytes, static_cast<char*>(chunks_[c].base) + off};
      return true;
    }
    return false;
  }
  // Returns every pending block whose events have all completed.
  void reclaim() {
    for (auto it = pending_.begin(); it != pending_.end();) {
      bool done = true;
      for (hipEvent_t e : it->events) {
        if (hipEventQuery(e) != hipSuccess) {  // not reached yet (or the query failed: keep the block)
          (void)hipGetLastError();
          done = false;
          break;
        }
      }
      if (!done) {
        ++it;
        continue;
      }
      (void)chunks_[it->block.chunk].alloc.release(it->block.off, it->block.bytes);
      recycle_events(it->events);
      it = pending_.erase(it);
    }
  }
  bool pinned_;
  uint64_t last_size_ = 0;  // size of the largest chunk: the next one doubles it
  std::vector<Chunk> chunks_;
  std::list<Pending> pending_;
  std::vector<Block> kept_;
  std::vector<hipEvent_t> events_;
};

// The pools of one device, and the lock that guards them.
struct DevicePools {
  std::mutex mu;
  ListPool dev{false}, pin{true};
};

std::mutex& pools_mu() {
  static std::mutex* mu = new std::mutex();
  return *mu;
}
std::vector<DevicePools*>& all_pools() {
  static std::vector<DevicePools*>* all = new std::vector<DevicePools*>();  // never destroyed
  return *all;
}

DevicePools& pools(int device) {
  std::lock_guard<std::mutex> lock(pools_mu());
  auto& all = all_pools();
  if (device >= static_cast<int>(all.size())) all.resize(device + 1, nullptr);
  if (all[device] == nullptr) all[device] = new DevicePools();
  return *all[device];
}

// After a device-wide synchronisation: gives back the memory of every list no longer held.
void trim_pools_after_sync() {
  std::vector<DevicePools*> all;
  {
    std::lock_guard<std::mutex> lock(pools_mu());
    all = all_pools();
  }
  for (DevicePools* p : all) {
    if (p == nullptr) continue;
    std::lock_guard<std::mutex> lock(p->mu);
    p->dev.trim_after_sync();
    p->pin.trim_after_sync();
  }
}

// Immutable device copies of work lists, keyed by everything that shapes them. Calls hold
// a shared reference from lookup until their launches are enqueued and the launches' event
// is recorded (note_use), so an entry evicted by another thread meanwhile stays alive; when
// the last reference goes, its device block returns to the pool after those events.
struct Plan {
  std::vector<int32_t> cu, cu_loop;  // offsets of the owned and the looped-over segments
  TileRule rule;                     // how block was chosen (part of the key)
  int heads = 0, block = 0, order = 0, device = 0, chunk = 0;
  Item* d_items = nullptr;  // n_items work items, then n_reduce split tiles (loop split)
  int n_items = 0, n_reduce = 0;
  ListPool::Block mem;             // d_items' block in the device pool
  hipEvent_t ready = nullptr;      // upload finished (from the device pool's event pool)
  std::vector<std::pair<hipStream_t, hipEvent_t>> uses;  // last launch reading d_items, per stream
  bool captured = false;  // a captured graph's launches read d_items
#if T2V_CHECKED
  std::vector<Item> host_items;  // checked builds: the list as uploaded, validated at every call
#endif
  ~Plan() {
    DevicePools& p = pools(device);
    std::lock_guard<std::mutex> lock(p.mu);
    std::vector<hipEvent_t> evs;
    if (ready != nullptr) evs.push_back(ready);
    for (auto& u : uses) evs.push_back(u.second);
    if (captured) {
      p.dev.keep(mem);
      mem = ListPool::Block{};
    }
    p.dev.release_after(mem, std::move(evs));
  }
};
using PlanRef = std::shared_ptr<Plan>;

// Records, on `stream`, the point after which the launches just enqueued no longer read the
// plan's list. Later launches on the same stream replace the earlier event (stream order). Captured
// launches run whenever their graph does: the list is then kept until t2v_release_cache.
int note_use(const PlanRef& plan, hipStream_t stream) {
  const bool capturing = is_capturing(stream);
  DevicePools& p = pools(plan->device);
  std::lock_guard<std::mutex> lock(p.mu);
  if (capturing) {
    plan->captured = true;
    return T2V_OK;
  }
  hipEvent_t ev = nullptr;
  hipError_t e = p.dev.take_event(&ev);
  if (e == hipSuccess) e = hipEventRecord(ev, stream);
  if (e != hipSuccess) {
    if (ev != nullptr) (void)hipEventDestroy(ev);
    // Without the event the list could be reused under a running kernel: keep it alive.
    (void)hipStreamSynchronize(stream);
    return hip_fail(e, "hipEventRecord after launch");
  }
  for (auto& u : plan->uses) {
    if (u.first == stream) {
      std::vector<hipEvent_t> old{u.second};
      p.dev.recycle_events(old);
      u.second = ev;
      return T2V_OK;
    }
  }
  plan->uses.push_back({stream, ev});
  return T2V_OK;
}

constexpr size_t kMaxPlans = 64;

class PlanCache {
 public:
  // Returns the plan (creating and uploading it on `stream` if new) with the
  // upload ordered before any later work on `stream`.
  // The tile rows follow `rule` (chosen once, when the plan is built; plan->block). chunk > 0:
  // the loop split of build_worklist, with the reduce list after the items.
  int get(const int32_t* cu, const int32_t* cu_loop, int nseq, int heads, const TileRule& rule, int order, int chunk,
          hipStream_t stream, PlanRef* out) {
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::list<PlanRef> evicted;  // declared before the lock: released after it
    std::unique_lock<std::mutex> lock(mu_);
    for (auto itr = plans_.begin(); itr != plans_.end(); ++itr) {
      Plan& p = **itr;
      if (p.heads == heads && p.rule.same(rule) && p.order == order && p.device == device && p.chunk == chunk &&
          p.cu.size() == static_cast<size_t>(nseq + 1) &&
          std::memcmp(p.cu.data(), cu, sizeof(int32_t) * (nseq + 1)) == 0 &&
          std::memcmp(p.cu_loop.data(), cu_loop, sizeof(int32_t) * (nseq + 1)) == 0) {
        plans_.splice(plans_.begin(), plans_, itr);  // most recently used first
        *out = *itr;
        if (p.ready == nullptr) return T2V_OK;
        if (is_capturing(stream)) {
          // The graph's launches would not wait for an event recorded outside it: the upload, queued
          // on another stream, is waited for here.
          lock.unlock();  // *out keeps the plan
          const RelaxedCapture relaxed(true);
          e = hipEventSynchronize(p.ready);
          return e == hipSuccess ? T2V_OK : hip_fail(e, "hipEventSynchronize");
        }
        e = hipStreamWaitEvent(stream, p.ready, 0);
        return e == hipSuccess ? T2V_OK : hip_fail(e, "hipStreamWaitEvent");
      }
    }
    PlanRef p = std::make_shared<Plan>();
    p->cu.assign(cu, cu + nseq + 1);
    p->cu_loop.assign(cu_loop, cu_loop + nseq + 1);
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
      (void)hipGetLastError();
      ncu = 0;
    }
    std::vector<Item> items;
    const int block = rows_of(rule, cu, cu_loop, nseq, heads, order, ncu, &items);
    p->rule = rule;
    p->heads = heads;
    p->block = block;
    p->order = order;
    p->device = device;
    p->chunk = chunk;
    if (items.empty() || chunk > 0)
      items = build_worklist(cu, cu_loop, nseq, heads, block, order, chunk, rule.kind == 3 ? short_weight : nullptr);
    p->n_items = static_cast<int>(items.size());
    if (chunk > 0) {
      const std::vector<Item> red = build_reduce_list(cu, cu_loop, nseq, heads, block, chunk);
      p->n_reduce = static_cast<int>(red.size());
      items.insert(items.end(), red.begin(), red.end());
    }
    const size_t bytes = items.size() * sizeof(Item);
#if T2V_CHECKED
    p->host_items = items;
#endif
    if (log_enabled()) {
      double ms = 0.0, lb = 0.0;
      plan_makespan(items.data(), p->n_items, block, ncu > 0 ? ncu : 1, &ms, &lb);
      std::fprintf(stderr,
                   "t2v: work list: %d sequences, %d heads, %d-row tiles, %s order: %d items, predicted makespan "
                   "%.4g (lower bound %.4g, ratio %.4f) on %d CUs",
                   nseq, heads, block, order == T2V_ORDER_NATURAL ? "pack" : "longest-first", p->n_items, ms, lb,
                   lb > 0.0 ? ms / lb : 1.0, ncu);
      if (chunk > 0) std::fprintf(stderr, "; loops split at %d rows, %d split tiles", chunk, p->n_reduce);
      std::fprintf(stderr, "\n");
    }
    if (bytes > 0) {
      const bool capturing = is_capturing(stream);
      const RelaxedCapture relaxed(capturing);  // for the pools' allocations and the upload
      DevicePools& dp = pools(device);
      std::lock_guard<std::mutex> plock(dp.mu);
      ListPool::Block staging;
      if (int st = dp.dev.alloc(bytes, &p->mem)) return st;
      if (int st = dp.pin.alloc(bytes, &staging)) {
        dp.dev.release_after(p->mem, {});
        p->mem = ListPool::Block{};
        return st;
      }
      p->d_items = static_cast<Item*>(p->mem.ptr);
      std::memcpy(staging.ptr, items.data(), bytes);
      if (capturing) {
        // Now, outside the graph: an eager call that finds the plan before the graph has run would
        // otherwise read a list that is not there yet.
        e = upload_now(p->d_items, staging.ptr, bytes);
        dp.pin.release_after(staging, {});
        if (e != hipSuccess) return hip_fail(e, "upload of the work list");
      } else {
        e = hipMemcpyAsync(p->d_items, staging.ptr, bytes, hipMemcpyHostToDevice, stream);
        hipEvent_t copied = nullptr;
        if (e == hipSuccess) e = dp.pin.take_event(&copied);
        if (e == hipSuccess) e = hipEventRecord(copied, stream);
        if (e != hipSuccess) {
          if (copied != nullptr) (void)hipEventDestroy(copied);
          (void)hipStreamSynchronize(stream);  // the staging block may still be read
          dp.pin.release_after(staging, {});
          return hip_fail(e, "upload of the work list");
        }
        dp.pin.release_after(staging, {copied});
        e = dp.dev.take_event(&p->ready);
        if (e == hipSuccess) e = hipEventRecord(p->ready, stream);
        if (e != hipSuccess) return hip_fail(e, "hipEventRecord of the work-list upload");
      }
    }
    plans_.push_front(p);
    *out = p;
    // An evicted plan's list returns to the pool (after its launches) when its last
    // reference goes: here after the lock is released, or later by a call still holding it.
    while (plans_.size() > kMaxPlans) {
      evicted.push_back(std::move(plans_.back()));
      plans_.pop_back();
    }
    return T2V_OK;
  }

  // Waits for the device, then drops every plan and frees the pools' memory.
  void clear() {
    std::list<PlanRef> old;
    {
      std::lock_guard<std::mutex> lock(mu_);
      old.swap(plans_);
    }
    old.clear();  // plans still referenced by a call in progress stay alive until it ends
  }

 private:
  std::mutex mu_;
  std::list<PlanRef> plans_;
};

PlanCache& cache() {
  static PlanCache* c = new PlanCache();  // never destroyed: no HIP calls at process exit
  return *c;
}

#if T2V_CHECKED
// ---------------------------------------------------------------- checked library
//
// Built from the same sources with T2V_CHECKED=1: before any kernel runs, every work list is
// validated on the host against the call's offsets (check_work_items: tile rows against
// cu_seqlens, heads, loop pieces, partial slots); after the launches the call waits for its
// kernels and reads back their device-side DMA row checks. Calls are serialised, since the
// device records belong to the kernel source files, not to calls. A violation returns
// T2V_ERR_BOUNDS naming the list item, or the kernel, workgroup, row and segment length.
std::mutex& checked_mu() {
  static std::mutex m;
  return m;
}

// T2V_CHECK_CANARY=n takes n rows off every bound the kernels check (a correct kernel then
// reports its segments' last rows), to show that the device-side checks report.
unsigned int check_canary() {
  const char* e = std::getenv("T2V_CHECK_CANARY");
  return e != nullptr ? static_cast<unsigned int>(std::max(0, std::atoi(e))) : 0u;
}

int check_list(const std::vector<Item>& items, int n_items, int n_reduce, const int32_t* cu_own,
               const int32_t* cu_loop, int nseq, int heads, int block, int64_t max_slots, const char* kernel) {
  std::string why = check_work_items(items.data(), n_items, cu_own, cu_loop, nseq, heads, block, max_slots, false);
  if (why.empty() && n_reduce > 0)
    why = check_work_items(items.data() + n_items, n_reduce, cu_own, cu_loop, nseq, heads, block, max_slots, true);
  if (!why.empty()) return set_error(T2V_ERR_BOUNDS, std::string("checked library: ") + kernel + " work list, " + why);
  return T2V_OK;
}

int check_plan(const PlanRef& p, const int32_t* cu_own, const int32_t* cu_loop, int nseq, int heads,
               int64_t max_slots, const char* kernel) {
  return check_list(p->host_items, p->n_items, p->n_reduce, cu_own, cu_loop, nseq, heads, p->block, max_slots,
                    kernel);
}

// Set by check_arm once a call is about to launch kernels: only such calls wait for the device
// afterwards (a call refused by validation, or with nothing to do, makes no device call).
thread_local bool t_check_armed = false;

// Clears the kernels' DMA row records and sets the canary, just before a call's first launch.
int check_arm() {
  const unsigned int canary = check_canary();
  unsigned int rec[4];
  for (auto take : {fwd_check_take, dkdv_check_take, dkdv_wide_check_take, dq_check_take, short_check_take}) {
    const hipError_t e = take(rec, canary);
    if (e != hipSuccess) return hip_fail(e, "clearing the DMA row checks");
  }
  t_check_armed = true;
  return T2V_OK;
}

// Waits for this call's kernels, then reports the first DMA row found outside its segment.
int check_collect(hipStream_t s) {
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "waiting for the checked kernels");
  const char* names[5] = {"forward", "dK/dV", "dK/dV", "dQ", "one-pass backward"};
  hipError_t (*takes[5])(unsigned int*, unsigned int) = {fwd_check_take, dkdv_check_take, dkdv_wide_check_take,
                                                         dq_check_take, short_check_take};
  int status = T2V_OK;
  for (int i = 0; i < 5; ++i) {
    unsigned int rec[4];
    e = takes[i](rec, 0u);
    if (e != hipSuccess) return hip_fail(e, "reading the DMA row checks");
    if (rec[0] != 0u && status == T2V_OK)
      status = set_error(T2V_ERR_BOUNDS, std::string("checked library: ") + names[i] + " kernel, workgroup " +
                                             std::to_string(rec[1]) + " copied row " +
                                             std::to_string(static_cast<int>(rec[2])) + " of a " +
                                             std::to_string(rec[3]) + "-row segment (" + std::to_string(rec[0]) +
                                             " rows outside their segments in this call)");
  }
  return status;
}
#endif

int64_t tensor_bytes(int64_t T, int heads, int head_dim) { return T * heads * head_dim * 2; }

// Optional per-kernel timing: events bracket each launch while enabled.
enum KernelSlot { kSlotFwd = 0, kSlotPre = 1, kSlotDkdv = 2, kSlotDq = 3, kNumSlots = 4 };

class KernelTimer {
 public:
  void set_enabled(bool on) {
    std::lock_guard<std::mutex> lock(mu_);
    drop_locked();
    enabled_ = on;
  }
  // Runs `launch` between two events on `stream` when timing is on.
  template <typename F>
  hipError_t run(int slot, hipStream_t stream, F&& launch) {
    if (!enabled_.load()) return launch();
    hipEvent_t a = nullptr, b = nullptr;
    hipError_t e = hipEventCreate(&a);
    if (e == hipSuccess) e = hipEventCreate(&b);
    if (e == hipSuccess) e = hipEventRecord(a, stream);
    if (e == hipSuccess) e = launch();
    if (e == hipSuccess) e = hipEventRecord(b, stream);
    if (e != hipSuccess) {
      if (a != nullptr) (void)hipEventDestroy(a);
      if (b != nullptr) (void)hipEventDestroy(b);
      return e;
    }
    std::lock_guard<std::mutex> lock(mu_);
    rec_.push_back({slot, a, b});
    return hipSuccess;
  }
  int read(double* ms, int* counts) {
    std::lock_guard<std::mutex> lock(mu_);
    for (int i = 0; i < kNumSlots; ++i) {
      ms[i] = 0.0;
      counts[i] = 0;
    }
    for (const auto& r : rec_) {
      hipError_t e = hipEventSynchronize(r.b);
      float t = 0.0f;
      if (e == hipSuccess) e = hipEventElapsedTime(&t, r.a, r.b);
      if (e != hipSuccess) {
        drop_locked();
        return hip_fail(e, "kernel timing events");
      }
      ms[r.slot] += t;
      counts[r.slot] += 1;
    }
    drop_locked();
    return T2V_OK;
  }

 private:
  struct Rec {
    int slot;
    hipEvent_t a, b;
  };
  void drop_locked() {
    for (const auto& r : rec_) {
      (void)hipEventSynchronize(r.b);
      (void)hipEventDestroy(r.a);
      (void)hipEventDestroy(r.b);
    }
    rec_.clear();
  }
  std::mutex mu_;
  std::atomic<bool> enabled_{false};
  std::vector<Rec> rec_;
};

KernelTimer& timer() {
  static KernelTimer* t = new KernelTimer();
  return *t;
}

// Optional per-workgroup trace: while armed, each MFMA kernel launch takes the next
// n_items records of the caller's buffer (4 uint64 each); a launch that does not fit is
// run untraced and counted as overflowed.
class WorkgroupTracer {
 public:
  void set(unsigned long long* buf, int64_t capacity) {
    std::lock_guard<std::mutex> lock(mu_);
    buf_ = buf;
    cap_ = buf != nullptr ? capacity : 0;
    used_ = 0;
    overflow_ = 0;
  }
  unsigned long long* reserve(int64_t n) {
    std::lock_guard<std::mutex> lock(mu_);
    if (buf_ == nullptr || n <= 0) return nullptr;
    if (used_ + n > cap_) {
      ++overflow_;
      return nullptr;
    }
    unsigned long long* p = buf_ + 4 * used_;
    used_ += n;
    return p;
  }
  void count(int64_t* used, int* overflow) {
    std::lock_guard<std::mutex> lock(mu_);
    *used = used_;
    *overflow = overflow_;
  }

 private:
  std::mutex mu_;
  unsigned long long* buf_ = nullptr;
  int64_t cap_ = 0, used_ = 0;
  int overflow_ = 0;
};

WorkgroupTracer& tracer() {
  static WorkgroupTracer* t = new WorkgroupTracer();
  return *t;
}

}  // namespace
}  // namespace t2v

namespace t2v {
namespace {

// Forward over queries at cu_q and keys at cu_k (the same array for self-attention).
int attn_fwd_impl(const void* q, const void* k, const void* v, const int32_t* cu_q, const int32_t* cu_k, int nseq,
                  int heads, int head_dim, float scale, void* out, float* lse, void* stream) {
  if (int st = check_offsets_on_host(cu_q, cu_k)) return st;
  int64_t Tq = 0, Tk = 0;
  if (cu_q == cu_k) {
    if (int st = validate_shape(cu_q, nseq, heads, head_dim, scale, &Tq)) return st;
    Tk = Tq;
  } else if (int st = validate_shape_qk(cu_q, cu_k, nseq, heads, head_dim, scale, &Tq, &Tk)) {
    return st;
  }
  if (Tq == 0) return T2V_OK;
  const int64_t qb = tensor_bytes(Tq, heads, head_dim), kb = tensor_bytes(Tk, heads, head_dim);
  const int64_t lb = Tq * heads * 4;
  if (int st = validate_pointers({{q, qb, "q"}, {k, kb, "k"}, {v, kb, "v"}}, {{out, qb, "out"}, {lse, lb, "lse"}}))
    return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  PlanRef plan;
  if (int st = cache().get(cu_q, cu_k, nseq, heads, fwd_rule(head_dim), order_from_env(), 0, s, &plan)) return st;
#if T2V_CHECKED
  if (int st = check_plan(plan, cu_q, cu_k, nseq, heads, 0, "forward")) return st;
#endif
  if (plan->n_items == 0) return T2V_OK;
#if T2V_CHECKED
  if (int st = check_arm()) return st;
#endif
  AttnArgs a{};
  a.q_rows = plan->block;
  a.q = q;
  a.k = k;
  a.v = v;
  a.heads = heads;
  a.head_dim = head_dim;
  a.total_tokens = Tq;
  a.scale = scale;
  a.trace = tracer().reserve(plan->n_items);
  a.persistent = persistent_enabled();
  hipError_t e = timer().run(kSlotFwd, s, [&] { return launch_fwd(a, out, lse, plan->d_items, plan->n_items, s); });
  const int used = note_use(plan, s);
  if (e != hipSuccess) return hip_fail(e, "forward kernel launch");
  return used;
}

// Device memory that a caller of t2v_attn_bwd_qk_ws offers for the partial sums of the one-pass
// backward, and what the call could use: {least, most} bytes.
struct Workspace {
  void* ptr;
  uint64_t bytes;
  uint64_t need[2];
};

// The one-pass backward, over as many heads at a time as the workspace has partial slots for.
// The pieces follow from the whole call's offsets and heads, so the results do not depend on how
// many batches of heads there are.
int attn_bwd_short(const AttnArgs& args, const int32_t* cu_q, const int32_t* cu_k, int nseq, int piece, int order,
                   Workspace* ws, hipStream_t s) {
  const uint64_t slot_bytes = static_cast<uint64_t>(short_partial_slot_bytes());
  const uint64_t per_head =
      static_cast<uint64_t>(split_slots(cu_k, cu_q, nseq, short_keys(), piece)) * slot_bytes;
  ws->need[0] = per_head;
  ws->need[1] = per_head * args.heads;
  int batch = args.heads;
  if (per_head > 0) {
    if (ws->bytes < per_head)
      return set_error(T2V_ERR_WORKSPACE, "the one-pass backward needs " + std::to_string(per_head) +
                                              " bytes of workspace or more, got " + std::to_string(ws->bytes));
    const int most = static_cast<int>(std::min<uint64_t>(ws->bytes / per_head, batch));
    const int n = (batch + most - 1) / most;
    batch = (batch + n - 1) / n;
  }
  for (int h0 = 0; h0 < args.heads; h0 += batch) {
    const int heads = std::min(batch, args.heads - h0);
    PlanRef plan;
    if (int st = cache().get(cu_k, cu_q, nseq, heads, short_rule(), order, piece, s, &plan)) return st;
#if T2V_CHECKED
    if (int st = check_plan(plan, cu_k, cu_q, nseq, heads, static_cast<int64_t>(ws->bytes / slot_bytes),
                            "one-pass backward"))
      return st;
    if (h0 == 0)
      if (int st = check_arm()) return st;
#endif
    if (plan->n_items == 0) continue;
    AttnArgs a = args;
    // Head h0 of a [T, H, D] bf16 tensor.
    const int64_t off = static_cast<int64_t>(h0) * args.head_dim * 2;
    auto in = [off](const void* p) { return static_cast<const char*>(p) + off; };
    auto grad = [off](void* p) { return static_cast<char*>(p) + off; };
    a.q = in(args.q);
    a.k = in(args.k);
    a.v = in(args.v);
    a.out = in(args.out);
    a.dout = in(args.dout);
    a.dq = grad(args.dq);
    a.dk = grad(args.dk);
    a.dv = grad(args.dv);
    a.lse += h0 * args.total_tokens;
    a.delta += h0 * args.total_tokens;
    a.partial = static_cast<float*>(ws->ptr);
    a.trace = tracer().reserve(plan->n_items);
    const hipError_t e = timer().run(kSlotDkdv, s, [&] {
      return launch_bwd_short(a, plan->d_items, plan->n_items, plan->d_items + plan->n_items, plan->n_reduce, s);
    });
    const int used = note_use(plan, s);
    if (e != hipSuccess) return hip_fail(e, "one-pass backward launch");
    if (used != T2V_OK) return used;
  }
  return T2V_OK;
}

// ws: the caller's workspace, with which the one-pass backward may be taken; nullptr: the general
// path, which needs none.
int attn_bwd_impl(const void* q, const void* k, const void* v, const void* out, const float* lse, const int32_t* cu_q,
                  const int32_t* cu_k, int nseq, int heads, int head_dim, float scale, const void* dout, void* dq,
                  void* dk, void* dv, float* delta_ws, void* stream, Workspace* ws = nullptr) {
  if (int st = check_offsets_on_host(cu_q, cu_k)) return st;
  int64_t Tq = 0, Tk = 0;
  if (cu_q == cu_k) {
    if (int st = validate_shape(cu_q, nseq, heads, head_dim, scale, &Tq)) return st;
    Tk = Tq;
  } else if (int st = validate_shape_qk(cu_q, cu_k, nseq, heads, head_dim, scale, &Tq, &Tk)) {
    return st;
  }
  if (Tq == 0) return T2V_OK;
  const int64_t qb = tensor_bytes(Tq, heads, head_dim), kb = tensor_bytes(Tk, heads, head_dim);
  const int64_t lb = Tq * heads * 4;
  std::vector<Range> outputs = {{dq, qb, "dq"}, {dk, kb, "dk"}, {dv, kb, "dv"}, {delta_ws, 2 * lb, "delta_ws"}};
  if (ws != nullptr && ws->bytes > 0) outputs.push_back({ws->ptr, static_cast<int64_t>(ws->bytes), "ws"});
  if (int st = validate_pointers(
          {{q, qb, "q"}, {k, kb, "k"}, {v, kb, "v"}, {out, qb, "out"}, {lse, lb, "lse"}, {dout, qb, "dout"}}, outputs))
    return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int order = order_from_env();
  AttnArgs a{};
  a.q = q;
  a.k = k;
  a.v = v;
  a.out = out;
  a.lse = lse;
  a.dout = dout;
  a.dq = dq;
  a.dk = dk;
  a.dv = dv;
  a.delta = delta_ws;
  a.heads = heads;
  a.head_dim = head_dim;
  a.total_tokens = Tq;
  a.scale = scale;
  if (const int piece = ws != nullptr ? short_piece(cu_q, cu_k, nseq, heads, head_dim, cu_count()) : 0)
    return attn_bwd_short(a, cu_q, cu_k, nseq, piece, order, ws, s);
  PlanRef pk, pq;
  // dK/dV tiles own keys and loop over queries; dQ tiles own queries and loop over keys.
  // Loops too long for the available parallelism (short keys, long queries) are split into
  // pieces whose fp32 partial sums go to slots in dq's memory: dq is an output that the dQ
  // kernel, launched after the reduce, overwrites, so the slots are capped at its size.
  const int kv_rows = dkdv_tile_rows(head_dim);
  int chunk = 0;
  if (split_enabled())
    chunk = choose_loop_split(cu_k, cu_q, nseq, heads, kv_rows, cu_count(), qb / dkdv_partial_slot_bytes(head_dim))
                .chunk;
  const TileRule kv_rule = dkdv_rule(head_dim, chunk, persistent_enabled());
  if (int st = cache().get(cu_k, cu_q, nseq, heads, kv_rule, order, chunk, s, &pk)) return st;
  if (int st = cache().get(cu_q, cu_k, nseq, heads, dq_rule(head_dim), order, 0, s, &pq)) return st;
#if T2V_CHECKED
  if (int st = check_plan(pk, cu_k, cu_q, nseq, heads, qb / dkdv_partial_slot_bytes(head_dim), "dK/dV")) return st;
  if (int st = check_plan(pq, cu_q, cu_k, nseq, heads, 0, "dQ")) return st;
#endif
  a.q_rows = pq->block;
  a.partial = static_cast<float*>(dq);
  a.persistent = persistent_enabled();
  a.kv_wide = pk->block != kv_rows;
#if T2V_CHECKED
  if (int st = check_arm()) return st;
#endif
  hipError_t e = timer().run(kSlotPre, s, [&] { return launch_bwd_pre(a, s); });
  if (e != hipSuccess) return hip_fail(e, "backward preprocess launch");
  if (pk->n_items > 0) {
    a.trace = tracer().reserve(pk->n_items);
    e = timer().run(kSlotDkdv, s, [&] {
      hipError_t r = launch_bwd_dkdv(a, pk->d_items, pk->n_items, s);
      if (r == hipSuccess && pk->n_reduce > 0) r = launch_bwd_dkdv_reduce(a, pk->d_items + pk->n_items, pk->n_reduce, s);
      return r;
    });
    const int used = note_use(pk, s);
    if (e != hipSuccess) return hip_fail(e, "dK/dV kernel launch");
    if (used != T2V_OK) return used;
  }
  if (pq->n_items > 0) {
    a.trace = tracer().reserve(pq->n_items);
    e = timer().run(kSlotDq, s, [&] { return launch_bwd_dq(a, pq->d_items, pq->n_items, s); });
    const int used = note_use(pq, s);
    if (e != hipSuccess) return hip_fail(e, "dQ kernel launch");
    if (used != T2V_OK) return used;
  }
  return T2V_OK;
}

// ------------------------------------------------------------ backward without allocation
//
// For callers that cannot allocate device memory: the [2, H, T] Delta / lse scratch and
// both work lists live in one static device array, `scratch`, instead of the caller's
// delta_ws and the library's list pool. Its device address is taken once per GPU (with
// that GPU current) and kept; host code uses only that address, never the array's name.
// Every call on a GPU shares the array, so calls that overlap on one GPU (different
// streams, or threads) race; calls on one stream are ordered by it. Nothing in it needs
// to start at zero: each call overwrites the parts it reads (the Delta pass writes the
// scratch rows, the list uploads the items).
constexpr size_t kScratchAlign = 256;

size_t align_up(size_t n) { return (n + kScratchAlign - 1) / kScratchAlign * kScratchAlign; }

int scratch_address(int device, unsigned char** out) {
  static std::mutex* mu = new std::mutex();
  static std::vector<unsigned char*>* ptrs = new std::vector<unsigned char*>();  // never destroyed
  std::lock_guard<std::mutex> lock(*mu);
  if (device >= static_cast<int>(ptrs->size())) ptrs->resize(device + 1, nullptr);
  if ((*ptrs)[device] == nullptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return set_error(T2V_ERR_HIP, std::string("hipGetSymbolAddress of the no-allocation scratch: ") +
                                        hipGetErrorString(e));
    }
    (*ptrs)[device] = static_cast<unsigned char*>(p);
  }
  *out = (*ptrs)[device];
  return T2V_OK;
}

struct HostLists {
  std::vector<Item> kv, ql;
};

// Host lists that captured graphs copy from.
class CapturedLists {
 public:
  void keep(std::shared_ptr<HostLists> l) {
    std::lock_guard<std::mutex> lock(mu_);
    lists_.push_back(std::move(l));
  }
  void clear() {
    std::lock_guard<std::mutex> lock(mu_);
    lists_.clear();
  }

 private:
  std::mutex mu_;
  std::vector<std::shared_ptr<HostLists>> lists_;
};

CapturedLists& captured_lists() {
  static CapturedLists* c = new CapturedLists();  // never destroyed
  return *c;
}

int attn_bwd_noalloc_impl(const void* q, const void* k, const void* v, const void* out, const float* lse,
                          const int32_t* cu, int nseq, int heads, int head_dim, float scale, const void* dout,
                          void* dq, void* dk, void* dv, void* stream) {
  if (int st = check_offsets_on_host(cu, cu)) return st;
  int64_t T = 0;
  if (int st = validate_shape(cu, nseq, heads, head_dim, scale, &T)) return st;
  if (T == 0) return T2V_OK;
  const int64_t tb = tensor_bytes(T, heads, head_dim), lb = T * heads * 4;
  if (int st = validate_pointers(
          {{q, tb, "q"}, {k, tb, "k"}, {v, tb, "v"}, {out, tb, "out"}, {lse, lb, "lse"}, {dout, tb, "dout"}},
          {{dq, tb, "dq"}, {dk, tb, "dk"}, {dv, tb, "dv"}}))
    return st;
  const size_t delta_bytes = align_up(static_cast<size_t>(2 * lb));
  auto too_big = [&](size_t need) {
    return set_error(T2V_ERR_INVALID_ARG,
                     "the no-allocation backward needs " + std::to_string(need) + " bytes of scratch (8 * heads * T "
                     "for Delta and lse, 32 per work item), more than its " +
                     std::to_string(kNoAllocScratchBytes) + "-byte array");
  };
  if (delta_bytes > kNoAllocScratchBytes) return too_big(delta_bytes);
  // The same work lists as t2v_attn_bwd (tile rules, order, loop split), built per call.
  const int order = order_from_env();
  const int kv_rows = dkdv_tile_rows(head_dim);
  const int ncu = cu_count();
  int chunk = 0;
  if (split_enabled()) chunk = choose_loop_split(cu, cu, nseq, heads, kv_rows, ncu, tb / dkdv_partial_slot_bytes(head_dim)).chunk;
  const TileRule kv_rule = dkdv_rule(head_dim, chunk, persistent_enabled());
  const auto lists = std::make_shared<HostLists>();
  std::vector<Item>&kv = lists->kv, &ql = lists->ql;
  const int kv_block = rows_of(kv_rule, cu, cu, nseq, heads, order, ncu, &kv);
  if (kv.empty()) kv = build_worklist(cu, cu, nseq, heads, kv_block, order, chunk);
  const int n_kv = static_cast<int>(kv.size());
  int n_reduce = 0;
  if (chunk > 0) {
    const std::vector<Item> red = build_reduce_list(cu, cu, nseq, heads, kv_rows, chunk);
    n_reduce = static_cast<int>(red.size());
    kv.insert(kv.end(), red.begin(), red.end());
  }
  const TileRule qr = dq_rule(head_dim);
  const int q_rows = rows_of(qr, cu, cu, nseq, heads, order, ncu, &ql);
  if (ql.empty()) ql = build_worklist(cu, cu, nseq, heads, q_rows, order);
#if T2V_CHECKED
  if (int st = check_list(kv, n_kv, n_reduce, cu, cu, nseq, heads, kv_block, tb / dkdv_partial_slot_bytes(head_dim),
                          "dK/dV"))
    return st;
  if (int st = check_list(ql, static_cast<int>(ql.size()), 0, cu, cu, nseq, heads, q_rows, 0, "dQ")) return st;
#endif
  const size_t kv_bytes = align_up(kv.size() * sizeof(Item)), q_bytes = align_up(ql.size() * sizeof(Item));
  if (delta_bytes + kv_bytes + q_bytes > kNoAllocScratchBytes) return too_big(delta_bytes + kv_bytes + q_bytes);
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  unsigned char* base = nullptr;
  if (int st = scratch_address(device, &base)) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  Item* d_kv = reinterpret_cast<Item*>(base + delta_bytes);
  Item* d_q = reinterpret_cast<Item*>(base + delta_bytes + kv_bytes);
  // Pageable sources: the runtime stages them itself, in stream order (the call returns once
  // the host arrays may be released). A graph copies them again on each replay, so under capture they
  // stay where they are until t2v_release_cache.
  if (is_capturing(s)) captured_lists().keep(lists);
  if (!kv.empty()) e = hipMemcpyAsync(d_kv, kv.data(), kv.size() * sizeof(Item), hipMemcpyHostToDevice, s);
  if (e == hipSuccess && !ql.empty()) e = hipMemcpyAsync(d_q, ql.data(), ql.size() * sizeof(Item), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail(e, "upload of the work lists into the no-allocation scratch");
  AttnArgs a{};
  a.q_rows = q_rows;
  a.partial = static_cast<float*>(dq);
  a.q = q;
  a.k = k;
  a.v = v;
  a.out = out;
  a.lse = lse;
  a.dout = dout;
  a.dq = dq;
  a.dk = dk;
  a.dv = dv;
  a.delta = reinterpret_cast<float*>(base);
  a.heads = heads;
  a.head_dim = head_dim;
  a.total_tokens = T;
  a.scale = scale;
  a.persistent = persistent_enabled();
  a.kv_wide = kv_block != kv_rows;
#if T2V_CHECKED
  if (int st = check_arm()) return st;
#endif
  e = timer().run(kSlotPre, s, [&] { return launch_bwd_pre(a, s); });
  if (e != hipSuccess) return hip_fail(e, "backward preprocess launch");
  if (n_kv > 0) {
    a.trace = tracer().reserve(n_kv);
    e = timer().run(kSlotDkdv, s, [&] {
      hipError_t r = launch_bwd_dkdv(a, d_kv, n_kv, s);
      if (r == hipSuccess && n_reduce > 0) r = launch_bwd_dkdv_reduce(a, d_kv + n_kv, n_reduce, s);
      return r;
    });
    if (e != hipSuccess) return hip_fail(e, "dK/dV kernel launch");
  }
  if (!ql.empty()) {
    a.trace = tracer().reserve(static_cast<int64_t>(ql.size()));
    e = timer().run(kSlotDq, s, [&] { return launch_bwd_dq(a, d_q, static_cast<int>(ql.size()), s); });
    if (e != hipSuccess) return hip_fail(e, "dQ kernel launch");
  }
  return T2V_OK;
}

// Runs f, turning host exceptions into statuses (none may cross the C ABI).
template <typename F>
int guarded(F&& f) {
  try {
    return f();
  } catch (const std::bad_alloc&) {
    return set_error(T2V_ERR_OOM, "host allocation failed");
  } catch (...) {
    return set_error(T2V_ERR_INVALID_ARG, "unexpected host exception");
  }
}

// Runs an attention call; in the checked library, serialised and followed by the kernels'
// device-side checks.
template <typename F>
int checked_call(void* stream, F&& f) {
#if T2V_CHECKED
  std::lock_guard<std::mutex> lock(checked_mu());
  t_check_armed = false;
  const int st = f();
  if (st != T2V_OK || !t_check_armed) return st;
  t_check_armed = false;
  return check_collect(static_cast<hipStream_t>(stream));
#else
  (void)stream;
  return f();
#endif
}

}  // namespace
}  // namespace t2v

namespace t2v {

int persistent_grid(const void* kernel, int threads, int n_items) {
  int per_cu = 0, ncu = cu_count();
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) {
    (void)hipGetLastError();
    per_cu = 1;
  }
  int grid = std::max(1, per_cu) * std::max(1, ncu);
  if (grid >= kNumXcd) grid -= grid % kNumXcd;
  return std::max(1, std::min(grid, n_items));
}

}  // namespace t2v

extern "C" {

int t2v_attn_fwd(const void* q, const void* k, const void* v, const int32_t* cu_seqlens, int nseq, int heads,
                 int head_dim, float scale, void* out, float* lse, void* stream) {
  return t2v::guarded([&] {
    return t2v::checked_call(stream, [&] {
      return t2v::attn_fwd_impl(q, k, v, cu_seqlens, cu_seqlens, nseq, heads, head_dim, scale, out, lse, stream);
    });
  });
}

int t2v_attn_bwd(const void* q, const void* k, const void* v, const void* out, const float* lse,
                 const int32_t* cu_seqlens, int nseq, int heads, int head_dim, float scale, const void* dout,
                 void* dq, void* dk, void* dv, float* delta_ws, void* stream) {
  return t2v::guarded([&] {
    return t2v::checked_call(stream, [&] {
      return t2v::attn_bwd_impl(q, k, v, out, lse, cu_seqlens, cu_seqlens, nseq, heads, head_dim, scale, dout, dq,
                                dk, dv, delta_ws, stream);
    });
  });
}

int t2v_attn_bwd_noalloc(const void* q, const void* k, const void* v, const void* out, const float* lse,
                         const int32_t* cu_seqlens, int nseq, int heads, int head_dim, float scale, const void* dout,
                         void* dq, void* dk, void* dv, void* stream) {
  return t2v::guarded([&] {
    return t2v::checked_call(stream, [&] {
      return t2v::attn_bwd_noalloc_impl(q, k, v, out, lse, cu_seqlens, nseq, heads, head_dim, scale, dout, dq, dk,
                                        dv, stream);
    });
  });
}

int t2v_attn_fwd_qk(const void* q, const void* k, const void* v, const int32_t* cu_seqlens_q,
                    const int32_t* cu_seqlens_k, int nseq, int heads, int head_dim, float scale, void* out, float* lse,
                    void* stream) {
  return t2v::guarded([&] {
    if (cu_seqlens_q == nullptr || cu_seqlens_k == nullptr)
      return t2v::set_error(T2V_ERR_INVALID_ARG, "cu_seqlens_q or cu_seqlens_k is NULL");
    return t2v::checked_call(stream, [&] {
      return t2v::attn_fwd_impl(q, k, v, cu_seqlens_q, cu_seqlens_k, nseq, heads, head_dim, scale, out, lse, stream);
    });
  });
}

int t2v_attn_bwd_qk(const void* q, const void* k, const void* v, const void* out, const float* lse,
                    const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k, int nseq, int heads, int head_dim,
                    float scale, const void* dout, void* dq, void* dk, void* dv, float* delta_ws, void* stream) {
  return t2v::guarded([&] {
    if (cu_seqlens_q == nullptr || cu_seqlens_k == nullptr)
      return t2v::set_error(T2V_ERR_INVALID_ARG, "cu_seqlens_q or cu_seqlens_k is NULL");
    return t2v::checked_call(stream, [&] {
      return t2v::attn_bwd_impl(q, k, v, out, lse, cu_seqlens_q, cu_seqlens_k, nseq, heads, head_dim, scale, dout,
                                dq, dk, dv, delta_ws, stream);
    });
  });
}

int t2v_attn_bwd_qk_ws(const void* q, const void* k, const void* v, const void* out, const float* lse,
                       const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k, int nseq, int heads, int head_dim,
                       float scale, const void* dout, void* dq, void* dk, void* dv, float* delta_ws, void* ws,
                       uint64_t ws_bytes, uint64_t* need, void* stream) {
  return t2v::guarded([&] {
    if (cu_seqlens_q == nullptr || cu_seqlens_k == nullptr)
      return t2v::set_error(T2V_ERR_INVALID_ARG, "cu_seqlens_q or cu_seqlens_k is NULL");
    t2v::Workspace w{ws, ws_bytes, {0, 0}};
    const int st = t2v::checked_call(stream, [&] {
      return t2v::attn_bwd_impl(q, k, v, out, lse, cu_seqlens_q, cu_seqlens_k, nseq, heads, head_dim, scale, dout,
                                dq, dk, dv, delta_ws, stream, &w);
    });
    if (need != nullptr) {
      need[0] = w.need[0];
      need[1] = w.need[1];
    }
    return st;
  });
}

int t2v_timing_enable(int on) {
  t2v::timer().set_enabled(on != 0);
  return T2V_OK;
}

int t2v_kernel_times(double* ms_out, int* counts_out) {
  if (ms_out == nullptr || counts_out == nullptr) return t2v::set_error(T2V_ERR_INVALID_ARG, "NULL output");
  return t2v::timer().read(ms_out, counts_out);
}

int t2v_trace_set(unsigned long long* dev_records, int64_t capacity) {
  if (capacity < 0 || (dev_records == nullptr && capacity != 0))
    return t2v::set_error(T2V_ERR_INVALID_ARG, "capacity must be >= 0, and 0 when dev_records is NULL");
  if (dev_records != nullptr && reinterpret_cast<uintptr_t>(dev_records) % 8 != 0)
    return t2v::set_error(T2V_ERR_INVALID_ARG, "dev_records is not 8-byte aligned");
  t2v::tracer().set(dev_records, capacity);
  return T2V_OK;
}

int t2v_trace_count(int64_t* n_records, int* n_overflowed) {
  if (n_records == nullptr || n_overflowed == nullptr) return t2v::set_error(T2V_ERR_INVALID_ARG, "NULL output");
  t2v::tracer().count(n_records, n_overflowed);
  return T2V_OK;
}

void t2v_release_cache(void) {
  (void)hipDeviceSynchronize();
  t2v::cache().clear();
  t2v::captured_lists().clear();
  t2v::trim_pools_after_sync();
}

}  // extern "C"
