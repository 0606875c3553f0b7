// Shared pieces of libcel: error state, scratch memory, input validation,
// prefix scans, CSR relabelling into position space and a segmented sort.
#include <chrono>
#include <cstdarg>
#include <cstring>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

#include "cel_internal.h"

namespace cel {

// ------------------------------------------------------------------ errors

static thread_local char g_msg[512] = "";

int set_error(int code, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_msg, sizeof g_msg, fmt, ap);
  va_end(ap);
  return code;
}

const char *last_error_text() { return g_msg; }

int status_error(const Status &h, const char *fn) {
  if (h.err & EB_ARG) return set_error(CEL_E_ARG, "%s: malformed graph or argument arrays", fn);
  if (h.err & EB_CYCLE) return set_error(CEL_E_CYCLE, "%s: the graph has a cycle", fn);
  if (h.err & EB_OVERFLOW)
    return set_error(CEL_E_OVERFLOW, "%s: sum(w) + sum over edges of c[src] reaches 2^62", fn);
  if (h.err & EB_ORDER)
    return set_error(CEL_E_ORDER, "%s: order/level/cluster arrays inconsistent with the graph", fn);
  if (h.err & EB_WAIT)
    return set_error(CEL_E_HIP, "%s: a bounded wait between waves of a sweep timed out", fn);
  return CEL_OK;
}

int check_host_graph(const cel_graph *g, const char *fn) {
  if (!g) return set_error(CEL_E_ARG, "%s: graph is NULL", fn);
  if (g->n < 0 || g->m < 0) return set_error(CEL_E_ARG, "%s: negative n or m", fn);
  if (!g->out_ptr || !g->in_ptr || (g->m > 0 && (!g->out_idx || !g->in_idx)) ||
      (g->n > 0 && (!g->w || !g->mem || !g->ob)))
    return set_error(CEL_E_ARG, "%s: NULL graph array", fn);
  return CEL_OK;
}

int check_host_devices(const cel_devices *d, const char *fn) {
  if (!d || !d->cap) return set_error(CEL_E_ARG, "%s: devices or caps NULL", fn);
  if (d->D < 1 || d->D > kMaxD) return set_error(CEL_E_ARG, "%s: D = %d not in [1, 255]", fn, d->D);
  if (d->bw <= 0 || d->lat < 0 || d->lat >= kLim)
    return set_error(CEL_E_ARG, "%s: need bw > 0 and 0 <= lat < 2^62", fn);
  for (int i = 0; i < d->D; i++)
    if (d->cap[i] < 0) return set_error(CEL_E_ARG, "%s: negative memory cap", fn);
  return CEL_OK;
}

// ----------------------------------------------------------------- scratch

struct Arena {
  std::mutex mu;  // held by the Scratch object of the running call
  std::vector<std::pair<char *, size_t>> blocks;
  size_t blk = 0, off = 0;  // bump position of the running call
  size_t need = 0;          // bytes the running call asked for in total
  size_t grow_to = 0;       // one block of this size replaces the chain at the next call
};

static std::mutex g_arenas_mu;
static std::map<std::pair<int, hipStream_t>, Arena *> g_arenas;
constexpr size_t kAlign = 256;
constexpr size_t kMinBlock = size_t(8) << 20;

Scratch::Scratch(hipStream_t s) : s_(s) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    err_ = set_error(CEL_E_HIP, "hipGetDevice failed");
    return;
  }
  {
    std::lock_guard<std::mutex> lk(g_arenas_mu);
    Arena *&a = g_arenas[{dev, s}];
    if (!a) a = new Arena();  // kept until the process ends
    a_ = a;
  }
  a_->mu.lock();
  a_->blk = a_->off = a_->need = 0;
  if (a_->grow_to > 0) {
    // the last call spilled into several blocks: replace them by one that
    // fits it, once the stream has drained (earlier kernels may use them)
    if (hipStreamSynchronize(s_) != hipSuccess) {
      err_ = set_error(CEL_E_HIP, "hipStreamSynchronize failed");
      return;
    }
    for (auto &b : a_->blocks) (void)hipFree(b.first);
    a_->blocks.clear();
    void *p = nullptr;
    if (hipMalloc(&p, a_->grow_to) != hipSuccess || !p) {
      err_ = set_error(CEL_E_NOMEM, "scratch arena of %zu bytes: allocation failed", a_->grow_to);
      a_->grow_to = 0;
      return;
    }
    a_->blocks.push_back({(char *)p, a_->grow_to});
    a_->grow_to = 0;
  }
}

int Scratch::raw(void **out, size_t bytes) {
  if (err_ != CEL_OK) return err_;
  const size_t sz = (bytes + kAlign - 1) / kAlign * kAlign;
  if (base_) {  // fixed range: bump, never allocate
    if (sz > cap_ - off_)
      return err_ = set_error(CEL_E_ARG, "the call needs more than the %zu bytes of fixed scratch",
                              cap_);
    *out = base_ + off_;
    off_ += sz;
    return CEL_OK;
  }
  a_->need += sz;
  while (a_->blk < a_->blocks.size() && a_->off + sz > a_->blocks[a_->blk].second) {
    a_->blk++;
    a_->off = 0;
  }
  if (a_->blk == a_->blocks.size()) {  // grow: a new block at the end of the chain
    const size_t bsz = sz > kMinBlock ? sz : kMinBlock;
    void *p = nullptr;
    if (hipMalloc(&p, bsz) != hipSuccess || !p)
      return err_ = set_error(CEL_E_NOMEM, "scratch allocation of %zu bytes failed", bytes);
    a_->blocks.push_back({(char *)p, bsz});
    a_->off = 0;
  }
  *out = a_->blocks[a_->blk].first + a_->off;
  a_->off += sz;
  return CEL_OK;
}

Scratch::Mark Scratch::mark() const {
  if (base_ || !a_) return Mark{0, off_};
  return Mark{a_->blk, a_->off};
}

void Scratch::release(const Mark &m) {
  if (err_ != CEL_OK) return;
  if (base_ || !a_) {
    off_ = m.off;
    return;
  }
  // `need` keeps counting every request: it sizes the single block that
  // replaces a spilled chain, and a bound from above is enough there
  a_->blk = m.blk;
  a_->off = m.off;
}

Scratch::~Scratch() {
  if (!a_) return;
  if (a_->blocks.size() > 1) a_->grow_to = a_->need;
  a_->mu.unlock();
}

int read_status(const Status *dst, Status *host, hipStream_t s) {
  CEL_HIP(hipMemcpyAsync(host, dst, sizeof(Status), hipMemcpyDeviceToHost, s));
  CEL_HIP(hipStreamSynchronize(s));
  return CEL_OK;
}

// ---------------------------------------------------- turn of the whole grids

static std::mutex g_turn_mu;
static std::map<int, std::timed_mutex *> g_turns;  // one a device, kept until the process ends
constexpr auto kTurnWait = std::chrono::seconds(1);

bool GridTurn::take() {
  if (mu_) return true;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  std::timed_mutex *m;
  {
    std::lock_guard<std::mutex> lk(g_turn_mu);
    std::timed_mutex *&t = g_turns[dev];
    if (!t) t = new std::timed_mutex();
    m = t;
  }
  if (late_ ? !m->try_lock() : !m->try_lock_for(kTurnWait)) {
    late_ = true;  // a call waits once
    return false;
  }
  mu_ = m;
  return true;
}

void GridTurn::done() {
  if (mu_) mu_->unlock();
  mu_ = nullptr;
}

GridTurn::~GridTurn() {
  if (!mu_) return;
  (void)hipStreamSynchronize(s_);
  done();
}

// ------------------------------------------------------------ side stream

static std::mutex g_side_mu;
static std::map<int, hipStream_t> g_side;

int SideFork::start(hipStream_t s) {
  int dev = 0;
  CEL_HIP(hipGetDevice(&dev));
  {
    std::lock_guard<std::mutex> lk(g_side_mu);
    hipStream_t &t = g_side[dev];
    if (!t) CEL_HIP(hipStreamCreateWithFlags(&t, hipStreamNonBlocking));
    side_ = t;
  }
  CEL_HIP(hipEventCreateWithFlags(&fork_, hipEventDisableTiming));
  CEL_HIP(hipEventCreateWithFlags(&join_, hipEventDisableTiming));
  CEL_HIP(hipEventRecord(fork_, s));
  CEL_HIP(hipStreamWaitEvent(side_, fork_, 0));
  s_ = s;
  joined_ = false;
  return CEL_OK;
}

int SideFork::join() {
  if (joined_) return CEL_OK;
  joined_ = true;
  CEL_HIP(hipEventRecord(join_, side_));
  CEL_HIP(hipStreamWaitEvent(s_, join_, 0));
  return CEL_OK;
}

SideFork::~SideFork() {
  if (!joined_ && join() != CEL_OK) (void)hipStreamSynchronize(side_);
  if (join_) {
    (void)hipEventSynchronize(join_);
    (void)hipEventDestroy(join_);
  }
  if (fork_) (void)hipEventDestroy(fork_);
}

// ------------------------------------------------------------- validation

// saturating add for the overflow bound
__device__ inline uint64_t sat_add(uint64_t a, uint64_t b) {
  uint64_t r = a + b;
  return (r < a || r > (uint64_t)kLim) ? (uint64_t)kLim : r;
}

// What a call's order array is checked against.
enum OrderKind { kNoOrder = 0, kLevelOrder = 1, kTopoOrder = 2 };
struct OrderCheck {
  const int32_t *order, *level, *level_ptr;
  int32_t L;
  int32_t *pos;
};

constexpr uint32_t kCheckGroups = 64;  // at most the block size
constexpr uint32_t kCheckStride = 32;  // counters 128 bytes apart

// Every call opens with these checks, and on a graph of a few thousand nodes
// a launch costs more than the work in it: two launches hold all of them
// (they were five for the graph and four more for an order).  Here: what
// reads one node or one position; k_check_edges: what follows edges or needs
// the inverse order.
//
// Node fields and row pointers; the block's part of the overflow bound; with
// an order, its ids in range, pos[order[p]] = p, and (level orders) level_ptr
// and the place of every node's level in it.  Clears k_check_edges' counters.
template <int KIND>
__global__ void k_check_nodes(cel_graph g, int64_t bw, int64_t lat, OrderCheck oc, Status *st,
                              uint64_t *part_out, uint32_t *groups) {
  __shared__ uint64_t part[4];
  if (blockIdx.x == 0 && threadIdx.x < kCheckGroups) groups[threadIdx.x * kCheckStride] = 0;
  const int32_t n = g.n, m = g.m;
  uint64_t acc = 0;
  uint32_t bad = 0;
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v <= n;
       v += (int64_t)gridDim.x * blockDim.x) {
    if (KIND == kLevelOrder && v <= oc.L) {  // 0 at the front, n at the back, non-decreasing
      const int32_t a = oc.level_ptr[v];
      if (v == 0 && a != 0) bad |= EB_ORDER;
      if (v == oc.L && a != n) bad |= EB_ORDER;
      if (v < oc.L && oc.level_ptr[v + 1] < a) bad |= EB_ORDER;
    }
    if (KIND != kNoOrder && v < n) {
      const int32_t u = oc.order[v];
      if (u < 0 || u >= n) {
        bad |= EB_ORDER;
      } else {
        // duplicates are found by k_check_edges: two positions naming one id
        // leave pos[id] at one of them, and the other does not read itself back
        oc.pos[u] = (int32_t)v;
        if (KIND == kLevelOrder) {
          const int32_t l = oc.level[u];
          if (l < 0 || l >= oc.L || v < oc.level_ptr[l] || v >= oc.level_ptr[l + 1])
            bad |= EB_ORDER;
        }
      }
    }
    if (v == 0 && (g.out_ptr[0] != 0 || g.in_ptr[0] != 0)) bad |= EB_ARG;
    if (v == n) {
      if (g.out_ptr[n] != m || g.in_ptr[n] != m) bad |= EB_ARG;
      continue;
    }
    int32_t o0 = g.out_ptr[v], o1 = g.out_ptr[v + 1], i0 = g.in_ptr[v], i1 = g.in_ptr[v + 1];
    if (o1 < o0 || i1 < i0) bad |= EB_ARG;
    int64_t w = g.w[v], mem = g.mem[v], ob = g.ob[v];
    if (w < 0 || mem < 0 || ob < 0) {
      bad |= EB_ARG;
      continue;
    }
    int64_t deg = o1 > o0 ? (int64_t)o1 - o0 : 0;
    int64_t c = comm_of(ob, bw, lat);  // ob >= 0, bw >= 1, lat < 2^62: no overflow
    uint64_t t = (uint64_t)w;
    if (deg > 0) t = (c >= kLim / deg) ? (uint64_t)kLim : sat_add(t, (uint64_t)(c * deg));
    acc = sat_add(acc, t);
  }
  // wave reduce (saturating) then block
  for (int off = 32; off > 0; off >>= 1) {
    uint64_t o = __shfl_down(acc, off);
    acc = sat_add(acc, o);
  }
  int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) part[wv] = acc;
  if (bad) raise_err(st, bad);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t tot = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) tot = sat_add(tot, part[i]);
    part_out[blockIdx.x] = tot;
  }
}

__device__ inline uint64_t mix64(uint64_t x) {  // SplitMix64 finaliser
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// CSR and CSC must hold the same edge multiset.  The CSR side adds a 64-bit
// hash of every (source, target) pair to one total and the CSC side takes it
// away; equal multisets leave 0, and any difference is caught with
// overwhelming probability.
__device__ inline uint64_t pair_hash(int32_t u, int32_t v) {
  return mix64(((uint64_t)(uint32_t)u << 32) | (uint32_t)v);
}

// After k_check_nodes.  Blocks [0, eb) take the out-edges (targets in range,
// pair hashes, source before target in the order), blocks [eb, 2 eb) the
// in-edges (sources in range, pair hashes), both edge-balanced; every block
// takes its share of the positions (pos[order[p]] = p: a permutation).  The
// last block to end compares the hash totals and, if asked, adds up the
// overflow bound.  Row pointers that failed leave the edges out, order ids
// out of range the positions; levels that failed are compared all the same
// (the call is refused already, and an argument error is reported before an
// order error whatever the checks after it find).
//
// Blocks store their part of the hash and count themselves in one of
// kCheckGroups counters, the last of a group in st->done.  The counting is
// relaxed, after a wait for the block's own store, and the last block reads
// the parts past the caches: a release in each of 3,200 blocks would write
// back an L2 each time (65 us for a kernel of 10), and that many adds to one
// address are no faster.
template <int KIND>
__global__ void __launch_bounds__(256) k_check_edges(cel_graph g, OrderCheck oc, int eb, int bound,
                                                     const uint64_t *part, int np, uint64_t *hs,
                                                     uint32_t *groups, Status *st) {
  __shared__ int32_t ptr[kRowsPB + 1], su[2];
  __shared__ uint64_t red[4], redh[4];
  __shared__ uint32_t s_err;
  __shared__ int s_last;
  const int32_t n = g.n;
  if (threadIdx.x == 0) s_err = __atomic_load_n(&st->err, __ATOMIC_RELAXED);
  __syncthreads();
  const uint32_t err = s_err;
  uint32_t bad = 0;
  uint64_t acc = 0;
  if (!(err & EB_ARG) && n > 0) {
    const bool out = (int)blockIdx.x < eb;
    if (out) {
      for_edges_slice(blockIdx.x, g.out_ptr, n, g.m, ptr, su, [&](int32_t u, int32_t e) {
        const int32_t t = g.out_idx[e];
        if (t < 0 || t >= n) {
          bad |= EB_ARG;
          return;
        }
        if (KIND == kLevelOrder && oc.level[t] <= oc.level[u]) bad |= EB_ORDER;
        if (KIND == kTopoOrder && oc.pos[t] <= oc.pos[u]) bad |= EB_ORDER;
        acc += pair_hash(u, t);
      });
    } else if ((int)blockIdx.x < 2 * eb) {
      for_edges_slice(blockIdx.x - eb, g.in_ptr, n, g.m, ptr, su, [&](int32_t v, int32_t k) {
        const int32_t u = g.in_idx[k];
        if (u < 0 || u >= n) {
          bad |= EB_ARG;
          return;
        }
        acc -= pair_hash(u, v);
      });
    }
  }
  if (KIND != kNoOrder && !(err & EB_ORDER))
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x)
      if (oc.pos[oc.order[p]] != (int32_t)p) bad |= EB_ORDER;
  if (bad) raise_err(st, bad);
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_store(&hs[blockIdx.x], red[0] + red[1] + red[2] + red[3], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the store is complete
    const uint32_t k = blockIdx.x % kCheckGroups;
    const uint32_t size = (gridDim.x - k + kCheckGroups - 1) / kCheckGroups;
    bool last = __hip_atomic_fetch_add(&groups[k * kCheckStride], 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT) == size - 1;
    if (last)
      last = __hip_atomic_fetch_add(&st->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
             (gridDim.x < kCheckGroups ? gridDim.x : kCheckGroups) - 1;
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  uint64_t tot = 0, hash = 0;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += blockDim.x)
    hash += __hip_atomic_load(&hs[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (bound)
    for (int i = threadIdx.x; i < np; i += blockDim.x) tot = sat_add(tot, part[i]);
  for (int off = 32; off > 0; off >>= 1) {
    tot = sat_add(tot, __shfl_down(tot, off));
    hash += __shfl_down(hash, off);
  }
  if ((threadIdx.x & 63) == 0) {  // red was read before the barrier
    red[threadIdx.x >> 6] = tot;
    redh[threadIdx.x >> 6] = hash;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (redh[0] + redh[1] + redh[2] + redh[3] != 0) raise_err(st, EB_ARG);
    if (bound) {
      uint64_t t = 0;
      for (int i = 0; i < 4; i++) t = sat_add(t, red[i]);
      st->total = t;
      if (t >= (uint64_t)kLim) raise_err(st, EB_OVERFLOW);
    }
  }
}

template <int KIND>
static int check_all(const cel_graph *g, int64_t bw, int64_t lat, bool bound, const OrderCheck &oc,
                     Status *st, Scratch &sc, hipStream_t s) {
  const int B = 256;
  const int nbk = grid_for((int64_t)g->n + 1, B, 2048);
  uint64_t *part;
  uint32_t *groups;
  CEL_TRY(sc.get(&part, nbk));
  CEL_TRY(sc.get(&groups, kCheckGroups * kCheckStride));
  k_check_nodes<KIND><<<nbk, B, 0, s>>>(*g, bw, lat, oc, st, part, groups);
  const int eb = (int)edge_blocks(g->m);
  int grid = 2 * eb;
  if (KIND != kNoOrder) {  // few edges and many positions: blocks for the positions alone
    const int pb = grid_for(g->n, B, 512);
    if (grid < pb) grid = pb;
  }
  uint64_t *hs;
  CEL_TRY(sc.get(&hs, grid));
  k_check_edges<KIND><<<grid, B, 0, s>>>(*g, oc, eb, bound ? 1 : 0, part, nbk, hs, groups,
                                         st);
  CEL_HIP(hipGetLastError());
  return CEL_OK;
}

int check_graph(const cel_graph *g, int64_t bw, int64_t lat, bool bound, Status *st, Scratch &sc,
                hipStream_t s) {
  return check_all<kNoOrder>(g, bw, lat, bound, OrderCheck{}, st, sc, s);
}

int check_graph_levels(const cel_graph *g, int64_t bw, int64_t lat, const int32_t *order,
                       const int32_t *level, const int32_t *level_ptr, int32_t L, int32_t *pos,
                       Status *st, Scratch &sc, hipStream_t s) {
  return check_all<kLevelOrder>(g, bw, lat, true, OrderCheck{order, level, level_ptr, L, pos}, st,
                                sc, s);
}

int check_graph_topo(const cel_graph *g, int64_t bw, int64_t lat, bool bound, const int32_t *order,
                     int32_t *pos, Status *st, Scratch &sc, hipStream_t s) {
  return check_all<kTopoOrder>(g, bw, lat, bound, OrderCheck{order, nullptr, nullptr, 0, pos}, st,
                               sc, s);
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ------------------------------------------------------------------- scans

constexpr int kScanB = 256, kScanItems = 16, kScanTile = kScanB * kScanItems;

template <class T>
__device__ T block_exclusive_scan(T x, T *wsum, T *total) {
  // 256 threads = 4 waves of 64
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  T inc = x;
  for (int off = 1; off < 64; off <<= 1) {
    T y = __shfl_up(inc, off);
    if (lane >= off) inc += y;
  }
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  T base = 0, tot = 0;
  for (int i = 0; i < kScanB / 64; i++) {
    if (i < wv) base += wsum[i];
    tot += wsum[i];
  }
  __syncthreads();
  *total = tot;
  return base + inc - x;
}

// What is summed: an array, or the row lengths of a CSR taken in the order of
// `order` (0 after a failed check, whose ids may be out of range).
template <class T>
struct ScanArray {
  const T *in;
  __device__ void open() {}
  __device__ T operator()(int64_t i) const { return in[i]; }
};
struct ScanRows {
  const int32_t *order, *ptr;
  const Status *st;
  bool ok;
  __device__ void open() { ok = !failed(st); }
  __device__ int32_t operator()(int64_t i) const {
    if (!ok) return 0;
    const int32_t v = order[i];
    return ptr[v + 1] - ptr[v];
  }
};

// A scan is one launch up to a tile of kScanTile values and two above: the
// blocks' sums, then the scan, in which every block adds up the sums before
// its own (up to kScanFlat of them; more are scanned first).
template <class T, class F>
__global__ void k_scan_reduce(F f, int64_t n, T *bsum) {
  __shared__ T wsum[kScanB / 64];
  int64_t base = (int64_t)blockIdx.x * kScanTile;
  T acc = 0;
  f.open();
  for (int i = threadIdx.x; i < kScanTile; i += kScanB) {
    int64_t k = base + i;
    if (k < n) acc += f(k);
  }
  T tot;
  (void)block_exclusive_scan<T>(acc, wsum, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// boff: the offset of every block; else bsum, the sums of the blocks (or one
// block, both null).  total, if given, takes the sum of all.
template <class T, class F>
__global__ void k_scan_apply(F f, T *out, int64_t n, const T *bsum, const T *boff, T *total) {
  __shared__ T buf[kScanTile];
  __shared__ T wsum[kScanB / 64];
  int64_t base = (int64_t)blockIdx.x * kScanTile;
  f.open();
  for (int i = threadIdx.x; i < kScanTile; i += kScanB) {
    int64_t k = base + i;
    buf[i] = k < n ? f(k) : (T)0;
  }
  T pre = boff ? boff[blockIdx.x] : (T)0;
  if (bsum) {  // uniform
    T a = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanB) a += bsum[i];
    (void)block_exclusive_scan<T>(a, wsum, &pre);
  }
  __syncthreads();
  T loc = 0;
  for (int k = 0; k < kScanItems; k++) loc += buf[threadIdx.x * kScanItems + k];
  T tot;
  T run = block_exclusive_scan<T>(loc, wsum, &tot) + pre;
  for (int k = 0; k < kScanItems; k++) {
    run += buf[threadIdx.x * kScanItems + k];
    buf[threadIdx.x * kScanItems + k] = run;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kScanTile; i += kScanB) {
    int64_t k = base + i;
    if (k < n) out[k + 1] = buf[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0;
  if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = pre + tot;
}

constexpr int64_t kScanFlat = 4096;  // block sums that a block adds up itself

template <class T, class F>
static int exclusive_scan(F f, T *out, int64_t n, Scratch &sc, hipStream_t s, T *total) {
  if (n <= 0) {
    k_scan_apply<T, F><<<1, kScanB, 0, s>>>(f, out, 0, nullptr, nullptr, total);
    CEL_HIP(hipGetLastError());
    return CEL_OK;
  }
  int64_t nb = (n + kScanTile - 1) / kScanTile;
  T *bsum = nullptr, *boff = nullptr;
  if (nb > 1) {
    CEL_TRY(sc.get(&bsum, nb));
    k_scan_reduce<T, F><<<(unsigned)nb, kScanB, 0, s>>>(f, n, bsum);
    if (nb > kScanFlat) {
      CEL_TRY(sc.get(&boff, nb + 1));
      CEL_TRY((exclusive_scan<T, ScanArray<T>>(ScanArray<T>{bsum}, boff, nb, sc, s, nullptr)));
      bsum = nullptr;
    }
  }
  k_scan_apply<T, F><<<(unsigned)nb, kScanB, 0, s>>>(f, out, n, bsum, boff, total);
  CEL_HIP(hipGetLastError());
  return CEL_OK;
}

int exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, Scratch &sc, hipStream_t s,
                       int32_t *total) {
  return exclusive_scan<int32_t>(ScanArray<int32_t>{in}, out, n, sc, s, total);
}
int exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, Scratch &sc, hipStream_t s,
                       int64_t *total) {
  return exclusive_scan<int64_t>(ScanArray<int64_t>{in}, out, n, sc, s, total);
}

// ---------------------------------------------------------------- relabel

// Output edges in edge-balanced blocks: slot k of row p (position p) takes
// edge k - pptr[p] of node order[p], so a row of huge degree is spread over
// many blocks.
__global__ void k_relabel_rows(int32_t n, int32_t m, const int32_t *order, const int32_t *pos,
                               const int32_t *ptr, const int32_t *idx, const int32_t *pptr,
                               int32_t *pidx, const Status *st) {
  __shared__ int32_t rp[kRowsPB + 1], su[2];
  if (failed(st)) return;
  for_edges_balanced(pptr, n, m, rp, su, [&](int32_t p, int32_t k) {
    pidx[k] = pos[idx[ptr[order[p]] + (k - pptr[p])]];
  });
}

int relabel_csr(int32_t n, int32_t m, const int32_t *order, const int32_t *pos,
                const int32_t *ptr, const int32_t *idx, int32_t *pptr, int32_t *pidx, Scratch &sc,
                hipStream_t s, const Status *st) {
  CEL_TRY(exclusive_scan<int32_t>(ScanRows{order, ptr, st, false}, pptr, n, sc, s, nullptr));
  if (n <= 0) return CEL_OK;
  k_relabel_rows<<<edge_blocks(m), 256, 0, s>>>(n, m, order, pos, ptr, idx, pptr, pidx, st);
  CEL_HIP(hipGetLastError());
  return CEL_OK;
}

// ------------------------------------------------------- segmented sort
//
// Device-only: tiles of at most kSortTile elements are bitonic-sorted in LDS,
// then segments longer than a tile are merged in passes of doubling run
// width.  Tile lists and pass counts come from device data and host-known
// upper bounds, so no host synchronisation is needed.

constexpr int kSortTile = 2048;

struct Tile {
  int32_t start, len;
};

__device__ inline bool kless(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib) {
  return ka < kb || (ka == kb && ia < ib);
}

// The tile list of segments [s0, s0 + kTileSegs) and the number of tiles
// before it: one block up to kTileSegs segments; above, the blocks' counts by
// k_tile_count, and every block adds up the counts before its own.
constexpr int kTileB = 1024, kTilePer = 16, kTileSegs = kTileB * kTilePer;

__device__ inline int32_t tiles_of(int32_t len) {
  return len > 1 ? (len + kSortTile - 1) / kSortTile : 0;
}

// the sum of x over the block's waves before this one plus the lanes before
// this one, and the block's total
__device__ inline int32_t tile_scan(int32_t x, int32_t *ws, int32_t *total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int32_t inc = x;
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t y = __shfl_up(inc, off);
    if (lane >= off) inc += y;
  }
  if (lane == 63) ws[wv] = inc;
  __syncthreads();
  int32_t base = 0, tot = 0;
  for (int i = 0; i < kTileB / 64; i++) {
    if (i < wv) base += ws[i];
    tot += ws[i];
  }
  __syncthreads();
  *total = tot;
  return base + inc - x;
}

__global__ void __launch_bounds__(kTileB) k_tile_count(const int32_t *seg, int32_t nseg,
                                                      int32_t *bcnt, const Status *st) {
  __shared__ int32_t ws[kTileB / 64];
  const bool ok = !failed(st);  // offsets not validated otherwise
  const int64_t s0 = (int64_t)blockIdx.x * kTileSegs;
  int32_t c = 0;
  for (int k = 0; ok && k < kTilePer; k++) {
    const int64_t i = s0 + k * kTileB + threadIdx.x;
    if (i < nseg) c += tiles_of(seg[i + 1] - seg[i]);
  }
  int32_t tot;
  (void)tile_scan(c, ws, &tot);
  if (threadIdx.x == 0) bcnt[blockIdx.x] = tot;
}

// tiles in any order (they are sorted one by one); *ntiles = 0 after a failed check
__global__ void __launch_bounds__(kTileB) k_tile_fill(const int32_t *seg, int32_t nseg,
                                                     const int32_t *bcnt, Tile *tiles,
                                                     int32_t *ntiles, const Status *st) {
  __shared__ int32_t ws[kTileB / 64];
  const bool ok = !failed(st);
  const int64_t s0 = (int64_t)blockIdx.x * kTileSegs;
  int32_t pre = 0;
  if (bcnt) {
    int32_t a = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kTileB) a += bcnt[i];
    (void)tile_scan(a, ws, &pre);
  }
  int32_t c = 0;
  for (int k = 0; ok && k < kTilePer; k++) {
    const int64_t i = s0 + k * kTileB + threadIdx.x;
    if (i < nseg) c += tiles_of(seg[i + 1] - seg[i]);
  }
  int32_t tot;
  int32_t t = pre + tile_scan(c, ws, &tot);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *ntiles = ok ? pre + tot : 0;
  for (int k = 0; ok && k < kTilePer; k++) {
    const int64_t i = s0 + k * kTileB + threadIdx.x;
    if (i >= nseg) break;
    const int32_t a = seg[i], len = seg[i + 1] - a;
    if (len <= 1) continue;
    for (int32_t o = 0; o < len; o += kSortTile, t++)
      tiles[t] = Tile{a + o, len - o < kSortTile ? len - o : kSortTile};
  }
}

// Bitonic sort of one tile (<= kSortTile elements) in LDS; blocks past the
// tile count (ntiles, on the device) exit.
__global__ void __launch_bounds__(256) k_sort_tiles(uint64_t *keys, uint32_t *ids,
                                                    const Tile *tiles, const int32_t *ntiles,
                                                    const Status *st) {
  __shared__ uint64_t sk[kSortTile];
  __shared__ uint32_t si[kSortTile];
  if (failed(st) || (int32_t)blockIdx.x >= *ntiles) return;
  const Tile t = tiles[blockIdx.x];
  int P = 2;
  while (P < t.len) P <<= 1;
  for (int i = threadIdx.x; i < P; i += blockDim.x) {
    if (i < t.len) {
      sk[i] = keys[t.start + i];
      si[i] = ids[t.start + i];
    } else {
      sk[i] = ~0ull;
      si[i] = ~0u;
    }
  }
  __syncthreads();
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < (P >> 1); i += blockDim.x) {
        int lo = 2 * stride * (i / stride) + (i % stride), hi = lo + stride;
        bool up = (lo & size) == 0;
        uint64_t ka = sk[lo], kb = sk[hi];
        uint32_t ia = si[lo], ib = si[hi];
        if (kless(kb, ib, ka, ia) == up) {
          sk[lo] = kb; sk[hi] = ka;
          si[lo] = ib; si[hi] = ia;
        }
      }
      __syncthreads();
    }
  }
  for (int i = threadIdx.x; i < t.len; i += blockDim.x) {
    keys[t.start + i] = sk[i];
    ids[t.start + i] = si[i];
  }
}

// segment of every element: last s with seg[s] <= i
__global__ void k_seg_of(const int32_t *seg, int32_t nseg, int64_t n, int32_t *sid,
                         const Status *st) {
  if (failed(st)) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    int32_t lo = 0, hi = nseg - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (seg[mid] <= i) lo = mid;
      else hi = mid - 1;
    }
    sid[i] = lo;
  }
}

// One merge round over the segments longer than a tile: runs of `width` are
// merged in pairs (each element finds its slot by counting the smaller
// elements of the partner run); segments already one run are copied.
__global__ void k_merge_pass(const uint64_t *kin, const uint32_t *iin, uint64_t *kout,
                             uint32_t *iout, const int32_t *seg, const int32_t *sid, int64_t n,
                             int64_t width, const Status *st) {
  if (failed(st)) return;
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int32_t s = sid[g];
    const int64_t base = seg[s], len = seg[s + 1] - base;
    if (len <= kSortTile) continue;  // sorted by its tile, never moves
    const uint64_t k = kin[g];
    const uint32_t id = iin[g];
    if (len <= width) {
      kout[g] = k;
      iout[g] = id;
      continue;
    }
    const int64_t off = g - base;
    const int64_t a0 = (off / (2 * width)) * (2 * width);
    const int64_t a1 = a0 + width < len ? a0 + width : len;
    const int64_t b1 = a0 + 2 * width < len ? a0 + 2 * width : len;
    int64_t r0, r1, own;
    if (off < a1) {
      r0 = a1; r1 = b1; own = off - a0;
    } else {
      r0 = a0; r1 = a1; own = off - a1;
    }
    int64_t l = r0, h = r1;  // partner elements smaller than (k, id)
    while (l < h) {
      const int64_t mid = (l + h) >> 1;
      if (kless(kin[base + mid], iin[base + mid], k, id)) l = mid + 1;
      else h = mid;
    }
    const int64_t dst = a0 + own + (l - r0);
    kout[base + dst] = k;
    iout[base + dst] = id;
  }
}

// elements of segments longer than a tile: copy back from the scratch copy
__global__ void k_copy_big(const uint64_t *kin, const uint32_t *iin, uint64_t *kout,
                           uint32_t *iout, const int32_t *seg, const int32_t *sid, int64_t n,
                           const Status *st) {
  if (failed(st)) return;
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int32_t s = sid[g];
    if (seg[s + 1] - seg[s] <= kSortTile) continue;
    kout[g] = kin[g];
    iout[g] = iin[g];
  }
}

int segmented_sort(uint64_t *keys, uint32_t *ids, const int32_t *seg, int32_t nseg, int64_t n,
                   Scratch &sc, hipStream_t s, const Status *st) {
  if (nseg <= 0 || n <= 1) return CEL_OK;
  int32_t *bcnt = nullptr, *ntiles;
  Tile *tiles;
  const int64_t maxtiles = (int64_t)nseg + n / kSortTile + 1;
  const unsigned nb = (unsigned)(((int64_t)nseg + kTileSegs - 1) / kTileSegs);
  CEL_TRY(sc.get(&ntiles, 1));
  CEL_TRY(sc.get(&tiles, maxtiles));
  if (nb > 1) {
    CEL_TRY(sc.get(&bcnt, nb));
    k_tile_count<<<nb, kTileB, 0, s>>>(seg, nseg, bcnt, st);
  }
  k_tile_fill<<<nb, kTileB, 0, s>>>(seg, nseg, bcnt, tiles, ntiles, st);
  k_sort_tiles<<<(unsigned)maxtiles, 256, 0, s>>>(keys, ids, tiles, ntiles, st);
  int passes = 0;  // enough for the longest possible segment (n)
  while (((int64_t)kSortTile << passes) < n) passes++;
  if (passes > 0) {
    int32_t *sid;
    uint64_t *k2;
    uint32_t *i2;
    CEL_TRY(sc.get(&sid, n));
    CEL_TRY(sc.get(&k2, n));
    CEL_TRY(sc.get(&i2, n));
    k_seg_of<<<grid_for(n, 256, 8192), 256, 0, s>>>(seg, nseg, n, sid, st);
    uint64_t *ka = keys, *kb = k2;
    uint32_t *ia = ids, *ib = i2;
    for (int p = 0; p < passes; p++) {
      k_merge_pass<<<grid_for(n, 256, 8192), 256, 0, s>>>(ka, ia, kb, ib, seg, sid, n,
                                                           (int64_t)kSortTile << p, st);
      std::swap(ka, kb);
      std::swap(ia, ib);
    }
    if (passes & 1)
      k_copy_big<<<grid_for(n, 256, 8192), 256, 0, s>>>(k2, i2, keys, ids, seg, sid, n, st);
  }
  CEL_HIP(hipGetLastError());
  return CEL_OK;
}

}  // namespace cel
