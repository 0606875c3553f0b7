// Makespans of K placements under the device models without insertion (and of
// batches of placements over narrow levels, cel_makespan), one workgroup each,
// in blocks of tasks in LDS.
//
// Without insertion every start time is the later of a few finish times fixed
// by the order alone: a node waits for the previous node on its device and for
// its inputs (on another device after the transfer), a transfer that is a task
// of its own waits for its producer and for the previous task on each channel
// or queue that it holds (Section 5.2 eq. 7 without insertion; Section 6.1).
// So the finish times are longest paths over the tasks in issue order (a node,
// then its transfers), val(t) = w(t) + max(base(t), max over predecessors of
// val + edge cost), each predecessor earlier in that order.
//
// The tasks are taken in blocks of up to kBkB = 2048.  Predecessors before the
// block are final and fold into base(t); inside it the values come by policy
// iteration in LDS: every task follows one predecessor (first the previous
// task on its device or channel) or none, pointer jumping sums the chains
// asynchronously (a (sum, next) pair is one 64-bit LDS word, so every version
// read is a true pair), and each task then switches to a strictly larger
// predecessor until none can: the values then satisfy the recurrence, whose
// solution is unique.  An Adjusting Placement of the 1.07M-node transformer
// graph with transfer tasks needs 3.4 iterations a block (691 blocks); over
// the whole graph at once it would need 228, on inception-600 1,150, since
// every switch is followed by a change further down the channels.
//
// What bounds it: one workgroup per placement, so the latency of a block:
// about 2.5 us of dependent loads and LDS (its own tasks are read a block
// ahead) and 2.9 us per iteration, of which the jumps' LDS traffic takes 1.7
// (counters: the CU's vector units issue in 54 % of the cycles, its LDS works in
// about half of them, 8 % of those on bank conflicts).
// Blocks of 1,024 and 4,096 tasks took 1.7 and 4 times as long per call (more
// blocks; more LDS traffic a round and register spills).  Whole calls, the walk
// in order (k_makespan_model) against the blocks: transfer tasks on the 1.07M-node
// graph 121 -> 8.4 ms, on inception-600 15.7 -> 1.3, on transformer-24 3.7 ->
// 0.40; FIFO devices on inception-600 10.0 -> 0.44; transfers on the compute
// queues there 15.2 -> 0.55.
//
// A block reserves list space in LDS for tasks of more than four inputs (of a
// long row for as many as the block can hold); where it does not suffice the
// block is taken again with half the tasks, and the next one with twice as many.
// A call
// whose values reach 2^47 (the packed words hold 48 bits), or that needs more
// iterations than the other method would cost, raises st->i1 and writes no
// result: the caller runs the other method.
#include "cel_internal.h"

namespace cel {

constexpr int kBkB = 2048;        // tasks of a block at most; chunks of the task order
constexpr int kBkT = 1024;        // threads
constexpr int kBkU = kBkB / kBkT; // tasks per thread
constexpr int kBkOv = 16384;      // list entries of tasks with more than four inputs
constexpr int kBkLight = 16;      // longer input rows are read by the whole wave
// Entries are named by their byte offset in s_e; the one past the block's last
// has value 0 and itself as next: chains end there, and a missing
// predecessor reads it (no arrival is below 0).
constexpr uint32_t kEnd = 8 * kBkB;

// Per task, within its chunk of kBkB tasks: the previous task on its first
// resource (+ 1, 0: none) in bits 0-12, on its second in bits 13-25, and
// whether it is the last on the first (bit 26) and on the second (bit 27).
constexpr uint32_t kBkLast1 = 1u << 26, kBkLast2 = 1u << 27;

__device__ inline int64_t bk_dur(int64_t w, int64_t tm) {  // ceil(w * tm / 1024)
  return (w >> 10) * tm + (((w & 1023) * tm + 1023) >> 10);
}
__device__ inline int64_t bk_link(int64_t ob, int32_t bw, int32_t lat) {
  return ob / bw + (ob % bw != 0 ? 1 : 0) + lat;
}

// lanes whose key equals x (kb bits), as ballots of the keys' bits
template <int KB>
__device__ inline uint64_t same_key(uint32_t x, const uint64_t (&bits)[KB], uint64_t act) {
  uint64_t m = act;
#pragma unroll
  for (int b = 0; b < KB; b++) m &= (x >> b) & 1u ? bits[b] : ~bits[b];
  return m;
}

// The info words.  TASKS: keys of two resources per task (255: none) from
// key[]; otherwise one resource, the device in devp[].  A workgroup takes one
// chunk: in every wave of 64 tasks the previous lane of the same key by
// ballots, across the chunk's 64 waves by a table of each wave's last task per
// key and a prefix maximum over it.
template <bool TASKS>
__global__ void __launch_bounds__(kBkT) k_bk_prev(int32_t n, int32_t nk, const uint8_t *devp,
                                                 const uint16_t *key, const int64_t *aoff,
                                                 uint32_t *info, const Status *st) {
  constexpr int KB = 8;
  __shared__ uint16_t s_last[kBkB / 64][256];  // task + 1, 0: none
  __shared__ uint16_t s_all[256];
  if (failed(st)) return;
  const int64_t k = blockIdx.y;
  const int64_t t0 = TASKS ? k * n + aoff[k * n] : k * n;
  const int64_t N = TASKS ? (k + 1) * (int64_t)n + aoff[(k + 1) * n] - t0 : n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1;
  for (int64_t cb = (int64_t)blockIdx.x * kBkB; cb < N; cb += (int64_t)gridDim.x * kBkB) {
    for (int i = threadIdx.x; i < kBkB / 64 * 128; i += kBkT) reinterpret_cast<uint32_t *>(s_last)[i] = 0;
    __syncthreads();
    uint32_t k1[kBkU], k2[kBkU];
    int32_t p1[kBkU], p2[kBkU];  // previous task + 1
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      const int32_t t = u * kBkT + threadIdx.x;
      const bool act = cb + t < N;
      k1[u] = k2[u] = 255;
      if (act) {
        if (TASKS) {
          const uint32_t x = key[t0 + cb + t];
          k1[u] = x & 255u;
          k2[u] = x >> 8;
        } else {
          k1[u] = devp[t0 + cb + t];
        }
      }
      const int sg = u * (kBkT / 64) + wave;
      uint64_t b1[KB], b2[KB];
      const uint64_t a1 = __ballot(act), a2 = TASKS ? __ballot(k2[u] != 255) : 0;
#pragma unroll
      for (int b = 0; b < KB; b++) {
        b1[b] = __ballot(act && (k1[u] >> b) & 1u);
        b2[b] = TASKS ? __ballot(k2[u] != 255 && (k2[u] >> b) & 1u) : 0;
      }
      uint64_t m1 = same_key<KB>(k1[u], b1, a1);
      if (TASKS && a2) m1 |= same_key<KB>(k1[u], b2, a2);
      p1[u] = m1 & lt ? t - lane + 64 - __builtin_clzll(m1 & lt) : 0;
      p2[u] = 0;
      // the wave's last task of every key
      if (act && !(m1 >> lane >> 1)) s_last[sg][k1[u]] = (uint16_t)(t + 1);
      if (TASKS && a2) {
        uint64_t m2 = same_key<KB>(k2[u], b1, a1) | same_key<KB>(k2[u], b2, a2);
        if (k2[u] == 255) m2 = 0;
        p2[u] = m2 & lt ? t - lane + 64 - __builtin_clzll(m2 & lt) : 0;
        if (k2[u] != 255 && !(m2 >> lane >> 1)) s_last[sg][k2[u]] = (uint16_t)(t + 1);
      }
    }
    __syncthreads();
    for (int x = wave; x < nk; x += kBkT / 64) {  // lane: a wave of 64 tasks
      constexpr int NW = kBkB / 64;
      int32_t v = lane < NW ? s_last[lane][x] : 0;
      for (int o = 1; o < NW; o <<= 1) {
        const int32_t y = __shfl_up(v, o);
        if (lane >= o && y > v) v = y;
      }
      if (lane == NW - 1) s_all[x] = (uint16_t)v;
      const int32_t before = __shfl_up(v, 1);
      if (lane < NW) s_last[lane][x] = (uint16_t)(lane ? before : 0);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      const int32_t t = u * kBkT + threadIdx.x;
      if (cb + t >= N) continue;
      const int sg = u * (kBkT / 64) + wave;
      uint32_t x = p1[u] ? (uint32_t)p1[u] : s_last[sg][k1[u]];
      if (s_all[k1[u]] == t + 1) x |= kBkLast1;
      if (TASKS && k2[u] != 255) {
        x |= (p2[u] ? (uint32_t)p2[u] : s_last[sg][k2[u]]) << 13;
        if (s_all[k2[u]] == t + 1) x |= kBkLast2;
      }
      info[t0 + cb + t] = x;
    }
    __syncthreads();
  }
}

// The task of node position p of placement k, from its first one: p plus the
// transfers of the positions before it.
__device__ inline int32_t bk_task(const int64_t *aoff, int64_t kn, int32_t p) {
  return p + (int32_t)(aoff[kn + p] - aoff[kn]);
}

// Tasks of K placements in issue order: weight, resources and the tasks of up
// to four inputs (rec: -1 past them; a node of more inputs on other devices has
// -2 - p in rec.w and reads its row again).  BLOCK: both resources of a
// transfer are device queues, and its producer is the one before it on the
// first; otherwise they are the send channel (D + device) and the receive
// channel (2 D + device).
template <bool HET, bool BLOCK>
__global__ void k_bk_tasks(int32_t K, int32_t n, int32_t D, const int32_t *iptr,
                           const int32_t *iidx, const int64_t *wp, const int64_t *cq,
                           const uint8_t *devp, const uint64_t *dmask, const int64_t *aoff,
                           const int64_t *tmul, const int64_t *lbw, const int64_t *llat, int4 *rec,
                           int64_t *wv, uint16_t *key, Status *st) {
  if (failed(st)) return;
  uint32_t bad = 0;
  for (int64_t k = blockIdx.y; k < K; k += gridDim.y) {
    const int64_t kn = k * n;
    for (int32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < n; p += gridDim.x * blockDim.x) {
      const int32_t d = devp[kn + p], t = bk_task(aoff, kn, p);
      const int64_t g = kn + aoff[kn] + t, c = cq[p];
      int32_t r[4] = {-1, -1, -1, -1};
      int32_t cnt = 0;
      for (int32_t e = iptr[p]; e < iptr[p + 1] && cnt <= 4; e++) {
        const int32_t u = iidx[e];
        if (devp[kn + u] == d) continue;
        const uint64_t m = dmask[kn + u];
        if (!((m >> d) & 1)) {  // CSR and CSC disagree
          bad |= EB_ARG;
          continue;
        }
        const int32_t x = bk_task(aoff, kn, u) + 1 + __builtin_popcountll(m & ((1ull << d) - 1));
        if (cnt == 0) r[0] = x;
        else if (cnt == 1) r[1] = x;
        else if (cnt == 2) r[2] = x;
        else if (cnt == 3) r[3] = x;
        cnt++;
      }
      rec[g] = cnt > 4 ? make_int4(-1, -1, -1, -2 - p) : make_int4(r[0], r[1], r[2], r[3]);
      wv[g] = HET ? bk_dur(wp[p], tmul[d]) : wp[p];
      key[g] = (uint16_t)(d | 255 << 8);
      int64_t x = g + 1;
      for (uint64_t m = dmask[kn + p]; m; m &= m - 1, x++) {
        const int b = __builtin_ctzll(m);
        rec[x] = make_int4(BLOCK ? -1 : t, -1, -1, -1);
        wv[x] = HET ? bk_link(c, (int32_t)lbw[d * D + b], (int32_t)llat[d * D + b]) : c;
        key[x] = (uint16_t)(BLOCK ? d | b << 8 : (D + d) | (2 * D + b) << 8);
      }
    }
  }
  if (bad) raise_err(st, bad);
}

// finish of every node from its task's value
__global__ void k_bk_gather(int32_t K, int32_t n, const int64_t *aoff, const int64_t *val,
                            int64_t *finp, const Status *st) {
  if (failed(st)) return;
  const int64_t tot = (int64_t)K * n;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < tot;
       i += (int64_t)gridDim.x * blockDim.x)
    finp[i] = val[i + aoff[i]];
}

struct BkArgs {
  int32_t n, D, nk, budget;
  int32_t fits;                 // values known to stay below 2^47 (else st->total decides)
  const int32_t *iptr, *iidx;   // predecessors in position space
  const int4 *ipre;             // first 4 of them (-1 past the row)
  const int64_t *wp, *cq;       // w and c (heterogeneous links: ob) by position
  const uint8_t *devp;          // [K][n]
  const int64_t *tmul, *lbw, *llat;
  const uint32_t *info;         // per task
  const int64_t *aoff;          // transfers: [K n + 1]
  const uint64_t *dmask;
  const int4 *rec;              // transfers: per task
  const int64_t *wv;
  const uint16_t *key;
  int64_t *val;                 // finish per task (no transfers: [K][n] by position)
  int64_t *makespan;            // [K]
};

// entries that other waves write meanwhile (relaxed atomics: plain LDS reads
// and writes of the whole word; volatile ones go through the flat path)
__device__ inline uint64_t lds_ld(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline void lds_st(uint64_t *p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// XFER: tasks with transfers; otherwise nodes alone, a cross-device input
// costing c (HET: its link's cost) on the edge.  (<false, true> spills 96 bytes a
// lane, outside the iterations: 1,024 threads leave a lane 128 registers.)
template <bool XFER, bool HET>
__global__ void __launch_bounds__(kBkT) k_ms_blocks(BkArgs a, Status *st) {
  constexpr int kKeys = XFER ? 192 : (HET ? 64 : 256);
  __shared__ uint64_t s_ent[2][kBkB + 1];           // value << 16 | next, by block parity
  __shared__ int64_t s_c[XFER ? 1 : kBkB + 1];      // c (or ob) of the block's nodes
  __shared__ uint8_t s_dev[XFER ? 1 : kBkB + 1];
  __shared__ uint16_t s_ov[kBkOv];
  __shared__ int64_t s_free[kKeys];                 // finish of the last task on each resource
  __shared__ int32_t s_bw[HET ? 64 * 64 : 1], s_lat[HET ? 64 * 64 : 1];
  __shared__ int64_t s_red[kBkT / 64];
  __shared__ int32_t s_ovn, s_f, s_chg[3];
  __shared__ int32_t s_blk;  // blocks that ended (thread 0; a register more costs 2 %)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) {
    s_f = failed(st) ? 1 : 0;
    if (!s_f && !a.fits && st->total >= (uint64_t(1) << 47)) {
      atomicOr(&st->i1, 1);
      s_f = 1;
    }
  }
  for (int i = tid; i < kKeys; i += kBkT) s_free[i] = 0;
  if (HET)
    for (int i = tid; i < a.D * a.D; i += kBkT) {
      s_bw[i] = (int32_t)a.lbw[i];
      s_lat[i] = (int32_t)a.llat[i];
    }
  __syncthreads();
  if (s_f) return;
  const int32_t n = a.n, D = a.D;
  const int64_t kn = (int64_t)blockIdx.x * n;
  const int64_t t0 = XFER ? kn + a.aoff[kn] : kn;  // the placement's first task
  const int32_t N = XFER ? (int32_t)(kn + n + a.aoff[kn + n] - t0) : n;
  const uint8_t *dev = a.devp + kn;
  int64_t *val = a.val + t0;
  int64_t span = 0;
  int32_t its = 0, nt = 0;
  int32_t pp0 = 0;  // the previous block's first task
  // The budget is spent.  (Written out at both places without transfers, once at
  // the end with them: all registers are in use, and the other way round either
  // kernel takes 3 to 4 % longer.)
  auto give_up = [&]() {
    if (tid == 0) {
      atomicOr(&st->i1, 1);
      atomicMax(&st->i2, its);
      atomicMax(&st->i3, s_blk);
    }
  };
  if (tid == 0) {
    s_ent[0][kBkB] = s_ent[1][kBkB] = kEnd;
    if (!XFER) {
      s_c[kBkB] = 0;
      s_dev[kBkB] = 0;
    }
    s_chg[0] = s_chg[1] = s_chg[2] = 0;
    s_blk = 0;
  }
  struct Task {  // a task's own data, read a block ahead
    int64_t wv, c;
    int4 q;
    uint32_t inf, kk;
    int32_t cnt;  // row length (not XFER)
  };
  auto load = [&](int32_t p) {
    Task x{0, 0, make_int4(-1, -1, -1, -1), 0, 255 << 8, 0};
    if (p < N) {
      x.inf = a.info[t0 + p];
      if (XFER) {
        x.q = a.rec[t0 + p];
        x.wv = a.wv[t0 + p];
        x.kk = a.key[t0 + p];
      } else {
        x.kk = (uint32_t)dev[p] | 255u << 8;
        x.q = a.ipre[p];
        x.cnt = a.iptr[p + 1] - a.iptr[p];
        x.wv = a.wp[p];
        x.c = a.cq[p];
      }
    }
    return x;
  };
  Task cur[kBkU];
#pragma unroll
  for (int u = 0; u < kBkU; u++) cur[u] = load(u * kBkT + tid);
  for (int32_t p0 = 0, lim = kBkB, par = 0; p0 < N;) {
    uint64_t *const s_e = s_ent[par];
    const uint64_t *const s_pe = s_ent[par ^ 1];
    // a final value before the block: the previous block's are read from LDS;
    // older ones were complete before the previous block's store_barrier
    auto final_val = [&](int32_t x) -> int64_t {
      return x >= pp0 ? (int64_t)(s_pe[x - pp0] >> 16) : val[x];
    };
    const int32_t cb = p0 & ~(kBkB - 1);  // the chunk's first task; blocks stay inside it
    nt = N - p0 < lim ? N - p0 : lim;
    if (cb + kBkB - p0 < nt) nt = cb + kBkB - p0;
    int64_t wv[kBkU], base[kBkU];
    uint32_t inf[kBkU], kk[kBkU], ch[kBkU];  // resources; slots of the previous tasks on them
    int4 q[kBkU];
    int32_t cnt[kBkU];   // row length (XFER: 0, or the row of a node with many inputs)
    uint32_t ovr[kBkU];  // list: start | entries << 16
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      const int32_t t = u * kBkT + tid;
      wv[u] = cur[u].wv;
      base[u] = 0;
      inf[u] = cur[u].inf;
      kk[u] = cur[u].kk;
      q[u] = cur[u].q;
      cnt[u] = cur[u].cnt;
      if (t >= nt) {
        inf[u] = cnt[u] = 0;
        kk[u] = 255 << 8;
        q[u] = make_int4(-1, -1, -1, -1);
      } else if (!XFER) {
        if (HET) wv[u] = bk_dur(wv[u], a.tmul[kk[u] & 255u]);
        s_dev[t] = (uint8_t)kk[u];
        s_c[t] = cur[u].c;
      }
    }
    if (tid == 0) s_ovn = 0;
    lds_barrier();
    // ---- previous tasks on the resources
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      const int32_t t = u * kBkT + tid;
      uint32_t c2[2] = {kEnd, kEnd};
#pragma unroll
      for (int x = 0; x < (XFER ? 2 : 1); x++) {
        const uint32_t key = x ? kk[u] >> 8 : kk[u] & 255u;
        if (t >= nt || key == 255) continue;
        const int32_t pr = (int32_t)((inf[u] >> (13 * x)) & 0x1FFFu) - 1;
        if (pr < 0) base[u] = max_nonneg(base[u], s_free[key]);
        else if (cb + pr >= p0) c2[x] = 8u * (uint32_t)(cb + pr - p0);
        else base[u] = max_nonneg(base[u], final_val(cb + pr));
      }
      ch[u] = c2[0] | c2[1] << 16;
    }
    // ---- inputs: before the block into base, inside it into slots
    uint32_t s01[kBkU], s23[kBkU];
    auto edge = [&](int64_t c, int32_t du, int32_t dv) -> int64_t {  // cross-device cost (not XFER)
      return HET ? bk_link(c, s_bw[du * D + dv], s_lat[du * D + dv]) : c;
    };
    // task of input u of a node on device d, or -1 on the same device (XFER)
    auto xtask = [&](int32_t v, int32_t d) -> int32_t {
      if (dev[v] == d) return -1;
      return bk_task(a.aoff, kn, v) + 1 + __builtin_popcountll(a.dmask[kn + v] & ((1ull << d) - 1));
    };
    // one input (XFER: its task): folded when before the block, its entry returned otherwise
    auto input = [&](int32_t x, int32_t d, int64_t &b) -> uint32_t {
      if (x < 0) return kEnd;
      if (XFER) {
        if (x >= p0) return 8u * (uint32_t)(x - p0);
        b = max_nonneg(b, final_val(x));
        return kEnd;
      }
      if (x >= p0) return s_dev[x - p0] == d ? kEnd : 8u * (uint32_t)(x - p0);
      const int32_t du = dev[x];
      const int64_t v = final_val(x), c = a.cq[x];
      if (du != d) b = max_nonneg(b, v + edge(c, du, d));
      return kEnd;
    };
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      const int32_t d = (int32_t)(kk[u] & 255u);
      int32_t hp = -1;  // the node's position when its row is read here
      if (XFER) {
        if (q[u].w < -1) {
          hp = -2 - q[u].w;
          cnt[u] = a.iptr[hp + 1] - a.iptr[hp];
        }
      } else if (cnt[u] > 4) {
        hp = p0 + u * kBkT + tid;
      }
      const bool row = hp >= 0;
      const bool heavy = row && cnt[u] > kBkLight;
      uint32_t sl[4] = {kEnd, kEnd, kEnd, kEnd};
      if (!(XFER && row) && !heavy) {
        sl[0] = input(q[u].x, d, base[u]);
        sl[1] = input(q[u].y, d, base[u]);
        sl[2] = input(q[u].z, d, base[u]);
        sl[3] = input(q[u].w, d, base[u]);
      }
      s01[u] = sl[0] | sl[1] << 16;
      s23[u] = sl[2] | sl[3] << 16;
      ovr[u] = 0;
      if (row && !heavy) {
        const int32_t e0 = a.iptr[hp] + (XFER ? 0 : 4), e1 = a.iptr[hp + 1];
        int32_t o = 0, m = 0;
        if (nt > 1) o = atomicAdd(&s_ovn, e1 - e0);
        for (int32_t e = e0; e < e1; e++) {
          const uint32_t s = input(XFER ? xtask(a.iidx[e], d) : a.iidx[e], d, base[u]);
          if (s != kEnd && o + m < kBkOv) s_ov[o + m++] = (uint16_t)s;
        }
        ovr[u] = (uint32_t)o | (uint32_t)m << 16;
      }
      for (uint64_t hv = __ballot(heavy); hv; hv &= hv - 1) {  // the whole wave reads one row
        const int l = __builtin_ctzll(hv);
        const int32_t ph = __builtin_amdgcn_readlane(hp, l), dh = __builtin_amdgcn_readlane(d, l);
        const int32_t e0 = a.iptr[ph], e1 = a.iptr[ph + 1];
        // at most nt - 1 of the inputs lie in the block, unless edges are parallel
        int32_t o = 0, m = 0, room = 0;
        if (nt > 1) {
          room = e1 - e0 < nt ? e1 - e0 : nt;
          if (lane == l) o = atomicAdd(&s_ovn, room);
          o = __builtin_amdgcn_readlane(o, l);
        }
        int64_t b = 0;
        for (int32_t e = e0; e < e1; e += 64) {
          uint32_t s = kEnd;
          if (e + lane < e1) s = input(XFER ? xtask(a.iidx[e + lane], dh) : a.iidx[e + lane], dh, b);
          const uint64_t in = __ballot(s != kEnd);
          const int32_t at = m + __popcll(in & ((1ull << lane) - 1));
          if (s != kEnd && at < room && o + at < kBkOv) s_ov[o + at] = (uint16_t)s;
          m += __popcll(in);
        }
        if (m > room && lane == l) atomicAdd(&s_ovn, kBkOv + 1);
        for (int x = 32; x > 0; x >>= 1) b = max_nonneg(b, (int64_t)__shfl_xor((long long)b, x));
        if (lane == l) {
          base[u] = max_nonneg(base[u], b);
          ovr[u] = (uint32_t)o | (uint32_t)m << 16;
        }
      }
    }
    // The previous block's values, stored about a block ago, are complete
    // behind this barrier: the next block reads them from memory.
    store_barrier();
    if (s_ovn > kBkOv) {  // too many listed inputs: half the tasks (nt = 1 lists none)
      lim = nt / 2;
      its++;          // about as long
      lds_barrier();  // every wave has read s_ovn before it is cleared
      continue;
    }
    // ---- policy iteration (LDS barriers only: the next block's data is on its way)
#pragma unroll
    for (int u = 0; u < kBkU; u++) cur[u] = load(p0 + nt + u * kBkT + tid);
    auto entry = [&](uint32_t off) -> uint64_t {
      return lds_ld(reinterpret_cast<const uint64_t *>(reinterpret_cast<const char *>(s_e) + off));
    };
    int64_t ec[kBkU], v[kBkU];
    uint32_t pol[kBkU];
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      pol[u] = ch[u] & 0xFFFFu;
      ec[u] = 0;
    }
    for (int32_t i = 0;; i = i == 2 ? 0 : i + 1) {
      uint64_t e[kBkU];
#pragma unroll
      for (int u = 0; u < kBkU; u++) {
        const int32_t t = u * kBkT + tid;
        e[u] = kEnd;
        if (t < nt) {
          e[u] = (uint64_t)(wv[u] + (pol[u] == kEnd ? base[u] : ec[u])) << 16 | pol[u];
          s_e[t] = e[u];
        }
      }
      lds_barrier();
      // Every jump moves a chain's end to an earlier task: the values add, the
      // next entry is the one read (a chain that has ended adds 0 and stays:
      // masking it out costs more than its reads and writes, 8.6 against 7.7 ms).
      for (bool any = true; any;) {
        uint32_t open = 0;
        uint64_t f[kBkU];
#pragma unroll
        for (int u = 0; u < kBkU; u++) f[u] = entry((uint32_t)e[u] & 0xFFFFu);
#pragma unroll
        for (int u = 0; u < kBkU; u++) {
          e[u] = (e[u] & ~uint64_t(0xFFFF)) + f[u];
          open |= ((uint32_t)e[u] & 0xFFFFu) ^ kEnd;
          if (u * kBkT + tid < nt) lds_st(&s_e[u * kBkT + tid], e[u]);
        }
        any = __ballot(open != 0) != 0;
      }
      lds_barrier();
      // ---- improvement: strictly larger arrivals only
      bool chg = false;
#pragma unroll
      for (int u = 0; u < kBkU; u++) {
        v[u] = (int64_t)(e[u] >> 16);
        const int32_t d = (int32_t)(kk[u] & 255u);
        const int64_t arr = v[u] - wv[u];
        int64_t best = arr;
        uint32_t np = pol[u];
        int64_t nc = ec[u];
        if (base[u] > best) {
          best = base[u];
          np = kEnd;
          nc = 0;
        }
        auto look = [&](uint32_t off, bool chain) {
          int64_t c = 0;
          if (!XFER && !chain) {
            c = edge(s_c[off >> 3], HET ? (int32_t)s_dev[off >> 3] : 0, d);
            if (HET && off == kEnd) c = 0;
          }
          const int64_t x = (int64_t)(entry(off) >> 16) + c;
          const bool b = x > best;
          best = b ? x : best;
          np = b ? off : np;
          nc = b ? c : nc;
        };
        look(ch[u] & 0xFFFFu, true);
        if (XFER) look(ch[u] >> 16, true);
        look(s01[u] & 0xFFFFu, false);
        look(s01[u] >> 16, false);
        if (__ballot(s23[u] != (kEnd | kEnd << 16))) {
          look(s23[u] & 0xFFFFu, false);
          look(s23[u] >> 16, false);
        }
        for (uint32_t x = 0; x < ovr[u] >> 16; x++) look(s_ov[(ovr[u] & 0xFFFFu) + x], false);
        if (u * kBkT + tid < nt && best > arr) {
          pol[u] = np;
          ec[u] = nc;
          chg = true;
        }
      }
      its++;
      if (__ballot(chg) && lane == 0) s_chg[i] = 1;
      if (tid == 0) s_chg[i == 2 ? 0 : i + 1] = 0;  // last read two iterations ago
      lds_barrier();
      if (!s_chg[i]) break;
      if (its > a.budget) {  // uniform: the caller runs the other method
        if (XFER) goto over;
        give_up();
        return;
      }
    }
    // ---- the block's finish times
#pragma unroll
    for (int u = 0; u < kBkU; u++) {
      const int32_t t = u * kBkT + tid;
      if (t >= nt) continue;
      val[p0 + t] = v[u];
      if (!XFER || kk[u] >> 8 == 255) span = max_nonneg(span, v[u]);
      if (inf[u] & kBkLast1) s_free[kk[u] & 255u] = v[u];
      if (XFER && (inf[u] & kBkLast2)) s_free[kk[u] >> 8] = v[u];
    }
    if (tid == 0) atomicAdd(&s_blk, 1);  // (no wait)
    pp0 = p0;
    p0 += nt;
    par ^= 1;
    lim = 2 * lim < kBkB ? 2 * lim : kBkB;
    lds_barrier();
    if (tid == 0) s_chg[0] = 0;  // the next block's first flag, read behind two more barriers
    if (its > a.budget && p0 < N) {  // whatever the block needed
      if (XFER) goto over;
      give_up();
      return;
    }
  }
  for (int o = 32; o > 0; o >>= 1) span = max_nonneg(span, (int64_t)__shfl_xor((long long)span, o));
  if (lane == 0) s_red[wave] = span;
  __syncthreads();
  if (tid == 0) {
    for (int i = 1; i < kBkT / 64; i++) span = max_nonneg(span, s_red[i]);
    a.makespan[blockIdx.x] = span;
    atomicMax(&st->i2, its);
    atomicMax(&st->i3, s_blk);
  }
  return;
over:
  give_up();
}

// ------------------------------------------------------------------- host

namespace {
struct BkInfo {
  int32_t path, iters, blocks;
};
thread_local BkInfo t_bk_info{1, 0, 0};
}  // namespace

void ms_blocks_info(const Status *h) {
  t_bk_info = h ? BkInfo{h->i1 ? 1 : 0, h->i2, h->i3} : BkInfo{1, 0, 0};
}

int ms_blocks(const MsBlocks &b, Scratch &sc, hipStream_t s, Status *st) {
  const int64_t Kn = (int64_t)b.K * b.n;
  BkArgs a{};
  a.n = b.n;
  a.D = b.D;
  a.budget = b.budget;
  a.fits = b.fits;
  a.iptr = b.iptr;
  a.iidx = b.iidx;
  a.ipre = b.ipre;
  a.wp = b.wp;
  a.cq = b.cq;
  a.devp = b.devp;
  a.tmul = b.tmul;
  a.lbw = b.lbw;
  a.llat = b.llat;
  a.aoff = b.aoff;
  a.dmask = b.dmask;
  a.makespan = b.makespan;
  const bool het = b.tmul != nullptr;
  uint32_t *info = b.info;
  const int gy = b.K < 1024 ? b.K : 1024;
  if (!b.aoff) {
    a.nk = b.D;
    a.val = b.finp;
    if (!info) CEL_TRY(sc.get(&info, Kn));
    k_bk_prev<false><<<dim3((b.n + kBkB - 1) / kBkB, b.K), kBkT, 0, s>>>(b.n, b.D, b.devp, nullptr,
                                                                        nullptr, info, st);
  } else {
    a.nk = b.block ? b.D : 3 * b.D;
    const int64_t tot = Kn + b.transfers;
    int4 *rec;
    int64_t *wv;
    uint16_t *key;
    CEL_TRY(sc.get(&info, tot));
    CEL_TRY(sc.get(&rec, tot));
    CEL_TRY(sc.get(&wv, tot));
    CEL_TRY(sc.get(&key, tot));
    CEL_TRY(sc.get(&a.val, tot));
    const dim3 gt(grid_for(b.n, 256, 4096), gy);
#define CEL_BK_TASKS(H, B)                                                                        \
  k_bk_tasks<H, B><<<gt, 256, 0, s>>>(b.K, b.n, b.D, b.iptr, b.iidx, b.wp, b.cq, b.devp, b.dmask, \
                                      b.aoff, b.tmul, b.lbw, b.llat, rec, wv, key, st)
    if (het && b.block) CEL_BK_TASKS(true, true);
    else if (het) CEL_BK_TASKS(true, false);
    else if (b.block) CEL_BK_TASKS(false, true);
    else CEL_BK_TASKS(false, false);
#undef CEL_BK_TASKS
    k_bk_prev<true><<<dim3((unsigned)(tot / b.K / kBkB + 1), b.K), kBkT, 0, s>>>(
        b.n, a.nk, nullptr, key, b.aoff, info, st);
    a.rec = rec;
    a.wv = wv;
    a.key = key;
  }
  a.info = info;
  {
    KTimer kt(s, b.timer);
    if (b.aoff) k_ms_blocks<true, false><<<b.K, kBkT, 0, s>>>(a, st);
    else if (het) k_ms_blocks<false, true><<<b.K, kBkT, 0, s>>>(a, st);
    else k_ms_blocks<false, false><<<b.K, kBkT, 0, s>>>(a, st);
  }
  if (b.aoff)
    k_bk_gather<<<grid_for(Kn, 256, 8192), 256, 0, s>>>(b.K, b.n, b.aoff, a.val, b.finp, st);
  CEL_HIP(hipGetLastError());
  return CEL_OK;
}

}  // namespace cel

extern "C" int cel_makespan_blocks_info(int32_t *info) {
  using namespace cel;
  if (!info) return set_error(CEL_E_ARG, "cel_makespan_blocks_info: NULL argument");
  info[0] = t_bk_info.path;
  info[1] = t_bk_info.iters;
  info[2] = t_bk_info.blocks;
  return CEL_OK;
}
