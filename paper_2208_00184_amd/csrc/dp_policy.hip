// The clustering DP (Section 5.1.3, eq. 4-6) by policy iteration.
//
// In position space, with PO the prefix sum of each node's out-going comm and
// Int(i, j) the comm of the edges with both ends in [i, j):
//   S(0) = 0,  S(j) = min over lo(j) <= i < j of S(i) + cost(i, j),
//   cost(i, j) = PO[j] - PO[i] - Int(i, j),
// a shortest path from 0 to every j over the breakpoint graph.  A policy is a
// back pointer P(j) in [lo(j), j) for every j; its values S_P(j) = S_P(P(j)) +
// cost(P(j), j) are sums along the pointers, found by pointer jumping.  Each
// j then switches to the candidate i of smallest S_P(i) + cost(i, j) when that
// is strictly below S_P(j).  Every policy's values are costs of real
// clusterings, a switch never raises a value, and when no j can switch the
// values satisfy the recurrence, whose solution is unique: S is exact.  The
// back pointers are then set to the smallest minimising i (the tie rule), so
// the breakpoints are those of the sequential DP.  Transformer-96 needs 9
// iterations where the blocked DP runs 16,728 dependent blocks.
// (k_dp_tiles below for values of 40 bits, k_dp_policy for larger ones.)
//
// Improvement: one thread per target j sweeps its candidates i = j - 1 down to
// lo(j), keeping Int(i, j) = Int(i + 1, j) + c(i) * #{successors of i at
// offsets below j - i}.  The offsets below R of each position's successors
// are packed four to a 64-bit word (14 bits each), or, for a position with
// more, kept as a table of counts below every d: every count is one load.
// Neighbouring threads read neighbouring candidates, so the window's data is
// read from the L1 cache; S - PO of the candidates is published behind a grid
// barrier with agent-scope fences (the plain, cached loads need them), every
// other value crossing workgroups goes through agent-scope atomics.
#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>

#include "cel_internal.h"

namespace cel {

constexpr int kDpB = 1024;
constexpr int kDpU = 4;          // nodes per thread with loads in flight together
constexpr uint32_t kDpOffMask = 0x3FFF;

// near successors: count per position (edge-balanced over the position CSR)
__global__ void k_dpn_count(int32_t n, int32_t m, int32_t R, const int32_t *sptr,
                            const int32_t *sidx, int32_t *ncnt, const Status *st) {
  __shared__ int32_t rp[kRowsPB + 1], su[2];
  if (failed(st)) return;
  for_edges_balanced(sptr, n, m, rp, su, [&](int32_t i, int32_t e) {
    const int32_t o = sidx[e] - i;
    if (o > 0 && o < R) atomicAdd(&ncnt[i], 1);
  });
}

__global__ void k_dpn_fill(int32_t n, int32_t m, int32_t R, const int32_t *sptr,
                           const int32_t *sidx, const int32_t *nptr, int32_t *ncnt,
                           uint16_t *noff, const Status *st) {
  __shared__ int32_t rp[kRowsPB + 1], su[2];
  if (failed(st)) return;
  for_edges_balanced(sptr, n, m, rp, su, [&](int32_t i, int32_t e) {
    const int32_t o = sidx[e] - i;
    if (o > 0 && o < R) noff[nptr[i] + atomicSub(&ncnt[i], 1) - 1] = (uint16_t)o;
  });
}

// Each position's offsets below R: up to four packed in a 64-bit word (14
// bits each, the unused ones kDpOffMask, above any offset); a position with
// more gets kDpHeavy | h, h its index among such positions, whose counts of
// offsets below d (d = 0..R, parallel edges counted each) form a table of
// R + 1 entries.
constexpr uint64_t kDpHeavy = uint64_t(1) << 62;

__global__ void k_dpn_heavy(int32_t n, const int32_t *nptr, int32_t *hflag, const Status *st) {
  if (failed(st)) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    hflag[i] = nptr[i + 1] - nptr[i] > 4 ? 1 : 0;
}

__global__ void k_dpn_pack(int32_t n, int32_t R, const int32_t *nptr, const uint16_t *noff,
                           const int32_t *hoff, uint64_t *nearw, uint32_t *hcnt,
                           const Status *st) {
  if (failed(st)) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t b = nptr[i], e = nptr[i + 1];
    if (e - b > 4) {
      const int64_t h = hoff[i];
      uint32_t *t = hcnt + h * (R + 1);
      for (int32_t d = 0; d <= R; d++) t[d] = 0;
      for (int32_t x = b; x < e; x++) t[noff[x] + 1]++;  // offsets < R: index <= R
      for (int32_t d = 1; d <= R; d++) t[d] += t[d - 1];  // t[d] = offsets below d
      nearw[i] = kDpHeavy | (uint64_t)h;
      continue;
    }
    uint16_t o[4] = {kDpOffMask, kDpOffMask, kDpOffMask, kDpOffMask};
    for (int32_t x = b; x < e; x++) o[x - b] = noff[x];
    uint64_t w = 0;
    for (int k = 0; k < 4; k++) w |= (uint64_t)o[k] << (16 * k);
    nearw[i] = w;
  }
}

struct DpArgs {
  int32_t n, R, cap, max_rounds;
  const int32_t *lo;          // [n + 1] first feasible i of a cluster ending at j
  const int64_t *PO;          // [n + 1]
  const int64_t *cq;          // [n] comm by position
  const uint64_t *nearw;      // [n] packed successor offsets below R, or a bitmask's index
  const uint32_t *hcnt;       // [H][R + 1] offsets below d of the positions with many
  int32_t *P;                 // [n + 1] back pointers (the output)
  int32_t *Parg;              // [n + 1] the smallest minimising i of the last improvement
  int64_t *cost;              // [n + 1] cost(P(j), j)
  int64_t *SP;                // [n + 1] S(i) - PO[i]
  LpE *e0, *e1;               // [n + 1] pointer-jumping entries
  int32_t *bar;
  Status *st;
};

// successors of a position at offsets below d (1 <= d <= R)
// (SWAR over the four 16-bit fields: a field b, an offset below 2^12 or the
// unused 0x3FFF, has bits 14-15 clear, so (0x8000 | d) - (b + 1) neither
// borrows nor carries across fields and keeps bit 15 exactly when b < d.)
__device__ inline int32_t dp_near_below(const DpArgs &a, uint64_t w, uint32_t d) {
  if (w & kDpHeavy) return (int32_t)a.hcnt[(int64_t)(uint32_t)w * (a.R + 1) + d];
  constexpr uint64_t kOnes = 0x0001000100010001ull, kHigh = 0x8000800080008000ull;
  const uint64_t t = (((uint64_t)d * kOnes) | kHigh) - (w + kOnes);
  return __popcll(t & kHigh);
}

// Values of any size: int64 sums, 16-byte pointer-jumping entries and
// synchronous rounds (PO[n] of 2^40 and more, positions past 2^24, or
// cel_policy_iteration(2)).
__global__ void __launch_bounds__(kDpB) k_dp_policy(DpArgs a) {
  __shared__ int32_t s_ok, s_bit;
  if (failed(a.st)) return;
  Status *st = a.st;
  const int32_t n = a.n;
  const int64_t gsz = (int64_t)gridDim.x * kDpB;
  const int64_t gid = (int64_t)blockIdx.x * kDpB + threadIdx.x;
  int32_t bar = 0, bit;
  // The first policy: clusters of half the window, R / 2 positions (fewer
  // where lo(j) binds), cost(P(j), j) from one scan of each window.  Chains
  // of n / (R / 2) pointers instead of the n of singleton clusters: on the
  // transformer graphs a third fewer pointer-jumping passes in all, with no
  // more iterations (any policy is a valid start; only the fixed point ends
  // the iteration).
  const int32_t h = a.R / 2 > 1 ? a.R / 2 : 1;
  for (int64_t j = gid; j <= n; j += gsz) {
    if (j == 0) {
      st32(&a.P[0], -1);
      st_coherent(&a.cost[0], 0);
      continue;
    }
    const int32_t lj = a.lo[j];
    const int32_t p = (int32_t)j - h > lj ? (int32_t)j - h : lj;
    int64_t Int = 0;
    for (int32_t i = (int32_t)j - 1; i >= p; i--)
      Int += a.cq[i] * dp_near_below(a, a.nearw[i], (uint32_t)(j - i));
    st32(&a.P[j], p);
    st_coherent(&a.cost[j], a.PO[j] - a.PO[p] - Int);
  }
  if (!grid_sync(a.bar, ++bar, 0, &s_ok, &s_bit, st, &bit)) return;
  LpE *cur = a.e0, *oth = a.e1;
  int32_t it = 0;
  bool done = false;
  for (; it < a.cap; it++) {
    // ---- evaluation: S(j) = sum of cost along the back pointers (P(j) = 0 ends a chain)
    int32_t more = 0;
    for (int64_t j0 = gid; j0 <= n; j0 += kDpU * gsz) {
      int32_t q[kDpU];
#pragma unroll
      for (int u = 0; u < kDpU; u++) {
        const int64_t j = j0 + u * gsz;
        q[u] = j <= n ? ld32(&a.P[j]) : -1;
      }
      int64_t cq_[kDpU];
      int32_t nq[kDpU];
#pragma unroll
      for (int u = 0; u < kDpU; u++) {
        cq_[u] = q[u] > 0 ? ld_coherent(&a.cost[q[u]]) : 0;
        nq[u] = q[u] > 0 ? ld32(&a.P[q[u]]) : -1;
      }
#pragma unroll
      for (int u = 0; u < kDpU; u++) {
        const int64_t j = j0 + u * gsz;
        if (j > n) continue;
        const int32_t nx = nq[u] > 0 ? nq[u] : -1;
        more |= nx >= 0;
        lpe_st(&cur[j], LpE{ld_coherent(&a.cost[j]) + cq_[u], nx, 0});
      }
    }
    more = __syncthreads_or(more);
    if (!grid_sync(a.bar, ++bar, more, &s_ok, &s_bit, st, &bit)) return;
    int32_t r = 1;
    while (bit) {
      if (r == a.max_rounds) {  // a pointer cycle: cannot happen (P(j) < j)
        raise_err(st, EB_ORDER);
        return;  // uniform: bit and r are the same in every workgroup
      }
      more = 0;
      for (int64_t j0 = gid; j0 <= n; j0 += kDpU * gsz) {
        LpE x[kDpU];
#pragma unroll
        for (int u = 0; u < kDpU; u++) {
          const int64_t j = j0 + u * gsz;
          x[u] = j <= n ? lpe_ld(&cur[j]) : LpE{0, -1, 1};
        }
        LpE y[kDpU];
#pragma unroll
        for (int u = 0; u < kDpU; u++) y[u] = x[u].nxt >= 0 ? lpe_ld(&cur[x[u].nxt]) : LpE{0, -1, 0};
#pragma unroll
        for (int u = 0; u < kDpU; u++) {
          const int64_t j = j0 + u * gsz;
          if (j > n || x[u].both) continue;
          if (x[u].nxt < 0) {
            lpe_st(&oth[j], LpE{x[u].v, -1, 1});
            st32(&cur[j].both, 1);
          } else {
            const LpE z{x[u].v + y[u].v, y[u].nxt, 0};
            more |= z.nxt >= 0;
            lpe_st(&oth[j], z);
          }
        }
      }
      more = __syncthreads_or(more);
      if (!grid_sync(a.bar, ++bar, more, &s_ok, &s_bit, st, &bit)) return;
      LpE *t = cur;
      cur = oth;
      oth = t;
      r++;
    }
    // S - PO for the candidates (plain stores, published by a fenced barrier)
    for (int64_t j = gid; j <= n; j += gsz)
      a.SP[j] = ld_coherent(&cur[j].v) - a.PO[j];
    if (!grid_sync_fenced(a.bar, ++bar, &s_ok, &s_bit, st)) return;
    // ---- improvement: the best candidate of every target
    int32_t chg = 0;
    for (int64_t j = gid + 1; j <= n; j += gsz) {
      const int32_t lj = a.lo[j];
      int64_t Int = 0, best = kInf, ib = 0;
      int32_t arg = (int32_t)j - 1;
      int32_t i = (int32_t)j - 1;
      for (; i >= lj + 3; i -= 4) {  // four candidates with their loads in flight
        uint64_t nw[4];
        int64_t ci[4], sp[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          nw[u] = a.nearw[i - u];
          ci[u] = a.cq[i - u];
          sp[u] = a.SP[i - u];
        }
        int32_t k[4];
#pragma unroll
        for (int u = 0; u < 4; u++) k[u] = dp_near_below(a, nw[u], (uint32_t)(j - (i - u)));
#pragma unroll
        for (int u = 0; u < 4; u++) {
          Int += ci[u] * k[u];
          const int64_t v = sp[u] - Int;
          if (v <= best) {
            best = v;
            arg = i - u;
            ib = Int;
          }
        }
      }
      for (; i >= lj; i--) {
        Int += a.cq[i] * dp_near_below(a, a.nearw[i], (uint32_t)(j - i));
        const int64_t v = a.SP[i] - Int;
        if (v <= best) {
          best = v;
          arg = i;
          ib = Int;
        }
      }
      st32(&a.Parg[j], arg);
      if (best < a.SP[j]) {  // PO[j] + best < S(j): strictly better
        st32(&a.P[j], arg);
        st_coherent(&a.cost[j], a.PO[j] - a.PO[arg] - ib);
        chg = 1;
      }
    }
    chg = __syncthreads_or(chg);
    if (!grid_sync(a.bar, ++bar, chg, &s_ok, &s_bit, st, &bit)) return;
    if (!bit) {
      done = true;
      break;
    }
  }
  if (!done) {
    if (gid == 0) {
      st->i2 = 0;
      st->i3 = it;
    }
    return;
  }
  // converged: the smallest minimising i of every target, and S(n)
  for (int64_t j = gid + 1; j <= n; j += gsz) a.P[j] = ld32(&a.Parg[j]);
  if (gid == 0) {
    st->s0 = a.SP[n] + a.PO[n];
    st->i2 = 1;
    st->i3 = it + 1;
  }
}

// ------------------------------------------- packed values, candidates in LDS
//
// The same iteration when PO[n] < 2^40 and n < 2^24: every value is an exact
// double, and a chain sum and its next position fit one 64-bit word.  An
// iteration has two phases, each ended by a grid barrier:
//  - jumps: asynchronous pointer jumping on the packed entries (pk_make) that
//    the previous phase wrote; the thread that finishes a position's chain
//    publishes S - PO of it and, per 64 positions, which of them moved by
//    another amount than their left neighbour since the last iteration;
//  - sweep: the best candidate of every target, new entries for all.
// A target all of whose candidates moved by one amount keeps its best one, so
// a wave none of whose targets saw anything else skips its sweep: over the
// iterations of the 1.07M-node transformer graph 4.6 sweeps of all targets
// remain of 12 (3.4 of 8 on inception-600, 4.5 of 7 on transformer-24).
//
// Sweep.  A workgroup takes tiles of 1024 T / SEG targets and stages the
// candidates' S - PO, comm and packed offsets in LDS once (24 B each).  T
// consecutive targets per lane share each candidate's three LDS reads (T odd:
// a wave's reads fall into different banks); with SEG > 1 the candidates of
// a target are split over SEG waves by distance, each with its own running
// sum and minimum, combined through LDS, so that small graphs use the whole
// GPU.  About 13 vector instructions per candidate and target, all 32-bit or
// double (the counts by SWAR over four 16-bit fields, the sums by one fma):
// the instruction rate bounds a sweep.  Over the whole kernel on the 1.07M-node
// graph the vector units issue in 34 % of the cycles: the waits of jumps,
// barriers and skipped sweeps take the rest (2.9 GB moved, 1.6 TB/s).  Reading
// the candidates from L1 with 64-bit
// integer products and sweeping everything every time, the kernel took 4.0 ms
// on the 1.07M-node graph, 0.83 ms on inception-600, 0.60 ms on
// transformer-24; this one 1.84, 0.28 and 0.19 ms.
struct DtArgs {
  int32_t n, R, cap;
  int32_t seg;                // waves per group of targets (T = 1 only)
  int32_t sub;                // tiles a workgroup takes at once (T > 1 only)
  const int32_t *lo;          // [n + 1]
  const int64_t *PO;          // [n + 1]
  const int64_t *cq;          // [n]
  const uint64_t *nearw;      // [n]
  const uint32_t *hcnt;
  int32_t *P, *Parg;          // [n + 1] back pointers; smallest minimising start
  int64_t *cost;              // [n + 1] cost(P(j), j)
  int64_t *sp0, *sp1;         // [n + 1] S - PO as doubles, by iteration parity
  uint64_t *E;                // [n + 1] packed entries
  uint64_t *chw;              // [n / 64 + 1] positions that moved unlike their left neighbour
  int64_t *dfl;               // [2 (n / 64 + 1)] how far each word's first and last moved
  int32_t *bar;
  Status *st;
};

__device__ inline double ld_f64(const int64_t *p) { return __longlong_as_double(ld_coherent(p)); }

constexpr int dt_pool(int T) { return T == 1 ? 16200 : 19600; }  // 8-byte words (1: beside the combining arrays)
constexpr int kDtTab = 512;                       // count tables of a tile in LDS at most
constexpr uint64_t kDtLocal = uint64_t(1) << 61;  // the table's index is one of those

template <int T>
__global__ void __launch_bounds__(kDpB) k_dp_tiles(DtArgs a) {
  // staged positions (three arrays), and in what they leave free the count
  // tables of the tile's positions with many near successors: read per lane
  // and step, a table in global memory cost a microsecond each time
  constexpr int kPool = dt_pool(T);
  __shared__ __align__(16) uint64_t s_pool[kPool];
  __shared__ int32_t s_hid[kDtTab], s_nh;
  __shared__ double s_m[T == 1 ? kDpB : 1], s_i[T == 1 ? kDpB : 1];
  __shared__ int32_t s_a[T == 1 ? kDpB : 1];
  __shared__ int32_t s_ok, s_bit;
  if (failed(a.st)) return;
  Status *st = a.st;
  const int32_t n = a.n, R = a.R, n1 = n + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t gsz = (int64_t)gridDim.x * kDpB;
  const int64_t gid = (int64_t)blockIdx.x * kDpB + threadIdx.x;
  const int S = T == 1 ? a.seg : 1, NS = T > 1 ? a.sub : 1;
  const int B = kDpB / NS, part = threadIdx.x / B, pt = threadIdx.x - part * B;  // threads of a tile
  const int32_t TT = B / S * T, ntiles = (n + TT - 1) / TT;
  const int grp = (pt >> 6) / S, seg = (pt >> 6) - grp * S, len = (R + S - 1) / S;
  const int np = TT + R + 1;  // a tile's staged positions at most
  double *const s_sp = reinterpret_cast<double *>(s_pool + 3 * np * part), *const s_c = s_sp + np;
  uint64_t *const s_nw = s_pool + 3 * np * part + 2 * np;
  uint16_t *const s_tab = reinterpret_cast<uint16_t *>(s_pool + 3 * np * NS);
  const int room = (kPool - 3 * np * NS) * 4 / (R + 1), ntab = room < kDtTab ? room : kDtTab;
  // a workgroup's tiles at one time lie far apart: the targets that still
  // need a sweep in the later iterations are runs of neighbours
  const int32_t tile0 = part * (int32_t)gridDim.x + (int32_t)blockIdx.x, tstep = NS * (int32_t)gridDim.x;
  int32_t bar = 0, bit, staged = -1;
  if (gid == 0) pk_st(a.E, pk_make(0, kPkEnd));

  // The sweep of one tile.  INIT: the first policy, clusters of half the
  // window (with S - PO taken as 0 and the window cut to it, the farthest
  // candidate is the best one: the running sum only grows).  Chains of n / (R
  // / 2) pointers, and on the transformer graphs fewer iterations than from
  // singletons or whole windows.
  const int32_t h = R / 2 > 1 ? R / 2 : 1;
  auto sweep = [&](int32_t tile, bool init, bool all, const int64_t *sp) -> int32_t {
    const int32_t J0 = tile * TT;                         // targets J0 + 1 .. J0 + TT
    const int32_t base = J0 + 1 - R > 0 ? J0 + 1 - R : 0; // first candidate staged
    const int32_t end = J0 + TT < n ? J0 + TT : n;        // last position staged
    const int32_t j0 = J0 + 1 + (grp * 64 + lane) * T;    // this lane's first target
    int32_t lo[T], lmin = INT32_MAX, lmax = 0;
#pragma unroll
    for (int k = 0; k < T; k++) {
      lo[k] = j0 + k;  // past n: no candidate
      if (j0 + k <= n) {
        lo[k] = a.lo[j0 + k];
        if (init && j0 + k - h > lo[k]) lo[k] = j0 + k - h;
      }
      lmin = lo[k] < lmin ? lo[k] : lmin;
      lmax = lo[k] > lmax ? lo[k] : lmax;
    }
    bool need = all;  // every target (the first policy's values: nothing to compare with)
    if (!all) {  // did any candidate of the wave's targets move unlike its neighbour?
      int32_t p0 = j0 <= n ? lmin + 1 : INT32_MAX, p1 = j0 <= n ? (j0 + T - 2 < n ? j0 + T - 2 : n - 1) : -1;
      for (int o = 32; o > 0; o >>= 1) {
        const int32_t q0 = __shfl_xor(p0, o), q1 = __shfl_xor(p1, o);
        p0 = q0 < p0 ? q0 : p0;
        p1 = q1 > p1 ? q1 : p1;
      }
      bool any = false;
      if (p0 <= p1)
        for (int32_t w = (p0 >> 6) + lane; w <= (p1 >> 6); w += 64) {
          uint64_t x = pk_ld(a.chw + w) & ~1ull;
          if (w > 0 && ld_coherent(a.dfl + 2 * w) != ld_coherent(a.dfl + 2 * w - 1)) x |= 1;
          if (w == (p0 >> 6)) x &= ~0ull << (p0 & 63);
          if (w == (p1 >> 6)) x &= ~0ull >> (63 - (p1 & 63));
          any |= x != 0;
        }
      need = __ballot(any) != 0;
    }
    if (__syncthreads_or(need)) {
      if (staged != tile) {
        if (threadIdx.x == 0) s_nh = 0;
        __syncthreads();
      }
      for (int32_t x = pt; x <= end - base; x += B) {
        s_sp[x] = init ? 0.0 : ld_f64(sp + base + x);
        if (staged != tile && base + x < n) {
          s_c[x] = (double)a.cq[base + x];
          uint64_t w = a.nearw[base + x];
          if ((w & kDpHeavy) && a.hcnt[(int64_t)(uint32_t)w * (R + 1) + R] < 65536u) {
            const int32_t l = atomicAdd(&s_nh, 1);
            if (l < ntab) {
              s_hid[l] = (int32_t)(uint32_t)w;
              w = kDpHeavy | kDtLocal | (uint64_t)l;
            }
          }
          s_nw[x] = w;
        }
      }
      if (staged != tile) {
        __syncthreads();
        const int32_t nt = s_nh < ntab ? s_nh : ntab;
        for (int32_t l = wave; l < nt; l += kDpB / 64)
          for (int32_t d = lane; d <= R; d += 64)
            s_tab[l * (R + 1) + d] = (uint16_t)a.hcnt[(int64_t)s_hid[l] * (R + 1) + d];
      }
      staged = tile;
      __syncthreads();
    }
    double Int[T], best[T];
    int32_t arg[T];
#pragma unroll
    for (int k = 0; k < T; k++) {
      Int[k] = 0.0;
      best[k] = INFINITY;
      arg[k] = j0 + k - 1;
    }
    // candidate i for the targets j0 + k, k >= k0, that hold it in their window
    auto cand = [&](int32_t i, int k0, auto masked) {
      const uint64_t w = s_nw[i - base];
      const double c = s_c[i - base], v0 = s_sp[i - base];
      constexpr uint32_t kOnes = 0x00010001u, kHigh = 0x80008000u;
      const uint32_t d0 = (uint32_t)(j0 - i) * kOnes + kHigh;
      const uint32_t tl = d0 - ((uint32_t)w + kOnes), th = d0 - ((uint32_t)(w >> 32) + kOnes);
      const bool heavy = (w & kDpHeavy) != 0;
      int32_t cnt[T];
      // (field by field, (0x8000 | d) - (b + 1) keeps bit 15 exactly when b < d)
#pragma unroll
      for (int k = 0; k < T; k++)
        cnt[k] = __popc((tl + k * kOnes) & kHigh) + __popc((th + k * kOnes) & kHigh);
      if (heavy) {  // entries past R: targets whose window does not hold i
        const int32_t d = j0 - i;
#pragma unroll
        for (int k = 0; k < T; k++) {
          const int32_t dk = d + k < 0 ? 0 : (d + k < R ? d + k : R);
          cnt[k] = w & kDtLocal ? (int32_t)s_tab[(uint32_t)w * (R + 1) + dk]
                                : (int32_t)a.hcnt[(int64_t)(uint32_t)w * (R + 1) + dk];
        }
      }
#pragma unroll
      for (int k = 0; k < T; k++) {
        if (k < k0 || (decltype(masked)::value && i < lo[k])) continue;
        Int[k] = fma(c, (double)cnt[k], Int[k]);
        const double v = v0 - Int[k];
        arg[k] = v <= best[k] ? i : arg[k];
        asm("v_min_f64 %0, %1, %2" : "=v"(best[k]) : "v"(best[k]), "v"(v));  // no NaN to quiet
      }
    };
    if (need) {
      if (T == 1) {
        int32_t i = j0 - 1 - seg * len;
        const int32_t ie = j0 - (seg + 1) * len > lo[0] ? j0 - (seg + 1) * len : lo[0];
        for (; i > ie; i -= 2) {  // two candidates' reads in flight
          cand(i, 0, std::false_type());
          cand(i - 1, 0, std::false_type());
        }
        if (i == ie) cand(i, 0, std::false_type());
      } else {
#pragma unroll
        for (int q = T - 2; q >= 0; q--)
          if (j0 + q < end) cand(j0 + q, q + 1, std::true_type());
        int32_t i = j0 - 1;
        if (i >= end) i = lmin - 1;  // no target
        for (; i >= lmax; i--) cand(i, 0, std::false_type());
        for (; i >= lmin; i--) cand(i, 0, std::true_type());
      }
    }
    if (T == 1 && S > 1) {
      s_m[threadIdx.x] = best[0];
      s_i[threadIdx.x] = Int[0];
      s_a[threadIdx.x] = arg[0];
      __syncthreads();
      if (seg == 0) {
        double pre = 0.0, b = INFINITY;
        for (int x = 0; x < S; x++) {  // nearest segment first: on ties the farther one
          const double v = s_m[threadIdx.x + 64 * x] - pre;
          if (v <= b && v < INFINITY) {
            b = v;
            arg[0] = s_a[threadIdx.x + 64 * x];
          }
          pre += s_i[threadIdx.x + 64 * x];
        }
        best[0] = b;
      }
    }
    int32_t chg = 0;
    if (seg == 0) {
#pragma unroll
      for (int k = 0; k < T; k++) {
        const int32_t j = j0 + k;
        if (j > n) continue;
        int32_t p;
        int64_t cost;
        bool set = false;
        if (need) {
          set = init || best[k] < s_sp[j - base];  // PO[j] + best < S(j): strictly better
          a.Parg[j] = arg[k];
        }
        if (set) {
          p = arg[k];
          // Int(p, j) = (S - PO)(p) - best
          cost = a.PO[j] - a.PO[p] - (int64_t)(s_sp[p - base] - best[k]);
          a.P[j] = p;
          a.cost[j] = cost;
          chg = 1;
        } else {
          p = a.P[j];
          cost = a.cost[j];
        }
        pk_st(a.E + j, pk_make(cost, p > 0 ? (uint32_t)p : kPkEnd));
      }
    }
    __syncthreads();  // the tile's LDS is free
    return chg;
  };

  // every part of a workgroup takes the same number of tiles (barriers inside)
  for (int32_t tile = tile0; tile - part * (int32_t)gridDim.x < ntiles; tile += tstep)
    (void)sweep(tile, true, true, nullptr);
  if (!grid_sync(a.bar, ++bar, 0, &s_ok, &s_bit, st, &bit)) return;
  int32_t it = 0;
  bool done = false;
  for (; it < a.cap; it++) {
    int64_t *sp = it & 1 ? a.sp1 : a.sp0;
    const int64_t *spo = it & 1 ? a.sp0 : a.sp1;
    // ---- jumps: position 0 ends a chain
    for (int64_t jb = gid; jb - lane < n1; jb += kPkU * gsz) {  // whole waves
      uint64_t e[kPkU];
#pragma unroll
      for (int u = 0; u < kPkU; u++) {
        const int64_t j = jb + u * gsz;
        e[u] = j <= n ? pk_ld(a.E + j) : pk_make(0, kPkEnd);
      }
      for (int32_t k = 0;; k++) {  // back pointers decrease: every chain ends
        uint64_t f[kPkU];
        bool any = false;
#pragma unroll
        for (int u = 0; u < kPkU; u++) {
          const uint32_t x = pk_next(e[u]);
          f[u] = x != kPkEnd ? pk_ld(a.E + x) : 0;
        }
#pragma unroll
        for (int u = 0; u < kPkU; u++) {
          if (pk_next(e[u]) == kPkEnd) continue;
          e[u] = pk_make(pk_val(e[u]) + pk_val(f[u]), pk_next(f[u]));
          pk_st(a.E + jb + u * gsz, e[u]);
          any |= pk_next(e[u]) != kPkEnd;
        }
        if (!any) break;
        if (k > n) {  // cannot happen (P(j) < j); bounded all the same
          raise_err(st, EB_ORDER);
          break;
        }
      }
#pragma unroll
      for (int u = 0; u < kPkU; u++) {
        const int64_t j = jb + u * gsz;
        if (j - lane >= n1) continue;  // uniform over the wave
        double v = 0.0, dl = 0.0;
        if (j <= n) {
          v = (double)(pk_val(e[u]) - a.PO[j]);
          dl = it > 0 ? v - ld_f64(spo + j) : 0.0;
          st_coherent(sp + j, __double_as_longlong(v));
        }
        const double left = __shfl_up(dl, 1);
        const uint64_t m = __ballot(j <= n && lane > 0 && dl != left);
        if (lane == 0) {
          pk_st(a.chw + (j >> 6), m);
          st_coherent(a.dfl + 2 * (j >> 6), __double_as_longlong(dl));
        }
        if (lane == 63) st_coherent(a.dfl + 2 * (j >> 6) + 1, __double_as_longlong(dl));
      }
    }
    if (!grid_sync(a.bar, ++bar, 0, &s_ok, &s_bit, st, &bit)) return;
    if (ld32(reinterpret_cast<const int32_t *>(&st->err))) return;  // uniform after the barrier
    // ---- sweep
    int32_t chg = 0;
    for (int32_t tile = tile0; tile - part * (int32_t)gridDim.x < ntiles; tile += tstep)
      chg |= sweep(tile, false, it == 0, sp);
    chg = __syncthreads_or(chg);
    if (!grid_sync(a.bar, ++bar, chg, &s_ok, &s_bit, st, &bit)) return;
    if (!bit) {
      done = true;
      break;
    }
  }
  if (done) {  // converged: the smallest minimising start of every target, and S(n)
    if (seg == 0)
      for (int32_t tile = tile0; tile < ntiles; tile += tstep) {
        const int32_t j0 = tile * TT + 1 + (grp * 64 + lane) * T;
        for (int k = 0; k < T; k++)
          if (j0 + k <= n) a.P[j0 + k] = a.Parg[j0 + k];  // written by this thread
      }
    if (gid == 0) st->s0 = (int64_t)ld_f64((it & 1 ? a.sp1 : a.sp0) + n) + a.PO[n];
  }
  if (gid == 0) {
    st->i2 = done ? 1 : 0;
    st->i3 = done ? it + 1 : it;
  }
}

// ------------------------------------------------------ cluster starts

// The cluster starts are the chain from n through the final back pointers P
// (each P(j) < j).  Doubling tables J_0 = P (J_0(0) = 0), J_{k+1} = J_k(J_k)
// are built until the 2^k-th ancestor of n is position 0; then M = {n}, and
// for l = k down to 0 every marked position marks J_l of itself: after level
// l the marks cover every distance along the chain from n that is a sum of
// distinct powers 2^l .. 2^k, so at the end every chain node is marked and
// nothing else (a mark another thread sets during a pass only adds ancestors).
// About 2 log2(C) whole-GPU passes where one thread would follow C pointers.
struct CmArgs {
  int32_t n, K;               // K levels allocated in J
  const int32_t *P;           // [n + 1]
  int32_t *J;                 // [K][n + 1]
  int32_t *M;                 // [n + 1]
  int32_t *flag;              // [n] 1 at the cluster starts
  int32_t *bar;
  Status *st;
};

__global__ void __launch_bounds__(kDpB) k_chain_marks(CmArgs a) {
  __shared__ int32_t s_ok, s_bit, s_red[kDpB / 64];
  Status *st = a.st;
  if (failed(st)) return;
  const int64_t n1 = (int64_t)a.n + 1;
  const int64_t gsz = (int64_t)gridDim.x * kDpB;
  const int64_t gid = (int64_t)blockIdx.x * kDpB + threadIdx.x;
  int32_t bar = 0, bit;
  for (int64_t j = gid; j < n1; j += gsz) {
    const int32_t pj = j > 0 ? a.P[j] : 0;
    if (j > 0 && (pj < 0 || pj >= j)) raise_err(st, EB_ORDER);  // not a back pointer
    st32(&a.J[j], j > 0 && pj >= 0 && pj < j ? pj : 0);
    st32(&a.M[j], j == a.n ? 1 : 0);
  }
  if (!grid_sync(a.bar, ++bar, 0, &s_ok, &s_bit, st, &bit)) return;
  int32_t k = 0;
  while (ld32(&a.J[(int64_t)k * n1 + a.n]) != 0 && k + 1 < a.K) {  // uniform after the barrier
    const int32_t *Jk = a.J + (int64_t)k * n1;
    int32_t *Jn = a.J + (int64_t)(k + 1) * n1;
    for (int64_t j = gid; j < n1; j += gsz) st32(&Jn[j], ld32(&Jk[ld32(&Jk[j])]));
    if (!grid_sync(a.bar, ++bar, 0, &s_ok, &s_bit, st, &bit)) return;
    k++;
  }
  for (int32_t l = k; l >= 0; l--) {
    const int32_t *Jl = a.J + (int64_t)l * n1;
    for (int64_t j = gid; j < n1; j += gsz)
      if (ld32(&a.M[j])) st32(&a.M[ld32(&Jl[j])], 1);
    if (!grid_sync(a.bar, ++bar, 0, &s_ok, &s_bit, st, &bit)) return;
  }
  int32_t c = 0;
  for (int64_t j = gid; j < a.n; j += gsz) {
    const int32_t m = ld32(&a.M[j]);
    a.flag[j] = m;
    c += m;
  }
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = 0;
    for (int i = 0; i < kDpB / 64; i++) t += s_red[i];
    atomicAdd(&st->i0, t);
  }
}

// ------------------------------------------------------------------- host

namespace {
std::mutex g_dp_mu;
std::map<int, int> g_dp_groups;  // device -> co-resident workgroups (one per CU at most)
std::map<int, int> g_cm_groups;  // the same for k_chain_marks
}  // namespace

int dp_policy(int32_t n, int32_t m, int32_t R, const int32_t *lo, const int64_t *PO,
              const int64_t *cq, const int32_t *sptr, const int32_t *sidx, int32_t *P,
              Scratch &sc, hipStream_t s, Status *st, GridTurn &turn, bool *launched) {
  *launched = false;
  if (n <= 0) return CEL_OK;
  int gmax = 0;
  {
    int dev = 0;
    CEL_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_dp_mu);
    auto it = g_dp_groups.find(dev);
    if (it == g_dp_groups.end()) {
      int cus = 0, nb = 0;
      CEL_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
      int fit = 1;  // one per CU at most, where every variant fits
      for (const void *f : {(const void *)k_dp_policy, (const void *)k_dp_tiles<1>,
                            (const void *)k_dp_tiles<3>, (const void *)k_dp_tiles<5>}) {
        CEL_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kDpB, 0));
        fit = nb < fit ? nb : fit;
      }
      it = g_dp_groups.emplace(dev, cus * fit).first;
    }
    gmax = it->second;
  }
  if (gmax < 1) return CEL_OK;
  int32_t *ncnt, *nptr, *Parg, *bar, *hflag, *hoff;
  uint16_t *noff;
  uint64_t *nearw;
  uint32_t *hcnt;
  int64_t *cost;
  CEL_TRY(sc.get(&ncnt, (int64_t)n + 2 + gmax));  // and the barrier's words: cleared together
  bar = ncnt + n;
  CEL_TRY(sc.get(&nptr, (int64_t)n + 1));
  CEL_TRY(sc.get(&noff, m));
  CEL_TRY(sc.get(&nearw, n));
  CEL_TRY(sc.get(&hflag, n));
  CEL_TRY(sc.get(&hoff, (int64_t)n + 1));
  CEL_TRY(sc.get(&Parg, (int64_t)n + 1));
  CEL_TRY(sc.get(&cost, (int64_t)n + 1));
  k_fill_i32<<<grid_for((int64_t)n + 2 + gmax, 256, 4096), 256, 0, s>>>(ncnt, (int64_t)n + 2 + gmax,
                                                                      0);
  // (bar[1]: the barriers' abort flag)
  if (policy_iteration_gives_up()) k_fill_i32<<<1, 64, 0, s>>>(bar + 1, 1, 1);
  k_dpn_count<<<edge_blocks(m), 256, 0, s>>>(n, m, R, sptr, sidx, ncnt, st);
  CEL_TRY(exclusive_scan_i32(ncnt, nptr, n, sc, s));
  k_dpn_fill<<<edge_blocks(m), 256, 0, s>>>(n, m, R, sptr, sidx, nptr, ncnt, noff, st);
  k_dpn_heavy<<<grid_for(n, 256, 4096), 256, 0, s>>>(n, nptr, hflag, st);
  CEL_TRY(exclusive_scan_i32(hflag, hoff, n, sc, s, &st->i1));
  Status hs;
  CEL_TRY(read_status(st, &hs, s));
  if (hs.err) return CEL_OK;  // the counts were not written; the caller reports it
  const int32_t H = hs.i1;  // positions with more than four offsets below R
  const int64_t total = hs.s1;
  if ((int64_t)H * (R + 1) * 4 > (int64_t(1) << 30)) return CEL_OK;  // tables too large: blocked DP
  CEL_TRY(sc.get(&hcnt, (int64_t)H * (R + 1)));
  k_dpn_pack<<<grid_for(n, 256, 4096), 256, 0, s>>>(n, R, nptr, noff, hoff, nearw, hcnt, st);
  CEL_HIP(hipGetLastError());
  const double blocked_us = 500.0 + 0.064 * n;  // the blocked DP: 64 ns per target
  // Values that fit 40 bits (S is at most PO[n], the comm of all edges): tiles
  // in LDS.  S, PO and every sum are then exact doubles.
  if (policy_iteration_packed() && n < (int32_t)kPkEnd - 1 && total >= 0 &&
      total < (int64_t(1) << 40)) {
    // Targets per lane and waves per target: one round of tiles over the
    // workgroups where possible.  Up to 1024 targets a workgroup one target
    // per lane, the candidates split over 2, 4, 8 or 16 waves while that
    // leaves workgroups idle; above, the fewest targets per lane, as far as
    // the window fits the staged positions.
    int T = 1, seg = 1;
    const int64_t per = ((int64_t)n + gmax - 1) / gmax;  // targets per workgroup in one round
    if (per <= kDpB) {
      while (seg < 16 && per * 2 * seg <= kDpB && 2 * seg <= R) seg *= 2;
    } else if (per > 3 * kDpB && 3 * (5 * kDpB + R + 1) <= dt_pool(5)) {
      T = 5;
    } else if (3 * (3 * kDpB + R + 1) <= dt_pool(3)) {
      T = 3;
    }
    int sub = 1;  // tiles at once, while their windows fit
    if (T > 1)
      while (sub < 4 && 3 * 2 * sub * (kDpB / (2 * sub) * T + R + 1) <= dt_pool(T)) sub *= 2;
    const int64_t span = (int64_t)kDpB / sub / seg * T;  // targets of a tile
    const int64_t tiles = ((int64_t)n + span - 1) / span;
    const int G = (int)(tiles < gmax ? tiles : gmax);
    DtArgs a{};
    a.n = n;
    a.R = R;
    a.seg = seg;
    a.sub = sub;
    // an iteration costs two barriers and the jumps (some 20 us) and at most
    // one sweep (0.6 ps per candidate and target)
    const double it_us = 20.0 + 0.6e-6 * R * (double)n;
    a.cap = (int32_t)(blocked_us / it_us);
    if (a.cap < 4) a.cap = 4;
    a.lo = lo;
    a.PO = PO;
    a.cq = cq;
    a.nearw = nearw;
    a.hcnt = hcnt;
    a.P = P;
    a.Parg = Parg;
    a.cost = cost;
    CEL_TRY(sc.get(&a.sp0, (int64_t)n + 1));
    CEL_TRY(sc.get(&a.sp1, (int64_t)n + 1));
    CEL_TRY(sc.get(&a.E, (int64_t)n + 1));
    CEL_TRY(sc.get(&a.chw, (int64_t)n / 64 + 1));
    CEL_TRY(sc.get(&a.dfl, 2 * ((int64_t)n / 64 + 1)));
    a.bar = bar;
    a.st = st;
    if (!turn.take()) return CEL_OK;
    {
      KTimer kt(s, "k_cluster_policy");
      if (T == 5) k_dp_tiles<5><<<G, kDpB, 0, s>>>(a);
      else if (T == 3) k_dp_tiles<3><<<G, kDpB, 0, s>>>(a);
      else k_dp_tiles<1><<<G, kDpB, 0, s>>>(a);
    }
    CEL_HIP(hipGetLastError());
    *launched = true;
    return CEL_OK;
  }
  const int64_t need = ((int64_t)n + 1 + kDpB - 1) / kDpB;
  const int G = (int)(need < gmax ? need : gmax);
  int32_t max_rounds = 2;
  while ((int64_t(1) << (max_rounds - 2)) < (int64_t)n + 1) max_rounds++;
  // Iterations allowed before the blocked DP is cheaper: an iteration costs
  // its pointer-jumping passes (a few us of barrier plus 48 bytes per node at
  // a few TB/s each) and a sweep of R candidates per target (about 0.5 ps per
  // candidate and target over the whole GPU).
  const double it_us = max_rounds * (5.0 + 48.0 * n / 4.0e6) + 10.0 + 0.5e-6 * R * (double)n;
  int32_t cap = (int32_t)(blocked_us / it_us);
  if (cap < 4) cap = 4;
  DpArgs a{};
  a.n = n;
  a.R = R;
  a.cap = cap;
  a.max_rounds = max_rounds;
  a.lo = lo;
  a.PO = PO;
  a.cq = cq;
  a.nearw = nearw;
  a.hcnt = hcnt;
  a.P = P;
  a.Parg = Parg;
  a.cost = cost;
  CEL_TRY(sc.get(&a.SP, (int64_t)n + 1));
  CEL_TRY(sc.get(&a.e0, (int64_t)n + 1));
  CEL_TRY(sc.get(&a.e1, (int64_t)n + 1));
  a.bar = bar;
  a.st = st;
  if (!turn.take()) return CEL_OK;
  {
    // at most one workgroup per CU, within the occupancy calculator's limit:
    // resident all at once on an idle GPU; the barriers' waits are bounded
    KTimer kt(s, "k_cluster_policy");
    k_dp_policy<<<G, kDpB, 0, s>>>(a);
  }
  CEL_HIP(hipGetLastError());
  *launched = true;
  return CEL_OK;
}

int chain_marks(int32_t n, const int32_t *P, int32_t *flag, Scratch &sc, hipStream_t s, Status *st,
                GridTurn &turn, bool *launched) {
  *launched = false;
  if (n <= 0) return CEL_OK;
  int gmax = 0;
  {
    int dev = 0;
    CEL_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_dp_mu);
    auto it = g_cm_groups.find(dev);
    if (it == g_cm_groups.end()) {
      int cus = 0, nb = 0;
      CEL_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
      CEL_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)k_chain_marks, kDpB,
                                                           0));
      it = g_cm_groups.emplace(dev, cus * (nb < 1 ? nb : 1)).first;
    }
    gmax = it->second;
  }
  if (gmax < 1 || !turn.take()) return CEL_OK;
  const int64_t need = ((int64_t)n + 1 + kDpB - 1) / kDpB;
  const int G = (int)(need < gmax ? need : gmax);
  int32_t K = 2;  // 2^(K - 1) > n: enough levels for a chain through every position
  while ((int64_t(1) << (K - 1)) <= (int64_t)n) K++;
  int32_t *J, *M, *bar;
  CEL_TRY(sc.get(&J, (int64_t)K * ((int64_t)n + 1)));
  CEL_TRY(sc.get(&M, (int64_t)n + 1));
  CEL_TRY(sc.get(&bar, 2 + (int64_t)G));
  k_fill_i32<<<1, 256, 0, s>>>(bar, 2 + (int64_t)G, 0);
  CmArgs a{};
  a.n = n;
  a.K = K;
  a.P = P;
  a.J = J;
  a.M = M;
  a.flag = flag;
  a.bar = bar;
  a.st = st;
  {
    // at most one workgroup per CU (bounded grid-barrier waits, as k_dp_policy)
    KTimer kt(s, "k_chain_marks");
    k_chain_marks<<<G, kDpB, 0, s>>>(a);
  }
  CEL_HIP(hipGetLastError());
  *launched = true;
  return CEL_OK;
}

}  // namespace cel
