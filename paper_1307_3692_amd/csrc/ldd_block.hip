// Workgroup-owned decomposition: one workgroup runs every round of one graph, with workgroup
// barriers between rounds and no grid-wide step.  This is the search of Sec. 5 (Algorithm 2 via
// the delayed-start breadth-first search), round by round, as the multi-block engine runs it:
//
//   preparation  Delta = max shift; labels INF; the vertices with arcs sorted by wake round
//                w(v) = (Delta - shift[v]) >> 20 (counting sort in LDS)
//   round r      wake: every vertex of bucket r offers its own label ((Delta - shift[v]) << B) | v;
//                top-down: every vertex u of F_{r-1} offers P(u) + (2^20 << B) along its arcs;
//                offers are applied with an atomic minimum on the 64-bit label (exact), and the
//                first offer a vertex receives appends it to F_r
//   empty F_r    the next round is the next non-empty wake bucket
//   output       centre = low B bits of the label (INF: an isolated vertex, its own centre) and
//                the cut (Def. 1.1)
//
// A round costs a few workgroup barriers and a handful of dependent cache accesses instead of a
// kernel launch and a grid-wide state exchange, so graphs with many rounds and small frontiers
// (small graphs, high-diameter graphs) run far faster here; a batch runs one graph per workgroup,
// the largest first, each workgroup taking the next graph when it finishes one.
//
// What a round costs is its chain of dependent memory accesses, so the frontier is kept in LDS with
// each vertex's first arc and degree: a round is columns, labels, and the row offsets of what it reached.
// A wave takes up to 64 rows and walks their arcs 64 at a time, whatever their degrees (walk_rows).
//
// A graph too large for one workgroup (a batch's largest graphs, or one large high-diameter graph)
// runs on a team of K workgroups, all resident at once: member m owns a slice of the vertices
// (its preparation, wake buckets, tail seed and output) and a share of every frontier, which is one
// queue in device memory.  The members meet at a barrier in device memory, where the queue's length
// and the error bits are read, once per step; a step is one round when the frontier is large or
// grows fast, else several (see team_steps).  The labels are then shared by several CUs, so their
// loads and atomics take device scope.
#include "ldd_block.h"

#include <climits>

namespace ldd {

namespace {

constexpr int BT = 1024;         // threads per workgroup
constexpr int BNW = BT / WAVE;   // waves per workgroup
constexpr int WPT = BLOCK_WCAP / BT;  // wake buckets per thread in the scans

// Frontier entries kept in LDS (double-buffered): alone 12 B each
// (vertex, first arc, degree), the rest of a larger frontier in the graph's queues; a team member
// 20 B each (and the label), the rest straight to the team's queue.
constexpr int LC = 1024;
constexpr int TC = 2048;
constexpr int TC1 = TEAM_Q_BYTES / 4;  // a team's step of one round: vertices only
static_assert(LC * 24 == ALONE_Q_BYTES && TC * 40 == TEAM_Q_BYTES, "the frontier's LDS");

constexpr int LONG_ROW = 32;      // rows of more arcs are taken by a wave at once ...
constexpr int HUGE_ROW = 4096;    // ... or, above this, listed for the whole workgroup
constexpr unsigned HCAP = 32;     // such rows listed per round (past that a wave takes them too)
constexpr int STEP_ROW = 1024;    // a team's steps are one round when there is a row of more arcs
constexpr int WALK_WORDS = WAVE * LONG_ROW / 64;

struct HeavyRow {
  u64 offer;
  int a0, deg;
};

constexpr int FIX_LONG_ROWS = 544;  // long rows of a graph held whole in LDS

struct BlockShared {
  unsigned nlong;
  unsigned short longv[FIX_LONG_ROWS];
  BlockJob j;                // the job in hand
  int woff[BLOCK_WCAP + 1];  // wake bucket offsets (exclusive prefix), then the scatter cursors
  u64 starts[BNW][WALK_WORDS];  // per wave: which of its arcs start a row (walk_rows)
  HeavyRow heavy[HCAP];
  u64 red64[BNW];
  unsigned red32[BNW];
  int job;
  int nxt;                   // next non-empty wake bucket (block minimum)
  unsigned cnt3[3];          // appends: round k counts in cnt3[k % 3], so one barrier per round
  unsigned nh3[3];           // heavy rows listed, likewise
  unsigned oc3[3];           // claims: a conflict in the round, likewise
  unsigned er3[3];           // errors the round's walks found, likewise: the next round's waves may be ahead of
                             // one that has yet to ask whether this one failed, and all have to leave together
  unsigned maxdeg;           // the largest degree (a team: if above STEP_ROW)
  unsigned err;              // the job's error bits; in a team's rounds the member's own (see terr)
  u64 delta, n_active;       // preparation results
  u64 settled, examined;     // round results
  long long rounds, sweeps;
  // team of several workgroups on one graph
  g_sync* ts;
  int tK, tm, tlo, thi;      // team size, this member, this member's vertex slice
  unsigned epoch;            // barriers passed
  unsigned tnf;              // the queue length the last team barrier published
  unsigned tcount;           // this member's appends to the shared queue in this step
  unsigned tbase;            // the staged appends' place in the shared queue
  unsigned spill;            // an append of this step did not fit the LDS before its last round
  unsigned tspill;           // ... in any member (published by the last barrier)
  unsigned terr;             // the error bits the last barrier published: what ends the rounds
  unsigned sfirst;           // vertices this member reached first in this step
  u64 tfirst;                // ... the team, in the last step
  u64 nz[BLOCK_WCAP / 64];   // non-empty wake buckets of the whole graph
};

__device__ __forceinline__ u64 block_max64(u64 v, BlockShared& sh) {
  v = wave_max_u64(v);
  __syncthreads();
  if (lane_id() == 0) sh.red64[threadIdx.x / WAVE] = v;
  __syncthreads();
  u64 m = 0;
#pragma unroll
  for (int w = 0; w < BNW; ++w) m = sh.red64[w] > m ? sh.red64[w] : m;
  return m;
}

__device__ __forceinline__ u64 block_sum64(u64 v, BlockShared& sh) {
  v = wave_sum_u64(v);
  __syncthreads();
  if (lane_id() == 0) sh.red64[threadIdx.x / WAVE] = v;
  __syncthreads();
  u64 s = 0;
#pragma unroll
  for (int w = 0; w < BNW; ++w) s += sh.red64[w];
  return s;
}

// exclusive prefix sum of x over the workgroup; *total receives the sum (all threads call)
__device__ __forceinline__ unsigned block_excl_scan(unsigned x, BlockShared& sh, unsigned* total) {
  const unsigned incl = wave_incl_scan(x);
  const unsigned wid = threadIdx.x / WAVE;
  __syncthreads();
  if (lane_id() == WAVE - 1) sh.red32[wid] = incl;
  __syncthreads();
  unsigned before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < BNW; ++w) {
    const unsigned t = sh.red32[w];
    before += w < (int)wid ? t : 0u;
    all += t;
  }
  *total = all;
  return before + incl - x;
}

// The first non-empty wake bucket at or after r (D + n + 1 when none is left: past the end);
// all threads call.  Found by a block-wide minimum over the bucket offsets.
__device__ __forceinline__ int next_nonempty(BlockShared& sh, int r, int D) {
  __syncthreads();
  if (threadIdx.x == 0) sh.nxt = 0x7fffffff;
  __syncthreads();
  for (int q = r + (int)threadIdx.x; q <= D; q += BT)
    if (sh.woff[q + 1] > sh.woff[q]) atomicMin(&sh.nxt, q);
  __syncthreads();
  const int q = sh.nxt;
  __syncthreads();
  return q <= D ? q : 0x3fffffff;
}

// A graph's labels are touched by its own workgroup only while it runs, so their loads and atomics
// need workgroup scope alone (all waves of a workgroup share one CU and its vector L1).  A team's
// labels are shared by its members' CUs, which may sit on different XCDs, each with its own L2.
// Within the rounds every access another member may read or write is itself coherent at device
// scope: the claims are device-scope atomics, the queue entries device-scope stores and loads, and
// the loads that decide something (an offer, a queue entry) device-scope loads; so the per-round
// barrier only has to wait for the member's own accesses to complete, with no L2 writeback or
// invalidation (which would also drop the cached CSR every round).  A label load that only filters
// atomics (is the label still larger than the offer?) stays at workgroup scope and may see an
// older value, which is never smaller (labels only decrease, and the preparation's barriers,
// which do write back and invalidate, order every cached copy after the labels' initialisation),
// so at worst it lets through an atomic that finds nothing to do.  The phases that use plain
// loads and stores on shared data (preparation, the tail's seed, the output) are bracketed by
// barriers or fences that do write back and invalidate.
constexpr int WG = __HIP_MEMORY_SCOPE_WORKGROUP;
constexpr int AG = __HIP_MEMORY_SCOPE_AGENT;

template <int SC>
__device__ __forceinline__ u64 lab_load(g_cu64* p) {
  return __hip_atomic_load(const_cast<g_u64*>(p), __ATOMIC_RELAXED, SC);
}
template <int SC>
__device__ __forceinline__ u64 lab_min(g_u64* p, u64 v) {
  return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, SC);
}
template <int SC>
__device__ __forceinline__ void lab_store(g_u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, SC);
}
__device__ __forceinline__ u64 wg_load(g_cu64* p) { return lab_load<WG>(p); }

// The job in hand (copied to LDS by the kernel), in scalar registers.
template <class T>
__device__ __forceinline__ T uniform(T v) {
  static_assert(sizeof(T) == 8, "a pointer or a 64-bit number");
  u64 x;
  __builtin_memcpy(&x, &v, 8);
  x = (u64)(unsigned)__builtin_amdgcn_readfirstlane((int)x) |
      (u64)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32;
  __builtin_memcpy(&v, &x, 8);
  return v;
}
__device__ __forceinline__ BlockJob job_of(const BlockShared& sh) {
  const BlockJob& s = sh.j;
  BlockJob j;
  j.n = __builtin_amdgcn_readfirstlane(s.n);
  j.nnz = uniform(s.nnz);
  j.row_ptr = uniform(s.row_ptr);
  j.col = uniform(s.col);
  j.shift = uniform(s.shift);
  j.centre = uniform(s.centre);
  j.P = uniform(s.P);
  j.wk = uniform(s.wk);
  j.wake = uniform(s.wake);
  j.q0 = uniform(s.q0);
  j.q1 = uniform(s.q1);
  j.tail_den = __builtin_amdgcn_readfirstlane(s.tail_den);
  j.team = __builtin_amdgcn_readfirstlane(s.team);
  j.sync = uniform(s.sync);
  j.deg_cap = __builtin_amdgcn_readfirstlane(s.deg_cap);
  return j;
}

// The slice loops (preparation, wake sort, output) are latency-bound with one vertex per thread at a
// time: a thread takes VU vertices at once (v, v + BT, ...), and in the output AU arcs of each,
// so that each of its loads has others in flight.
constexpr int VU = 4, AU = 2;

// Vertices v0 + k * BT (k < VU) below hi: has[k] when the vertex has arcs, key[k] = Delta - shift.
__device__ __forceinline__ void slice_load(const int* __restrict__ rp, const long long* __restrict__ shift, int v0,
                                           int hi, u64 delta, u64 (&key)[VU], bool (&has)[VU]) {
  int a0[VU], a1[VU];
  long long sv[VU];
#pragma unroll
  for (int k = 0; k < VU; ++k) {
    const int v = v0 + k * BT;
    a0[k] = a1[k] = 0;
    sv[k] = 0;
    if (v < hi) {
      a0[k] = rp[v];
      a1[k] = rp[v + 1];
      sv[k] = shift[v];
    }
  }
#pragma unroll
  for (int k = 0; k < VU; ++k) {
    has[k] = a1[k] > a0[k];
    key[k] = delta - (u64)sv[k];
  }
}

// Wake buckets of the vertices with arcs in [lo, hi): counting sort by w(v) = (Delta - shift) >> 20
// in LDS; the vertices' own labels ((Delta - shift[v]) << B) | v go to wk[lo ...] in bucket order
// (a wake then needs no shift load) and sh.woff[q] is bucket q's offset from lo (all threads call).
__device__ __forceinline__ void wake_sort(const BlockJob& j, BlockShared& sh, int lo, int hi, u64 delta) {
  g_cint* __restrict__ rp = j.row_ptr;
  g_ci64* __restrict__ shift = j.shift;
  const int tid = threadIdx.x;
  const int B = j.n > 1 ? 32 - __builtin_clz((unsigned)(j.n - 1)) : 1;
  for (int q = tid; q <= BLOCK_WCAP; q += BT) sh.woff[q] = 0;
  __syncthreads();
  for (int v0 = lo + tid; v0 < hi; v0 += VU * BT) {
    u64 key[VU];
    bool has[VU];
    slice_load(rp, shift, v0, hi, delta, key, has);
#pragma unroll
    for (int k = 0; k < VU; ++k)
      if (has[k]) atomicAdd(&sh.woff[(int)(key[k] >> FIX)], 1);
  }
  __syncthreads();
  {
    unsigned loc[WPT], sum = 0;
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      loc[i] = (unsigned)sh.woff[tid * WPT + i];
      sum += loc[i];
    }
    unsigned total;
    unsigned run = block_excl_scan(sum, sh, &total);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const unsigned c = loc[i];
      sh.woff[tid * WPT + i] = (int)run;
      run += c;
    }
    if (tid == 0) sh.woff[BLOCK_WCAP] = (int)total;
  }
  __syncthreads();
  // scatter: woff[q] serves as bucket q's cursor (it ends at the start of bucket q + 1) and is
  // shifted back by one bucket afterwards
  for (int v0 = lo + tid; v0 < hi; v0 += VU * BT) {
    u64 key[VU];
    bool has[VU];
    slice_load(rp, shift, v0, hi, delta, key, has);
#pragma unroll
    for (int k = 0; k < VU; ++k)
      if (has[k]) j.wk[lo + atomicAdd(&sh.woff[(int)(key[k] >> FIX)], 1)] = (key[k] << B) | (u64)(v0 + k * BT);
  }
  __syncthreads();
  {
    int vals[WPT];
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int q = tid * WPT + i;
      vals[i] = q == 0 ? 0 : sh.woff[q - 1];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WPT; ++i) sh.woff[tid * WPT + i] = vals[i];
    __syncthreads();
  }
}

// Checks, Delta and the count of vertices with arcs over [lo, hi), which also get label INF
// (all threads call; results are the workgroup's: *dmax and *active reduced, errors in sh.err,
// which the caller cleared).
__device__ __forceinline__ void prepare_scan(const BlockJob& j, BlockShared& sh, int lo, int hi, bool ends,
                                             u64* dmax_out, u64* active_out, u64* degmax_out = nullptr) {
  const int n = j.n;
  const long long nnz = j.nnz;
  g_cint* __restrict__ rp = j.row_ptr;
  g_ci64* __restrict__ shift = j.shift;
  g_u64* P = j.P;
  const int tid = threadIdx.x;
  unsigned err = 0;
  u64 dmax = 0, active = 0, degmax = 0;
  if (ends && n > 0 && (rp[0] != 0 || (long long)rp[n] != nnz) && tid == 0) err |= ERR_BAD_ROWPTR;
  for (int v0 = lo + tid; v0 < hi; v0 += VU * BT) {
    long long sv[VU];
    int a0[VU], a1[VU];
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      sv[k] = 0;
      a0[k] = a1[k] = 0;
      if (v < hi) {
        sv[k] = shift[v];
        a0[k] = rp[v];
        a1[k] = rp[v + 1];
      }
    }
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      if (v < hi) {
        if (sv[k] < 0 || sv[k] > (1ll << 52)) err |= ERR_BAD_SHIFT;
        if (a1[k] < a0[k]) err |= ERR_BAD_ROWPTR;
        active += a1[k] > a0[k];
        dmax = (u64)sv[k] > dmax ? (u64)sv[k] : dmax;
        degmax = a1[k] > a0[k] && (u64)(a1[k] - a0[k]) > degmax ? (u64)(a1[k] - a0[k]) : degmax;
        P[v] = INF;
      }
    }
  }
  if (err) atomicOr(&sh.err, err);
  *dmax_out = block_max64(dmax, sh);
  *active_out = block_sum64(active, sh);
  if (degmax_out) *degmax_out = block_max64(degmax, sh);
  __syncthreads();
}

// The checks that need Delta: labels fit 64 bits, and the shifts span fewer than BLOCK_WCAP units.
__device__ __forceinline__ unsigned range_err(int n, u64 delta) {
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  if ((delta + ((u64)1 << FIX)) >= ((u64)1 << (64 - B))) return BLK_OVERFLOW;
  if ((delta >> FIX) >= (u64)BLOCK_WCAP) return BLK_WIDE;
  return 0;
}

// Preparation of one graph: checks, Delta, the vertices with arcs, labels INF, and the wake
// buckets.  Results in sh (delta, n_active, err, woff).
__device__ __attribute__((noinline)) void block_prepare(BlockShared& sh) {
  const BlockJob j = job_of(sh);
  if (threadIdx.x == 0) sh.err = 0;
  __syncthreads();
  u64 delta, n_active, degmax;
  prepare_scan(j, sh, 0, j.n, true, &delta, &n_active, &degmax);
  if (threadIdx.x == 0) {
    unsigned e = sh.err;
    if (!e) e = range_err(j.n, delta);
    sh.err = e;
    sh.delta = delta;
    sh.n_active = n_active;
    sh.maxdeg = (unsigned)degmax;
  }
  __syncthreads();
  if (sh.err) return;
  wake_sort(j, sh, 0, j.n, delta);
}

// The LDS of frontiers and small graphs.  A fixed array: the address of dynamic LDS is not a constant
// outside the kernel's own body, and every access of these functions loaded it from memory first.
__shared__ __attribute__((aligned(16))) unsigned char blk_dyn[BLOCK_LDS_BYTES];

// Two consecutive row offsets as one access (4-byte aligned).
struct __attribute__((packed, aligned(4))) RowEnds {
  int a0, a1;
};
__device__ __forceinline__ void row_of(g_cint* rp, int v, int* a0, int* deg) {
  const RowEnds e = *reinterpret_cast<const LDD_GLOBAL RowEnds*>(rp + v);
  *a0 = e.a0;
  *deg = e.a1 - e.a0;
}

// One row's arcs first, first + stride, ..., two at a time.
template <class Arcs>
__device__ __forceinline__ void walk_row(const BlockJob& j, BlockShared& sh, int ci, int a0, int deg, u64 o, int first,
                                         int stride, const Arcs& arcs) {
  const u64 offer[2] = {o, o};
#pragma unroll 1
  for (int x = first; x < deg; x += 2 * stride) {
    int w[2];
    bool go[2], bad = false;
    go[0] = true;
    go[1] = x + stride < deg;
    w[0] = j.col[a0 + x];
    w[1] = go[1] ? j.col[a0 + x + stride] : 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      bad |= go[k] && (unsigned)w[k] >= (unsigned)j.n;
      go[k] = go[k] && (unsigned)w[k] < (unsigned)j.n;
    }
    if (bad) atomicOr(&sh.er3[ci], ERR_BAD_COL);
    arcs.template run<2>(w, go, offer);
  }
}

// U passes of 64 of a wave's arcs, from word c0 of its start bits on (see walk_rows).
template <int U, class Arcs>
__device__ __forceinline__ void walk_pass(const BlockJob& j, BlockShared& sh, int ci, const u64* starts, int c0, int total,
                                          int& row, int adj, u64 offer, const Arcs& arcs) {
  int w[U];
  bool go[U], bad = false;
  u64 off[U];
#pragma unroll
  for (int k = 0; k < U; ++k) {
    const u64 word = (c0 + k) * 64 < total ? starts[c0 + k] : 0;
    const int t = (c0 + k) * 64 + (int)lane_id();
    // the arc's row: the row starts at or before it
    const int r = row + (int)rank_below(word) + (int)((word >> lane_id()) & 1) - 1;
    row += __builtin_popcount(__builtin_amdgcn_readfirstlane((int)word)) +
           __builtin_popcount(__builtin_amdgcn_readfirstlane((int)(word >> 32)));
    const int at = __shfl(adj, r, WAVE);
    off[k] = shfl_u64(offer, r);
    go[k] = t < total && at != INT_MIN;
    w[k] = go[k] ? j.col[at + t] : 0;
  }
#pragma unroll
  for (int k = 0; k < U; ++k) {
    bad |= go[k] && (unsigned)w[k] >= (unsigned)j.n;
    go[k] = go[k] && (unsigned)w[k] < (unsigned)j.n;
  }
  if (bad) atomicOr(&sh.er3[ci], ERR_BAD_COL);
  arcs.template run<U>(w, go, off);
}

// The frontier's nf rows.  What bounds this is instructions: with a lane (or eight) per row half of the lanes
// idle on uneven degrees, and each instruction of a wave costs its SIMD four cycles whether they do or not
// (RGG with 200,000 vertices, 1400 rows: 18 us a round with eight lanes per row).  So a wave takes up
// to 64 rows, one per lane, and walks their arcs 64 at a time: a bit per arc in LDS marks where a row starts,
// and an arc's row is the number of bits up to it.  Neighbouring lanes read neighbouring columns.
// entry(i) gives row i's first arc, degree and offer; arcs.run gets U far ends per lane with their
// offers.  Few rows are spread over all waves, from the last one down (the round's wake runs in
// the first).  A row of more than LONG_ROW arcs is walked by its wave alone, one of more than HUGE_ROW listed in slot
// ci for walk_heavy.  Rows lie in [0, nnz] (checked by the preparation); columns are checked here (sh.er3[ci]).
template <class Entry, class Arcs>
__device__ __forceinline__ void walk_rows(const BlockJob& j, BlockShared& sh, int ci, unsigned nf, const Entry& entry,
                                          const Arcs& arcs, unsigned& examined) {
  const unsigned lane = lane_id(), wid = BNW - 1 - threadIdx.x / WAVE;
  const unsigned per = (nf + BNW - 1) / BNW, rows = per < (unsigned)WAVE ? per : (unsigned)WAVE;  // rows per wave and pass
  u64* starts = sh.starts[wid];
  for (unsigned i0 = wid * rows; i0 < nf; i0 += BNW * rows) {
    int a0 = 0, deg = 0;
    u64 offer = 0;
    const bool mine = lane < rows && i0 + lane < nf;
    if (mine) entry(i0 + lane, &a0, &deg, &offer);
    examined += (unsigned)deg;
    bool alone = deg > LONG_ROW;
    if (deg > HUGE_ROW) {
      const unsigned h = atomicAdd(&sh.nh3[ci], 1u);
      if (h < HCAP) {
        sh.heavy[h] = HeavyRow{offer, a0, deg};
        alone = false;
        deg = 0;
      }
    }
    for (u64 m = __ballot(alone); m; m &= m - 1) {
      const int src = __ffsll((long long)m) - 1;
      walk_row(j, sh, ci, __builtin_amdgcn_readlane(a0, src), __builtin_amdgcn_readlane(deg, src), shfl_u64(offer, src),
               (int)lane, WAVE, arcs);
    }
    // rows taken elsewhere keep one arc, which is skipped (so that every row has a start)
    const bool none = alone || deg == 0;
    const int d = mine ? (none ? 1 : deg) : 0;
    const int incl = (int)wave_incl_scan((unsigned)d), pre = incl - d;
    const int total = __builtin_amdgcn_readlane(incl, WAVE - 1);
    if (lane < (unsigned)WALK_WORDS) starts[lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (mine) atomicOr(reinterpret_cast<unsigned*>(starts) + (pre >> 5), 1u << (pre & 31));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int adj = none ? INT_MIN : a0 - pre;
    int row = 0;
    if (total <= 64) {
      walk_pass<1>(j, sh, ci, starts, 0, total, row, adj, offer, arcs);
    } else {
#pragma unroll 1
      for (int c = 0; c * 64 < total; c += 4) walk_pass<4>(j, sh, ci, starts, c, total, row, adj, offer, arcs);
    }
  }
}

// The rows listed in slot ci, each by the whole workgroup (all threads call, after a barrier; ends
// without one).
template <class Arcs>
__device__ __forceinline__ void walk_heavy(const BlockJob& j, BlockShared& sh, int ci, const Arcs& arcs) {
  const unsigned nh = sh.nh3[ci] < HCAP ? sh.nh3[ci] : HCAP;
#pragma unroll 1
  for (unsigned h = 0; h < nh; ++h) {
    const HeavyRow e = sh.heavy[h];
    walk_row(j, sh, ci, e.a0, e.deg, e.offer, (int)threadIdx.x, BT, arcs);
  }
}

// Offers applied to the labels in memory.  filter: a far end's label is loaded first and the atomic is left
// out when it cannot drop; without it the chain is one access shorter, which pays while few rows
// are in flight.  Every label that may have dropped goes to won(w, first arc of w, degree of w, old
// label, offer); EAGER: w's row offsets are read while the atomic is in flight (else 0, 0).  With filter an offer
// is left out, too, when seen(w, offer) knows of one as good.
struct SeenNone {
  __device__ __forceinline__ bool operator()(int, u64) const { return false; }
};
template <int SC, bool EAGER, class Won, class Seen = SeenNone>
struct Relax {
  const BlockJob& j;
  bool filter;
  const Won& won;
  Seen seen = Seen{};
  template <int U>
  __device__ __forceinline__ void run(const int (&w)[U], const bool (&in)[U], const u64 (&offer)[U]) const {
    u64 pw[U], old[U];
    int b0[U], bd[U];
    bool go[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      go[k] = in[k];
      if (filter && in[k]) go[k] = !seen(w[k], offer[k]);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) pw[k] = filter && go[k] ? wg_load(&j.P[w[k]]) : INF;
#pragma unroll
    for (int k = 0; k < U; ++k) {
      go[k] = go[k] && pw[k] > offer[k];
      b0[k] = bd[k] = 0;
      if (go[k]) {
        old[k] = lab_min<SC>(&j.P[w[k]], offer[k]);
        if (EAGER) row_of(j.row_ptr, w[k], &b0[k], &bd[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (go[k]) won(w[k], b0[k], bd[k], old[k], offer[k]);
  }
};
constexpr unsigned FILTER_MIN = 64;  // frontiers of more rows load the label first

// A frontier's entries in LDS: buffer b of v (vertex), a (first arc), d (degree), and l (label).
template <int CAP>
struct Frontier {
  __device__ static u64& l(int b, int i) { return reinterpret_cast<u64*>(blk_dyn)[b * CAP + i]; }
  template <int OFF>
  __device__ static int& at(int b, int i) { return reinterpret_cast<int*>(blk_dyn + OFF)[b * CAP + i]; }
};
struct AloneQ : Frontier<LC> {
  __device__ static int& v(int b, int i) { return at<0>(b, i); }
  __device__ static int& a(int b, int i) { return at<8 * LC>(b, i); }
  __device__ static int& d(int b, int i) { return at<16 * LC>(b, i); }
};
struct TeamQ : Frontier<TC> {
  __device__ static int& v(int b, int i) { return at<16 * TC>(b, i); }
  __device__ static int& a(int b, int i) { return at<24 * TC>(b, i); }
  __device__ static int& d(int b, int i) { return at<32 * TC>(b, i); }
  // a step of one round stages vertices only, in all of it
  __device__ static int& one(unsigned i) { return reinterpret_cast<int*>(blk_dyn)[i]; }
};

// ---- rounds of a workgroup alone on labels in memory (more than CLAIM_N vertices, and the tail) -----
// Appends to the next frontier: the first LC entries in LDS (buffer b), the rest in
// `next` (at most one entry per vertex: n are enough).
struct AloneAppend {
  unsigned* cnt;
  g_int* next;
  int b;
  __device__ __forceinline__ void operator()(int v, int a0, int deg) const {
    const unsigned i = atomicAdd(cnt, 1u);
    if (i < (unsigned)LC) {
      AloneQ::v(b, (int)i) = v;
      AloneQ::a(b, (int)i) = a0;
      AloneQ::d(b, (int)i) = deg;
    } else {
      next[i - LC] = v;
    }
  }
};

// One round (or tail sweep): the wake bucket wk[0 .. nw) and the nf entries of the
// frontier (buffer b, then cur) offer their labels; what they reach goes to `app`.  A round appends a
// vertex reached for the first time (old label INF); a sweep one whose label dropped, once per sweep
// (its stamp takes the sweep's tag).  All threads call; ends with a barrier.
template <bool SWEEP>
__device__ __forceinline__ unsigned alone_round(const BlockJob& j, BlockShared& sh, g_cu64* wk, int nw, unsigned nf, int b,
                                                g_cint* cur, u64 mask, u64 unit, int tag, int ci, const AloneAppend& app) {
  unsigned examined = 0;
  const auto won = [&](int w, int a0, int deg, u64 old, u64 offer) {
    if (SWEEP) {
      if (old > offer && __hip_atomic_exchange(&j.wake[w], tag, __ATOMIC_RELAXED, WG) != tag) app(w, a0, deg);
    } else if (old == INF) {
      app(w, a0, deg);
    }
  };
  const Relax<WG, true, decltype(won)> relax{j, nf > FILTER_MIN, won}, heavy{j, true, won};
  for (int t = (int)threadIdx.x; t < nw; t += BT) {  // a load first: a vertex reached with a smaller label needs no atomic
    const u64 self = wk[t];
    const int v = (int)(self & mask);
    if (wg_load(&j.P[v]) > self) {
      int a0, deg;
      const u64 old = lab_min<WG>(&j.P[v], self);
      row_of(j.row_ptr, v, &a0, &deg);
      if (old == INF) app(v, a0, deg);
    }
  }
  walk_rows(
      j, sh, ci, nf,
      [&](unsigned i, int* a0, int* deg, u64* offer) {
        int v;
        if (i < (unsigned)LC) {
          v = AloneQ::v(b, (int)i);
          *a0 = AloneQ::a(b, (int)i);
          *deg = AloneQ::d(b, (int)i);
        } else {
          v = cur[i - LC];
          row_of(j.row_ptr, v, a0, deg);
        }
        *offer = wg_load(&j.P[v]) + unit;
      },
      relax, examined);
  __syncthreads();
  if (sh.nh3[ci]) {
    walk_heavy(j, sh, ci, heavy);
    __syncthreads();
  }
  return examined;
}

// Whether the label-correcting tail takes over: few vertices are left, many rounds remain, and the frontier
// is small against what is left.  A frontier that still moves reaches it in a few more rounds, for less than
// the tail's sweeps (256^3 grid, beta 0.02: 4.5 ms with the tail entered at an eighth of what is left, 4.1 ms
// at a 64th); what is left once it has died down are small components, each waking in its own round.
// Or the frontier is large against what is left (teams, with a clean queue): the tail's first step lets
// those left pull instead of expanding the whole frontier to reach them (Erdos-Renyi, 464249 vertices of
// degree 6.6: the last two rounds offer the arcs of 114531 vertices to 3000, 28 us;
// entered at twice and at eight times what is left, 270 and 268 us instead of 289; two million vertices of degree 5,
// 588 instead of 623; 40000, 180 instead of 200).
constexpr int TAIL_MIN_LEFT = 16;
constexpr u64 TAIL_IDLE = 64;
constexpr u64 TAIL_FLOOD = 2;

__device__ __forceinline__ bool tail_next(const BlockJob& j, u64 n_active, u64 settled, unsigned nf, int left_rounds,
                                          bool flood = false) {
  const u64 left = n_active - settled;
  return j.tail_den > 0 && left > 0 && left * (u64)j.tail_den <= n_active && left_rounds > TAIL_MIN_LEFT &&
         ((u64)nf * TAIL_IDLE <= left || (flood && nf >= left * TAIL_FLOOD));
}
// The tail's seed walks a row on one thread (0.7 us an arc), and the other members of a team wait for it no longer
// than their barrier allows: a team with a row of more arcs runs its rounds to the end.
constexpr int TAIL_ROW = 1 << 18;
// A workgroup alone pays the tail's scan of every vertex against rounds of about 2.5 us each.
constexpr int TAIL_SCAN = 4096;

// ---- rounds of a workgroup alone, claimed in LDS --------------------------------------------
// Global atomics bound a workgroup's rounds: a 64-bit atomic minimum costs a CU 1.7 ns alone and 9.4 ns
// when every CU issues them (27 G/s over the GPU, whatever the scope and size), a load from L2
// 0.5 - 1 ns.  So a graph of at most CLAIM_N vertices keeps two bits per vertex in LDS, "settled before
// this round" and "reached": an arc to a settled vertex costs no memory access beyond its column, and
// the first offer to a vertex is seen without asking its label.  The offers of a round meet in a
// direct-mapped table in LDS.  They all lie in one round, so an entry is 56 bits: the vertex, and below
// it the fraction and centre of its smallest offer; one LDS minimum enters an offer.  Of two
// vertices of one slot the larger loses it and takes a second slot, whose loser goes to its label in memory
// by an atomic minimum (a conflict).  When the round ends its vertices' labels are written once, with plain stores.
// A round whose frontier outweighs the vertices left, of a graph without long rows, pulls instead:
// each unsettled vertex reads its row, tests its neighbours' frontier bits in LDS and loads the labels
// of those in the frontier (no atomics).
constexpr int TABLE = 4096;     // slots for CLAIM_N vertices (twice as many fit beside the bits of half as many)
constexpr int FC = 2048;        // entries of the frontier kept in LDS; the rest in the graph's queue
constexpr int PULL_DEG = 64;    // pull only when no vertex has more arcs
constexpr unsigned PULL_MIN = 2048, PULL_X = 3;  // pull when frontier > PULL_MIN and > unsettled / PULL_X
constexpr int LOW = 38;         // bits of a fraction and a centre: 20 + 18
constexpr int PULL_U = 8;       // arcs a pulling lane has in flight
constexpr int PULL_WIN = 8192;  // vertices listed at a time in a pull

struct ClaimLds {  // LDS: the frontier, the table, the vertices' bits
  static constexpr int FL = 0, FV = FL + 8 * FC, FA = FV + 4 * FC, FD = FA + 4 * FC, TAB = FD + 4 * FC,
                       END = TAB + 8 * TABLE + CLAIM_N / 4;
  static_assert(END == CLAIM_Q_BYTES && CLAIM_N <= 1 << (LOW - FIX), "the frontier's LDS");
  static_assert(CLAIM_N / 8 <= 8 * TABLE && 2 * PULL_WIN <= 8 * FC, "a pull's bits and list take the table's and labels' place");
  // the bits from the end down, so that their place does not depend on the table's size
  __device__ static unsigned& bits(unsigned i) { return reinterpret_cast<unsigned*>(blk_dyn + END)[~(int)i]; }
  __device__ static u64& tab(unsigned i) { return reinterpret_cast<u64*>(blk_dyn + TAB)[i]; }
  __device__ static unsigned& fbits(unsigned i) { return reinterpret_cast<unsigned*>(blk_dyn + TAB)[i]; }
  __device__ static u64& fl(unsigned i) { return reinterpret_cast<u64*>(blk_dyn + FL)[i]; }  // frontier: label,
  __device__ static int& fv(unsigned i) { return reinterpret_cast<int*>(blk_dyn + FV)[i]; }  // vertex (of the next one,
  __device__ static int& fa(unsigned i) { return reinterpret_cast<int*>(blk_dyn + FA)[i]; }  // while it is built),
  __device__ static int& fd(unsigned i) { return reinterpret_cast<int*>(blk_dyn + FD)[i]; }  // first arc, degree
  __device__ static unsigned short& list(unsigned i) { return reinterpret_cast<unsigned short*>(blk_dyn + FL)[i]; }
};
constexpr unsigned REACHED = 1, SETTLED = 2;

__device__ __forceinline__ unsigned vertex_bits(unsigned v) { return ClaimLds::bits(v >> 4) >> ((v & 15) * 2) & 3u; }
static_assert(TABLE == 1 << 12, "Claim::shift");
static_assert(8 * TABLE == CLAIM_N / 8, "twice the slots beside the bits of half the vertices");

struct Claim {  // what a round's offers need
  g_u64* P;
  g_int* over;     // the next frontier's entries past FC
  unsigned* cnt;   // its length
  unsigned* conf;  // set by a conflict
  u64 base;        // the round's first label
  int shift;       // 32 - log2 of the table's slots
  __device__ __forceinline__ unsigned slot(unsigned v) const { return v * 2654435761u >> shift; }
  __device__ __forceinline__ unsigned slot2(unsigned v) const { return v * 2246822519u >> shift; }
  __device__ __forceinline__ void reach(int w) const {
    const unsigned i = atomicAdd(cnt, 1u);
    if (i < (unsigned)FC) ClaimLds::fv(i) = w;
    else over[i - FC] = w;
  }
  // the offer's place in the table; what it pushed out (or met) when the slot is another vertex's
  __device__ __forceinline__ u64 enter(int w, u64 offer) const {
    return atomicMin(&ClaimLds::tab(slot((unsigned)w)), (u64)w << LOW | (offer - base));
  }
  // the loser of a shared slot takes its vertex's second slot; the loser of that one goes to memory
  __device__ __forceinline__ void place_loser(int w, u64 offer, u64 old) const {
    if (old == INF || (int)(old >> LOW) == w) return;
    const u64 mine = (u64)w << LOW | (offer - base);
    u64 lost = mine > old ? mine : old;
    const unsigned v = (unsigned)(lost >> LOW);
    const u64 second = atomicMin(&ClaimLds::tab(slot2(v)), lost);
    if (second == INF || (unsigned)(second >> LOW) == v) return;
    lost = lost > second ? lost : second;
    (void)lab_min<WG>(&P[lost >> LOW], base + (lost & (((u64)1 << LOW) - 1)));
    *conf = 1;
  }
};

struct ClaimArcs {  // offers along arcs, to their unsettled far ends
  const Claim& c;
  template <int U>
  __device__ __forceinline__ void run(const int (&w)[U], const bool (&in)[U], const u64 (&offer)[U]) const {
    unsigned f[U];
    u64 old[U];
#pragma unroll
    for (int k = 0; k < U; ++k) f[k] = in[k] ? vertex_bits((unsigned)w[k]) : SETTLED;
#pragma unroll
    for (int k = 0; k < U; ++k) {
      old[k] = INF;
      if (!(f[k] & SETTLED)) old[k] = c.enter(w[k], offer[k]);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (f[k] == 0) {
        const unsigned s = ((unsigned)w[k] & 15) * 2;
        if (!(atomicOr(&ClaimLds::bits((unsigned)w[k] >> 4), REACHED << s) >> s & REACHED)) c.reach(w[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) c.place_loser(w[k], offer[k], old[k]);
  }
};

// A round's offers: the wake bucket wk[0 .. nw) and the frontier's nf entries, the first FC in LDS, the rest
// in cur.  All threads call; ends with a barrier.
__device__ __forceinline__ unsigned claim_round(const BlockJob& j, BlockShared& sh, const Claim& c, g_cu64* wk, int nw,
                                                unsigned nf, g_cint* cur, u64 mask, u64 unit, int ci) {
  unsigned examined = 0;
  const ClaimArcs arcs{c};
  for (int t = (int)threadIdx.x; t < nw; t += BT) {
    const u64 self[1] = {wk[t]};
    const int v[1] = {(int)(self[0] & mask)};
    const bool in[1] = {true};
    arcs.run<1>(v, in, self);
  }
  walk_rows(
      j, sh, ci, nf,
      [&](unsigned i, int* a0, int* deg, u64* offer) {
        if (i < (unsigned)FC) {
          *a0 = ClaimLds::fa(i);
          *deg = ClaimLds::fd(i);
          *offer = ClaimLds::fl(i) + unit;
        } else {
          const int v = cur[i - FC];
          row_of(j.row_ptr, v, a0, deg);
          *offer = wg_load(&j.P[v]) + unit;
        }
      },
      arcs, examined);
  __syncthreads();
  if (sh.nh3[ci]) {
    walk_heavy(j, sh, ci, arcs);
    __syncthreads();
  }
  return examined;
}

__device__ __forceinline__ void table_clear(int slots) {
  for (int i = threadIdx.x; i < slots; i += BT) ClaimLds::tab((unsigned)i) = INF;
}

// A pulled round: the wake bucket's unsettled vertices take their own labels, then every unsettled
// vertex the best offer of its neighbours in the frontier.  Labels go straight to memory (a conflict, for
// the settling).  All threads call; ends with a barrier.
__device__ __forceinline__ u64 pull_round(const BlockJob& j, BlockShared& sh, const Claim& c, g_cu64* wk, int nw, unsigned nf,
                                          g_cint* cur, u64 mask, u64 unit, int ci) {
  const int n = j.n;
  g_cint* __restrict__ rp = j.row_ptr;
  g_cint* __restrict__ col = j.col;
  g_u64* P = j.P;
  const int tid = threadIdx.x;
  for (int i = tid; i < (n + 31) / 32; i += BT) ClaimLds::fbits((unsigned)i) = 0;
  for (int t = tid; t < nw; t += BT) {
    const u64 self = wk[t];
    const unsigned v = (unsigned)(self & mask);
    if (!(vertex_bits(v) & SETTLED)) lab_store<WG>(&P[v], self);  // INF until now
  }
  __syncthreads();
  for (unsigned i = tid; i < nf; i += BT) {
    const unsigned v = (unsigned)(i < (unsigned)FC ? ClaimLds::fv(i) : cur[i - FC]);
    atomicOr(&ClaimLds::fbits(v >> 5), 1u << (v & 31));
  }
  if (tid == 0) *c.conf = 1;
  u64 examined = 0;
  for (int v0 = 0; v0 < n; v0 += PULL_WIN) {  // the window's unsettled vertices are listed, then pull
    __syncthreads();
    if (tid == 0) sh.nxt = 0;
    __syncthreads();
    const int hi = n - v0 < PULL_WIN ? n - v0 : PULL_WIN;
    for (int i = tid; i < hi; i += BT)
      if (!(vertex_bits((unsigned)(v0 + i)) & SETTLED))
        ClaimLds::list((unsigned)atomicAdd(&sh.nxt, 1)) = (unsigned short)i;
    __syncthreads();
    const int cnt = sh.nxt;
    for (int i = tid; i < cnt; i += BT) {
      const int v = v0 + ClaimLds::list((unsigned)i);
      const int a0 = rp[v], a1 = rp[v + 1];
      if (a0 == a1) continue;
      const u64 p = wg_load(&P[v]);
      u64 best = p;
      examined += (u64)(a1 - a0);
      for (int a = a0; a < a1; a += PULL_U) {
        int w[PULL_U];
        u64 pw[PULL_U];
        bool bad = false;
#pragma unroll
        for (int k = 0; k < PULL_U; ++k) w[k] = a + k < a1 ? col[a + k] : v;  // (v is not in the frontier)
#pragma unroll
        for (int k = 0; k < PULL_U; ++k) {
          const bool ok = (unsigned)w[k] < (unsigned)n;
          bad |= !ok;
          const bool in = ok && ((ClaimLds::fbits((unsigned)w[k] >> 5) >> (w[k] & 31)) & 1u);
          pw[k] = in ? wg_load(&P[w[k]]) + unit : INF;
        }
#pragma unroll
        for (int k = 0; k < PULL_U; ++k) best = pw[k] < best ? pw[k] : best;
        if (bad) atomicOr(&sh.er3[ci], ERR_BAD_COL);
      }
      if (best < p) lab_store<WG>(&P[v], best);
      if (best != INF) c.reach(v);
    }
  }
  __syncthreads();
  table_clear(1 << (32 - c.shift));
  __syncthreads();
  return examined;
}

// The rounds of one prepared graph of at most CLAIM_N vertices until all are settled or the tail may
// start (returned), with the state of block_rounds.
__device__ __forceinline__ bool claim_rounds(const BlockJob& j, BlockShared& sh, g_int* cur, g_int* next, int& r, u64& settled,
                                             u64& examined, long long& rounds, unsigned& err) {
  const int n = j.n;
  g_u64* P = j.P;
  const int tid = threadIdx.x;
  const int shift = n <= CLAIM_N / 2 ? 19 : 20;
  const u64 delta = sh.delta, n_active = sh.n_active;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const int D = (int)(delta >> FIX);
  const u64 unit = (u64)1 << (FIX + B), mask = ((u64)1 << B) - 1;
  for (int i = tid; i < (n + 15) / 16; i += BT) ClaimLds::bits((unsigned)i) = 0;
  table_clear(1 << (32 - shift));
  if (tid < 3) sh.oc3[tid] = 0;
  __syncthreads();
  unsigned nf = 0;
  int ci = 0;
  while (settled < n_active && r <= D + n && rounds <= (long long)D + n + 2) {
    const int w0 = r <= D ? sh.woff[r] : 0, nw = r <= D ? sh.woff[r + 1] - w0 : 0;
    const Claim c{P, next, &sh.cnt3[ci], &sh.oc3[ci], (u64)r << (FIX + B), shift};
    if (nf > PULL_MIN && sh.maxdeg <= PULL_DEG && (u64)nf * PULL_X > n_active - settled)
      examined += pull_round(j, sh, c, j.wk + w0, nw, nf, cur, mask, unit, ci);
    else
      examined += claim_round(j, sh, c, j.wk + w0, nw, nf, cur, mask, unit, ci);
    // the round's vertices are settled: their labels to memory, their rows to the frontier's entries
    nf = sh.cnt3[ci];
    const bool conf = sh.oc3[ci] != 0;
    for (unsigned i = tid; i < nf; i += BT) {
      const unsigned v = (unsigned)(i < (unsigned)FC ? ClaimLds::fv(i) : next[i - FC]);
      const unsigned h1 = c.slot(v), h2 = c.slot2(v);
      const u64 t1 = ClaimLds::tab(h1), t2 = ClaimLds::tab(h2);
      int a0, deg;
      row_of(j.row_ptr, (int)v, &a0, &deg);
      const u64 seen = conf ? wg_load(&P[v]) : INF;
      u64 t = INF;
      if ((unsigned)(t1 >> LOW) == v) {
        t = t1;
        ClaimLds::tab(h1) = INF;
      }
      if ((unsigned)(t2 >> LOW) == v) {
        t = t2 < t ? t2 : t;
        ClaimLds::tab(h2) = INF;
      }
      u64 p = t == INF ? INF : c.base + (t & (((u64)1 << LOW) - 1));
      if (p < seen) lab_store<WG>(&P[v], p);
      else p = seen;
      atomicOr(&ClaimLds::bits(v >> 4), (SETTLED | REACHED) << ((v & 15) * 2));
      if (i < (unsigned)FC) {
        ClaimLds::fl(i) = p;
        ClaimLds::fa(i) = a0;
        ClaimLds::fd(i) = deg;
      }
    }
    if (tid == 0) {
      const int old = ci == 0 ? 2 : ci - 1;
      sh.cnt3[old] = sh.oc3[old] = sh.nh3[old] = sh.er3[old] = 0;
    }
    __syncthreads();
    err = sh.er3[ci];
    if (err) break;
    ci = ci == 2 ? 0 : ci + 1;
    settled += nf;
    ++rounds;
    g_int* t = cur;
    cur = next;
    next = t;
    if (nf) ++r;
    else r = next_nonempty(sh, r + 1, D);
    if (tail_next(j, n_active, settled, nf, D - r - n / TAIL_SCAN)) return true;
  }
  return false;
}

// The rounds of one prepared graph (results in sh: settled, examined, rounds, sweeps, err).
// Once few vertices are left (unreached vertices * tail_den <= vertices with arcs) and more than
// TAIL_MIN_LEFT rounds remain, the tail finishes by label correction: every unreached vertex
// takes the best of its own label and its neighbours' in F_{r-1} (the only settled vertices
// whose offers are still pending), then sweeps relax the changed labels until none drops.  The
// labels are the unique fixpoint of P(v) = min(own label, min_w P(w) + unit), so the result is
// the same exact one.
__device__ __attribute__((noinline)) void block_rounds(BlockShared& sh) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  g_cint* __restrict__ rp = j.row_ptr;
  g_cint* __restrict__ col = j.col;
  g_ci64* __restrict__ shift = j.shift;
  g_u64* P = j.P;
  const int tid = threadIdx.x;
  const u64 delta = sh.delta, n_active = sh.n_active;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const int D = (int)(delta >> FIX);
  const u64 unit = (u64)1 << (FIX + B);
  g_int* cur = j.q0;
  g_int* next = j.q1;
  int b = 0;  // the frontier's buffer in LDS
  unsigned nf = 0;
  u64 settled = 0, examined = 0;
  long long rounds = 0, sweeps = 0;
  const u64 mask = ((u64)1 << B) - 1;
  if (tid < 3) sh.cnt3[tid] = sh.nh3[tid] = sh.er3[tid] = 0;
  int ci = 0;  // this round's counters: cnt3[ci], nh3[ci], er3[ci]; those of (ci + 2) % 3 are cleared for two rounds on
  int r = next_nonempty(sh, 0, D);
  bool tail = false;
  unsigned err = 0;  // of the last round (the same in every thread)
  // after a round's barrier: its appends are the frontier; the counters of round k - 1 (read by every
  // thread before that barrier) are cleared for round k + 2
  const auto advance = [&]() {
    nf = sh.cnt3[ci];
    err = sh.er3[ci];
    if (tid == 0) {
      const int old = ci == 0 ? 2 : ci - 1;
      sh.cnt3[old] = sh.nh3[old] = sh.er3[old] = 0;
    }
    ci = ci == 2 ? 0 : ci + 1;
    g_int* t = cur;
    cur = next;
    next = t;
    b ^= 1;
  };
  const bool claims = n <= CLAIM_N;
  if (claims) {
    tail = claim_rounds(j, sh, cur, next, r, settled, examined, rounds, err);
    __syncthreads();
    if (tid < 3) sh.cnt3[tid] = sh.nh3[tid] = sh.er3[tid] = 0;
    __syncthreads();
  }
  while (!claims && settled < n_active && r <= D + n && rounds <= (long long)D + n + 2) {
    const int w0 = r <= D ? sh.woff[r] : 0, w1 = r <= D ? sh.woff[r + 1] : 0;
    const AloneAppend app{&sh.cnt3[ci], next, b ^ 1};
    examined += alone_round<false>(j, sh, j.wk + w0, w1 - w0, nf, b, cur, mask, unit, 0, ci, app);
    advance();
    if (err) break;
    settled += nf;
    ++rounds;
    if (nf) ++r;
    else r = next_nonempty(sh, r + 1, D);
    if (tail_next(j, n_active, settled, nf, D - r - n / TAIL_SCAN)) {
      tail = true;
      break;
    }
  }
  if (tail) {
    // seed: F_{r-1} is the frontier (final labels); every unreached vertex with arcs takes the best of
    // its own label and its neighbours' in F_{r-1}, and is queued for the first sweep
    const AloneAppend app{&sh.cnt3[ci], next, b ^ 1};
    const u64 prev_round = (u64)(r - 1);
    for (int v = tid; v < n; v += BT) {
      const int a0 = rp[v], a1 = rp[v + 1];
      if (a1 == a0 || wg_load(&P[v]) != INF) continue;
      u64 best = ((delta - (u64)shift[v]) << B) | (u64)v;
      for (int a = a0; a < a1; ++a) {
        const int u = col[a];
        if ((unsigned)u >= (unsigned)n) {
          atomicOr(&sh.er3[ci], ERR_BAD_COL);
          break;
        }
        const u64 pu = wg_load(&P[u]);
        if (pu != INF && (pu >> (FIX + B)) == prev_round && pu + unit < best) best = pu + unit;
      }
      examined += (u64)(a1 - a0);
      lab_store<WG>(&P[v], best);
      j.wake[v] = -1;  // the stamp of the first sweep
      app(v, a0, a1 - a0);
    }
    __syncthreads();
    advance();
    // sweeps: sweep k relaxes the labels queued by the step before and queues those that drop
    for (int k = 1; nf && !err && sweeps <= n; ++k) {
      const AloneAppend app{&sh.cnt3[ci], next, b ^ 1};
      examined += alone_round<true>(j, sh, nullptr, 0, nf, b, cur, mask, unit, -(k + 1), ci, app);
      advance();
      ++sweeps;
    }
    settled = n_active;
  }
  __syncthreads();
  examined = block_sum64(examined, sh);
  if (tid == 0) {
    sh.err |= err;
    sh.settled = settled;
    sh.examined = examined;
    sh.rounds = rounds;
    sh.sweeps = sweeps;
  }
  __syncthreads();
}

// The cut arcs of a listed row (output_slice): its vertex and centre come as its offer.
struct CutRow {
  const BlockJob& j;
  u64 mask;
  u64& cut2;
  template <int U>
  __device__ __forceinline__ void run(const int (&w)[U], const bool (&in)[U], const u64 (&row)[U]) const {
    bool far[U];
    u64 pw[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      far[k] = in[k] && w[k] > (int)(row[k] >> 32);
      pw[k] = far[k] ? wg_load(&j.P[w[k]]) : 0;
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      cut2 += far[k] && (pw[k] == INF ? w[k] : (int)(pw[k] & mask)) != (int)(unsigned)row[k] ? 2u : 0u;
  }
};

// Centres and cut arcs of the vertices [lo, hi), added to *cut2 and *pieces; an arc to a vertex out
// of range (arcs of the last frontier were not read by a round) sets ERR_BAD_COL.  The graph is symmetric, so
// an edge is looked at from its smaller end alone and counts as two arcs: the far ends' labels are what
// bounds this pass (random accesses: with every CU busy 2.3 ns an arc, half of a random graph's
// whole time, when both arcs loaded one).
// A row of more than HUGE_ROW arcs is listed for the whole workgroup: a thread takes 0.36 us an arc, and the
// members of a team waited longer than their barrier allows for one with millions.  The caller has cleared
// slot 0 of nh3 and er3 before a barrier; all threads call, and thread 0 adds the rows' errors to sh.err last.
__device__ __forceinline__ void output_slice(const BlockJob& j, BlockShared& sh, int lo, int hi, u64 mask, u64* cut2,
                                             u64* pieces) {
  const int n = j.n;
  g_cint* __restrict__ rp = j.row_ptr;
  g_cint* __restrict__ col = j.col;
  g_cu64* P = j.P;
  for (int v0 = lo + (int)threadIdx.x; v0 < hi; v0 += VU * BT) {
    int a[VU], a1[VU], c[VU];
    u64 p[VU];
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      a[k] = a1[k] = 0;
      p[k] = INF;
      if (v < hi) {
        a[k] = rp[v];
        a1[k] = rp[v + 1];
        p[k] = wg_load(&P[v]);
      }
    }
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      c[k] = p[k] == INF ? v : (int)(p[k] & mask);
      if (v < hi) {
        j.centre[v] = c[k];
        *pieces += c[k] == v;
      }
      if (__builtin_expect(a1[k] - a[k] > HUGE_ROW, 0)) {
        const unsigned h = atomicAdd(&sh.nh3[0], 1u);
        if (h < HCAP) {
          sh.heavy[h] = HeavyRow{(u64)(unsigned)v << 32 | (unsigned)c[k], a[k], a1[k] - a[k]};
          a[k] = a1[k];
        }
      }
    }
    bool bad = false;
    for (bool more = true; more;) {  // AU arcs of each vertex per pass
      int w[VU][AU];
      bool has[VU][AU];
#pragma unroll
      for (int k = 0; k < VU; ++k)
#pragma unroll
        for (int t = 0; t < AU; ++t) {
          has[k][t] = a[k] + t < a1[k];
          w[k][t] = has[k][t] ? col[a[k] + t] : 0;
        }
      u64 pw[VU][AU];
#pragma unroll
      for (int k = 0; k < VU; ++k)
#pragma unroll
        for (int t = 0; t < AU; ++t) {
          const bool ok = (unsigned)w[k][t] < (unsigned)n;
          bad |= has[k][t] && !ok;
          has[k][t] = has[k][t] && ok && w[k][t] > v0 + k * BT;
          pw[k][t] = has[k][t] ? wg_load(&P[w[k][t]]) : 0;
        }
      more = false;
#pragma unroll
      for (int k = 0; k < VU; ++k) {
#pragma unroll
        for (int t = 0; t < AU; ++t)
          *cut2 += has[k][t] && (pw[k][t] == INF ? w[k][t] : (int)(pw[k][t] & mask)) != c[k] ? 2u : 0u;
        a[k] += AU;
        more |= a[k] < a1[k];
      }
    }
    if (bad) atomicOr(&sh.err, ERR_BAD_COL);
  }
  __syncthreads();
  if (__builtin_expect(sh.nh3[0] != 0, 0)) {
    walk_heavy(j, sh, 0, CutRow{j, mask, *cut2});
    __syncthreads();
    if (threadIdx.x == 0) sh.err |= sh.er3[0];
  }
}

// The same with the centres (at most 16 bits) kept in LDS.  Centres of the vertices [lo, hi) (INF: an isolated vertex, its own
// centre), four per thread at a time; put(v, centre) is called for each.
template <class Put>
__device__ __forceinline__ void output_centres(const BlockJob& j, int lo, int hi, u64 mask, u64* pieces, const Put& put) {
  for (int v0 = lo + (int)threadIdx.x; v0 < hi; v0 += VU * BT) {
    u64 p[VU];
#pragma unroll
    for (int k = 0; k < VU; ++k) p[k] = v0 + k * BT < hi ? wg_load(&j.P[v0 + k * BT]) : 0;
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      if (v < hi) {
        const int c = p[k] == INF ? v : (int)(p[k] & mask);
        j.centre[v] = c;
        *pieces += c == v;
        put(v, c);
      }
    }
  }
}

// Arcs of the rows [lo, hi) whose ends have different centres (of(v): v's centre, known once
// output_centres is done), added to *cut2.  An arc to a vertex out of range (arcs of the last frontier were
// not read by a round) sets ERR_BAD_COL in sh.err (by thread 0, with no barrier after it).  The rows are walked as
// a frontier's: a lane per row took 0.94 ns an arc, most of it idle lanes on uneven degrees.
template <class Of>
struct CutArcs {
  const Of& of;
  u64& cut2;
  template <int U>
  __device__ __forceinline__ void run(const int (&w)[U], const bool (&in)[U], const u64 (&c)[U]) const {
    int cw[U];
#pragma unroll
    for (int k = 0; k < U; ++k) cw[k] = in[k] ? of(w[k]) : 0;
#pragma unroll
    for (int k = 0; k < U; ++k) cut2 += in[k] && cw[k] != (int)c[k];
  }
};
template <class Of>
__device__ __forceinline__ void output_cut(const BlockJob& j, BlockShared& sh, int lo, int hi, const Of& of, u64* cut2) {
  if (threadIdx.x == 0) sh.nh3[0] = sh.er3[0] = 0;
  __syncthreads();
  const CutArcs<Of> arcs{of, *cut2};
  unsigned examined = 0;
  walk_rows(
      j, sh, 0, (unsigned)(hi - lo),
      [&](unsigned i, int* a0, int* deg, u64* c) {
        row_of(j.row_ptr, lo + (int)i, a0, deg);
        *c = (u64)(unsigned)of(lo + (int)i);
      },
      arcs, examined);
  __syncthreads();
  walk_heavy(j, sh, 0, arcs);
  __syncthreads();
  if (threadIdx.x == 0) sh.err |= sh.er3[0];
}

__device__ __attribute__((noinline)) void block_output(BlockShared& sh, BlockOut* out) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  const int tid = threadIdx.x;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const u64 mask = ((u64)1 << B) - 1;
  const unsigned e0 = sh.err | (sh.settled < sh.n_active ? ERR_WATCHDOG : 0u);
  if (tid == 0) sh.nh3[0] = sh.er3[0] = 0;
  __syncthreads();  // every thread has read sh.err: the passes below may add to it
  u64 cut2 = 0, pieces = 0;
  if (!e0) {
    // centres of up to 16 bits are kept in LDS (a load from L2 costs a CU 0.5 - 1 ns), others read as written
    unsigned short* lc = reinterpret_cast<unsigned short*>(blk_dyn);
    static_assert(CLAIM_Q_BYTES >= 2 << 16, "centres in LDS");
    if (n <= 1 << 16) {
      output_centres(j, 0, n, mask, &pieces, [&](int v, int c) { lc[v] = (unsigned short)c; });
      __syncthreads();
      output_cut(j, sh, 0, n, [&](int v) { return (int)lc[v]; }, &cut2);
    } else {
      output_slice(j, sh, 0, n, mask, &cut2, &pieces);
    }
  }
  cut2 = block_sum64(cut2, sh);
  pieces = block_sum64(pieces, sh);
  if (tid == 0) {
    out->err = e0 | sh.err;
    out->cut_arcs = cut2;
    out->pieces = pieces;
    out->delta = sh.delta;
    out->n_active = sh.n_active;
    out->rounds = sh.rounds;
    out->sweeps = sh.sweeps;
    out->examined = sh.examined;
  }
}

// One graph, the whole workgroup.
__device__ void block_graph(BlockShared& sh, BlockOut* out) {
  block_prepare(sh);
  if (sh.err) {
    if (threadIdx.x == 0) {
      out->err = sh.err;
      out->delta = sh.delta;
    }
    return;
  }
  block_rounds(sh);
  block_output(sh, out);
}

// One small graph whose labels and CSR fit the LDS, the whole workgroup: every vertex
// starts from its own label ((Delta - shift) << B) | v and the labels are relaxed,
// P(v) = min(P(v), min over arcs (v, u) of P(u) + unit), in place, until a pass lowers none.
// That is the unique fixpoint the rounds reach (the minimum over centres of the shifted
// distance, ties to the smaller centre; Sec. 5's search, by label correction from every source at
// once), so the result is the same; no wake buckets, frontier or queue, and every access but
// the first loads of the CSR and shifts stays in LDS.  A pass costs about n / 1024 vertices per
// thread; there are at most as many passes as the largest number of hops from a vertex to its
// centre, plus one block of passes (fewer, since labels lowered early in a pass are read later in
// the same pass).
// Labels are 8-byte LDS words written whole, so a concurrent read sees the old or the new label.
//
// What bounds a pass is its LDS accesses and instructions.  A thread keeps its first FIX_V vertices' labels
// (it alone writes them) and the first RD columns of each, as 16-bit ids, in registers, so that an arc
// costs one LDS read and a 64-bit minimum; a missing arc reads the vertex itself, whose offer is
// never lower.  With row offsets and columns read from LDS in every pass (the columns of 64 rows of four
// in conflicting banks) a pass of the 64 x 64 grid took 2.2 us, so 0.9: its 20 label accesses per thread are
// 0.55 us of the LDS's 128 bytes a cycle.  A decomposition of that grid at beta 0.1 (40 passes) went from 113 to
// 61 us, 46 of them this kernel.  Two or eight passes between barriers measure the same within 2 us.
constexpr int FIX_V = 6;
constexpr int FIX_BLOCK = 4;  // passes between two barriers
// A row of more than FIX_LONG arcs is relaxed by a wave, 64 arcs at a time, not by its thread arc after arc
// (R-MAT 11, 4 edges per vertex: 518 us with each hub's row on one thread, and 167; R-MAT 10: 269 and 82).
constexpr int FIX_LONG = 64;
static_assert(BLOCK_LDS_BYTES / 4 / FIX_LONG <= FIX_LONG_ROWS, "every long row can be listed");

struct FixGraph {
  u64* P;           // LDS: labels
  const int* rp;    // LDS: row offsets, columns
  const int* col;
  int n, degmax, B;
  u64 unit;
  const unsigned short* longv;  // LDS: the vertices of long rows
  int nlong;
};

// The passes and the output.  Passes run FIX_BLOCK at a time with no barrier between them (in-place
// relaxation is exact in any interleaving); a block of passes in which no thread lowered any label
// read only final labels, so the labels are the fixpoint.
template <int RD>
__device__ __forceinline__ void fix_passes(const FixGraph& g, g_int* centre, g_u64* labels, long long* passes_out,
                                           bool* converged_out, u64* cut2, u64* pieces) {
  const int n = g.n, tid = threadIdx.x;
  u64* P = g.P;
  const int* __restrict__ rp = g.rp;   // the CSR in LDS is never written during the passes
  const int* __restrict__ col = g.col;
  const bool rest = g.degmax > RD;
  unsigned id[FIX_V][RD / 2];
  u64 p[FIX_V];
#pragma unroll
  for (int k = 0; k < FIX_V; ++k) {
    const int v = tid + k * BT, a0 = v < n ? rp[v] : 0, a1 = v < n ? rp[v + 1] : 0;
    p[k] = v < n && a1 - a0 <= FIX_LONG ? P[v] : 0;  // 0: never lowered here
#pragma unroll
    for (int e = 0; e < RD / 2; ++e) {
      const int x = a0 + 2 * e < a1 ? col[a0 + 2 * e] : v, y = a0 + 2 * e + 1 < a1 ? col[a0 + 2 * e + 1] : v;
      id[k][e] = (unsigned)x | (unsigned)y << 16;
    }
  }
  long long passes = 0;
  bool converged = false;
  for (;;) {
    int changed = 0;
    for (int i = 0; i < FIX_BLOCK; ++i) {
#pragma unroll
      for (int k = 0; k < FIX_V; ++k) {
        const int v = tid + k * BT;
        if (v < n) {
          u64 best = INF;
#pragma unroll
          for (int e = 0; e < RD / 2; ++e) {
            const u64 q = P[id[k][e] & 0xffff], t = P[id[k][e] >> 16];
            const u64 m = q < t ? q : t;
            best = m < best ? m : best;
          }
          if (rest && p[k]) {
            const int a1 = rp[v + 1];
            for (int a = rp[v] + RD; a < a1; ++a) {
              const u64 q = P[col[a]];
              best = q < best ? q : best;
            }
          }
          best += g.unit;
          if (best < p[k]) {
            P[v] = p[k] = best;
            changed = 1;
          }
        }
      }
      for (int v = tid + FIX_V * BT; v < n; v += BT) {
        const int a1 = rp[v + 1];
        if (a1 - rp[v] > FIX_LONG) continue;
        const u64 own = P[v];
        u64 best = own;
        for (int a = rp[v]; a < a1; ++a) {
          const u64 q = P[col[a]] + g.unit;
          best = q < best ? q : best;
        }
        if (best < own) {
          P[v] = best;
          changed = 1;
        }
      }
      for (int t = tid / WAVE; t < g.nlong; t += BT / WAVE) {  // one wave each: the only writer of the label
        const int v = g.longv[t], a1 = rp[v + 1];
        u64 best = INF;
        for (int a = rp[v] + (int)lane_id(); a < a1; a += WAVE) {
          const u64 q = P[col[a]];
          best = q < best ? q : best;
        }
        best = wave_min_u64(best) + g.unit;
        if (best < P[v]) {
          if (lane_id() == 0) P[v] = best;
          changed = 1;
        }
      }
    }
    passes += FIX_BLOCK;
    converged = !__syncthreads_or(changed);
    if (converged || passes > (long long)n + 1 + FIX_BLOCK) break;
  }
  // centres, pieces, cut; the labels to the graph's label array
  const u64 mask = ((u64)1 << g.B) - 1;
  for (int v = tid; v < n; v += BT) {
    const u64 q = P[v];
    const int c = (int)(q & mask);
    centre[v] = c;
    labels[v] = q;
    *pieces += c == v;
    const int a1 = rp[v + 1];
    if (a1 - rp[v] > FIX_LONG) continue;
    for (int a = rp[v]; a < a1; ++a) *cut2 += (int)(P[col[a]] & mask) != c;
  }
  for (int t = tid / WAVE; t < g.nlong; t += BT / WAVE) {
    const int v = g.longv[t], c = (int)(P[v] & mask), a1 = rp[v + 1];
    for (int a = rp[v] + (int)lane_id(); a < a1; a += WAVE) *cut2 += (int)(P[col[a]] & mask) != c;
  }
  *passes_out = passes;
  *converged_out = converged;
}

__device__ __attribute__((noinline)) void block_graph_fix(BlockShared& sh, BlockOut* out) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  const long long nnz = j.nnz;
  g_cint* __restrict__ rp = j.row_ptr;
  g_cint* __restrict__ col = j.col;
  g_ci64* __restrict__ shift = j.shift;
  const int tid = threadIdx.x;
  u64* P = reinterpret_cast<u64*>(blk_dyn);
  int* lrp = reinterpret_cast<int*>(P + n);
  int* lcol = lrp + n + 1;
  if (tid == 0) sh.err = sh.nlong = 0;
  __syncthreads();
  unsigned err = 0;
  u64 dmax = 0;
  if (tid == 0 && n > 0 && (rp[0] != 0 || (long long)rp[n] != nnz)) err |= ERR_BAD_ROWPTR;
  u64 active = 0, degmax = 0;
  for (int v0 = tid; v0 < n; v0 += VU * BT) {
    long long s[VU];
    int a0[VU], deg[VU];
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      s[k] = 0;
      a0[k] = deg[k] = 0;
      if (v < n) {
        s[k] = shift[v];
        row_of(rp, v, &a0[k], &deg[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      const int v = v0 + k * BT;
      if (v < n) {
        if (s[k] < 0 || s[k] > (1ll << 52)) err |= ERR_BAD_SHIFT;
        if (deg[k] < 0) err |= ERR_BAD_ROWPTR;
        lrp[v] = a0[k];
        P[v] = (u64)s[k];  // the shift, until Delta is known
        active += deg[k] > 0;
        if (deg[k] > FIX_LONG && !err) {  // (offsets that are no offsets may claim more of them than there can be)
          const unsigned i = atomicAdd(&sh.nlong, 1u);
          if (i < (unsigned)FIX_LONG_ROWS) sh.longv[i] = (unsigned short)v;
          else err |= ERR_BAD_ROWPTR;
        }
        degmax = deg[k] > 0 && (u64)deg[k] > degmax ? (u64)deg[k] : degmax;
        dmax = (u64)s[k] > dmax ? (u64)s[k] : dmax;
      }
    }
  }
  if (tid == 0) lrp[n] = (int)nnz;
  for (long long a0 = tid; a0 < nnz; a0 += VU * BT) {
    int c[VU];
#pragma unroll
    for (int k = 0; k < VU; ++k) c[k] = a0 + k * BT < nnz ? col[a0 + k * BT] : 0;
#pragma unroll
    for (int k = 0; k < VU; ++k) {
      if ((unsigned)c[k] >= (unsigned)n) err |= ERR_BAD_COL;
      if (a0 + k * BT < nnz) lcol[a0 + k * BT] = c[k];
    }
  }
  if (err) atomicOr(&sh.err, err);
  const u64 delta = block_max64(dmax, sh);
  const u64 n_active = block_sum64(active, sh);
  degmax = block_max64(degmax, sh);
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  __syncthreads();
  if (tid == 0) {
    unsigned e = sh.err;
    if (!e && (delta + ((u64)1 << FIX)) >= ((u64)1 << (64 - B))) e |= BLK_OVERFLOW;
    sh.err = e;
  }
  __syncthreads();
  if (sh.err) {
    if (tid == 0) {
      out->err = sh.err;
      out->delta = delta;
    }
    return;
  }
  for (int v = tid; v < n; v += BT) P[v] = ((delta - P[v]) << B) | (u64)v;
  __syncthreads();
  const FixGraph g{P, lrp, lcol, n, (int)degmax, B, (u64)1 << (FIX + B), sh.longv, (int)sh.nlong};
  long long passes = 0;
  bool converged = false;
  u64 cut2 = 0, pieces = 0;
  if (degmax <= 4) fix_passes<4>(g, j.centre, j.P, &passes, &converged, &cut2, &pieces);
  else fix_passes<8>(g, j.centre, j.P, &passes, &converged, &cut2, &pieces);
  cut2 = block_sum64(cut2, sh);
  pieces = block_sum64(pieces, sh);
  if (tid == 0) {
    out->err = converged ? 0u : (unsigned)ERR_WATCHDOG;
    out->cut_arcs = cut2;
    out->pieces = pieces;
    out->delta = delta;
    out->n_active = n_active;
    out->rounds = passes;
    out->sweeps = 0;
    out->examined = (u64)passes * (u64)nnz;
  }
}

// ---- a team of workgroups on one graph ----------------------------------------------------

// Member 0 clears the words of the next step's slot before it arrives at this step's barrier:
// every member read them (as the slot of the step before last) before arriving at the last
// barrier, and the next step uses them only after this step's barrier (all threads call).
__device__ __forceinline__ void team_clear_next(BlockShared& sh) {
  if (sh.tm != 0) return;
  const int nx = (int)((sh.epoch + 1) % 3);
  const int ng = (sh.tK + TEAM_GROUP - 1) / TEAM_GROUP;
  if ((int)threadIdx.x < ng) __hip_atomic_store(&sh.ts->gw[nx][threadIdx.x].v, 0ull, __ATOMIC_RELAXED, AG);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&sh.ts->tw[nx].v, 0ull, __ATOMIC_RELAXED, AG);
    __hip_atomic_store(&sh.ts->qcnt[nx], 0ull, __ATOMIC_RELAXED, AG);
    __hip_atomic_store(&sh.ts->first[nx], 0ull, __ATOMIC_RELAXED, AG);
  }
}

// The team's barrier k (all threads call; k = sh.epoch, slot k % 3).  Every wave first waits for
// its own stores and atomics to complete (a workgroup barrier does not wait for other waves'
// stores to leave the CU).  Then thread 0 arrives, adding (1 << 44) | (spill ? 1 << 38 : 0) |
// (error ? 1 << 32 : 0) | (its appends this step) to its group's word; the group's last arrival adds
// the group's sums to the team's word, and the team's last arrival publishes the step's queue length
// (the sum of the appends, bit 31: some member spilled; 0xffffffff if any member had an error) with the
// barrier's number in gen, which the others wait for.  In a team of at most TEAM_GROUP members the
// arrivals go to the team's word directly.  full: arrivals are acquire-release read-modify-writes,
// gen a release store and the wait ends with an acquire, so every plain write of the members before
// the barrier is visible to plain loads after it (each member writes back and invalidates its L2).
// Otherwise everything is relaxed: the members' shared accesses are device-scope themselves and
// complete before the arrival (the waits above), and every load after the barrier is issued after
// the wait observed gen.  A bounded wait raises ERR_BARRIER instead of hanging.  Returns the queue
// length (and in sh.tspill, sh.tfirst the step's spill and the vertices it reached first); after an
// error in any member every member has the team's error bits in sh.terr and in sh.err.  The rounds end on
// sh.terr, which changes at a barrier only: sh.err may already hold what a faster wave found in the next step.
template <bool FULL>
__device__ unsigned team_barrier(BlockShared& sh) {
  constexpr int RMW = FULL ? __ATOMIC_ACQ_REL : __ATOMIC_RELAXED;
  constexpr int PUB = FULL ? __ATOMIC_RELEASE : __ATOMIC_RELAXED;
  team_clear_next(sh);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    g_sync* ts = sh.ts;
    const unsigned K = (unsigned)sh.tK, g = (unsigned)sh.tm / TEAM_GROUP;
    const unsigned ng = (K + TEAM_GROUP - 1) / TEAM_GROUP;
    const unsigned in_g = K - g * TEAM_GROUP < (unsigned)TEAM_GROUP ? K - g * TEAM_GROUP : (unsigned)TEAM_GROUP;
    const unsigned e1 = sh.epoch + 1;
    const int slot = (int)(sh.epoch % 3);
    sh.err |= sh.er3[0] | sh.er3[1] | sh.er3[2];
    if (sh.err) __hip_atomic_fetch_or(&ts->err, sh.err, __ATOMIC_RELAXED, AG);
    constexpr int ARR = 44, SPILL = 38, ERR = 32;  // at most 32 groups or members: six bits each
    const u64 mine = (1ull << ARR) | ((u64)(sh.spill != 0) << SPILL) | ((u64)(sh.err != 0) << ERR) | (u64)sh.tcount;
    const auto bits = [](u64 sum) {  // one error and one spill whatever their count
      return (sum & 0xffffffffu) | ((u64)(((sum >> ERR) & 63) != 0) << ERR) | ((u64)(((sum >> SPILL) & 63) != 0) << SPILL);
    };
    bool last = false;
    u64 sum = 0;
    if (ng == 1) {
      const u64 old = __hip_atomic_fetch_add(&ts->tw[slot].v, mine, RMW, AG);
      last = (old >> ARR) + 1 == K;
      sum = bits(old + mine);
    } else {
      const u64 old = __hip_atomic_fetch_add(&ts->gw[slot][g].v, mine, RMW, AG);
      if ((old >> ARR) + 1 == in_g) {
        const u64 grp = (1ull << ARR) | bits(old + mine);
        const u64 top = __hip_atomic_fetch_add(&ts->tw[slot].v, grp, RMW, AG);
        last = (top >> ARR) + 1 == ng;
        sum = bits(top + grp);
      }
    }
    u64 word;
    if (last) {
      const unsigned nf = ((sum >> ERR) & 1) ? 0xffffffffu : (unsigned)sum | (unsigned)((sum >> SPILL) & 1) << 31;
      word = ((u64)nf << 32) | e1;
      __hip_atomic_store(&ts->gen, word, PUB, AG);
    } else {
      unsigned spins = 0;
      while ((unsigned)(word = __hip_atomic_load(&ts->gen, __ATOMIC_RELAXED, AG)) < e1) {
        __builtin_amdgcn_s_sleep(1);
        if (++spins > (1u << 22)) {  // seconds: far beyond any round, or a member's late start
          __hip_atomic_fetch_or(&ts->err, (unsigned)ERR_BARRIER, __ATOMIC_RELAXED, AG);
          word = (u64)0xffffffffu << 32;
          break;
        }
      }
    }
    if (FULL) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    unsigned nf = (unsigned)(word >> 32);
    sh.tspill = 0;
    sh.terr = 0;
    if (nf == 0xffffffffu) {
      const unsigned e = __hip_atomic_load(&ts->err, __ATOMIC_RELAXED, AG);
      sh.terr = e ? e : (unsigned)ERR_BARRIER;
      sh.err |= sh.terr;
      nf = 0;
    } else {
      sh.tspill = nf >> 31;
      nf &= 0x7fffffffu;
    }
    sh.tfirst = __hip_atomic_load(&ts->first[slot], __ATOMIC_RELAXED, AG);
    sh.tnf = nf;
    sh.tcount = 0;
    sh.spill = 0;
    sh.epoch = e1;
  }
  __syncthreads();
  return sh.tnf;
}

// The c entries staged in LDS (buffer b; ONE: of a step of one round) go to the team's shared queue behind
// one reservation (all threads call; ends with a barrier).  Entries past the queue's n are dropped with
// BLK_QUEUE.
template <bool ONE>
__device__ __forceinline__ void team_flush(BlockShared& sh, int n, g_int* next, g_u64* gcnt, int b, unsigned c) {
  if (threadIdx.x == 0) {
    sh.tbase = (unsigned)__hip_atomic_fetch_add(gcnt, (u64)c, __ATOMIC_RELAXED, AG);
    sh.tcount += c;
  }
  __syncthreads();
  const unsigned base = sh.tbase;
  for (unsigned i = threadIdx.x; i < c; i += BT) {
    const int v = ONE ? TeamQ::one(i) : TeamQ::v(b, (int)i);
    if (base + i < (unsigned)n) __hip_atomic_store(&next[base + i], v, __ATOMIC_RELAXED, AG);
    else atomicOr(&sh.err, BLK_QUEUE);
  }
  __syncthreads();
}

// End of a member's step: what its last round staged (buffer b, cnt entries counted) goes to the shared
// queue `next`, then the barrier, which returns the queue's length, the same in every member (all
// threads call, after a barrier).
template <bool FULL, bool ONE>
__device__ __forceinline__ unsigned team_step_end(BlockShared& sh, int n, g_int* next, g_u64* gcnt, int b, unsigned cnt) {
  constexpr unsigned CAP = ONE ? TC1 : TC;
  const unsigned c = cnt < CAP ? cnt : CAP;
  if (threadIdx.x == 0 && sh.sfirst) {
    __hip_atomic_fetch_add(&sh.ts->first[sh.epoch % 3], (u64)sh.sfirst, __ATOMIC_RELAXED, AG);
    sh.sfirst = 0;
  }
  if (c) team_flush<ONE>(sh, n, next, gcnt, b, c);
  const unsigned nf = team_barrier<FULL>(sh);
  if (threadIdx.x < 3) sh.cnt3[threadIdx.x] = sh.nh3[threadIdx.x] = sh.er3[threadIdx.x] = 0;
  __syncthreads();
  return nf;
}

// Before plain loads of labels that other members wrote since the last full barrier: an acquire
// that invalidates this CU's L1 and its XCD's L2 (all threads call).
__device__ __forceinline__ void team_acquire() {
  if (threadIdx.x == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __syncthreads();
}

// The first non-empty wake bucket of the whole graph at or after r, from the bitmap sh.nz (D + n +
// 1 past the end, as next_nonempty; all threads call).
__device__ __forceinline__ int team_next_nonempty(BlockShared& sh, int r, int D) {
  __syncthreads();
  if (threadIdx.x == 0) sh.nxt = 0x7fffffff;
  __syncthreads();
  const int w = (int)threadIdx.x;
  if (w < BLOCK_WCAP / 64 && r < BLOCK_WCAP) {
    const int b0 = w * 64;
    u64 bits = sh.nz[w];
    if (b0 + 63 < r) bits = 0;
    else if (b0 < r) bits &= ~0ull << (r - b0);
    if (bits) atomicMin(&sh.nxt, b0 + __builtin_ctzll(bits));
  }
  __syncthreads();
  const int q = sh.nxt;
  __syncthreads();
  return q <= D ? q : 0x3fffffff;
}

// Team preparation: every member scans its slice (checks, labels INF, Delta and the vertices with
// arcs, combined by atomics in the team's record) and sorts its slice's wake buckets; the members'
// non-empty buckets are ORed into the record and read back after a second barrier.
__device__ __attribute__((noinline)) void team_prepare(BlockShared& sh) {
  const BlockJob j = job_of(sh);
  const int tid = threadIdx.x;
  g_sync* ts = sh.ts;
  if (tid == 0) {
    sh.err = 0;
    sh.spill = 0;
    sh.sfirst = 0;
  }
  if (tid < 3) sh.er3[tid] = 0;
  __syncthreads();
  u64 dmax, active, degmax;
  prepare_scan(j, sh, sh.tlo, sh.thi, sh.tm == 0, &dmax, &active, &degmax);
  if (tid == 0) {
    if (degmax > (u64)STEP_ROW || (j.deg_cap > 0 && degmax > (u64)j.deg_cap))
      __hip_atomic_fetch_max(&ts->maxdeg, degmax, __ATOMIC_RELAXED, AG);
    if (dmax) __hip_atomic_fetch_max(&ts->delta, dmax, __ATOMIC_RELAXED, AG);
    if (active) __hip_atomic_fetch_add(&ts->active, active, __ATOMIC_RELAXED, AG);
    if (sh.err) __hip_atomic_fetch_or(&ts->err, sh.err, __ATOMIC_RELAXED, AG);
  }
  team_barrier<true>(sh);
  const u64 delta = __hip_atomic_load(&ts->delta, __ATOMIC_RELAXED, AG);
  const u64 n_active = __hip_atomic_load(&ts->active, __ATOMIC_RELAXED, AG);
  unsigned e = __hip_atomic_load(&ts->err, __ATOMIC_RELAXED, AG);
  if (!e) e = range_err(j.n, delta);
  const u64 maxdeg = __hip_atomic_load(&ts->maxdeg, __ATOMIC_RELAXED, AG);
  if (!e && j.deg_cap > 0 && maxdeg > (u64)j.deg_cap) e = BLK_SKEW;
  __syncthreads();
  if (tid == 0) {
    sh.err |= e;
    sh.maxdeg = (unsigned)maxdeg;
    if (maxdeg > (u64)TAIL_ROW) sh.j.tail_den = 0;
    sh.delta = delta;
    sh.n_active = n_active;
  }
  __syncthreads();
  if (sh.err) return;
  wake_sort(j, sh, sh.tlo, sh.thi, delta);
  if (tid < BLOCK_WCAP / 64) {
    u64 bits = 0;
    for (int b = 0; b < 64; ++b) {
      const int q = tid * 64 + b;
      bits |= (u64)(sh.woff[q + 1] > sh.woff[q]) << b;
    }
    if (bits) __hip_atomic_fetch_or(&ts->nz[tid], bits, __ATOMIC_RELAXED, AG);
  }
  team_barrier<true>(sh);
  if (tid < BLOCK_WCAP / 64) sh.nz[tid] = __hip_atomic_load(&ts->nz[tid], __ATOMIC_RELAXED, AG);
  __syncthreads();
}

// What a team member reaches in a round: staged in LDS (ONE: TC1 vertices; else TC entries of buffer b), the
// rest straight to the team's queue, each behind its own reservation (an entry past the queue's n is
// dropped with BLK_QUEUE).  early: the entry is expected in LDS by a later round of this step (a spill).
template <bool ONE>
struct TeamAppend {
  BlockShared* sh;
  unsigned* cnt;
  g_int* next;
  g_u64* gcnt;
  int n, b;
  bool early;
  __device__ __forceinline__ void operator()(int v, int a0, int deg, u64 label) const {
    const unsigned i = atomicAdd(cnt, 1u);
    if (ONE && i < (unsigned)TC1) {
      TeamQ::one(i) = v;
      return;
    }
    if (!ONE && i < (unsigned)TC) {
      TeamQ::v(b, (int)i) = v;
      TeamQ::a(b, (int)i) = a0;
      TeamQ::d(b, (int)i) = deg;
      TeamQ::l(b, (int)i) = label;
      return;
    }
    const u64 at = __hip_atomic_fetch_add(gcnt, 1ull, __ATOMIC_RELAXED, AG);
    if (at < (u64)n) __hip_atomic_store(&next[at], v, __ATOMIC_RELAXED, AG);
    else atomicOr(&sh->err, BLK_QUEUE);
    atomicAdd(&sh->tcount, 1u);
    if (early) sh->spill = 1;
  }
};

// The wake of round r in a team member: the vertices of its own bucket offer their labels (lane t of nw).
template <class Won>
__device__ __forceinline__ void team_wake(const BlockJob& j, g_cu64* wk, u64 mask, const Won& won) {
  const u64 self = *wk;
  const int v = (int)(self & mask);
  if (wg_load(&j.P[v]) > self) {  // a load first: a vertex reached earlier with a smaller label needs no atomic
    const u64 old = lab_min<AG>(&j.P[v], self);
    int a0, deg;
    row_of(j.row_ptr, v, &a0, &deg);
    won(v, a0, deg, old, self);
  }
}

// Entry cur[i] of the shared queue: its row, and its label plus `unit` (device-scope loads: the team's
// relaxed barrier invalidates nothing).
__device__ __forceinline__ void team_entry(const BlockJob& j, BlockShared& sh, g_cint* cur, unsigned i, u64 unit, int* a0,
                                           int* deg, u64* offer) {
  const int u = __hip_atomic_load(const_cast<g_int*>(&cur[i]), __ATOMIC_RELAXED, AG);
  *a0 = *deg = 0;
  *offer = 0;
  if ((unsigned)u < (unsigned)j.n) {
    *offer = lab_load<AG>(&j.P[u]) + unit;
    row_of(j.row_ptr, u, a0, deg);
  } else {
    atomicOr(&sh.err, ERR_QUEUE);
  }
}

// A step of one round (or tail sweep) of a team member: its bucket of round r wakes, and its share [e0, e1) of
// the frontier is relaxed.  first_only: the frontier is final, so a vertex is appended when it is reached
// first (its label is final when the round ends, and is read again in the next one), else whenever
// its label drops.  A sweep appends a vertex once (its stamp takes the tag).  All threads call; returns
// the queue's length.
template <bool SWEEP>
__device__ __forceinline__ unsigned team_step1(BlockShared& sh, g_cint* cur, g_int* nxt, unsigned e0, unsigned e1,
                                                         int r, int D, bool first_only, int tag, u64& examined) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const u64 unit = (u64)1 << (FIX + B), mask = ((u64)1 << B) - 1;
  g_u64* gcnt = &sh.ts->qcnt[sh.epoch % 3];
  const TeamAppend<true> app{&sh, &sh.cnt3[0], nxt, gcnt, n, 0, false};
  unsigned firsts = 0, ex = 0;
  const auto won = [&](int w, int a0, int deg, u64 old, u64 offer) {
    firsts += old == INF;
    if (SWEEP) {
      if (old > offer && __hip_atomic_exchange(&j.wake[w], tag, __ATOMIC_RELAXED, AG) != tag) app(w, a0, deg, offer);
    } else if (first_only ? old == INF : old > offer) {
      app(w, a0, deg, offer);
    }
  };
  const Relax<AG, false, decltype(won)> relax{j, e1 - e0 > FILTER_MIN, won}, heavy{j, true, won};
  if (!SWEEP && r <= D) {
    const int w1 = sh.woff[r + 1];
    for (int t = sh.woff[r] + (int)threadIdx.x; t < w1; t += BT) team_wake(j, j.wk + sh.tlo + t, mask, won);
  }
  for (unsigned c0 = e0; c0 < e1; c0 += BT) {  // BT rows at a time: the staging has room for what they reach
    const unsigned cn = e1 - c0 < (unsigned)BT ? e1 - c0 : (unsigned)BT;
    walk_rows(
        j, sh, 0, cn,
        [&](unsigned i, int* a0, int* deg, u64* offer) { team_entry(j, sh, cur, c0 + i, unit, a0, deg, offer); }, relax, ex);
    if (c0 + BT < e1) {
      __syncthreads();
      const unsigned c = sh.cnt3[0];
      if (c > (unsigned)TC1 / 2) {
        team_flush<true>(sh, n, nxt, gcnt, 0, c < (unsigned)TC1 ? c : (unsigned)TC1);
        if (threadIdx.x == 0) sh.cnt3[0] = 0;
      }
      __syncthreads();
    }
  }
  __syncthreads();
  if (sh.nh3[0]) {
    walk_heavy(j, sh, 0, heavy);
    __syncthreads();
  }
  examined += ex;
  firsts = (unsigned)wave_sum_u64(firsts);
  if (lane_id() == 0 && firsts) atomicAdd(&sh.sfirst, firsts);
  __syncthreads();
  return team_step_end<false, true>(sh, n, nxt, gcnt, 0, sh.cnt3[0]);
}

// Rounds per step.  A step of one round costs the team a barrier and the queue's way through device memory
// (about 6 us in all) beside its rounds' chains (about 3 us each); STEP_MAX rounds share them.  But a
// member alone relaxes what it reached in the step, so the frontier must not grow fast (a random
// graph's explosion would stay in few members and overflow their LDS, and reach most vertices by
// detours) and must fit their LDS: the rounds double while the frontier grows by less than half a step
// (plus STEP_SLACK entries) and a member's share stays below STEP_SHARE, and halve otherwise; shares of at
// most STEP_SMALL rows take up to STEP_MAX_SMALL rounds (1000^2 grid: 1.84 ms with 8, 1.58 with 16; the 256^3
// grid's larger shares drift apart in 16: 3.7 against 3.9 ms).
// The slack lets small frontiers through whose growth says little; two rounds from them may reach the slack times
// the square of the degree, so above STEP_DEGREE arcs per vertex it falls with that square (0 from 23 on).  With the
// whole slack the first waves of a dense graph went into the last round of a step from several members, each vertex
// queued by most of them: the queue overflowed and the launch engine ran the graph again (batches of eight
// Erdos-Renyi graphs, us: 1500 vertices of degree 50 623, and 178 now; 4000 of degree 300 577 and 327; geometric
// graphs up to degree 40 the same).
// A row of more than STEP_ROW arcs: one round per step.  The member that reaches such a vertex inside a step expands
// the row and what it reaches by itself (batches of eight R-MAT graphs, us, steps of several rounds and of one: scale
// 14 with 8 edges per vertex 1541 - 1619 and 1255 - 1286, scale 15 with 3 1142 - 1462 and 1097 - 1135; a 600 x 600 grid with a
// vertex of 3000 arcs 1420 and 1555, with steps of one round for rows of more than 256 a 200 x 200 grid with one of 1000
// 559 and 613).
// MIN_SHARE: a small frontier is left to fewer members, so that each has a connected patch of it (random
// geometric graph of 150,001 vertices: 0.65 / 0.60 / 0.58 ms at 32 / 16 / 8 rows).
constexpr int STEP_MAX = 8, STEP_MAX_SMALL = 16, STEP_BITS = 4;
static_assert(STEP_MAX <= 1 << STEP_BITS && STEP_MAX_SMALL <= 1 << STEP_BITS, "");
constexpr unsigned STEP_SMALL = 64;
constexpr unsigned STEP_SLACK = 8;
constexpr long long STEP_DEGREE = 8;
constexpr unsigned STEP_SHARE = 1024;
constexpr unsigned MIN_SHARE = 8;

// The offers a team member made in this step, one per slot in LDS: a patch of a mesh's frontier offers the
// same label to a vertex from up to three sides, and each would load that label and send an atomic
// (27 G/s over the GPU).  The vertex is known by its slot (its low bits, folded) and its high bits, which
// lie above the offer's distance from the step's first label: 2 B + 12 bits for steps of up to 16 rounds.  A
// slot keeps the smallest entry; an offer that finds its own vertex with one as good is left out (256^3 grid:
// 4.1 -> 3.7 ms, 32.5 million atomics for 16.8 million labels).
constexpr int SEEN = 4096;  // slots, beside the queues
static_assert(TEAM_Q_BYTES + 8 * SEEN <= BLOCK_LDS_BYTES, "");
struct SeenOffers {
  u64 base;
  int bits;  // of an offer's distance from base; 0: none is kept (labels too wide, or of any round)
  __device__ static u64& at(unsigned i) { return reinterpret_cast<u64*>(blk_dyn + TEAM_Q_BYTES)[i]; }
  __device__ static void clear() {
    for (int i = threadIdx.x; i < SEEN; i += BT) at((unsigned)i) = INF;
  }
  __device__ __forceinline__ bool operator()(int w, u64 offer) const {
    const u64 off = offer - base;
    // not kept: what lies further off (an entry left over from an earlier step may offer less than base), and the
    // furthest distance, which with 64 bits in all (B = 26) would make the highest vertices' entries an empty slot
    if (off >= ((u64)1 << bits) - 1) return false;
    const u64 mine = (u64)((unsigned)w >> 12) << bits | off;
    const u64 old = atomicMin(&at(((unsigned)w ^ (unsigned)w >> 12) & (SEEN - 1)), mine);
    return old <= mine && old >> bits == mine >> bits;
  }
};

// A step of several rounds r, r + 1, ... (or tail sweeps): the first relaxes the member's share [e0, e1)
// of the shared frontier, each later one what the member itself lowered in the round before (entries
// in LDS, with the label they were given); each wakes the member's own bucket of that round.  What the last
// round lowers goes to the shared queue.  All threads call; returns the queue's length.
//
// Several rounds per step are exact.  Claim: a vertex whose final label lies in round r + i gets it
// from some member in that member's own round i of the step or an earlier one.  A vertex whose own label is
// the final one wakes in that round in its owner; any other has a neighbour with a final label one
// round below, whose last lowering queued it with that label in a member that relaxes it one round later
// at the latest.  So after the step every label below r + rounds is final, as after that many single
// rounds.  Labels above their final value are passed on too and lowered again later, which costs
// work, never the result: whoever lowers a label queues the vertex (it may then be queued twice).
// The claim needs every entry to stay in LDS.  A member whose LDS is full before the last round (a
// spill) leaves entries to the next step, and the rounds go on as label correction until the queue is
// empty; offers stay below r + rounds all the same (an entry of the queue lies below r), so no
// vertex is given a label above its own one before its wake round.
template <bool SWEEP>
__device__ __forceinline__ unsigned team_steps(BlockShared& sh, g_cint* cur, g_int* nxt, unsigned e0, unsigned e1,
                                                         int r, int D, int rounds, u64& examined) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const u64 unit = (u64)1 << (FIX + B), mask = ((u64)1 << B) - 1;
  g_u64* gcnt = &sh.ts->qcnt[sh.epoch % 3];
  unsigned firsts = 0, ex = 0;
  int ci = 0;
  const SeenOffers seen{(u64)r << (FIX + B), !SWEEP && 2 * B + 12 <= 64 ? FIX + B + STEP_BITS : 0};
  bool filled = false;  // (cleared when the first round that filters begins)
#pragma unroll 1
  for (int k = 0; k < rounds; ++k) {
    const int ib = k & 1;  // the LDS buffer read; the other one is written
    const TeamAppend<false> app{&sh, &sh.cnt3[ci], nxt, gcnt, n, ib ^ 1, k + 1 < rounds};
    unsigned nin = e1 - e0;
    if (k) {
      nin = sh.cnt3[ci == 0 ? 2 : ci - 1];
      nin = nin < (unsigned)TC ? nin : (unsigned)TC;
    }
    const auto won = [&](int w, int a0, int deg, u64 old, u64 offer) {
      firsts += old == INF;
      if (old > offer) app(w, a0, deg, offer);
    };
    if (!filled && nin > FILTER_MIN) {
      SeenOffers::clear();
      __syncthreads();
      filled = true;
    }
    const Relax<AG, true, decltype(won), SeenOffers> relax{j, nin > FILTER_MIN, won, seen};
    if (!SWEEP && r + k <= D) {
      const int w1 = sh.woff[r + k + 1];
      for (int t = sh.woff[r + k] + (int)threadIdx.x; t < w1; t += BT) team_wake(j, j.wk + sh.tlo + t, mask, won);
    }
    walk_rows(
        j, sh, ci, nin,
        [&](unsigned i, int* a0, int* deg, u64* offer) {
          if (k) {
            *a0 = TeamQ::a(ib, (int)i);
            *deg = TeamQ::d(ib, (int)i);
            *offer = TeamQ::l(ib, (int)i) + unit;
          } else {
            team_entry(j, sh, cur, e0 + i, unit, a0, deg, offer);
          }
        },
        relax, ex);
    __syncthreads();
    if (sh.nh3[ci]) {
      walk_heavy(j, sh, ci, relax);
      __syncthreads();
    }
    if (k + 1 < rounds) {
      if (threadIdx.x == 0) {  // the counters of the round before, read by every thread: free for round k + 2
        const int old = ci == 0 ? 2 : ci - 1;
        sh.cnt3[old] = 0;
        sh.nh3[old] = 0;
      }
      ci = ci == 2 ? 0 : ci + 1;
    }
  }
  examined += ex;
  firsts = (unsigned)wave_sum_u64(firsts);
  if (lane_id() == 0 && firsts) atomicAdd(&sh.sfirst, firsts);
  __syncthreads();
  return team_step_end<false, false>(sh, n, nxt, gcnt, rounds & 1, sh.cnt3[ci]);
}

__device__ __forceinline__ unsigned step_slack(const BlockJob& j) {
  const long long most = STEP_DEGREE * j.n;
  const float x = j.nnz > most ? (float)most / (float)j.nnz : 1.0f;
  return (unsigned)((float)STEP_SLACK * x * x);
}

// most_rows: frontiers of as many take one round per step (0: all do).
__device__ __forceinline__ int next_rounds(int rounds, unsigned before, unsigned nf, bool spill, int K, unsigned most_rows,
                                           unsigned slack) {
  if (spill || nf >= most_rows) return 1;
  const int most = nf > STEP_SMALL * (unsigned)K ? STEP_MAX : STEP_MAX_SMALL;
  if (nf <= before + before / 2 + slack) return 2 * rounds < most ? 2 * rounds : most;
  return rounds > 1 ? rounds / 2 : 1;
}

// The member's share [e0, e1) of a frontier of nf entries.
__device__ __forceinline__ void team_share(unsigned nf, unsigned K, unsigned m, unsigned* e0, unsigned* e1) {
  const unsigned want = (nf + MIN_SHARE - 1) / MIN_SHARE, ks = want < K ? want : K;
  *e0 = m < ks ? (unsigned)((u64)nf * m / ks) : 0u;
  *e1 = m < ks ? (unsigned)((u64)nf * (m + 1) / ks) : 0u;
}

// The rounds of a team: the same rounds and tail as block_rounds, in steps of one or more rounds
// (team_step1, team_steps) with one barrier each.
__device__ __attribute__((noinline)) void team_rounds(BlockShared& sh) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  g_cint* __restrict__ rp = j.row_ptr;
  g_cint* __restrict__ col = j.col;
  g_ci64* __restrict__ shift = j.shift;
  g_u64* P = j.P;
  const int tid = threadIdx.x;
  const int K = sh.tK, m = sh.tm, lo = sh.tlo, hi = sh.thi;
  const u64 delta = sh.delta, n_active = sh.n_active;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const int D = (int)(delta >> FIX);
  const u64 unit = (u64)1 << (FIX + B);
  g_int* cur = j.q0;
  g_int* nxt = j.q1;
  unsigned nf = 0, e0, e1;
  u64 settled = 0, examined = 0;
  long long rounds = 0, sweeps = 0;
  if (tid < 3) sh.cnt3[tid] = sh.nh3[tid] = 0;
  int r = team_next_nonempty(sh, 0, D);
  int step = 1;        // rounds of the next step
  const unsigned slack = step_slack(j);
  const unsigned most_rows = sh.maxdeg > (unsigned)STEP_ROW ? 0 : STEP_SHARE * (unsigned)K;
  bool clean = true;   // no entry of the queue was left over by a spill
  bool tail = false;
  // at most D / 1 steps wake, and every step moves every queued label one round on
  for (long long steps = 0; steps <= (long long)D + n + 2; ++steps) {
    if (settled >= n_active && (clean || nf == 0)) break;
    if (nf == 0 && r > D) break;
    team_share(nf, (unsigned)K, (unsigned)m, &e0, &e1);
    const unsigned before = nf;
    if (step > 1) nf = team_steps<false>(sh, cur, nxt, e0, e1, r, D, step, examined);
    else nf = team_step1<false>(sh, cur, nxt, e0, e1, r, D, clean, 0, examined);
    if (sh.terr) break;
    settled += sh.tfirst;
    rounds += min(step, max(0, D + 1 - r));  // a step may reach past the last round
    if (sh.tspill) clean = false;
    g_int* t = cur;
    cur = nxt;
    nxt = t;
    r = r > D ? r : r + step;
    if (nf == 0) {
      clean = true;
      r = team_next_nonempty(sh, r, D);
    }
    step = next_rounds(step, before, nf, sh.tspill, K, most_rows, slack);
    if (tail_next(j, n_active, settled, nf, D - r, clean)) {
      tail = true;
      break;
    }
  }
  if (tail) {
    // seed over the member's slice (see block_rounds): every unreached vertex takes the best of its own
    // label and what its reached neighbours offer.  With a clean queue their offers are the only ones
    // pending (every other neighbour of the frontier is final), else the frontier stays queued too.
    g_u64* gcnt = &sh.ts->qcnt[sh.epoch % 3];
    const TeamAppend<true> app{&sh, &sh.cnt3[0], nxt, gcnt, n, 0, false};
    team_acquire();
    const auto room = [&]() {  // after each pass of at most BT appends
      __syncthreads();
      const unsigned c = sh.cnt3[0];
      if (c > (unsigned)(TC1 - BT)) {
        team_flush<true>(sh, n, nxt, gcnt, 0, c < (unsigned)TC1 ? c : (unsigned)TC1);
        if (tid == 0) sh.cnt3[0] = 0;
      }
      __syncthreads();
    };
    for (int v0 = lo; v0 < hi; v0 += BT) {  // the same passes in every thread
      const int v = v0 + tid;
      const int a0 = v < hi ? rp[v] : 0, a1 = v < hi ? rp[v + 1] : 0;
      if (v < hi) j.wake[v] = -1;  // the stamp of the first sweep
      if (a1 > a0 && wg_load(&P[v]) == INF) {
        u64 best = ((delta - (u64)shift[v]) << B) | (u64)v;
        for (int a = a0; a < a1; ++a) {
          const int u = col[a];
          if ((unsigned)u >= (unsigned)n) {
            atomicOr(&sh.err, ERR_BAD_COL);
            break;
          }
          const u64 pu = wg_load(&P[u]);
          if (pu != INF && pu + unit < best) best = pu + unit;
        }
        examined += (u64)(a1 - a0);
        lab_store<AG>(&P[v], best);
        app(v, 0, 0, 0);
      }
      room();
    }
    if (!clean) {
      team_share(nf, (unsigned)K, (unsigned)m, &e0, &e1);
      for (unsigned i0 = e0; i0 < e1; i0 += BT) {
        const unsigned i = i0 + (unsigned)tid;
        if (i < e1) app(__hip_atomic_load(&cur[i], __ATOMIC_RELAXED, AG), 0, 0, 0);
        room();
      }
    }
    nf = team_step_end<true, true>(sh, n, nxt, gcnt, 0, sh.cnt3[0]);
    step = 1;
    for (int k = 1; nf && !sh.terr && k <= n + 1; ++k) {
      g_int* t = cur;
      cur = nxt;
      nxt = t;
      team_share(nf, (unsigned)K, (unsigned)m, &e0, &e1);
      const unsigned before = nf;
      if (step > 1) nf = team_steps<true>(sh, cur, nxt, e0, e1, 0, 0, step, examined);
      else nf = team_step1<true>(sh, cur, nxt, e0, e1, 0, 0, false, -(k + 1), examined);
      sweeps += step;
      step = next_rounds(step, before, nf, sh.tspill, K, most_rows, slack);
    }
    settled = n_active;
  }
  __syncthreads();
  examined = block_sum64(examined, sh);
  if (tid == 0) {
    sh.settled = settled;
    sh.examined = examined;
    sh.rounds = rounds;
    sh.sweeps = sweeps;
  }
  __syncthreads();
}

// Centres and cut of the member's slice, summed in the team's record; after a last barrier,
// member 0 writes the graph's result.
__device__ __attribute__((noinline)) void team_output(BlockShared& sh, BlockOut* out) {
  const BlockJob j = job_of(sh);
  const int n = j.n;
  g_sync* ts = sh.ts;
  const int tid = threadIdx.x;
  const int B = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 1;
  const u64 mask = ((u64)1 << B) - 1;
  const unsigned e0 = sh.err | (sh.settled < sh.n_active ? ERR_WATCHDOG : 0u);
  u64 cut2 = 0, pieces = 0;
  if (tid == 0) sh.nh3[0] = sh.er3[0] = 0;
  team_acquire();
  if (!e0) {
    output_slice(j, sh, sh.tlo, sh.thi, mask, &cut2, &pieces);
  }
  cut2 = block_sum64(cut2, sh);
  pieces = block_sum64(pieces, sh);
  __syncthreads();
  if (tid == 0) {
    if (cut2) __hip_atomic_fetch_add(&ts->cut, cut2, __ATOMIC_RELAXED, AG);
    if (pieces) __hip_atomic_fetch_add(&ts->pieces, pieces, __ATOMIC_RELAXED, AG);
    if (sh.examined) __hip_atomic_fetch_add(&ts->examined, sh.examined, __ATOMIC_RELAXED, AG);
    if (e0 | sh.err) __hip_atomic_fetch_or(&ts->err, e0 | sh.err, __ATOMIC_RELAXED, AG);
  }
  team_barrier<true>(sh);
  if (tid == 0 && sh.tm == 0) {
    out->err = __hip_atomic_load(&ts->err, __ATOMIC_RELAXED, AG) | sh.err;
    out->cut_arcs = __hip_atomic_load(&ts->cut, __ATOMIC_RELAXED, AG);
    out->pieces = __hip_atomic_load(&ts->pieces, __ATOMIC_RELAXED, AG);
    out->examined = __hip_atomic_load(&ts->examined, __ATOMIC_RELAXED, AG);
    out->delta = sh.delta;
    out->n_active = sh.n_active;
    out->rounds = sh.rounds;
    out->sweeps = sh.sweeps;
  }
}

// Member m of the graph's team: the slice of 64-aligned vertices it owns, then the three phases.
__device__ void team_graph(BlockShared& sh, BlockOut* out, int m) {
  const int n = sh.j.n, K = sh.j.team;
  const int chunk = (int)((((long long)n + K - 1) / K + 63) & ~63ll);
  if (threadIdx.x == 0) {
    sh.ts = sh.j.sync;
    sh.tK = K;
    sh.tm = m;
    sh.tlo = (int)min((long long)n, (long long)m * chunk);
    sh.thi = (int)min((long long)n, (long long)sh.tlo + chunk);
    sh.epoch = 0;
    sh.tcount = 0;
  }
  __syncthreads();
  team_prepare(sh);
  if (sh.err) {
    if (threadIdx.x == 0 && m == 0) {
      out->err = sh.err;
      out->delta = sh.delta;
    }
    return;
  }
  team_rounds(sh);
  team_output(sh, out);
}

}  // namespace

// (BT, 4): four waves per SIMD, one workgroup per CU, up to 128 VGPRs (at 64, the bound that two
// workgroups per CU would need, the team and round loops spilled to scratch).
// With a job list each workgroup takes the next job of `order` (a graph, or one member of a
// graph's team) from the shared counter until none is left; without one, block b runs member b of
// the single graph.
// A team's members are consecutive jobs: a member that starts early waits at the team's first
// barrier for workgroups that finish their current job, which every resident workgroup does, so
// the team size must not exceed the resident workgroups (the host keeps it within the grid).
__global__ __launch_bounds__(BT, 4) void k_block_decompose(const BlockJob* __restrict__ jobs,
                                                           const TeamJob* __restrict__ order, int njobs,
                                                           unsigned* next_job, BlockOut* outs, BlockJob single) {
  __shared__ BlockShared sh;
  for (;;) {
    int g = 0, m = (int)blockIdx.x;
    if (order) {
      if (threadIdx.x == 0) sh.job = (int)atomicAdd(next_job, 1u);
      __syncthreads();
      const int k = sh.job;
      __syncthreads();
      if (k >= njobs) return;
      g = order[k].g;
      m = order[k].m;
    }
    if (threadIdx.x == 0) sh.j = order ? jobs[g] : single;
    __syncthreads();
    const u64 t0 = wall_clock64();
    if (sh.j.team > 1) team_graph(sh, &outs[g], m);
    else if (fix_lds_bytes(sh.j.n, sh.j.nnz) <= BLOCK_LDS_BYTES) block_graph_fix(sh, &outs[g]);
    else block_graph(sh, &outs[g]);
    if (threadIdx.x == 0 && m == 0) {
      outs[g].t_begin = t0;
      outs[g].t_end = wall_clock64();
    }
    if (!order) {
      // one graph: member 0 announces the result once every write of its workgroup (centres,
      // labels, the result record) has completed; the other members' writes completed before
      // they arrived at the team's last barrier
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (threadIdx.x == 0 && m == 0) {
        __threadfence_system();
        __hip_atomic_store(&outs[0].ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
      return;
    }
    __syncthreads();
  }
}

// Per-graph job descriptors of a batch in one offset CSR (graph g's rows at row_ptr[vo[g] + g]);
// team[2 g] = graph g's team size, team[2 g + 1] its TeamSync.
__global__ void k_block_jobs(int G, long long N, const long long* vo, const long long* ao, const int* row_ptr,
                             const int* col, const long long* shift, int* centre, u64* P, int* wq, int tail_den,
                             const int* team, TeamSync* sync, BlockJob* jobs) {
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < G; g += gridDim.x * blockDim.x) {
    BlockJob j;
    const long long v0 = vo[g];
    j.n = (int)(vo[g + 1] - v0);
    j.nnz = ao[g + 1] - ao[g];
    j.row_ptr = (g_cint*)(row_ptr + v0 + g);
    j.col = (g_cint*)(col + ao[g]);
    j.shift = (g_ci64*)(shift + v0);
    j.centre = (g_int*)(centre + v0);
    j.P = (g_u64*)(P + v0);
    j.wk = (g_u64*)wq + v0;
    j.wake = (g_int*)(j.wk);
    j.q0 = (g_int*)wq + 2 * N + v0;
    j.q1 = (g_int*)wq + 3 * N + v0;
    j.tail_den = tail_den;
    j.team = team ? team[2 * g] : 1;
    j.sync = j.team > 1 ? (g_sync*)(sync + team[2 * g + 1]) : nullptr;
    j.deg_cap = 0;
    jobs[g] = j;
  }
}

}  // namespace ldd
