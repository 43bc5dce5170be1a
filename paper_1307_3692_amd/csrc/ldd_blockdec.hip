// Block decomposition in the sense of Linial and Saks (Sec. 2): the edges are split into levels
// by running the (beta, O(log n / beta)) decomposition again and again on the edges not placed
// yet, beta = 1/2 by default.  Level L holds the edges whose endpoints fall into one piece of the
// L-th decomposition; the cut edges go on to level L + 1.  Each decomposition cuts an edge with
// probability below beta (Cor. 4.5), so the remaining edges shrink geometrically and O(log m)
// levels place them all; inside a level, every connected set of that level's edges lies in one
// piece, whose vertices are within O(log n / beta) of its centre (Lemma 4.2).
//
// Each level: shifts drawn on the device (the library's sampler, seed + level), one
// decomposition of the remaining graph (the single-graph engines), then one pass over the
// remaining arcs that assigns the level to arcs inside a piece and compacts the others into the
// next level's CSR (row counts, an exclusive scan, a scatter that keeps each arc's original id).
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <vector>

#include "../../include/ldd.h"
#include "ldd_device.h"
#include "ldd_internal.h"

using namespace ldd;

namespace {

#define BD_TRY(expr)                                                                            \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess) {                                                                     \
      ldd_set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
      status = LDD_ERR_HIP;                                                                     \
      goto done;                                                                                \
    }                                                                                           \
  } while (0)

// Rows are shared out by their length: a lane walks its row alone up to LANE_ARCS arcs, the lanes of a wave
// walk longer ones of its 64 rows together, one after another, and the block those of more than WAVE_ARCS.
// With every row on one lane the largest row of an R-MAT graph (thousands of arcs, a chain of
// dependent loads each) was a level's whole time (R-MAT 17, 12 edges per vertex: 5.86 ms, and 0.94 now).
constexpr int LV_T = 256;
constexpr int LANE_ARCS = 32;
constexpr int WAVE_ARCS = 1024;

struct LevelGraph {
  int n;
  const int* rp;
  const int* col;
  const int* orig;  // original arc ids; nullptr: the positions themselves (the first level)
  const int* centre;
};

// Arcs a0 + first, + stride, ... of a row whose centre is cu: on(arc, kept) for each, four columns and
// four centres in flight; every lane of the group calls on the same number of times, with arc < 0 past the end.
template <class On>
__device__ __forceinline__ void level_row(const LevelGraph& g, int a0, int a1, int cu, int first, int stride, const On& on) {
  const unsigned end = (unsigned)a1;  // positions past the end may exceed an int
  for (unsigned b = (unsigned)a0; b < end; b += 4u * stride) {
    int v[4], c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned a = b + (unsigned)(k * stride + first);
      v[k] = a < end ? g.col[a] : -1;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = v[k] >= 0 ? g.centre[v[k]] : cu;
#pragma unroll
    for (int k = 0; k < 4; ++k) on(v[k] >= 0 ? (int)(b + (unsigned)(k * stride + first)) : -1, v[k], c[k] != cu);
  }
}

// The rows of one block of LV_T consecutive vertices by length: lane(u, a0, a1, cu), wave(...) and block(...).
template <class Lane, class Wave, class Block>
__device__ __forceinline__ void level_rows(const LevelGraph& g, long long base, const Lane& lane_row, const Wave& wave_row,
                                           const Block& block_row) {
  __shared__ int heavy[LV_T];
  __shared__ int nheavy;
  const int tid = threadIdx.x;
  if (tid == 0) nheavy = 0;
  __syncthreads();
  const long long u = base + tid;
  int a0 = 0, a1 = 0, cu = 0;
  if (u < g.n) {
    a0 = g.rp[u];
    a1 = g.rp[u + 1];
    cu = g.centre[u];
  }
  const int deg = a1 - a0;
  if (u < g.n && deg <= LANE_ARCS) lane_row((int)u, a0, a1, cu);
  for (unsigned long long m = __ballot(deg > LANE_ARCS && deg <= WAVE_ARCS); m; m &= m - 1) {
    const int src = __ffsll((long long)m) - 1;
    wave_row((int)__builtin_amdgcn_readlane((int)u, src), __builtin_amdgcn_readlane(a0, src),
             __builtin_amdgcn_readlane(a1, src), __builtin_amdgcn_readlane(cu, src));
  }
  if (deg > WAVE_ARCS) heavy[atomicAdd(&nheavy, 1)] = tid;
  __syncthreads();
  const int nh = nheavy;
  for (int i = 0; i < nh; ++i) {
    const int h = (int)base + heavy[i];
    block_row(h, g.rp[h], g.rp[h + 1], g.centre[h]);
  }
  __syncthreads();  // the list is read
}

// Arcs of row u whose ends share a centre take the level; the others are counted for the next
// level's row u.
__global__ __launch_bounds__(LV_T) void k_level_mark(LevelGraph g, int level, int* __restrict__ arc_level,
                                                     int* __restrict__ keep_cnt, unsigned long long* placed) {
  __shared__ int kept;
  __shared__ unsigned long long total;
  const unsigned lane = threadIdx.x % WAVE;
  unsigned long long mine = 0;
  if (threadIdx.x == 0) {
    kept = 0;
    total = 0;
  }
  const long long stride = (long long)gridDim.x * LV_T;
  for (long long base = (long long)blockIdx.x * LV_T; base < g.n; base += stride) {
    int keep = 0;
    auto on = [&](int a, int, bool other) {
      if (a >= 0) {
        if (!other) arc_level[g.orig ? g.orig[a] : a] = level;
        mine += !other;
        keep += other;
      }
    };
    level_rows(
        g, base,
        [&](int u, int a0, int a1, int cu) {
          keep = 0;
          level_row(g, a0, a1, cu, 0, 1, on);
          keep_cnt[u] = keep;
        },
        [&](int u, int a0, int a1, int cu) {
          keep = 0;
          level_row(g, a0, a1, cu, (int)lane, WAVE, on);
          const unsigned k = (unsigned)wave_sum_u64((u64)keep);
          if (lane == 0) keep_cnt[u] = (int)k;
        },
        [&](int u, int a0, int a1, int cu) {
          keep = 0;
          level_row(g, a0, a1, cu, (int)threadIdx.x, LV_T, on);
          const unsigned k = (unsigned)wave_sum_u64((u64)keep);
          if (lane == 0 && k) atomicAdd(&kept, (int)k);
          __syncthreads();
          if (threadIdx.x == 0) {
            keep_cnt[u] = kept;
            kept = 0;
          }
          __syncthreads();
        });
  }
  mine = wave_sum_u64(mine);
  if (lane == 0 && mine) atomicAdd(&total, mine);
  __syncthreads();
  if (threadIdx.x == 0 && total) atomicAdd(placed, total);
}

// The kept arcs of row u, in order, to the next level's CSR (new_rp from the exclusive scan); clears the
// next level's count of placed arcs.
__global__ __launch_bounds__(LV_T) void k_level_compact(LevelGraph g, const int* __restrict__ new_rp,
                                                        int* __restrict__ new_col, int* __restrict__ new_orig,
                                                        unsigned long long* next_placed) {
  constexpr int NWL = LV_T / WAVE;
  __shared__ int wcnt[2][NWL];
  const unsigned lane = threadIdx.x % WAVE, wid = threadIdx.x / WAVE;
  if (blockIdx.x == 0 && threadIdx.x == 0) *next_placed = 0;
  const long long stride = (long long)gridDim.x * LV_T;
  for (long long base = (long long)blockIdx.x * LV_T; base < g.n; base += stride) {
    int o = 0, par = 0;
    auto put = [&](int at, int a, int v) {
      new_col[at] = v;
      new_orig[at] = g.orig ? g.orig[a] : a;
    };
    level_rows(
        g, base,
        [&](int u, int a0, int a1, int cu) {
          o = new_rp[u];
          level_row(g, a0, a1, cu, 0, 1, [&](int a, int v, bool other) {
            if (a >= 0 && other) put(o++, a, v);
          });
        },
        [&](int u, int a0, int a1, int cu) {
          o = new_rp[u];
          level_row(g, a0, a1, cu, (int)lane, WAVE, [&](int a, int v, bool other) {
            const bool k = a >= 0 && other;
            const u64 m = __ballot(k);
            if (k) put(o + (int)rank_below(m), a, v);
            o += (int)__popcll(m);
          });
        },
        [&](int u, int a0, int a1, int cu) {
          o = new_rp[u];
          level_row(g, a0, a1, cu, (int)threadIdx.x, LV_T, [&](int a, int v, bool other) {
            const bool k = a >= 0 && other;
            const u64 m = __ballot(k);
            if (lane == 0) wcnt[par][wid] = (int)__popcll(m);
            __syncthreads();  // counts alternate: a wave may be one call ahead of another's reads
            int at = o, all = 0;
#pragma unroll
            for (int w = 0; w < NWL; ++w) {
              const int x = wcnt[par][w];
              if (w < (int)wid) at += x;
              all += x;
            }
            if (k) put(at + (int)rank_below(m), a, v);
            o += all;
            par ^= 1;
          });
        });
  }
}

__global__ void k_fill_i32(int* p, long long count, int value) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = value;
}

int grid_of(long long items, int threads, int cap) {
  long long g = (items + threads - 1) / threads;
  return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

extern "C" ldd_status ldd_block_decompose(const ldd_csr* g, double beta, uint64_t seed, int32_t max_levels,
                                          int32_t* arc_level, int32_t* levels, int64_t* level_edges,
                                          const ldd_options* opt, void* hip_stream) {
  if (!g || g->n < 0 || g->nnz < 0 || g->nnz >= (1ll << 31) || max_levels < 1 || !levels ||
      (g->n > 0 && !g->row_ptr) || (g->nnz > 0 && (!g->col_idx || !arc_level))) {
    ldd_set_error("ldd_block_decompose: bad graph, output or max_levels");
    return LDD_ERR_INVALID_ARG;
  }
  if (beta == 0.0) beta = 0.5;
  if (!(beta > 0.0 && beta < 1.0)) {
    ldd_set_error("ldd_block_decompose: beta must lie in (0, 1)");
    return LDD_ERR_INVALID_ARG;
  }
  const int n = g->n;
  const long long nnz = g->nnz;
  hipStream_t st = (hipStream_t)hip_stream;
  ldd_status status = LDD_OK;
  unsigned char* base = nullptr;
  *levels = 0;
  if (n == 0 || nnz == 0) return LDD_OK;  // no edge to place: zero levels
  {
    // one allocation for the call (an allocation and its release cost 20 to 40 us, and there are twelve parts)
    size_t tmp_bytes = 0, bytes = 0;
    BD_TRY(hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_bytes, (int*)nullptr, (int*)nullptr, n + 1, st));
    auto part = [&](size_t want) {
      const size_t at = bytes;
      bytes = (bytes + want + 255) & ~(size_t)255;
      return at;
    };
    size_t off[6];  // two generations of the remaining graph: row offsets, columns, original arc ids
    for (int i = 0; i < 6; ++i) off[i] = part((i % 3 ? (size_t)nnz : (size_t)n + 1) * 4);
    const size_t o_shifts = part((size_t)n * 8), o_centre = part((size_t)n * 4), o_cnt = part(((size_t)n + 1) * 4),
                 o_placed = part(16), o_tmp = part(tmp_bytes);
    BD_TRY(hipMalloc(&base, bytes));
    int* buf[6];
    for (int i = 0; i < 6; ++i) buf[i] = (int*)(base + off[i]);
    long long* const shifts = (long long*)(base + o_shifts);
    int* const centre = (int*)(base + o_centre);
    int* const cnt = (int*)(base + o_cnt);
    unsigned long long* const placed = (unsigned long long*)(base + o_placed);  // arcs placed, by generation
    void* const tmp = base + o_tmp;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_of(nnz, 256, 4096)), dim3(256), 0, st, arc_level, nnz, -1);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, (int*)placed, 4ll, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, cnt + n, 1ll, 0);  // stays 0
    // the level's graph: the input first, then the compacted generations in turn
    const int* rp = g->row_ptr;
    const int* col = g->col_idx;
    const int* orig = nullptr;
    long long remaining = nnz;
    int gen = 0;
    ldd_options o{};
    if (opt) o = *opt;
    for (int level = 0; level < max_levels && remaining > 0; ++level) {
      ldd_status s = ldd_make_shifts_device(n, beta, seed + (uint64_t)level, (int64_t*)shifts, st);
      if (s == LDD_OK) {
        ldd_csr lg{n, remaining, rp, col};
        s = ldd_decompose(&lg, (const int64_t*)shifts, beta, centre, nullptr, &o, nullptr, st);
      }
      if (s != LDD_OK) {
        status = s;
        goto done;
      }
      const LevelGraph lv{n, rp, col, orig, centre};
      const int grid = grid_of(n, LV_T, 1024);
      hipLaunchKernelGGL(k_level_mark, dim3(grid), dim3(LV_T), 0, st, lv, level, arc_level, cnt, placed + gen);
      int* nrp = buf[gen ? 0 : 3];
      int* ncol = buf[gen ? 1 : 4];
      int* norig = buf[gen ? 2 : 5];
      BD_TRY(hipcub::DeviceScan::ExclusiveSum(tmp, tmp_bytes, cnt, nrp, n + 1, st));
      hipLaunchKernelGGL(k_level_compact, dim3(grid), dim3(LV_T), 0, st, lv, (const int*)nrp, ncol, norig,
                         placed + (gen ^ 1));
      BD_TRY(hipGetLastError());
      unsigned long long placed_h = 0;
      BD_TRY(hipMemcpyAsync(&placed_h, placed + gen, 8, hipMemcpyDeviceToHost, st));
      BD_TRY(hipStreamSynchronize(st));
      if (level_edges) level_edges[level] = (int64_t)(placed_h / 2);
      remaining -= (long long)placed_h;
      *levels = level + 1;
      rp = nrp;
      col = ncol;
      orig = norig;
      gen ^= 1;
    }
    if (remaining > 0) {
      ldd_set_error("%lld arcs not placed after %d levels (their level stays -1)", remaining, max_levels);
      status = LDD_ERR_RETRIES;
    }
  }
done:
  (void)hipFree(base);
  return status;
}
