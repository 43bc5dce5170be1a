// The workgroup-owned engine (one workgroup, or a team of a few workgroups, runs every round of
// one graph): job and result records and the kernels.
#pragma once
#include "ldd_device.h"

namespace ldd {

// wake buckets a workgroup sorts in LDS: graphs whose shifts span this many units of distance
// or more (floor(Delta / 2^20) >= BLOCK_WCAP) are left to the multi-block engine
constexpr int BLOCK_WCAP = 4096;

// LDS of the workgroup engine beside its control record (one workgroup per CU is resident: its
// registers allow no more).  A graph run alone whose labels and CSR fit (8 B per vertex,
// 4 B per row offset and per arc) is decomposed by a label-correcting iteration in LDS (block_graph_fix),
// its labels copied to the graph's label array at the end.  The rounds of other graphs take
// CLAIM_Q_BYTES alone on at most CLAIM_N vertices (two bits per vertex, the table of
// a round's offers and the frontier's entries), ALONE_Q_BYTES above; in a team TEAM_Q_BYTES.
constexpr int BLOCK_LDS_BYTES = 136 * 1024;
constexpr int CLAIM_N = 1 << 18;
constexpr int CLAIM_Q_BYTES = CLAIM_N / 4 + 8 * 4096 + 20 * 2048;
constexpr int ALONE_Q_BYTES = 24 * 1024;
constexpr int TEAM_Q_BYTES = 80 * 1024;
static_assert(CLAIM_Q_BYTES <= BLOCK_LDS_BYTES && ALONE_Q_BYTES <= BLOCK_LDS_BYTES && TEAM_Q_BYTES <= BLOCK_LDS_BYTES, "");
__device__ constexpr long long fix_lds_bytes(long long n, long long nnz) { return 12 * n + 4 * nnz + 4; }

// error bits of a workgroup job beyond ERR_*: the labels would not fit 64 bits; the shift range
// needs more wake buckets than the workgroup sorts; a team was asked to refuse a graph with a
// vertex of more than deg_cap arcs, and it has one; a team's queue had more entries than vertices
// (repeated ones: see team_steps).  The last three leave the graph to the multi-block engine.
enum : unsigned { BLK_OVERFLOW = 64u, BLK_WIDE = 128u, BLK_SKEW = 256u, BLK_QUEUE = 512u };

// A graph too large for one workgroup runs on a team of K workgroups (all resident at once) that
// meet at a barrier in device memory once per step of one or more rounds.  Per team, in device memory, zeroed before
// the launch: the barrier's words (below), the OR of the members' error bits, the append counters
// of the shared frontier queue, the preparation's and the output's sums, the largest degree (0: no row is
// long), and the OR of the members' non-empty wake buckets.  Its size does not
// depend on K.  A batch gives a team at most TEAM_MAX workgroups; one graph alone may take every
// resident workgroup.
constexpr int TEAM_MAX = 16;

constexpr int TEAM_GROUP = 16;   // barrier arrivals are counted per group of 16 members, then per group
constexpr int TEAM_GROUPS = 32;  // a team has at most TEAM_GROUP * TEAM_GROUPS = 512 members

struct TeamLine {
  alignas(128) u64 v;
};

// Barrier k of a team uses the words of slot k % 3; member 0 clears slot (k + 1) % 3 before it
// arrives at barrier k.  An arrival adds (1 << 44) | (spill ? 1 << 38 : 0) | (error ? 1 << 32 : 0) |
// (its appends) to its group's word, the group's last arrival adds the group's sums (one arrival, at
// most one error and spill) to the team's word, and the team's last arrival publishes the step's
// queue length with the barrier's number in gen.
struct TeamSync {
  TeamLine gw[3][TEAM_GROUPS];  // per step slot: the groups' arrivals, errors, spills and appends
  TeamLine tw[3];               // per step slot: the team's (arrivals are groups)
  alignas(128) u64 gen;         // (spill << 31 | queue length, or 0xffffffff after an error) << 32 | barriers passed
  alignas(128) unsigned err;    // OR of every member's error bits
  alignas(128) u64 qcnt[3];     // per step slot: the shared queue's reservations
  alignas(128) u64 first[3];    // per step slot: vertices reached for the first time
  alignas(128) u64 delta;
  alignas(128) u64 active;
  alignas(128) u64 cut, pieces, examined;
  alignas(128) u64 maxdeg;
  alignas(128) u64 nz[BLOCK_WCAP / 64];
};

// Pointers the device code knows to be global memory.  Through plain pointers every access of the engine
// compiled to a flat one (the pointers come out of a record in memory), which also counts as an LDS
// access: every wait for LDS data then waited for the loads and atomics in flight too.
#if defined(__HIP_DEVICE_COMPILE__)
#define LDD_GLOBAL __attribute__((address_space(1)))
#else
#define LDD_GLOBAL
#endif
typedef LDD_GLOBAL int g_int;
typedef LDD_GLOBAL u64 g_u64;
typedef const LDD_GLOBAL int g_cint;
typedef const LDD_GLOBAL u64 g_cu64;
typedef const LDD_GLOBAL long long g_ci64;
typedef LDD_GLOBAL TeamSync g_sync;

struct BlockJob {
  int n;
  long long nnz;
  g_cint* row_ptr;       // [n + 1]
  g_cint* col;           // [nnz], local ids
  g_ci64* shift;
  g_int* centre;         // OUT [n]
  g_u64* P;              // workspace [n]: labels
  g_u64* wk;             // workspace [n]: own labels of the vertices with arcs, by wake round
  g_int* wake;           // the first 4n bytes of wk: the tail's sweep stamps (once no wake is left)
  g_int* q0;             // workspace [n]: frontier queues
  g_int* q1;
  int tail_den;          // label-correcting tail once unreached * tail_den <= vertices with arcs (0: never)
  int team;              // workgroups on this graph (1: alone)
  g_sync* sync;          // team > 1: the team's barrier and counters
  int deg_cap;           // team > 1: refuse (BLK_SKEW) a graph with a vertex of more arcs (0: never)
};

struct BlockOut {
  unsigned err;
  u64 cut_arcs;   // arcs whose ends have different centres (twice the cut)
  u64 pieces;
  u64 delta;
  u64 n_active;
  long long rounds;
  long long sweeps;  // label-correcting sweeps of the tail (0: the rounds ran to the end)
  u64 examined;   // arcs read by the rounds, the seed and the sweeps
  u64 t_begin;    // device wall clock (constant-rate counter) when the workgroup took the graph
  u64 t_end;      // ... and when it finished it
  unsigned ready; // one graph without a job list: set last, at system scope (the host waits for it)
};

// One job of the kernel's list: graph g, member m of its team.
struct TeamJob {
  int g, m;
};

// order != NULL: workgroups take jobs (order[k], njobs of them) from *next_job; order == NULL: one
// job per workgroup, member blockIdx.x of the graph `single`.
__global__ void k_block_decompose(const BlockJob* jobs, const TeamJob* order, int njobs, unsigned* next_job, BlockOut* outs,
                                  BlockJob single);
__global__ void k_block_jobs(int G, long long N, const long long* vo, const long long* ao, const int* row_ptr,
                             const int* col, const long long* shift, int* centre, u64* P, int* wq, int tail_den,
                             const int* team, TeamSync* sync, BlockJob* jobs);

}  // namespace ldd
