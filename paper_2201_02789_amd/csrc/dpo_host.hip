// Host driver and C ABI of the nested-parallel BFS / SSSP library.
//
// Who runs what:
//   dpo_bfs           start kernel; then narrow levels in one workgroup (the
//                     narrow kernel runs as many as follow each other) and wide
//                     ones as a level step or a bottom-up level, as the narrow
//                     kernel's verdict says, which the host polls in pinned
//                     memory (run_narrow_and_wide)
//   dpo_bfs_noalloc   the same, the verdict read from a copy of the state
//   dpo_sssp          small graphs: the solo kernel alone; sparse graphs up to
//                     NEAR_VERTICES: the near-far kernel alone, unless a level
//                     outgrows it; others: start kernel and replays
//   batches, engines  init and admit kernels, the symmetry check (BFS by
//                     found bytes), replays
//   counters, phase timing, the flat and the one-grid-per-parent form: replays
// A replay is a HIP graph of K captured level steps and the advance kernel,
// which writes the level and the done flag to pinned memory.  The kernels read
// their level, frontier and counters from the workspace, so one instantiated
// graph serves every call with the same arguments; graphs are cached by their
// exact kernel arguments.
#include <hip/hip_runtime.h>
#include <sys/random.h>

#include <algorithm>
#include <chrono>
#include <deque>
#include <map>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "dpo.h"
#include "dpo_internal.h"
#include "dpo_pair.h"

namespace dpo {
namespace {

constexpr int kDefaultSteps = 16;
// A batch of dense graphs is done in one or two replays of so many steps; one of
// many levels gets two replays at a time from the third on, and a batch of sparse
// graphs, which mostly is one, kDefaultSteps in a replay (8 road-like graphs, some
// 200 levels: 3,130 us in replays of 8, 3,050 two at a time, 2,865 in replays of 16).
constexpr int kBatchSteps = 8;
constexpr int kMaxCachedGraphs = 64;

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
  size_t state, queries, qlist, qmap, grp_packed, grp_done, front0, front1, visit, dist2, rec, rec_q,
      rec_slot, ser, desc, stats, sercnt, total;
  int32_t ngroups_cap, desc_cap, fcap;
};

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t round32(int64_t x) { return (x + 31) & ~(int64_t)31; }

// Byte offset of the found bytes in the visit region (BFS: after the two
// bitmaps and the per-XCD copies)
size_t found_offset(int64_t slots) { return align_up((size_t)(2 + NHINT) * cdiv(slots, 32) * 4); }

int gran_of(const dpo_options& o) {
  if (o.mode == DPO_MODE_FLAT) return AGG_FLAT;
  switch (o.agg) {
    case DPO_AGG_NONE: return AGG_NONE;
    case DPO_AGG_WAVE: return AGG_WAVE;
    case DPO_AGG_BLOCK: return AGG_BLOCK;
    case DPO_AGG_MULTIBLOCK: return AGG_MULTI;
    case DPO_AGG_GRID: return AGG_MULTI;  // one group holding every virtual block
    default: return -1;
  }
}

// Blocks per multi-block group: agg_blocks, or every virtual block of the level
// for grid granularity.
int64_t group_blocks(const dpo_options& o, int64_t slots) {
  return o.agg == DPO_AGG_GRID ? std::max<int64_t>(cdiv(slots, PB), 1) : o.agg_blocks;
}


// Workspace for `slots` output slots (frontier entries) and `nq` queries.
Layout layout_for(int64_t slots, int32_t nq, const dpo_options& o) {
  Layout L{};
  const int gran = gran_of(o);
  const int64_t nvb = cdiv(slots, PB);
  const int64_t k = (gran == AGG_MULTI) ? group_blocks(o, slots) : 1;
  L.ngroups_cap = (gran == AGG_MULTI) ? (int32_t)cdiv(nvb, k) : 1;
  // descriptors per queue: virtual block vb publishes to queue vb % NQD
  // (multi-block group g to queue g % NQD)
  // an aggregation threshold lets every parent of a wave / block launch alone
  const bool solo = o.agg_threshold > 0 && (gran == AGG_WAVE || gran == AGG_BLOCK);
  switch (solo ? AGG_NONE : gran) {
    case AGG_NONE: L.desc_cap = (int32_t)(PB * cdiv(nvb, NQD)); break;
    case AGG_WAVE: L.desc_cap = (int32_t)(NW * cdiv(nvb, NQD)); break;
    case AGG_BLOCK: L.desc_cap = (int32_t)cdiv(nvb, NQD); break;
    case AGG_MULTI: L.desc_cap = (int32_t)cdiv(L.ngroups_cap, NQD); break;
    default: L.desc_cap = 1; break;
  }
  L.fcap = (int32_t)(2 * cdiv(slots, NQF) + 64);
  const size_t fslots = (size_t)NQF * L.fcap + (size_t)slots;
  size_t off = 0;
  L.state = off; off = align_up(off + sizeof(State));
  L.queries = off; off = align_up(off + (size_t)nq * sizeof(Query));
  L.qlist = off; off = align_up(off + (size_t)(2 * nq + 1) * 4);  // list + workgroup prefix
  L.qmap = off; off = align_up(off + (size_t)cdiv(slots, 32) * 4);
  L.grp_packed = off; off = align_up(off + 3 * (size_t)L.ngroups_cap * 8);
  L.grp_done = off; off = align_up(off + 3 * (size_t)L.ngroups_cap * 4);
  L.front0 = off; off = align_up(off + fslots * 4);
  L.front1 = off; off = align_up(off + fslots * 4);
  // SSSP stamps / two BFS bitmaps and the NHINT per-XCD copies; then the found
  // bytes (which SSSP, having no stamps when it uses them, lets overlap these)
  L.visit = off; off = align_up(off + std::max((size_t)slots * 4, found_offset(slots) + (size_t)cdiv(slots, 32) * 32));
  L.dist2 = off; off = align_up(off + (size_t)slots * 4);  // SSSP second distance array
  L.rec = off; off = align_up(off + (size_t)slots * 16);
  L.rec_q = off; off = align_up(off + (size_t)slots * 4);
  L.rec_slot = off; off = align_up(off + (size_t)slots * 4);  // SSSP
  L.ser = off; off = align_up(off + (size_t)cdiv(slots, PB) * PB * 16);
  L.desc = off; off = align_up(off + (size_t)NQD * L.desc_cap * 16);
  L.stats = off; off = align_up(off + (size_t)MAX_GRID * NSTAT * 8);
  L.sercnt = off; off = align_up(off + (size_t)MAX_GRID * 4);
  L.total = off;
  return L;
}

dpo_status check_options(const dpo_options& o) {
  if (o.mode != DPO_MODE_NESTED && o.mode != DPO_MODE_FLAT) return DPO_ERR_ARG;
  if (o.threshold < 0) return DPO_ERR_ARG;
  if (o.coarsen != 1 && o.coarsen != 2 && o.coarsen != 4 && o.coarsen != 8 && o.coarsen != 16)
    return DPO_ERR_ARG;
  if (o.agg < DPO_AGG_NONE || o.agg > DPO_AGG_GRID) return DPO_ERR_ARG;
  if (o.agg_threshold < 0) return DPO_ERR_ARG;
  if (o.split_min < 0) return DPO_ERR_ARG;
  if (o.serial_wave != 0 && o.serial_wave != 1) return DPO_ERR_ARG;
  if (o.dyn_share < 0 || o.dyn_share > 100) return DPO_ERR_ARG;
  if (o.claim_hint < DPO_HINT_AUTO || o.claim_hint > DPO_HINT_OFF) return DPO_ERR_ARG;
  if (o.agg == DPO_AGG_MULTIBLOCK && (o.agg_blocks < 2 || o.agg_blocks > 1024)) return DPO_ERR_ARG;
  if (o.child_block != 64 && o.child_block != 128 && o.child_block != 256) return DPO_ERR_ARG;
  if (o.steps_per_replay < 0 || o.steps_per_replay > 1024) return DPO_ERR_ARG;
  return DPO_OK;
}

dpo_status check_graph(const dpo_csr* g, bool need_w) {
  if (!g || g->n < 1 || g->m < 0 || !g->row_ptr) return DPO_ERR_ARG;
  if (g->m > 0 && !g->col_idx) return DPO_ERR_ARG;
  if (need_w && g->m > 0 && !g->weights) return DPO_ERR_ARG;
  return DPO_OK;
}

struct CachedGraph {
  const void* parent;
  const void* child;
  const void* third;
  const void* fourth;
  int pgrid, cgrid, tgrid, fgrid, steps;
  Args args;
  uint32_t* flags;
  hipGraphExec_t exec;
  uint64_t last_use;
};

struct GridEntry {
  const void* first;
  int second;
  unsigned third;
};

constexpr int kMaxGridEntries = 64;

struct Runtime {
  std::mutex mu;
  std::vector<CachedGraph> graphs;
  uint64_t tick = 0;
  uint32_t* host_flags = nullptr;  // pinned: base, done, error, levels_run; [8]: verdict
  uint32_t ticket = 0;             // of the last narrow launch that posted a verdict (24 bits)
  uint64_t drawn = 0;              // keys drawn without the system's help (draw_key)
  unsigned long long* host_stats = nullptr;  // pinned: MAX_GRID * NSTAT
  Query* host_q = nullptr;                   // pinned: MAX_QUERIES query records
  int32_t* host_list = nullptr;              // pinned: MAX_QUERIES query indices + prefix
  int cu_count = 0;
  // persistent grid sizes per kernel (fixed storage: the no-allocation entry
  // point uses them too)
  GridEntry grids[kMaxGridEntries];
  int ngrids = 0;
};

Runtime& rt() {
  static Runtime r;
  return r;
}

dpo_status hip_ok(hipError_t e) { return e == hipSuccess ? DPO_OK : DPO_ERR_HIP; }

// Compute-unit count of the current device (no allocation).
dpo_status ensure_device(Runtime& r) {
  if (r.cu_count > 0) return DPO_OK;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return DPO_ERR_HIP;
  if (hipDeviceGetAttribute(&r.cu_count, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return DPO_ERR_HIP;
  return DPO_OK;
}

dpo_status ensure_runtime(Runtime& r) {
  if (r.host_flags) return DPO_OK;
  if (ensure_device(r) != DPO_OK) return DPO_ERR_HIP;
  void* p = nullptr;
  const size_t qbytes = (size_t)MAX_QUERIES * (sizeof(Query) + 8) + 4;
  if (hipHostMalloc(&p, 256 + (size_t)MAX_GRID * NSTAT * 8 + qbytes, hipHostMallocDefault) !=
      hipSuccess)
    return DPO_ERR_HIP;
  r.host_flags = (uint32_t*)p;
  r.host_stats = (unsigned long long*)((char*)p + 256);
  r.host_q = (Query*)((char*)p + 256 + (size_t)MAX_GRID * NSTAT * 8);
  r.host_list = (int32_t*)(r.host_q + MAX_QUERIES);
  return DPO_OK;
}

// Persistent grid: as many workgroups as can be resident at once.
int persistent_grid(Runtime& r, const void* kernel, unsigned shmem = 0) {
  for (int i = 0; i < r.ngrids; ++i)
    if (r.grids[i].first == kernel && r.grids[i].third == shmem) return r.grids[i].second;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, PB, shmem) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  if (per_cu > 8) per_cu = 8;
  int grid = per_cu * r.cu_count;
  if (grid > MAX_GRID) grid = MAX_GRID;
  if (r.ngrids < kMaxGridEntries) r.grids[r.ngrids++] = GridEntry{kernel, grid, shmem};
  return grid;
}

dpo_status add_node(hipGraph_t graph, hipGraphNode_t* prev, const void* fn, int grid, int block,
                    void** params, unsigned shmem = 0) {
  hipKernelNodeParams kp{};
  kp.func = const_cast<void*>(fn);
  kp.gridDim = dim3(grid);
  kp.blockDim = dim3(block);
  kp.sharedMemBytes = shmem;
  kp.kernelParams = params;
  kp.extra = nullptr;
  hipGraphNode_t node;
  if (hipGraphAddKernelNode(&node, graph, *prev ? prev : nullptr, *prev ? 1 : 0, &kp) !=
      hipSuccess)
    return DPO_ERR_HIP;
  *prev = node;
  return DPO_OK;
}

// K level steps (BU_QUERIES: the tally and the bottom-up kernels first; parent kernel, then child kernel unless flat, then the third
// kernel if any: SSSP's thresholded children, on the parent kernel's grid, or
// BFS's harvest; then the fourth if any: SSSP's harvest) and the advance of the
// level base, which reports to `flags` (host, pinned), as one instantiated
// graph.
dpo_status get_exec(Runtime& r, const void* parent, const void* child, const void* third,
                    const void* fourth, int pgrid, int cgrid, int tgrid, int fgrid, int steps,
                    const Args& args, uint32_t* flags, hipGraphExec_t* out, bool cached = true) {
  for (auto& e : r.graphs) {
    if (!cached) break;
    if (e.parent == parent && e.child == child && e.third == third && e.fourth == fourth &&
        e.pgrid == pgrid && e.cgrid == cgrid && e.tgrid == tgrid && e.fgrid == fgrid &&
        e.steps == steps && e.flags == flags && std::memcmp(&e.args, &args, sizeof(Args)) == 0) {
      e.last_use = ++r.tick;
      *out = e.exec;
      return DPO_OK;
    }
  }
  hipGraph_t graph;
  if (hipGraphCreate(&graph, 0) != hipSuccess) return DPO_ERR_HIP;
  Args a = args;
  std::vector<uint32_t> step_ids(steps);
  hipGraphNode_t prev = nullptr;
  dpo_status s = DPO_OK;
  for (int i = 0; i < steps && s == DPO_OK; ++i) {
    step_ids[i] = (uint32_t)i;
    void* params[] = {&a, &step_ids[i]};
    if (a.bottom_up == BU_QUERIES) {
      s = add_node(graph, &prev, tally_kernel_ptr(), 2 * r.cu_count, PB, params);
      if (s == DPO_OK)
        s = add_node(graph, &prev, bottom_up_words_kernel_ptr(), r.cu_count, QB, params);
      if (s == DPO_OK)
        s = add_node(graph, &prev, bottom_up_queries_kernel_ptr(),
                     persistent_grid(r, bottom_up_queries_kernel_ptr()), PB, params);
    }
    if (s == DPO_OK) s = add_node(graph, &prev, parent, pgrid, PB, params);
    if (s == DPO_OK && child) s = add_node(graph, &prev, child, cgrid, PB, params);
    if (s == DPO_OK && third) s = add_node(graph, &prev, third, tgrid, PB, params);
    if (s == DPO_OK && fourth) s = add_node(graph, &prev, fourth, fgrid, PB, params);
  }
  State* st = a.st;
  uint32_t k = (uint32_t)steps;
  void* aparams[] = {&st, &k, &flags};
  if (s == DPO_OK) s = add_node(graph, &prev, advance_kernel_ptr(), 1, 64, aparams);
  hipGraphExec_t exec;
  if (s == DPO_OK && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess)
    s = DPO_ERR_HIP;
  (void)hipGraphDestroy(graph);
  if (s != DPO_OK) return s;
  if (!cached) {  // owned by the caller
    *out = exec;
    return DPO_OK;
  }
  if ((int)r.graphs.size() >= kMaxCachedGraphs) {
    size_t victim = 0;
    for (size_t i = 1; i < r.graphs.size(); ++i)
      if (r.graphs[i].last_use < r.graphs[victim].last_use) victim = i;
    (void)hipGraphExecDestroy(r.graphs[victim].exec);
    r.graphs.erase(r.graphs.begin() + victim);
  }
  r.graphs.push_back(
      CachedGraph{parent, child, third, fourth, pgrid, cgrid, tgrid, fgrid, steps, args, flags,
                  exec, ++r.tick});
  *out = exec;
  return DPO_OK;
}

// One set of queries run together: per-query tables, workspace carving and
// the replay loop shared by the single, batch and serving entry points.
struct SetRun {
  int problem = PROB_BFS;
  Layout lay{};
  Args a{};
  const void* parent = nullptr;
  const void* child = nullptr;
  // after the child kernel: SSSP's thresholded children, or BFS's harvest
  // (per-XCD copies); then SSSP's harvest (found bytes)
  const void* third = nullptr;
  const void* fourth = nullptr;
  int pgrid = 0, cgrid = 0, tgrid = 0, fgrid = 0, steps = kDefaultSteps;
  bool short_steps = false;  // kBatchSteps by default
  int32_t n = 0;  // vertices of the graph (the arena)
  hipStream_t stream = nullptr;
  int32_t* qlist = nullptr;  // device: indices of the queries being admitted
};

// Queries of `slots` vertices in all, over the graphs of g, go bottom-up by
// themselves, if g is symmetric: the check reads all of g (about 8 times as fast
// per entry as a traversal), and a level step of such queries is three kernels
// longer (BU_QUERIES_EDGES).
bool queries_pay(const dpo_csr& g, int64_t slots) {
  return slots >= g.n && (double)slots / g.n * g.m >= (double)BU_QUERIES_EDGES;
}

bool dense_graph(const dpo_csr& g) { return g.m >= (int64_t)HINT_AUTO_MIN_DEGREE * g.n; }

// tm: phase-timing rows; non-null selects the timed instantiations of the
// level kernels, run at the grid sizes of the product ones (same schedule).
dpo_status prepare_set(Runtime& r, int problem, const dpo_csr* g, const dpo_options& o,
                       int64_t slots, int32_t nq, void* out, void* ws, size_t ws_bytes,
                       void* stream, bool count_stats, SetRun* sr,
                       unsigned long long* tm = nullptr, bool batch_call = false) {
  if (slots < 1 || slots > INT32_MAX || nq < 1 || nq > MAX_QUERIES) return DPO_ERR_ARG;
  const Layout lay = layout_for(slots, nq, o);
  if (ws_bytes < lay.total) return DPO_ERR_WORKSPACE;
  const int gran = gran_of(o);
  sr->problem = problem;
  sr->n = g->n;
  sr->lay = lay;
  // Found bytes and the harvest (BFS: with per-XCD copies): single traversals,
  // the serving engine, SSSP batches (64 queries over 16 graphs 856 -> 805 us)
  // and BFS batches whose queries go bottom-up, on graphs whose average degree is
  // at least HINT_AUTO_MIN_DEGREE, unless the options say otherwise.  The harvest
  // adds a kernel launch to every level step; a graph of low average degree runs
  // many narrow levels and rarely a wide one.
  const bool dense = dense_graph(*g);
  const bool bfs = problem == PROB_BFS;
  // Queries that go bottom-up by themselves: a batch of enough work, and a serving
  // engine while enough is running.  They use found bytes (as do those of a large
  // batch that turns out directed: 512 queries over directed graphs 4,050 -> 3,700
  // us, 80 over larger ones 1,080 -> 670).
  const bool by_query = bfs && (batch_call ? queries_pay(*g, slots) : nq > 1) && gran != AGG_FLAT &&
                        gran != AGG_NONE && !count_stats && !tm;
  const bool hint = o.claim_hint == DPO_HINT_ON ||
                    (o.claim_hint == DPO_HINT_AUTO && (!batch_call || by_query || !bfs) && dense);
  sr->parent = parent_kernel_ptr(problem, gran);
  sr->child = gran == AGG_FLAT ? nullptr : child_kernel_ptr(problem, false, hint && !batch_call);
  sr->third = bfs ? (hint ? harvest_kernel_ptr(problem) : nullptr) : serial_kernel_ptr(problem, gran);
  sr->fourth = !bfs && hint ? harvest_kernel_ptr(problem) : nullptr;
  if (!sr->parent) return DPO_ERR_UNSUPPORTED;
  char* base = (char*)ws;
  Args& a = sr->a;
  std::memset(&a, 0, sizeof(a));  // padding too: cached graphs are keyed by these bytes
  a.rp = g->row_ptr;
  a.col = g->col_idx;
  a.w = g->weights;
  a.level = problem == PROB_BFS ? (int32_t*)out : nullptr;
  a.dist = problem == PROB_SSSP ? (uint32_t*)out : nullptr;
  a.st = (State*)(base + lay.state);
  a.q = (Query*)(base + lay.queries);
  a.grp_packed = (unsigned long long*)(base + lay.grp_packed);
  a.grp_done = (uint32_t*)(base + lay.grp_done);
  a.front0 = (int32_t*)(base + lay.front0);
  a.front1 = (int32_t*)(base + lay.front1);
  a.visit = (uint32_t*)(base + lay.visit);
  // SSSP with found bytes has no iteration stamps: the bytes overlap them
  a.found = (uint8_t*)(base + lay.visit + found_offset(slots));
  // in front of them, where BFS has its bitmaps
  a.bound = !bfs && hint && slots >= BOUND_MIN_SLOTS ? (uint8_t*)(base + lay.visit) : nullptr;
  a.dist2 = problem == PROB_SSSP ? (uint32_t*)(base + lay.dist2) : nullptr;
  a.vwords = (int32_t)cdiv(slots, 32);
  a.rec = (int4*)(base + lay.rec);
  a.rec_q = (int32_t*)(base + lay.rec_q);
  a.rec_slot = (int32_t*)(base + lay.rec_slot);
  a.ser = (int4*)(base + lay.ser);
  a.qmap = (int32_t*)(base + lay.qmap);
  a.desc = (int4*)(base + lay.desc);
  a.stats = (unsigned long long*)(base + lay.stats);
  a.sercnt = (uint32_t*)(base + lay.sercnt);
  a.slots = (int32_t)slots;
  a.n = g->n;
  a.m = g->m;
  a.nq = nq;
  a.CB = o.child_block;
  a.k = (gran == AGG_MULTI) ? (int32_t)group_blocks(o, slots) : 1;
  a.agg_threshold = o.agg_threshold;
  a.split_min = o.split_min;
  a.serial_wave = o.serial_wave;
  a.dyn_pct = o.dyn_share;
  a.hint = hint ? 1 : 0;
  a.ngroups_cap = lay.ngroups_cap;
  a.desc_cap = lay.desc_cap;
  a.fcap = lay.fcap;
  a.count_stats = count_stats ? 1 : 0;
  static_assert(TALLIES * MAX_QUERIES * 4 < MAX_GRID * NSTAT * 8, "the tallies take the counters' place");
  a.bottom_up = by_query && hint ? BU_QUERIES : BU_OFF;
  a.tally = (uint32_t*)(base + lay.stats);
  sr->qlist = (int32_t*)(base + lay.qlist);
  sr->pgrid = persistent_grid(r, sr->parent);
  // the thresholded children's kernel walks the lists of the parent kernel's
  // workgroups: one grid for both, all of it resident in either
  if (sr->third && !bfs) sr->pgrid = std::min(sr->pgrid, persistent_grid(r, sr->third));
  sr->cgrid = sr->child ? persistent_grid(r, sr->child) : 0;
  // the harvest: as many workgroups as its rounds need, at most those resident
  // (a small graph's many narrow levels launch it empty)
  const int hgrid = (int)std::min<int64_t>(persistent_grid(r, harvest_kernel_ptr(problem)),
                                           cdiv(slots, (int64_t)PB * HARVEST_RUNS));
  sr->tgrid = !sr->third ? 0 : bfs ? hgrid : sr->pgrid;
  sr->fgrid = sr->fourth ? hgrid : 0;
  sr->short_steps = batch_call && dense && o.steps_per_replay == 0;
  sr->steps = o.steps_per_replay ? o.steps_per_replay : sr->short_steps ? kBatchSteps : kDefaultSteps;
  sr->stream = (hipStream_t)stream;
  if (tm) {
    sr->parent = parent_kernel_ptr(problem, gran, true);
    sr->child = sr->child ? child_kernel_ptr(problem, true, hint) : nullptr;
    sr->third = bfs ? (hint ? harvest_kernel_ptr(problem, true) : nullptr)
                    : serial_kernel_ptr(problem, gran, true);
    sr->fourth = !bfs && hint ? harvest_kernel_ptr(problem, true) : nullptr;
    // a timed kernel that needs more registers than its product one runs on
    // the grid that is resident at its own occupancy (a larger grid would run
    // in two rounds and time the second round's wait as work)
    sr->pgrid = std::min(sr->pgrid, persistent_grid(r, sr->parent));
    if (sr->third && !bfs) sr->pgrid = std::min(sr->pgrid, persistent_grid(r, sr->third));
    if (sr->child) sr->cgrid = std::min(sr->cgrid, persistent_grid(r, sr->child));
    sr->tgrid = !sr->third ? 0 : !bfs ? sr->pgrid
                : std::min(sr->tgrid, persistent_grid(r, sr->third));
    if (sr->fourth) sr->fgrid = std::min(sr->fgrid, persistent_grid(r, sr->fourth));
    a.tm = tm;
  }
  return DPO_OK;
}

int init_grid(Runtime& r, int64_t work) {
  int64_t gsz = cdiv(std::max<int64_t>(work, (int64_t)MAX_GRID * NSTAT), PB);
  if (gsz > 4 * r.cu_count) gsz = 4 * r.cu_count;
  return (int)std::max<int64_t>(gsz, 1);
}

// Admit workgroups: hlist[count + k] = first workgroup of query hlist[k]
// (one per ADMIT_CHUNK of its slots, at least one); returns the total.
int32_t admit_prefix(const Query* hq, int32_t* hlist, int32_t count) {
  int32_t* pre = hlist + count;
  int64_t t = 0;
  for (int32_t k = 0; k < count; ++k) {
    pre[k] = (int32_t)t;
    t += std::max<int64_t>(1, cdiv(hq[hlist[k]].n, ADMIT_CHUNK));
  }
  pre[count] = (int32_t)t;
  return (int32_t)t;
}

dpo_status launch_admit(SetRun& sr, int32_t* hlist, int32_t count, int32_t groups) {
  if (hipMemcpyAsync(sr.qlist, hlist, (size_t)(2 * count + 1) * 4, hipMemcpyHostToDevice,
                     sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  int32_t* dl = sr.qlist;
  void* p1[] = {&sr.a, &dl, &count};
  if (hipLaunchKernel(admit_kernel_ptr(sr.problem), dim3((unsigned)groups), dim3(PB), p1, 0,
                      sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  void* p2[] = {&sr.a, &dl, &count};
  if (hipLaunchKernel(admit_sources_kernel_ptr(), dim3((unsigned)cdiv(count, PB)), dim3(PB), p2, 0,
                      sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  return DPO_OK;
}

// Start the queries hlist[0 .. count) whose records are already in hq (host,
// pinned; hlist has room for 2 * count + 1 entries): upload the table of nq
// records, the index list and the workgroup prefix, then the admit kernels.  (The
// records of running queries are the device's own, as of the end of its last
// replay: one upload of all costs less than one for each new record.)
dpo_status admit(SetRun& sr, const Query* hq, int32_t nq, int32_t* hlist, int32_t count) {
  if (count <= 0) return DPO_OK;
  if (hipMemcpyAsync(sr.a.q, hq, (size_t)nq * sizeof(Query), hipMemcpyHostToDevice, sr.stream) !=
      hipSuccess)
    return DPO_ERR_HIP;
  return launch_admit(sr, hlist, count, admit_prefix(hq, hlist, count));
}

dpo_status start_set(Runtime& r, SetRun& sr) {
  void* p[] = {&sr.a};
  if (hipLaunchKernel(init_kernel_ptr(sr.problem), dim3(init_grid(r, sr.lay.ngroups_cap)), dim3(PB),
                      p, 0, sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  return DPO_OK;
}

// A key that nothing about the graph can have to do with: the system's random
// bytes, or, should it have none to give, the clock and a counter.
PairKey draw_key(Runtime& r) {
  PairKey key;
  if (getrandom(&key, sizeof(key), 0) == (ssize_t)sizeof(key)) return key;
  uint64_t x = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() + (uint64_t)(uintptr_t)&r;
  for (uint32_t& k : key.k) {
    x = (x + ++r.drawn) * 0x9E3779B97F4A7C15ull;
    x ^= x >> 29;
    k = (uint32_t)(x >> 32);
  }
  return key;
}

// Symmetry check of the graph; vbase, ngraphs: of the graphs of an arena (device).
dpo_status launch_symmetry(Runtime& r, SetRun& sr, const uint32_t* vbase = nullptr,
                           uint32_t ngraphs = 0) {
  uint32_t n = (uint32_t)sr.n;
  PairKey key = draw_key(r);
  void* p[] = {&sr.a, &n, &key, &vbase, &ngraphs};
  const int64_t grid = std::min<int64_t>(cdiv(sr.a.m, (int64_t)NW * SYM_EDGES), 8 * (int64_t)r.cu_count);
  return hip_ok(hipLaunchKernel(symmetry_kernel_ptr(vbase != nullptr), dim3((unsigned)std::max<int64_t>(grid, 1)),
                                dim3(PB), p, 0, sr.stream));
}

// The same for an arena, its result into the state
// (BU_QUERIES) and, as V_BOTTOM_UP or V_TOP_DOWN under `ticket`, into the pinned
// word `verdict`.  *asked: false for an arena of more graphs than the space behind
// the tallies holds, which stays unchecked.
dpo_status check_symmetry(Runtime& r, SetRun& sr, const int32_t* graph_vbase, int32_t ngraphs,
                          uint32_t ticket, uint32_t* verdict, bool* asked) {
  uint32_t* vbase = sr.a.tally + TALLIES * sr.a.nq;
  *asked = (size_t)(TALLIES * sr.a.nq + ngraphs + 1) * 4 <= (size_t)MAX_GRID * NSTAT * 8;
  if (!*asked) return DPO_OK;
  // (pageable memory: copied before the call returns)
  if (hipMemcpyAsync(vbase, graph_vbase, (size_t)(ngraphs + 1) * 4, hipMemcpyHostToDevice, sr.stream) !=
      hipSuccess)
    return DPO_ERR_HIP;
  dpo_status s = launch_symmetry(r, sr, vbase, (uint32_t)ngraphs);
  void* p[] = {&sr.a.st, &ticket, &verdict};
  return s != DPO_OK ? s
                     : hip_ok(hipLaunchKernel(settle_symmetry_kernel_ptr(), dim3(1), dim3(64), p, 0, sr.stream));
}

// Start of a single traversal (one launch instead of init and admission).
dpo_status start_single(Runtime& r, SetRun& sr, const Query& q) {
  Query Q = q;
  void* p[] = {&sr.a, &Q};
  const int64_t work = std::max<int64_t>(sr.a.slots, 3 * (int64_t)sr.lay.ngroups_cap);
  const int64_t grid = std::min<int64_t>(cdiv(work, PB), 8 * (int64_t)r.cu_count);
  return hip_ok(hipLaunchKernel(start_kernel_ptr(sr.problem), dim3((unsigned)grid), dim3(PB), p, 0,
                                sr.stream));
}

// One replay of K level steps; its last kernel reports base, done, error and
// levels_run to the host's flags.
dpo_status replay(Runtime& r, SetRun& sr, hipGraphExec_t exec) {
  if (hipGraphLaunch(exec, sr.stream) != hipSuccess) return DPO_ERR_HIP;
  if (hipStreamSynchronize(sr.stream) != hipSuccess) return DPO_ERR_HIP;
  if (r.host_flags[2] != 0) return (dpo_status)(-(int32_t)r.host_flags[2]);
  return DPO_OK;
}

// Runs replays until every query has finished.
dpo_status run_to_completion(Runtime& r, SetRun& sr, int64_t max_levels) {
  hipGraphExec_t exec;
  dpo_status s =
      get_exec(r, sr.parent, sr.child, sr.third, sr.fourth, sr.pgrid, sr.cgrid, sr.tgrid, sr.fgrid,
               sr.steps, sr.a, r.host_flags, &exec);
  if (s != DPO_OK) return s;
  const int64_t max_replays = max_levels / sr.steps + 2;
  for (int64_t rep = 0; rep < max_replays;) {
    // short replays end a traversal of few levels early; one that has had
    // kDefaultSteps levels by then gets as many at a time
    const int count = sr.short_steps && rep * sr.steps >= kDefaultSteps ? kDefaultSteps / sr.steps : 1;
    for (int i = 1; i < count; ++i)
      if (hipGraphLaunch(exec, sr.stream) != hipSuccess) return DPO_ERR_HIP;
    s = replay(r, sr, exec);
    if (s != DPO_OK) return s;
    if (r.host_flags[1]) return DPO_OK;
    rep += count;
  }
  return DPO_ERR_TIMEOUT;
}

// The kernels of one level step, launched one by one.
dpo_status launch_step(SetRun& sr, uint32_t step) {
  void* p[] = {&sr.a, &step};
  if (hipLaunchKernel(sr.parent, dim3((unsigned)sr.pgrid), dim3(PB), p, 0, sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  if (sr.child &&
      hipLaunchKernel(sr.child, dim3((unsigned)sr.cgrid), dim3(PB), p, 0, sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  if (sr.third &&
      hipLaunchKernel(sr.third, dim3((unsigned)sr.tgrid), dim3(PB), p, 0, sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  if (sr.fourth &&
      hipLaunchKernel(sr.fourth, dim3((unsigned)sr.fgrid), dim3(PB), p, 0, sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  return DPO_OK;
}

// The narrow levels' kernel: one workgroup.  after: the level steps run since the
// last one, or AFTER_BOTTOM_UP.  verdict: pinned word it reports to, or nullptr.
dpo_status launch_narrow(SetRun& sr, uint32_t after, uint32_t ticket, uint32_t* verdict) {
  void* p[] = {&sr.a, &after, &ticket, &verdict};
  return hip_ok(hipLaunchKernel(narrow_kernel_ptr(sr.a.slots), dim3(1), dim3(NARROW_BLOCK), p, 0,
                                sr.stream));
}

// A bottom-up level of a single traversal, if one is due; check: the symmetry
// check first, if due.
dpo_status launch_bottom_up(Runtime& r, SetRun& sr, bool check) {
  dpo_status s = check ? launch_symmetry(r, sr) : DPO_OK;
  if (s != DPO_OK) return s;
  void* p[] = {&sr.a};
  const int64_t grid = std::min<int64_t>(cdiv(sr.a.slots, PB), persistent_grid(r, bottom_up_kernel_ptr()));
  return hip_ok(hipLaunchKernel(bottom_up_kernel_ptr(), dim3((unsigned)grid), dim3(PB), p, 0, sr.stream));
}

// Levels may be run by other kernels than the level step's (narrow, bottom-up,
// solo), except where the caller asks for the level step itself: the paper's two
// literal forms (flat, and one grid per parent), its counters, its phase timing.
bool any_kernel(const dpo_options& o, bool stats, bool timed) {
  return o.mode == DPO_MODE_NESTED && o.agg != DPO_AGG_NONE && !stats && !timed;
}

// Ticket of the next narrow launch that posts to `verdict`, which holds no
// other's from here on.  Never 0: the solo and near-far kernels post to the same
// word under ticket 0, and 0 is what the word is cleared to.
uint32_t next_ticket(Runtime& r, uint32_t* verdict) {
  r.ticket = r.ticket % 0xFFFFFFu + 1;
  __atomic_store_n(verdict, 0u, __ATOMIC_RELAXED);
  return r.ticket;
}

// Result of a solo or near-far launch that has ended, from its verdict.
dpo_status ended(uint32_t verdict) {
  const uint32_t code = verdict & 15u;
  if (code == V_DONE) return DPO_OK;
  return code == V_ERROR ? (dpo_status)(-(int32_t)((verdict >> 4) & 15u)) : DPO_ERR_HIP;
}

// SSSP on a small graph.
dpo_status launch_solo(SetRun& sr, int32_t source, int32_t threshold, uint32_t* verdict) {
  uint32_t src = (uint32_t)source, T = (uint32_t)threshold;
  void* p[] = {&sr.a, &src, &T, &verdict};
  return hip_ok(hipLaunchKernel(solo_kernel_ptr(sr.a.m >= SOLO_FAR_EDGES), dim3(1), dim3(NARROW_BLOCK),
                                p, 0, sr.stream));
}

// Waits for the verdict of narrow launch `ticket`.  The word is polled: a
// stream synchronisation per narrow launch would cost more than most of them.
// Every 2 ms the stream is asked too, so that a failed launch ends the wait.
dpo_status wait_verdict(const uint32_t* verdict, uint32_t ticket, hipStream_t stream, uint32_t* out) {
  auto look = [&] {
    *out = __atomic_load_n(verdict, __ATOMIC_ACQUIRE);
    return (*out >> 8) == ticket;
  };
  auto asked = std::chrono::steady_clock::now();
  for (uint32_t i = 1;; ++i) {
    if (look()) return DPO_OK;
    if (i % 256) continue;
    const auto now = std::chrono::steady_clock::now();
    if (now - asked < std::chrono::milliseconds(2)) continue;
    asked = now;
    const hipError_t e = hipStreamQuery(stream);
    if (e == hipErrorNotReady) {
      (void)hipGetLastError();  // not an error of the caller's
      continue;
    }
    return e == hipSuccess && look() ? DPO_OK : DPO_ERR_HIP;
  }
}

// The verdict from a copy of the state (on the stack: no pinned memory).
dpo_status copy_verdict(SetRun& sr, uint32_t* out) {
  uint32_t head[offsetof(State, plan) / 4 + 1];
  if (hipMemcpyAsync(head, sr.a.st, sizeof(head), hipMemcpyDeviceToHost, sr.stream) != hipSuccess ||
      hipStreamSynchronize(sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  const uint32_t done = head[offsetof(State, done) / 4], error = head[offsetof(State, error) / 4];
  *out = error << 4 | (error ? V_ERROR : done ? V_DONE : head[offsetof(State, plan) / 4]);
  return DPO_OK;
}

// A single traversal: narrow levels in one launch, then a wide one.  The host
// learns from the narrow kernel's verdict which kernels that takes.  Bottom-up
// levels follow each other more often than not: two are launched at a time, the
// second of which finds out by itself whether it is due.  A run of wide levels
// that go top-down takes as many level steps at a time as it has had (any level may
// run as a level step), so that the host's look and the narrow launch of each level
// cost little on a graph whose levels are all wide, and the steps past the run's
// end no more than the run (us, one step at a time / half as many as it has had /
// as many: a 160^3 grid of 480 levels 7,710 / 5,055 / 5,020, without allocation a
// 90^3 grid 7,630 / 3,500 / 3,400, a band of 1 M vertices 890 / 795 / 747, R-MAT
// of 1 M with each edge one way 373 / 373 / 359).
// verdict: pinned word for it, or nullptr where none may be allocated; the state
// is copied then, which takes about 15 us each time.
dpo_status run_narrow_and_wide(Runtime& r, SetRun& sr, int64_t max_levels, uint32_t* verdict) {
  uint32_t after = 0;
  uint32_t run = 0;  // wide levels run top-down one after another
  for (int64_t rep = 0; rep < max_levels + 2; ++rep) {
    const uint32_t ticket = verdict ? next_ticket(r, verdict) : 0u;
    dpo_status s = launch_narrow(sr, after, ticket, verdict);
    uint32_t v = 0;
    if (s == DPO_OK)
      s = verdict ? wait_verdict(verdict, ticket, sr.stream, &v) : copy_verdict(sr, &v);
    if (s != DPO_OK) return s;
    const uint32_t code = v & 15u;
    if (code == V_DONE || code == V_ERROR) {
      if (verdict && hipStreamSynchronize(sr.stream) != hipSuccess) return DPO_ERR_HIP;
      return code == V_DONE ? DPO_OK : (dpo_status)(-(int32_t)((v >> 4) & 15u));
    }
    run = code == V_STILL && after != AFTER_BOTTOM_UP ? run + after : 0;
    after = 0;
    if (code == V_TOP_DOWN || code == V_STILL) {
      after = std::min<uint32_t>(std::max<uint32_t>(run, 1), kDefaultSteps);
      for (uint32_t i = 0; i < after && s == DPO_OK; ++i) s = launch_step(sr, i);
    } else if (code == V_BOTTOM_UP || code == V_CHECK) {
      after = AFTER_BOTTOM_UP;
      s = launch_bottom_up(r, sr, code == V_CHECK);
      if (s == DPO_OK) s = launch_narrow(sr, after, 0u, nullptr);
      if (s == DPO_OK) s = launch_bottom_up(r, sr, false);
    }
    if (s != DPO_OK) return s;
  }
  return DPO_ERR_TIMEOUT;
}

dpo_status read_stats(Runtime& r, SetRun& sr, dpo_stats* st) {
  if (!st) return DPO_OK;
  if (hipMemcpyAsync(r.host_stats, sr.a.stats, (size_t)MAX_GRID * NSTAT * 8, hipMemcpyDeviceToHost,
                     sr.stream) != hipSuccess ||
      hipMemcpyAsync(r.host_flags, sr.a.st, 16, hipMemcpyDeviceToHost, sr.stream) != hipSuccess ||
      hipStreamSynchronize(sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  int64_t sum[NSTAT] = {0};
  for (int w = 0; w < MAX_GRID; ++w)
    for (int k = 0; k < NSTAT; ++k) sum[k] += (int64_t)r.host_stats[w * NSTAT + k];
  std::memset(st, 0, sizeof(*st));
  st->levels = (int32_t)r.host_flags[3];
  st->frontier_total = sum[S_FRONT];
  st->serial_parents = sum[S_SERIAL];
  st->records = sum[S_REC];
  st->child_blocks = sum[S_CHILD];
  st->edges_serial = sum[S_ESER];
  st->edges_child = sum[S_ECHILD];
  st->descriptors = sum[S_DESC];
  return DPO_OK;
}

dpo_status traverse(int problem, const dpo_csr* g, int32_t source, const dpo_options* o,
                    void* out, void* ws, size_t ws_bytes, void* stream, dpo_stats* st,
                    unsigned long long* tm = nullptr) {
  if (!o || !out || !ws) return DPO_ERR_ARG;
  dpo_status s = check_graph(g, problem == PROB_SSSP);
  if (s != DPO_OK) return s;
  s = check_options(*o);
  if (s != DPO_OK) return s;
  if (source < 0 || source >= g->n) return DPO_ERR_SOURCE;
  if (ws_bytes < layout_for(round32(g->n), 1, *o).total) return DPO_ERR_WORKSPACE;
  Runtime& r = rt();
  std::lock_guard<std::mutex> lock(r.mu);
  s = ensure_runtime(r);
  if (s != DPO_OK) return s;
  SetRun sr;
  s = prepare_set(r, problem, g, *o, round32(g->n), 1, out, ws, ws_bytes, stream, st != nullptr, &sr,
                  tm);
  if (s != DPO_OK) return s;
  if (tm && hipMemsetAsync(tm, 0, DPO_TIMING_BYTES, sr.stream) != hipSuccess) return DPO_ERR_HIP;
  const bool any = any_kernel(*o, st != nullptr, tm != nullptr);
  const bool narrow = any && problem == PROB_BFS;
  if (any && problem == PROB_SSSP && g->n <= SOLO_VERTICES && g->m <= SOLO_EDGES) {
    uint32_t* verdict = r.host_flags + 8;
    *verdict = 0;
    if ((s = launch_solo(sr, source, o->threshold, verdict)) != DPO_OK) return s;
    if (hipStreamSynchronize(sr.stream) != hipSuccess) return DPO_ERR_HIP;
    return ended(*verdict);
  }
  sr.a.bottom_up = narrow && sr.a.hint ? BU_SINGLE : BU_OFF;
  s = start_single(r, sr, Query{0, g->n, 0, 0, o->threshold, o->coarsen, 0, source});
  if (s != DPO_OK) return s;
  if (any && problem == PROB_SSSP && g->n <= NEAR_VERTICES && !dense_graph(*g)) {
    uint32_t* verdict = r.host_flags + 8;
    *verdict = 0;
    uint32_t src = (uint32_t)source;
    void* p[] = {&sr.a, &src, &verdict};
    if (hipLaunchKernel(near_kernel_ptr(), dim3(1), dim3(NARROW_BLOCK), p, 0, sr.stream) != hipSuccess ||
        hipStreamSynchronize(sr.stream) != hipSuccess)
      return DPO_ERR_HIP;
    if ((*verdict & 15u) != V_TOP_DOWN) return ended(*verdict);
  }
  s = narrow ? run_narrow_and_wide(r, sr, g->n, r.host_flags + 8) : run_to_completion(r, sr, g->n);
  return s != DPO_OK ? s : read_stats(r, sr, st);
}

dpo_status check_arena(const dpo_arena* ar, bool need_w) {
  if (!ar || ar->ngraphs < 1 || !ar->graph_vbase) return DPO_ERR_ARG;
  dpo_status s = check_graph(&ar->csr, need_w);
  if (s != DPO_OK) return s;
  if (ar->graph_vbase[0] != 0 || ar->graph_vbase[ar->ngraphs] != ar->csr.n) return DPO_ERR_ARG;
  for (int32_t g = 0; g < ar->ngraphs; ++g)
    if (ar->graph_vbase[g + 1] <= ar->graph_vbase[g]) return DPO_ERR_ARG;
  return DPO_OK;
}

// Output slots of a batch: query q occupies [slot0[q], slot0[q] + n_{graph(q)}),
// slot0 32-aligned, in query order.  Returns the total, or -1 on bad input.
int64_t batch_slots(const dpo_arena* ar, const dpo_query* qs, int32_t nq, int64_t* slot0) {
  int64_t tot = 0;
  for (int32_t i = 0; i < nq; ++i) {
    const int32_t g = qs[i].graph;
    if (g < 0 || g >= ar->ngraphs) return -1;
    if (slot0) slot0[i] = tot;
    tot += round32(ar->graph_vbase[g + 1] - ar->graph_vbase[g]);
  }
  if (slot0) slot0[nq] = tot;
  return tot;
}

dpo_status traverse_batch(int problem, const dpo_arena* ar, const dpo_query* qs, int32_t nq,
                          const dpo_options* bopts, int32_t nb, void* out, void* ws,
                          size_t ws_bytes, void* stream, dpo_stats* st) {
  if (!qs || !bopts || nb < 1 || !out || !ws || nq < 1 || nq > MAX_QUERIES) return DPO_ERR_ARG;
  dpo_status s = check_arena(ar, problem == PROB_SSSP);
  if (s != DPO_OK) return s;
  for (int32_t b = 0; b < nb; ++b)
    if ((s = check_options(bopts[b])) != DPO_OK) return s;
  const int64_t slots = batch_slots(ar, qs, nq, nullptr);
  if (slots < 0) return DPO_ERR_ARG;
  for (int32_t i = 0; i < nq; ++i) {
    const int32_t g = qs[i].graph;
    const int32_t n = ar->graph_vbase[g + 1] - ar->graph_vbase[g];
    if (qs[i].source < 0 || qs[i].source >= n) return DPO_ERR_SOURCE;
    if (qs[i].bucket < 0 || qs[i].bucket >= nb) return DPO_ERR_ARG;
  }
  if (ws_bytes < layout_for(slots, nq, bopts[0]).total) return DPO_ERR_WORKSPACE;
  Runtime& r = rt();
  std::lock_guard<std::mutex> lock(r.mu);
  s = ensure_runtime(r);
  if (s != DPO_OK) return s;
  SetRun sr;
  s = prepare_set(r, problem, &ar->csr, bopts[0], slots, nq, out, ws, ws_bytes, stream,
                  st != nullptr, &sr, nullptr, /*batch_call=*/true);
  if (s != DPO_OK) return s;
  Query* hq = r.host_q;
  int64_t slot = 0;
  for (int32_t i = 0; i < nq; ++i) {
    const int32_t g = qs[i].graph;
    const int32_t n = ar->graph_vbase[g + 1] - ar->graph_vbase[g];
    const dpo_options& bo = bopts[qs[i].bucket];
    hq[i] = Query{(int32_t)slot, n, ar->graph_vbase[g], 0, bo.threshold, bo.coarsen, 0,
                  qs[i].source};
    slot += round32(n);
  }
  int32_t* hl = r.host_list;
  for (int32_t i = 0; i < nq; ++i) hl[i] = i;
  if ((s = start_set(r, sr)) != DPO_OK) return s;
  // bottom-up only if the arena is symmetric: its check runs before the admission,
  // during which the host learns the answer and picks the replay
  uint32_t ticket = 0, verdict = V_TOP_DOWN;
  bool asked = false;
  if (sr.a.bottom_up) {
    ticket = next_ticket(r, r.host_flags + 8);
    s = check_symmetry(r, sr, ar->graph_vbase, ar->ngraphs, ticket, r.host_flags + 8, &asked);
    if (s != DPO_OK) return s;
  }
  if ((s = admit(sr, hq, nq, hl, nq)) != DPO_OK) return s;
  if (asked && (s = wait_verdict(r.host_flags + 8, ticket, sr.stream, &verdict)) != DPO_OK) return s;
  if ((verdict & 15u) != V_BOTTOM_UP) sr.a.bottom_up = BU_OFF;
  if ((s = run_to_completion(r, sr, slots)) != DPO_OK) return s;
  return read_stats(r, sr, st);
}


// ------------------------------------------------------------ no allocation
// Workspace of dpo_bfs_noalloc: a static device array that every GPU the
// library runs on holds until the process ends.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the
// symbol); it uses the device address that hipGetSymbolAddress returns, kept
// per device.
static __device__ __align__(256) unsigned char scratch[DPO_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` per device (under r.mu)

dpo_status scratch_of_current_device(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DPO_ERR_HIP;
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DPO_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return DPO_OK;
}

dpo_status traverse_noalloc(int problem, const dpo_csr* g, int32_t source, const dpo_options* o,
                            void* out, void* stream) {
  if (!o || !out) return DPO_ERR_ARG;
  dpo_status s = check_graph(g, problem == PROB_SSSP);
  if (s != DPO_OK) return s;
  if ((s = check_options(*o)) != DPO_OK) return s;
  if (source < 0 || source >= g->n) return DPO_ERR_SOURCE;
  // the static workspace bounds the graph size (checked before any HIP call)
  if (layout_for(round32(g->n), 1, *o).total > (size_t)DPO_NOALLOC_SCRATCH_BYTES)
    return DPO_ERR_WORKSPACE;
  Runtime& r = rt();
  std::lock_guard<std::mutex> lock(r.mu);
  if ((s = ensure_device(r)) != DPO_OK) return s;
  void* ws = nullptr;
  if ((s = scratch_of_current_device(&ws)) != DPO_OK) return s;
  SetRun sr;
  s = prepare_set(r, problem, g, *o, round32(g->n), 1, out, ws, DPO_NOALLOC_SCRATCH_BYTES, stream,
                  false, &sr);
  if (s != DPO_OK) return s;
  // the start kernel clears the state, the level sets, the group counters, the
  // outputs and the visited state, so nothing left in the array by an earlier
  // call is read
  const bool narrow = any_kernel(*o, false, false);
  sr.a.bottom_up = narrow && sr.a.hint ? BU_SINGLE : BU_OFF;
  s = start_single(r, sr, Query{0, g->n, 0, 0, o->threshold, o->coarsen, 0, source});
  if (s != DPO_OK) return s;
  if (narrow) return run_narrow_and_wide(r, sr, g->n, nullptr);
  uint32_t flags[4] = {0, 0, 0, 0};  // base, done, error, levels_run
  const int64_t max_replays = (int64_t)g->n / sr.steps + 2;
  State* st = sr.a.st;
  uint32_t k = (uint32_t)sr.steps;
  uint32_t* no_flags = nullptr;  // no pinned memory here: the flags are copied
  for (int64_t rep = 0; rep < max_replays; ++rep) {
    for (int i = 0; i < sr.steps; ++i)
      if ((s = launch_step(sr, (uint32_t)i)) != DPO_OK) return s;
    void* ap[] = {&st, &k, &no_flags};
    if (hipLaunchKernel(advance_kernel_ptr(), dim3(1), dim3(64), ap, 0, sr.stream) != hipSuccess)
      return DPO_ERR_HIP;
    if (hipMemcpyAsync(flags, st, sizeof(flags), hipMemcpyDeviceToHost, sr.stream) != hipSuccess ||
        hipStreamSynchronize(sr.stream) != hipSuccess)
      return DPO_ERR_HIP;
    if (flags[2] != 0) return (dpo_status)(-(int32_t)flags[2]);
    if (flags[1]) return DPO_OK;
  }
  return DPO_ERR_TIMEOUT;
}

// ------------------------------------------------------------ serving engine
// Continuous batching: queries are admitted at replay boundaries while
// others are running, as long as their output slots (footprint) and a query
// table entry are free; finished queries are retired and their slots reused.
struct Pending {
  uint64_t ticket;
  int32_t graph, source;
  void* out;
};

struct Running {
  bool used = false;
  uint64_t ticket = 0;
  void* out = nullptr;
  bool copied = true;  // the result goes to `out` by a copy command
  int32_t n = 0;
  int64_t slot0 = 0;
  int64_t footprint = 0;
};

}  // namespace
}  // namespace dpo

struct dpo_engine {
  int problem = dpo::PROB_BFS;
  dpo_csr csr{};
  std::vector<int32_t> vbase;
  std::vector<dpo_options> bopts;
  std::vector<int32_t> gbucket;
  dpo::SetRun sr;
  int32_t max_queries = 0;
  int64_t max_slots = 0;
  char* out_arena = nullptr;
  std::map<int64_t, int64_t> free_slots;  // start -> length, 32-aligned
  std::vector<dpo::Running> run;
  std::vector<int32_t> free_q;
  std::deque<dpo::Pending> pending;
  std::deque<uint64_t> completed;
  std::vector<uint64_t> landing;  // tickets whose results are being copied
  uint64_t next_ticket = 1;
  int32_t running = 0;
  bool inflight = false;
  hipGraphExec_t exec = nullptr;
  hipGraphExec_t plain = nullptr;  // BU_QUERIES: the replay where they would not pay
  dpo::Query* hq = nullptr;   // pinned mirror of the device query table
  int32_t* hlist = nullptr;   // pinned
  uint32_t* hflags = nullptr; // pinned
  uint4* hretire = nullptr;   // pinned: queries being retired, then their workgroup prefix
  std::vector<int32_t> hretire_pre, hretire_q;
  hipEvent_t retired = nullptr;
  int device = 0;
  int64_t running_n = 0;  // vertices of the running queries
  // since the engine was last idle: was the arena's symmetry asked for (the answer
  // is in hflags[4] once that step's replay has ended); was the last replay `exec`;
  // has one been followed by `plain`
  bool asked = false, tallied = false, stale = false;
};

namespace dpo {
namespace {

bool slots_alloc(dpo_engine* e, int64_t len, int64_t* start) {
  for (auto it = e->free_slots.begin(); it != e->free_slots.end(); ++it) {
    if (it->second >= len) {
      *start = it->first;
      const int64_t rest = it->second - len;
      const int64_t nstart = it->first + len;
      e->free_slots.erase(it);
      if (rest > 0) e->free_slots[nstart] = rest;
      return true;
    }
  }
  return false;
}

void slots_free(dpo_engine* e, int64_t start, int64_t len) {
  auto it = e->free_slots.emplace(start, len).first;
  auto nx = std::next(it);
  if (nx != e->free_slots.end() && it->first + it->second == nx->first) {
    it->second += nx->second;
    e->free_slots.erase(nx);
  }
  if (it != e->free_slots.begin()) {
    auto pv = std::prev(it);
    if (pv->first + pv->second == it->first) {
      pv->second += it->second;
      e->free_slots.erase(it);
    }
  }
}

// May retire_kernel store to `out`?  Words of the engine's device's memory;
// results for anything else (another device's memory, the host's) go by a copy
// command each, which takes any address.
bool storable(const dpo_engine* e, const void* out) {
  if ((uintptr_t)out % 4 != 0) return false;
  hipPointerAttribute_t at{};
  if (hipPointerGetAttributes(&at, out) != hipSuccess) {
    (void)hipGetLastError();  // not an error of the caller's
    return false;
  }
  return at.type == hipMemoryTypeDevice && at.device == e->device;
}

// Copies the results of the queries in e->hretire to their callers.  The list
// goes where the level steps put their records (a query has at least 32 slots,
// of 16 bytes each there).
dpo_status launch_retire(dpo_engine* e, int32_t count, int32_t groups) {
  SetRun& sr = e->sr;
  uint4* list = (uint4*)sr.a.rec;
  int32_t* pre = (int32_t*)(list + count);
  std::memcpy(e->hretire + count, e->hretire_pre.data(), (size_t)count * 4);
  if (hipMemcpyAsync(list, e->hretire, (size_t)count * 20, hipMemcpyHostToDevice, sr.stream) != hipSuccess)
    return DPO_ERR_HIP;
  const char* slots = e->out_arena;
  void* p[] = {&slots, &list, &pre, &count};
  return hip_ok(hipLaunchKernel(retire_kernel_ptr(), dim3((unsigned)groups), dim3(PB), p, 0, sr.stream));
}

// Retires, admits and launches.
dpo_status engine_enqueue(dpo_engine* e) {
  Runtime& r = rt();
  SetRun& sr = e->sr;
  dpo_status s = DPO_OK;
  if (e->inflight) {
    if (hipStreamSynchronize(sr.stream) != hipSuccess) return DPO_ERR_HIP;
    if (e->hflags[2] != 0) {
      e->inflight = false;
      return (dpo_status)(-(int32_t)e->hflags[2]);
    }
    // queries without frontier entries at the last level run have finished
    const int32_t last_level = (int32_t)e->hflags[0] - 1;
    const bool all_done = e->hflags[1] != 0;
    int64_t groups = 0;
    int32_t retired = 0, listed = 0;
    for (int32_t q = 0; q < e->max_queries; ++q) {
      const Running& ru = e->run[q];
      if (!ru.used || !(all_done || e->hq[q].last < last_level)) continue;
      e->hretire_q[retired++] = q;
      // (should a copy fail, all stay as they are and the next step tries again)
      if (ru.copied) {
        if (hipMemcpyAsync(ru.out, e->out_arena + ru.slot0 * 4, (size_t)ru.n * 4, hipMemcpyDeviceToDevice,
                           sr.stream) != hipSuccess)
          return DPO_ERR_HIP;
        continue;
      }
      const uint64_t out = (uint64_t)ru.out;
      e->hretire[listed] = uint4{(uint32_t)out, (uint32_t)(out >> 32), (uint32_t)ru.slot0, (uint32_t)ru.n};
      e->hretire_pre[listed++] = (int32_t)groups;
      groups += cdiv(ru.n, ADMIT_CHUNK);
    }
    if (listed && (s = launch_retire(e, listed, (int32_t)groups)) != DPO_OK) return s;
    if (retired && hipEventRecord(e->retired, sr.stream) != hipSuccess) return DPO_ERR_HIP;
    e->inflight = false;
    for (int32_t k = 0; k < retired; ++k) {
      Running& ru = e->run[e->hretire_q[k]];
      slots_free(e, ru.slot0, ru.footprint);
      e->running_n -= ru.n;
      e->landing.push_back(ru.ticket);
      ru = Running{};
      e->free_q.push_back(e->hretire_q[k]);
      --e->running;
    }
  }
  // admit in arrival order while a table entry and the footprint fit
  int32_t count = 0;
  const bool reset = e->running == 0;
  while (!e->pending.empty() && !e->free_q.empty()) {
    const Pending& p = e->pending.front();
    const int32_t n = e->vbase[p.graph + 1] - e->vbase[p.graph];
    int64_t slot0;
    if (!slots_alloc(e, round32(n), &slot0)) break;
    const int32_t q = e->free_q.back();
    e->free_q.pop_back();
    const dpo_options& bo = e->bopts[e->gbucket[p.graph]];
    e->hq[q] = Query{(int32_t)slot0, n, e->vbase[p.graph], 0, bo.threshold, bo.coarsen, 0,
                     p.source};
    Running& ru = e->run[q];
    ru.used = true;
    ru.ticket = p.ticket;
    ru.out = p.out;
    ru.n = n;
    ru.slot0 = slot0;
    ru.footprint = round32(n);
    e->hlist[count++] = q;
    e->running_n += n;
    ++e->running;
    e->pending.pop_front();
  }
  if (count) {
    if (reset) {
      // nothing was running: restart the level sets (and their counters)
      if ((s = start_set(r, sr)) != DPO_OK) return s;
      e->asked = e->tallied = e->stale = false;
    }
    if ((s = admit(sr, e->hq, e->max_queries, e->hlist, count)) != DPO_OK) return s;
  }
  if (e->running > 0) {
    // Bottom-up nodes while the running queries are enough work (see prepare_set)
    // and the arena is not known to be asymmetric; the answer holds until the
    // engine is idle.
    bool up = !e->plain;
    if (e->plain && queries_pay(e->csr, e->running_n)) {
      if (!e->asked) {
        e->hflags[4] = 0;
        bool asked;
        s = check_symmetry(r, sr, e->vbase.data(), (int32_t)e->vbase.size() - 1, 0, e->hflags + 4, &asked);
        if (s != DPO_OK) return s;
        if (!asked) e->hflags[4] = V_TOP_DOWN;
        e->asked = true;
      }
      up = __atomic_load_n(e->hflags + 4, __ATOMIC_RELAXED) != V_TOP_DOWN;
    }
    // the tallies of a query are zero from its admission until the first replay
    // that makes them; those of a level are cleared by the level before it, if that
    // one makes them too
    e->stale |= e->tallied && !up;
    if (up && e->stale) {
      e->stale = false;
      void* cp[] = {&sr.a};
      if (hipLaunchKernel(clear_tally_kernel_ptr(), dim3((unsigned)cdiv(2 * sr.a.nq, PB)), dim3(PB), cp, 0,
                          sr.stream) != hipSuccess)
        return DPO_ERR_HIP;
    }
    e->tallied = up;
    if (hipGraphLaunch(up ? e->exec : e->plain, sr.stream) != hipSuccess) return DPO_ERR_HIP;
    if (hipMemcpyAsync(e->hq, sr.a.q, (size_t)e->max_queries * sizeof(Query),
                       hipMemcpyDeviceToHost, sr.stream) != hipSuccess)
      return DPO_ERR_HIP;
    e->inflight = true;
    // (while the replay runs: 0.3 us each)
    for (int32_t k = 0; k < count; ++k) e->run[e->hlist[k]].copied = !storable(e, e->run[e->hlist[k]].out);
  }
  return DPO_OK;
}

dpo_status engine_step(dpo_engine* e) {
  const dpo_status s = engine_enqueue(e);
  // the retired queries' results are with their callers before dpo_engine_poll
  // can report them; admission and the next replay were enqueued behind them
  if (!e->landing.empty()) {
    if (hipEventSynchronize(e->retired) != hipSuccess) return DPO_ERR_HIP;
    e->completed.insert(e->completed.end(), e->landing.begin(), e->landing.end());
    e->landing.clear();
  }
  return s;
}

}  // namespace
}  // namespace dpo

extern "C" {

size_t dpo_engine_workspace_bytes(const dpo_options* o, int32_t max_queries, int64_t max_slots) {
  if (!o || dpo::check_options(*o) != DPO_OK || max_queries < 1 ||
      max_queries > dpo::MAX_QUERIES || max_slots < 32 || max_slots > INT32_MAX)
    return 0;
  return dpo::layout_for(dpo::round32(max_slots), max_queries, *o).total;
}

dpo_status dpo_engine_create(const dpo_arena* arena, int32_t kind, const dpo_options* bucket_opts,
                             int32_t nbuckets, const int32_t* graph_bucket, int32_t max_queries,
                             int64_t max_slots, void* ws, size_t ws_bytes, void* out_arena,
                             void* stream, dpo_engine** out) {
  using namespace dpo;
  if (!out || !bucket_opts || nbuckets < 1 || !ws || !out_arena || (kind != 0 && kind != 1))
    return DPO_ERR_ARG;
  *out = nullptr;
  const int problem = kind == 0 ? PROB_BFS : PROB_SSSP;
  dpo_status s = check_arena(arena, problem == PROB_SSSP);
  if (s != DPO_OK) return s;
  for (int32_t b = 0; b < nbuckets; ++b)
    if ((s = check_options(bucket_opts[b])) != DPO_OK) return s;
  if (max_queries < 1 || max_queries > MAX_QUERIES || max_slots < 32 || max_slots > INT32_MAX)
    return DPO_ERR_ARG;
  max_slots = round32(max_slots);
  if (ws_bytes < layout_for(max_slots, max_queries, bucket_opts[0]).total) return DPO_ERR_WORKSPACE;
  if (graph_bucket)
    for (int32_t g = 0; g < arena->ngraphs; ++g)
      if (graph_bucket[g] < 0 || graph_bucket[g] >= nbuckets) return DPO_ERR_ARG;
  Runtime& r = rt();
  std::lock_guard<std::mutex> lock(r.mu);
  if ((s = ensure_runtime(r)) != DPO_OK) return s;
  dpo_engine* e = new dpo_engine();
  e->problem = problem;
  (void)hipGetDevice(&e->device);
  e->csr = arena->csr;
  e->vbase.assign(arena->graph_vbase, arena->graph_vbase + arena->ngraphs + 1);
  e->bopts.assign(bucket_opts, bucket_opts + nbuckets);
  e->gbucket.assign(arena->ngraphs, 0);
  if (graph_bucket) e->gbucket.assign(graph_bucket, graph_bucket + arena->ngraphs);
  e->max_queries = max_queries;
  e->max_slots = max_slots;
  e->out_arena = (char*)out_arena;
  e->free_slots[0] = max_slots;
  e->run.assign(max_queries, Running{});
  e->hretire_pre.resize(max_queries);
  e->hretire_q.resize(max_queries);
  e->landing.reserve(max_queries);
  for (int32_t q = max_queries - 1; q >= 0; --q) e->free_q.push_back(q);
  s = prepare_set(r, problem, &e->csr, bucket_opts[0], max_slots, max_queries, out_arena, ws,
                  ws_bytes, stream, false, &e->sr);
  void* p = nullptr;
  if (s == DPO_OK &&
      hipHostMalloc(&p, 64 + (size_t)max_queries * (20 + sizeof(Query) + 8) + 4, hipHostMallocDefault) !=
          hipSuccess)
    s = DPO_ERR_HIP;
  if (s == DPO_OK) s = hip_ok(hipEventCreateWithFlags(&e->retired, hipEventDisableTiming));
  if (s == DPO_OK) {
    e->hflags = (uint32_t*)p;
    e->hretire = (uint4*)((char*)p + 64);
    e->hq = (Query*)((char*)e->hretire + (size_t)max_queries * 20);
    e->hlist = (int32_t*)(e->hq + max_queries);
    std::memset(e->hq, 0, (size_t)max_queries * sizeof(Query));
    s = get_exec(r, e->sr.parent, e->sr.child, e->sr.third, e->sr.fourth, e->sr.pgrid,
                 e->sr.cgrid, e->sr.tgrid, e->sr.fgrid, e->sr.steps, e->sr.a, e->hflags,
                 &e->exec, false);
    if (s == DPO_OK && e->sr.a.bottom_up) {
      Args a = e->sr.a;
      a.bottom_up = BU_OFF;
      s = get_exec(r, e->sr.parent, e->sr.child, e->sr.third, e->sr.fourth, e->sr.pgrid,
                   e->sr.cgrid, e->sr.tgrid, e->sr.fgrid, e->sr.steps, a, e->hflags, &e->plain, false);
    }
  }
  if (s == DPO_OK) s = start_set(r, e->sr);
  if (s == DPO_OK && e->sr.a.hint) {
    // no query has been admitted to any slot yet: no found vertex anywhere
    void* cp[] = {&e->sr.a};
    if (hipLaunchKernel(clear_found_kernel_ptr(), dim3(init_grid(r, max_slots / 4)), dim3(PB), cp,
                        0, e->sr.stream) != hipSuccess)
      s = DPO_ERR_HIP;
  }
  if (s == DPO_OK &&
      hipMemcpyAsync(e->sr.a.q, e->hq, (size_t)max_queries * sizeof(Query), hipMemcpyHostToDevice,
                     e->sr.stream) != hipSuccess)
    s = DPO_ERR_HIP;
  if (s == DPO_OK && hipStreamSynchronize(e->sr.stream) != hipSuccess) s = DPO_ERR_HIP;
  if (s != DPO_OK) {
    if (e->exec) (void)hipGraphExecDestroy(e->exec);
    if (e->plain) (void)hipGraphExecDestroy(e->plain);
    if (e->retired) (void)hipEventDestroy(e->retired);
    if (p) (void)hipHostFree(p);
    delete e;
    return s;
  }
  *out = e;
  return DPO_OK;
}

dpo_status dpo_engine_submit(dpo_engine* e, int32_t graph, int32_t source, void* out,
                             uint64_t* ticket) {
  if (!e || !out || graph < 0 || graph >= (int32_t)e->vbase.size() - 1) return DPO_ERR_ARG;
  const int32_t n = e->vbase[graph + 1] - e->vbase[graph];
  if (source < 0 || source >= n) return DPO_ERR_SOURCE;
  if (dpo::round32(n) > e->max_slots) return DPO_ERR_CAPACITY;
  const uint64_t t = e->next_ticket++;
  e->pending.push_back(dpo::Pending{t, graph, source, out});
  if (ticket) *ticket = t;
  return DPO_OK;
}

dpo_status dpo_engine_step(dpo_engine* e, int32_t* running, int32_t* pending) {
  if (!e) return DPO_ERR_ARG;
  dpo::Runtime& r = dpo::rt();
  dpo_status s;
  {
    std::lock_guard<std::mutex> lock(r.mu);
    s = dpo::engine_step(e);
  }
  if (running) *running = e->running;
  if (pending) *pending = (int32_t)e->pending.size();
  return s;
}

int32_t dpo_engine_poll(dpo_engine* e, uint64_t* tickets, int32_t cap) {
  if (!e || !tickets || cap < 1) return 0;
  int32_t k = 0;
  while (k < cap && !e->completed.empty()) {
    tickets[k++] = e->completed.front();
    e->completed.pop_front();
  }
  return k;
}

void dpo_engine_destroy(dpo_engine* e) {
  if (!e) return;
  if (e->inflight) (void)hipStreamSynchronize(e->sr.stream);
  if (e->exec) (void)hipGraphExecDestroy(e->exec);
  if (e->plain) (void)hipGraphExecDestroy(e->plain);
  if (e->retired) (void)hipEventDestroy(e->retired);
  if (e->hflags) (void)hipHostFree(e->hflags);
  delete e;
}

}  // extern "C"


extern "C" {

void dpo_default_options(dpo_options* o) {
  if (!o) return;
  o->mode = DPO_MODE_NESTED;
  o->threshold = 128;
  o->coarsen = 8;
  o->agg = DPO_AGG_MULTIBLOCK;
  o->agg_blocks = 4;
  o->child_block = 256;
  o->steps_per_replay = 0;
  o->agg_threshold = 0;
  o->split_min = 65536;
  o->serial_wave = 1;
  o->dyn_share = 0;
  o->claim_hint = DPO_HINT_AUTO;
}

size_t dpo_workspace_bytes(const dpo_csr* g, const dpo_options* o) {
  if (!g || !o || g->n < 1 || dpo::check_options(*o) != DPO_OK) return 0;
  return dpo::layout_for(dpo::round32(g->n), 1, *o).total;
}

int64_t dpo_batch_slots(const dpo_arena* ar, const dpo_query* q, int32_t nq, int64_t* slot0) {
  if (!q || nq < 1 || dpo::check_arena(ar, false) != DPO_OK) return -1;
  return dpo::batch_slots(ar, q, nq, slot0);
}

size_t dpo_batch_workspace_bytes(const dpo_arena* ar, const dpo_query* q, int32_t nq,
                                 const dpo_options* o) {
  if (!o || dpo::check_options(*o) != DPO_OK || nq < 1 || nq > dpo::MAX_QUERIES) return 0;
  const int64_t slots = dpo_batch_slots(ar, q, nq, nullptr);
  if (slots < 1) return 0;
  return dpo::layout_for(slots, nq, *o).total;
}

dpo_status dpo_bfs_batch(const dpo_arena* ar, const dpo_query* q, int32_t nq,
                         const dpo_options* bucket_opts, int32_t nbuckets, int32_t* levels,
                         void* ws, size_t ws_bytes, void* stream, dpo_stats* st) {
  return dpo::traverse_batch(dpo::PROB_BFS, ar, q, nq, bucket_opts, nbuckets, levels, ws, ws_bytes,
                             stream, st);
}

dpo_status dpo_sssp_batch(const dpo_arena* ar, const dpo_query* q, int32_t nq,
                          const dpo_options* bucket_opts, int32_t nbuckets, uint32_t* dist,
                          void* ws, size_t ws_bytes, void* stream, dpo_stats* st) {
  return dpo::traverse_batch(dpo::PROB_SSSP, ar, q, nq, bucket_opts, nbuckets, dist, ws, ws_bytes,
                             stream, st);
}

dpo_status dpo_bfs(const dpo_csr* g, int32_t source, const dpo_options* o, int32_t* levels,
                   void* ws, size_t ws_bytes, void* stream, dpo_stats* st) {
  return dpo::traverse(dpo::PROB_BFS, g, source, o, levels, ws, ws_bytes, stream, st);
}

dpo_status dpo_sssp(const dpo_csr* g, int32_t source, const dpo_options* o, uint32_t* dist,
                    void* ws, size_t ws_bytes, void* stream, dpo_stats* st) {
  return dpo::traverse(dpo::PROB_SSSP, g, source, o, dist, ws, ws_bytes, stream, st);
}

dpo_status dpo_bfs_noalloc(const dpo_csr* g, int32_t source, const dpo_options* o, int32_t* levels,
                           void* stream) {
  return dpo::traverse_noalloc(dpo::PROB_BFS, g, source, o, levels, stream);
}

dpo_status dpo_traverse_timed(int32_t kind, const dpo_csr* g, int32_t source, const dpo_options* o,
                              void* out, void* ws, size_t ws_bytes, void* stream, void* timing,
                              size_t timing_bytes) {
  if ((kind != 0 && kind != 1) || !timing || timing_bytes < (size_t)DPO_TIMING_BYTES)
    return DPO_ERR_ARG;
  return dpo::traverse(kind == 0 ? dpo::PROB_BFS : dpo::PROB_SSSP, g, source, o, out, ws, ws_bytes,
                       stream, nullptr, (unsigned long long*)timing);
}

const char* dpo_strerror(int32_t status) {
  switch (status) {
    case DPO_OK: return "ok";
    case DPO_ERR_ARG: return "invalid argument";
    case DPO_ERR_SOURCE: return "source vertex out of range";
    case DPO_ERR_WORKSPACE: return "workspace too small";
    case DPO_ERR_CAPACITY: return "device queue capacity exceeded";
    case DPO_ERR_TIMEOUT: return "device wait exceeded its watchdog or level cap";
    case DPO_ERR_HIP: return "HIP runtime error";
    case DPO_ERR_UNSUPPORTED: return "option combination not built";
    default: return "unknown status";
  }
}

}  // extern "C"
