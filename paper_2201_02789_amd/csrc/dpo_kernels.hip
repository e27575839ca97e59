// Device code: level-synchronous nested-parallel BFS / SSSP for gfx950.
//
// A level step is two kernels, the parent kernel and the child kernel; for SSSP
// the parent kernel's second pass (the thresholded children) runs as a third
// kernel after the child kernel, and with found bytes (Args::hint) a harvest
// kernel ends the level.  Levels for which that is not the shortest way are run
// by other kernels, each described where it stands: narrow BFS levels by one
// workgroup (narrow_kernel), wide ones of a symmetric graph bottom-up
// (bottom_up_kernel; queries of a batch or engine: tally_kernel,
// bottom_up_words_kernel, bottom_up_queries_kernel; symmetry_kernel checks the
// graph), whole SSSP traversals of small graphs (solo_kernel) and of sparse ones
// (near_kernel) by one workgroup.
//
// Parent kernel: the parent grid.  Workgroups (256 lanes = 4 wave64) take
// virtual parent blocks of 256 frontier entries (fewer when a BFS frontier would
// leave workgroups without one) in a grid-stride loop; lane i
// is the parent thread of frontier vertex u with child-thread count deg(u)
// (Sec. III-D):
//
//   deg == 0            nothing to do
//   0 < deg < T         thresholding (Sec. III-B): the parent runs the child
//                       body for each neighbour itself, serially
//   deg >= max(T, 1)    launch: gDim = ceil(deg / CB) original child blocks,
//                       coarsened to ceil(gDim / CF) blocks (Sec. IV-B); the
//                       parent writes a launch record {row start, deg, scanned
//                       offset, parent value} and takes part in aggregation
//
// Aggregation (Sec. II-B, V-A) fuses the child grids of a group of parents
// into one grid: an exclusive scan of the coarsened grid sizes gives each
// record its offset.  Granularities: none (each parent publishes its own
// grid), wave (64 parents), block (256 parents) and multi-block (k blocks).
// Multi-block groups take their record slot and offset from one packed 64-bit
// atomic per group (hi = records, lo = child blocks; Sec. V-A increments both
// counters as one integer), pre-aggregated per block; a group-wide done
// counter picks the last block, which publishes the aggregated grid.
//
// HIP has no device-side launch.  "Publishing" appends a descriptor {record
// base, record count, child-block base} to one of eight queues through a
// packed 64-bit counter (hi = descriptors, lo = child blocks), so block bases
// grow with the descriptor index.  The launch itself is the stream-ordered
// child kernel that follows: the kernel boundary makes records visible
// without the release/acquire fences an in-kernel hand-off would need.
//
// Child kernel: the aggregated child grids.  Workgroup w runs a contiguous
// share of the child blocks, finds the parent of its first block by 64-ary
// wave searches of the descriptor bases and the scanned record offsets (the
// disaggregation of Sec. V-A), then advances along the scanned offsets.  Each
// coarsened block runs the coarsening loop over CF original blocks of CB lanes
// (Sec. IV-B) with coalesced col_idx reads.
//
// Child body: BFS probes a visited bitmap (one bit per output slot,
// L2-resident), claims v in a second bitmap and writes its level; SSSP relaxes
// a second distance array with atomicMin and queues v once per iteration
// through an iteration stamp, or, with found bytes (single traversals, batches
// and engines of dense graphs), records v as found and leaves the queueing to
// the harvest kernel.
// The probed and the updated copies swap every level.  BFS with found bytes
// instead gives each XCD a probed copy of its own on wide levels and records
// discoveries as bytes, which the harvest kernel turns into levels and the next
// frontier (Vis, vis_of, harvest_kernel).
//
// Queries: a launch may carry many traversals ("queries") over graphs packed
// in one CSR arena.  Query q owns the output slots [slot0, slot0 + n) (slot0 a
// multiple of 32, so bitmap words never straddle queries); frontier entries
// are slots.  A single traversal is a batch of one.  Queries may start at
// different level indices (continuous batching): a vertex found at level
// index L + 1 gets level L + 1 - lstart.  New frontier vertices are
// staged per wave in LDS and appended to one of 64 frontier queues with one
// atomic per flush, so no counter sees more than a few dozen atomics a level.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dpo_internal.h"
#include "dpo_pair.h"

namespace dpo {

__device__ __forceinline__ uint32_t lane_rank(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  return x;
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Keeps the compiler from moving the first use of a loaded value up into the
// branch that loads it.  Where a batch's loads (or atomics) are predicated, it
// does that whenever a use is needed on that branch only, and each of them then
// waits for its own round trip before the next is issued.
__device__ __forceinline__ void pin(uint32_t& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(int32_t& x) { asm volatile("" : "+v"(x)); }

template <int U, typename T>
__device__ __forceinline__ void pin(T (&x)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) pin(x[u]);
}

__device__ __forceinline__ void set_error(State* st, uint32_t code) {
  atomicCAS(&st->error, 0u, code);
}

__device__ __forceinline__ uint32_t ceil_div(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

// ------------------------------------------------------------ frontier queues
// Next frontier = NQF queues of fcap slots plus an overflow queue of n slots.
struct Reserve {
  uint32_t q, pos, inseg, obase;
};

// Reserve `cnt` slots in queue q (one lane).  Slots past fcap spill into the
// overflow queue.
__device__ __forceinline__ Reserve reserve_slots(const Args& a, LevelSet* ls, uint32_t q,
                                                 uint32_t cnt) {
  Reserve r{q, 0u, 0u, 0u};
  const uint32_t old = atomicAdd(&ls->fcnt[q], cnt);
  r.pos = old;
  r.inseg = old >= (uint32_t)a.fcap ? 0u : min(cnt, (uint32_t)a.fcap - old);
  if (r.inseg < cnt) {
    const uint32_t rest = cnt - r.inseg;
    r.obase = atomicAdd(&ls->fcnt[NQF], rest);
    if ((uint64_t)r.obase + rest > (uint64_t)a.slots) set_error(a.st, ERR_CAPACITY);
  }
  return r;
}

__device__ __forceinline__ void put_slot(const Args& a, int32_t* buf, const Reserve& r, uint32_t p,
                                         int32_t v) {
  if (p < r.inseg) {
    buf[(size_t)r.q * a.fcap + r.pos + p] = v;
  } else {
    const uint32_t o = r.obase + (p - r.inseg);
    if (o < (uint32_t)a.slots) buf[(size_t)NQF * a.fcap + o] = v;
  }
}

struct Stage {
  int32_t* buf;  // STAGE LDS slots owned by this wave
  uint32_t cnt;  // wave-uniform fill
};

// Flush one wave's staged vertices (wave-uniform call).
__device__ __forceinline__ void stage_flush(Stage& s, const Args& a, LevelSet* ls, int32_t* fout,
                                         int lane) {
  if (s.cnt == 0) return;
  Reserve r{0u, 0u, 0u, 0u};
  if (lane == 0) r = reserve_slots(a, ls, blockIdx.x % NQF, s.cnt);
  r.q = __shfl(r.q, 0, 64);
  r.pos = __shfl(r.pos, 0, 64);
  r.inseg = __shfl(r.inseg, 0, 64);
  r.obase = __shfl(r.obase, 0, 64);
  wave_lds_sync();
  for (uint32_t i = lane; i < s.cnt; i += 64) put_slot(a, fout, r, i, s.buf[i]);
  wave_lds_sync();
  s.cnt = 0;
}

// Wave-uniform call: every lane of the wave must reach it.
__device__ __forceinline__ void stage_push(Stage& s, bool found, int32_t v, const Args& a,
                                           LevelSet* ls, int32_t* fout, int lane) {
  const unsigned long long m = __ballot(found);
  if (m == 0) return;
  const uint32_t c = (uint32_t)__popcll(m);
  if (s.cnt + c > STAGE) stage_flush(s, a, ls, fout, lane);
  if (found) s.buf[s.cnt + lane_rank(m)] = v;
  s.cnt += c;
}

// End of kernel: one reservation for the whole workgroup.  Block-uniform call.
__device__ __forceinline__ void block_flush(Stage& s, const Args& a, LevelSet* ls, int32_t* fout, int tid,
                            uint32_t* s_cnt /* LDS [NW + 5] */) {
  const int lane = tid & 63, wave = tid >> 6;
  if (lane == 0) s_cnt[wave] = s.cnt;
  __syncthreads();
  if (tid == 0) {
    uint32_t tot = 0;
    for (int w = 0; w < NW; ++w) tot += s_cnt[w];
    Reserve r{0u, 0u, 0u, 0u};
    if (tot) r = reserve_slots(a, ls, blockIdx.x % NQF, tot);
    s_cnt[NW] = tot;
    s_cnt[NW + 1] = r.q;
    s_cnt[NW + 2] = r.pos;
    s_cnt[NW + 3] = r.inseg;
    s_cnt[NW + 4] = r.obase;
  }
  __syncthreads();
  if (s_cnt[NW] == 0) return;
  const Reserve r{s_cnt[NW + 1], s_cnt[NW + 2], s_cnt[NW + 3], s_cnt[NW + 4]};
  uint32_t off = 0;
  for (int w = 0; w < wave; ++w) off += s_cnt[w];
  for (uint32_t i = lane; i < s.cnt; i += 64) put_slot(a, fout, r, off + i, s.buf[i]);
  s.cnt = 0;
}

// ------------------------------------------------------------ child body
// Per-element context: query bounds and where its outputs live.
struct Elem {
  int32_t vbase;  // graph vertex 0 in the CSR arena
  int32_t n;      // graph vertices
  int32_t sbase;  // slot0 - vbase: slot of global vertex v is v + sbase
  int32_t lv;     // level value written for a discovery (BFS)
  uint32_t du;    // parent distance (SSSP)
};

// Visited state in two copies.  Device atomics on lines that other waves keep
// probing with plain loads run more than ten times slower on this chip than
// atomics on lines that only atomics touch.  So a level with a wide frontier
// probes one copy, read-only for the whole level, and sends its atomics to the
// other ("split"); the copies swap at the next level.  A level with a narrow
// frontier probes and updates one copy, which keeps the atomic next to the
// probed line and the level short.  At the start of a level the probed copy is
// complete.  A split level folds its frontier's own vertices (the previous
// level's discoveries / improvements) into the copy it updates, which then
// lacks exactly those; SSSP folds at every level, so the unprobed array always
// lacks just the frontier's improvements.  A one-copy BFS level skips the fold
// and marks the other bitmap stale (it only ever holds visited vertices); the
// next split level then folds every non-zero word of the probed bitmap.
// BFS: buffer i is the bitmap visit + i * vwords.  SSSP: buffer 0 is the
// output distance array, buffer 1 the workspace one; both hold the result at
// the end (the last level improves nothing, so its fold leaves them equal).
struct Vis {
  const uint32_t* probe;  // read with plain loads
  uint32_t* claim;        // the level's claims / atomicMin
  uint32_t* fold;         // receives the frontier's vertices / distances
  bool split;
  uint32_t* own;          // BFS with per-XCD copies: this XCD's copy (= probe)
};

// BFS with per-XCD copies (Args::hint): bitmap c is the visited set (0, until a
// bottom-up level leaves it in the other one).  On a wide level (split) it does
// not change until the harvest kernel, and each XCD
// (workgroup % 8) probes its own bitmap, which holds bitmap 0 as of the
// level's start plus the vertices this XCD has found since, kept with plain
// loads and stores that stay in its L2; a narrow level probes and claims
// bitmap c with atomics and appends in place.
template <int P>
__device__ __forceinline__ Vis vis_of(const Args& a, uint32_t c, bool split) {
  if (P == PROB_BFS && a.hint) {
    uint32_t* all = a.visit + (size_t)c * (uint32_t)a.vwords;
    if (!split) return Vis{all, all, nullptr, false, nullptr};
    uint32_t* own = a.visit + (size_t)(2u + (blockIdx.x & (NHINT - 1))) * (uint32_t)a.vwords;
    return Vis{own, all, nullptr, false, own};
  }
  uint32_t* b0 = P == PROB_BFS ? a.visit : a.dist;
  uint32_t* b1 = P == PROB_BFS ? a.visit + a.vwords : a.dist2;
  uint32_t* pb = c ? b1 : b0;
  uint32_t* ob = c ? b0 : b1;
  return Vis{pb, split ? ob : pb, ob, split, nullptr};
}

__device__ __forceinline__ uint32_t coherent_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// SSSP bounds (Args::bound): a byte per vertex, not decreasing in the distance:
// three bits below the leading one (exact up to 16, then eight steps an octave).
// A sum whose byte is above that of any distance the vertex has had is above
// that distance itself.
__device__ __forceinline__ uint32_t bound_of(uint32_t d) {
  const int32_t b = (int32_t)(__float_as_uint((float)d) >> 20) - (127 << 3);
  return (uint32_t)min(max(b, 0), 255);
}

// Child body for U neighbours per lane (v < 0: none), all probes issued before
// any atomic so that the U round trips overlap.  BFS: probe, then claim the
// unvisited ones and write their level (per-XCD copies: record them as found).
// SSSP: relax (atomicMin) the edges that improve on the probed distance; an
// improved vertex joins the next frontier once per level (iteration stamp
// exchanged atomically, or a found byte that the harvest kernel reads).
// out[u] is the slot to append to the next frontier, or -1.
template <int P, int U>
__device__ __forceinline__ void visit_batch(const Args& a, const Vis& vis, const int32_t (&v)[U],
                                            const uint32_t (&w)[U], const Elem (&c)[U],
                                            uint32_t L, int32_t (&out)[U]) {
  int32_t sl[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    sl[u] = -1;
    if (v[u] >= 0) {
      const int32_t loc = v[u] - c[u].vbase;
      if ((uint32_t)loc >= (uint32_t)c[u].n) set_error(a.st, ERR_ARG);
      else sl[u] = v[u] + c[u].sbase;
    }
    out[u] = -1;
  }
  if (P == PROB_BFS) {
    const uint32_t* pb = vis.probe;
    uint32_t* cb = vis.claim;
    uint32_t word[U];
#pragma unroll
    for (int u = 0; u < U; ++u) word[u] = sl[u] >= 0 ? pb[(uint32_t)sl[u] >> 5] : ~0u;
    pin(word);
    // Per-XCD copies (wide level): a candidate records itself in its XCD's
    // copy and in the found bytes, both plain stores, and nothing else: no
    // atomic, no level, no append.  The harvest kernel after the level takes
    // every found vertex that bitmap 0 (visited before the level) lacks, so
    // the level's discoveries cost no device atomics, which the chip runs at
    // a few tens of G/s for random addresses.  A set bit in the copy means a
    // lane of this XCD found the vertex at this level, or it was visited
    // before; a stale or lost bit only lets a second found store through.
    if (vis.own) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t bit = 1u << (sl[u] & 31);
        if (sl[u] >= 0 && !(word[u] & bit)) {
          vis.own[(uint32_t)sl[u] >> 5] = word[u] | bit;
          a.found[sl[u]] = 1;
        }
      }
      return;
    }
    // Two shared copies (split level): vertices found earlier in this level
    // are still clear in the probed bitmap; a batch with many candidates reads
    // the claim words with coherent loads first, with few that round trip
    // would only add latency.
    bool filter = false;
    if (vis.split) {
      uint32_t ncand = 0;
#pragma unroll
      for (int u = 0; u < U; ++u)
        ncand += (uint32_t)__popcll(__ballot(sl[u] >= 0 && !(word[u] & (1u << (sl[u] & 31)))));
      filter = ncand > PRECHECK_MIN;
    }
    if (filter) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (sl[u] >= 0 && !(word[u] & (1u << (sl[u] & 31))))
          word[u] = coherent_load(&cb[(uint32_t)sl[u] >> 5]);
      pin(word);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t bit = 1u << (sl[u] & 31);
      if (sl[u] >= 0 && !(word[u] & bit)) word[u] = atomicOr(&cb[(uint32_t)sl[u] >> 5], bit);
      else word[u] = ~0u;
    }
    pin(word);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!(word[u] & (1u << (sl[u] & 31)))) {
        a.level[sl[u]] = c[u].lv;
        out[u] = sl[u];
      }
    }
  } else {
    const uint32_t* dp = vis.probe;
    uint32_t* dl = vis.claim;
    uint32_t nd[U], cur[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // saturating: a walk of 2^32 - 1 or more never improves a distance, so
      // no wrapped sum can undercut the true one
      const uint32_t sum = c[u].du + w[u];
      nd[u] = sum < c[u].du ? 0xFFFFFFFFu : sum;
    }
    // Most edges improve nothing, and most of those miss by far: a byte per
    // vertex, which each L2 holds for all of them, tells before the distance is
    // read.
    if (a.bound) {
#pragma unroll
      for (int u = 0; u < U; ++u) cur[u] = sl[u] >= 0 ? a.bound[sl[u]] : 0u;
      pin(cur);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (sl[u] >= 0 && bound_of(nd[u]) > cur[u]) sl[u] = -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = sl[u] >= 0 ? dp[sl[u]] : 0u;
    pin(cur);
    // Many candidates: the claim array first, with coherent loads, so that an
    // atomic is issued only for what is still an improvement.  Found bytes on few
    // slots: no lane waits for the atomic then, and that round trip costs more than
    // it saves (us, with / without: Erdos-Renyi of 1 M vertices, degree 16, 1,890 /
    // 1,675, R-MAT of 250 K 820 / 792, a batch of 64 796 / 782; at scale 21, where
    // the atomics leave L2, 1,860 / 1,884).
    uint32_t ncand = 0;
    if (vis.split && (!a.hint || a.bound)) {
#pragma unroll
      for (int u = 0; u < U; ++u) ncand += (uint32_t)__popcll(__ballot(sl[u] >= 0 && nd[u] < cur[u]));
    }
    const bool pre = ncand > PRECHECK_MIN;
    if (pre) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (sl[u] >= 0 && nd[u] < cur[u]) cur[u] = coherent_load(&dl[sl[u]]);
      pin(cur);
    }
    // Found bytes (Args::hint): an improved vertex is recorded with a plain
    // byte store and queued once by the harvest kernel after the level.  No lane
    // waits for its atomicMin: a candidate that comes second was undercut during
    // this level (what it read was no lower than the distance at the level's
    // start), by a lane that set the same byte.
    // R-MAT of 70,001 vertices 791 -> 765 us, of 1 M 1,729 -> 1,658.
    if (a.hint) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (sl[u] >= 0 && nd[u] < cur[u]) {
          atomicMin(&dl[sl[u]], nd[u]);
          a.found[sl[u]] = 1;
        }
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (sl[u] >= 0 && nd[u] < cur[u]) cur[u] = atomicMin(&dl[sl[u]], nd[u]);
      else cur[u] = 0u;
    }
    pin(cur);
    const uint32_t it = L + 1;
    uint32_t stamp[U];
#pragma unroll
    for (int u = 0; u < U; ++u) stamp[u] = (pre && nd[u] < cur[u]) ? coherent_load(&a.visit[sl[u]]) : 0u;
    pin(stamp);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (nd[u] < cur[u] && stamp[u] != it) stamp[u] = atomicExch(&a.visit[sl[u]], it);
      else stamp[u] = it;
    }
    pin(stamp);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (stamp[u] != it) out[u] = sl[u];
  }
}

struct Counters {
  uint32_t front, serial, rec, child, eser, echild, desc;
};

// Per-workgroup counters: one row per workgroup, summed on the host.
__device__ __forceinline__ void add_stats(const Args& a, unsigned long long* s_stats,
                                          const Counters& c, int tid) {
  if (!a.count_stats) return;
  if (c.front) atomicAdd(&s_stats[S_FRONT], (unsigned long long)c.front);
  if (c.serial) atomicAdd(&s_stats[S_SERIAL], (unsigned long long)c.serial);
  if (c.rec) atomicAdd(&s_stats[S_REC], (unsigned long long)c.rec);
  if (c.child) atomicAdd(&s_stats[S_CHILD], (unsigned long long)c.child);
  if (c.eser) atomicAdd(&s_stats[S_ESER], (unsigned long long)c.eser);
  if (c.echild) atomicAdd(&s_stats[S_ECHILD], (unsigned long long)c.echild);
  if (c.desc) atomicAdd(&s_stats[S_DESC], (unsigned long long)c.desc);
  __syncthreads();
  if (tid < NSTAT && blockIdx.x < MAX_GRID) a.stats[blockIdx.x * NSTAT + tid] += s_stats[tid];
}

// Phase clock of one wave, for the timed instantiations (ON = false: empty).
// mark(p) charges the shader-clock cycles since the previous mark to phase p,
// after the wave's outstanding memory operations have completed, so each
// phase pays for the loads and stores it issued.  Marks sit only at points
// that every lane of the wave reaches together, so the clock values stay
// wave-uniform.
template <bool ON>
struct PhaseClock {
  uint64_t last = 0;
  uint64_t acc[TP_N] = {0, 0, 0, 0, 0};
  __device__ __forceinline__ void start() {
    if (ON) last = __builtin_amdgcn_s_memtime();
  }
  __device__ __forceinline__ void mark(int p) {
    if (!ON) return;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    const uint64_t now = __builtin_amdgcn_s_memtime();
    acc[p] += now - last;
    last = now;
    __builtin_amdgcn_sched_barrier(0);
  }
};

__device__ __forceinline__ uint64_t realtime() { return __builtin_amdgcn_s_memrealtime(); }

// Timed instantiations: the workgroup's row (entry / exit realtime, cycles per
// phase summed over its waves, the busiest wave's total).  Block-uniform call.
template <bool ON>
__device__ __forceinline__ void tm_write(const Args& a, const PhaseClock<ON>& pc, int kind,
                                         uint32_t L, uint64_t t_entry, int tid) {
  if (!ON) return;
  __shared__ unsigned long long s_tm[NW][TP_N];
  const int lane = tid & 63, wave = tid >> 6;
  if (lane == 0)
    for (int p = 0; p < TP_N; ++p) s_tm[wave][p] = pc.acc[p];
  __syncthreads();
  if (tid == 0 && L < (uint32_t)TM_LEVELS && blockIdx.x < (uint32_t)MAX_GRID) {
    unsigned long long sum[TP_N] = {0, 0, 0, 0, 0}, mx = 0;
    for (int w = 0; w < NW; ++w) {
      unsigned long long t = 0;
      for (int p = 0; p < TP_N; ++p) {
        sum[p] += s_tm[w][p];
        t += s_tm[w][p];
      }
      mx = t > mx ? t : mx;
    }
    unsigned long long* row =
        a.tm + ((size_t)(L * TM_KINDS + (uint32_t)kind) * MAX_GRID + blockIdx.x) * TM_ROW;
    row[0] = t_entry;
    row[1] = realtime();
    for (int p = 0; p < TP_N; ++p) row[2 + p] = sum[p];
    row[7] = mx;
  }
}

// A level of a single traversal that the bottom-up kernel runs.  Uniform over a
// launch: the symmetry check's sums are complete when its kernel ends.
__device__ __forceinline__ bool found_symmetric(const State* st) {
  unsigned long long sum = 0;
  for (int i = 0; i < 8; ++i) sum += st->sym_sum[i];
  return sum == 0 && !st->asymmetric;
}

__device__ __forceinline__ bool goes_bottom_up(const State* st) {
  return st->plan == V_BOTTOM_UP || (st->plan == V_CHECK && found_symmetric(st));
}

// Does query q go bottom-up at level L?  Its frontier's edges against those it
// has not run, and against what the level would read and find, as for a single
// traversal (BU_ALPHA, BU_QUERY_READ).  The tallies do not change between the tally
// kernel of a level and the next level's.
__device__ __forceinline__ bool query_goes_bottom_up(const Args& a, uint32_t q, uint32_t L) {
  const uint32_t* t = a.tally;
  const uint32_t nq = (uint32_t)a.nq, E = t[(L & 1) * nq + q];
  if (E < BU_QUERY_EDGES) return false;
  const uint32_t before = t[2 * nq + q] - E, m = t[3 * nq + q];
  return (uint64_t)E * BU_ALPHA >= (m > before ? m - before : 0u) &&
         (uint64_t)t[4 * nq + q] * 2 <= ((uint64_t)E + t[5 * nq + q]) * BU_QUERY_READ;
}

// Append one aggregated grid to descriptor queue q (one lane).
__device__ __forceinline__ void publish(const Args& a, LevelSet* ls, uint32_t q, uint32_t rec_base,
                                        uint32_t nrec, uint32_t total) {
  const unsigned long long old =
      atomicAdd(&ls->qctr[q], ((unsigned long long)1 << 32) | (unsigned long long)total);
  const uint32_t d = (uint32_t)(old >> 32);
  if (d >= (uint32_t)a.desc_cap) {
    set_error(a.st, ERR_CAPACITY);
    return;
  }
  a.desc[(size_t)q * a.desc_cap + d] = make_int4((int32_t)rec_base, (int32_t)nrec, (int32_t)old, 0);
}

// Launch record `r` of the level: the parent's row, child count, scanned
// offset of its coarsened grid and distance; its query; for SSSP its slot.
template <int P>
__device__ __forceinline__ void put_record(const Args& a, uint32_t r, int32_t start, int32_t deg,
                                           uint32_t off, uint32_t du, int32_t q, int32_t slot) {
  a.rec[r] = make_int4(start, deg, (int32_t)off, (int32_t)du);
  a.rec_q[r] = q;
  if (P == PROB_SSSP) a.rec_slot[r] = slot;
}

// Frontier entry i of level L: queue q with s_fpre[q] <= i < s_fpre[q + 1].
__device__ __forceinline__ int32_t frontier_at(const Args& a, const int32_t* fin,
                                               const uint32_t* s_fpre, uint32_t i) {
  uint32_t lo = 0, hi = NQF + 1;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (s_fpre[mid] <= i) lo = mid; else hi = mid;
  }
  return fin[(size_t)lo * a.fcap + (i - s_fpre[lo])];
}


// One parent thread: its query, vertex, row and parameters.
struct Parent {
  int32_t start, deg, T, CF, slot;
  uint32_t q;
  Elem e;
};

template <int P>
__device__ __forceinline__ Parent load_parent(const Args& a, const int32_t* fin,
                                              const uint32_t* s_fpre, uint32_t i, uint32_t L) {
  Parent p;
  p.slot = frontier_at(a, fin, s_fpre, i);
  p.q = (uint32_t)a.qmap[(uint32_t)p.slot >> 5];
  const Query Q = a.q[p.q];
  const int32_t vg = Q.vbase + (p.slot - Q.slot0);
  p.start = a.rp[vg];
  p.deg = a.rp[vg + 1] - p.start;
  p.T = Q.T;
  p.CF = Q.CF;
  p.e.vbase = Q.vbase;
  p.e.n = Q.n;
  p.e.sbase = Q.slot0 - Q.vbase;
  p.e.lv = (int32_t)(L + 1) - Q.lstart;
  p.e.du = 0;
  return p;
}

// Multi-block groups: virtual block vb of the level's nvb is through; true for
// its group's last one (one lane), which publishes the group's grid.
__device__ __forceinline__ bool group_block_done(const Args& a, uint32_t vb, uint32_t nvb, uint32_t L) {
  const uint32_t g = vb / (uint32_t)a.k;
  const uint32_t in_group = min((uint32_t)a.k, nvb - g * (uint32_t)a.k);
  return atomicAdd(&a.grp_done[(L % 3) * a.ngroups_cap + g], 1u) == in_group - 1;
}

// epb: frontier entries per virtual block
__device__ __forceinline__ void publish_group(const Args& a, LevelSet* ls, uint32_t vb, uint32_t epb,
                                              uint32_t L, uint32_t& descs) {
  const uint32_t g = vb / (uint32_t)a.k;
  const unsigned long long tot = atomicAdd(&a.grp_packed[(L % 3) * a.ngroups_cap + g], 0ull);
  const uint32_t nrec = (uint32_t)(tot >> 32);
  if (nrec == 0) return;
  publish(a, ls, g % NQD, g * (uint32_t)a.k * epb, nrec, (uint32_t)tot);
  ++descs;
}

// ------------------------------------------------------------ parent kernel
// Pass 1 reads each frontier entry once, decides it (threshold), aggregates
// the launching ones and writes their records (block barriers) and lists the
// thresholded ones; pass 2 runs the listed parents' serial children with no
// barrier, so waves do not wait on each other.
//
// PH = PH_BOTH runs both passes.  PH_LIST runs pass 1 only and leaves the
// workgroup's list length in a.sercnt; PH_SERIAL, launched after the level's
// child kernel on the same grid, runs pass 2 over that list (SSSP: its parents
// are then checked against every improvement the launched children made).
template <int P, int G, int PH, bool TM>
__global__ __launch_bounds__(PB) void parent_kernel(Args a, uint32_t step) {
  __shared__ int32_t s_stage[NW][STAGE];
  __shared__ uint32_t s_fpre[NQF + 2];
  __shared__ uint32_t s_scan[2 * NW];
  __shared__ uint32_t s_bc[NW + 8];
  __shared__ unsigned long long s_stats[NSTAT];
  __shared__ uint32_t s_live[MAX_QUERIES / 32];  // queries seen at this level
  __shared__ uint32_t s_up[P == PROB_BFS ? MAX_QUERIES / 32 : 1];  // queries that go bottom-up
  // virtual blocks with entries of others (wrapping round: a bit too many only
  // costs its block's time)
  constexpr int SOME_WORDS = P == PROB_BFS ? 32 : 1;
  __shared__ uint32_t s_some[SOME_WORDS];
  __shared__ uint32_t s_ser[2];                  // serial list: length, next entry
  __shared__ uint32_t s_soff[NW][64];            // per wave: scanned child sizes of a group
  __shared__ uint32_t s_lpre[PH == PH_SERIAL ? MAX_GRID + 1 : 1];  // prefix of list lengths

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  State* st = a.st;
  uint64_t t_entry = 0;
  if (TM) t_entry = realtime();
  PhaseClock<TM> pc;
  pc.start();
  if (st->done || st->error) return;
  const uint32_t L = st->base + step;
  LevelSet* prv = &st->set[(L + 2) % 3];  // fills of frontier L
  LevelSet* cur = &st->set[L % 3];        // this level: next-frontier fills, queues, groups
  const int32_t* fin = (L & 1) ? a.front1 : a.front0;
  int32_t* fout = (L & 1) ? a.front0 : a.front1;

  // frontier L = queues 0..NQF-1 then overflow; prefix of their fills
  if (wave == 0) {
    const uint32_t c = min(prv->fcnt[lane], (uint32_t)a.fcap);
    const uint32_t incl = wave_incl_scan(c, lane);
    s_fpre[lane + 1] = incl;
    if (lane == 0) s_fpre[0] = 0;
    if (lane == 63) s_fpre[NQF + 1] = incl + prv->fcnt[NQF];
  }
  if (tid < NSTAT) s_stats[tid] = 0;
  for (int i = tid; i < (a.nq + 31) / 32; i += PB) s_live[i] = 0;
  __syncthreads();
  const uint32_t F = s_fpre[NQF + 1];
  if (F == 0) {
    if (PH != PH_SERIAL && blockIdx.x == 0 && tid == 0) st->done = 1;
    return;
  }
  // Each vertex enters a frontier at most once per level (the claim atomic,
  // the SSSP stamp, the harvest of found bytes), and the launch records,
  // serial lists and group counters of a level are sized for that; a larger
  // frontier is an error, never an index past them.
  if (F > (uint32_t)a.slots) {
    if (tid == 0) set_error(st, ERR_CAPACITY);
    return;
  }
  // visited copies of this level (every workgroup derives the same choice)
  const uint32_t vc = st->vsel[L & 1];
  // (found bytes of queries that go bottom-up are harvested on split levels)
  const bool by_query = P == PROB_BFS && a.bottom_up == BU_QUERIES && st->symmetric == 1 && F >= TALLY_MIN;
  const bool split = F >= (uint32_t)a.split_min || by_query;
  const bool stale = st->vstale[L & 1] != 0;
  const Vis vis = vis_of<P>(a, vc, split);
  if (PH != PH_SERIAL && blockIdx.x == 0) {
    LevelSet* z = &st->set[(L + 1) % 3];  // idle until level L + 1
    if (tid <= NQF) z->fcnt[tid] = 0;
    if (tid < NQD) z->qctr[tid] = 0;
    if (tid < NQD) z->cclaim[tid][0] = 0;
    if (tid == 0) {
      st->levels_run = L + 1;
      cur->vmode = vc | (split ? 2u : 0u);  // for this level's child kernel
      st->vsel[(L + 1) & 1] = vc ^ (split && !(P == PROB_BFS && a.hint) ? 1u : 0u);
      st->vstale[(L + 1) & 1] = (P == PROB_BFS && !split) ? 1u : 0u;
    }
  }
  if (P == PROB_BFS && a.bottom_up == BU_QUERIES)
    for (int i = blockIdx.x * PB + tid; i < a.nq; i += gridDim.x * PB)
      a.tally[((L + 1) & 1) * a.nq + i] = 0;
  if (G == AGG_MULTI && PH != PH_SERIAL) {
    const uint32_t nz = (L + 1) % 3;
    for (int i = blockIdx.x * PB + tid; i < a.ngroups_cap; i += gridDim.x * PB) {
      a.grp_packed[nz * a.ngroups_cap + i] = 0;
      a.grp_done[nz * a.ngroups_cap + i] = 0;
    }
  }

  if (by_query)
    for (int i = tid; i < (a.nq + 63) / 64 * 64; i += PB) {
      const unsigned long long m = __ballot(i < a.nq && query_goes_bottom_up(a, (uint32_t)i, L));
      if ((lane & 31) == 0) s_up[i >> 5] = (uint32_t)(m >> (lane & 32));
    }

  Stage s{s_stage[wave], 0u};
  Counters cn{0, 0, 0, 0, 0, 0, 0};
  // Frontier entries per virtual block, and per wave of it: PB and 64, or fewer
  // where that would leave workgroups of the grid without a block while waves
  // have more than SPREAD_EDGES edges on average (a single
  // traversal's level that claims in the bitmap it probes: over ONE_COPY_BLOCKS at
  // most).  The groups, lists and records
  // of a level are sized for slots / PB blocks of PB entries, so never more
  // blocks than that.  A run that counts or times grids keeps blocks of PB
  // parents, and so does SSSP, whose thresholded parents are shared out evenly
  // after the lists are complete (spread as well, a batch of 64 took 2 % longer:
  // more and smaller grids).
  uint32_t epb = PB;
  if (P == PROB_BFS && PH == PH_BOTH && !TM && !a.count_stats) {
    const uint32_t most = min(split || a.nq > 1 ? gridDim.x : ONE_COPY_BLOCKS, (uint32_t)a.slots / PB);
    while ((uint64_t)epb * (uint32_t)a.m > (uint64_t)SPREAD_EDGES * NW * (uint32_t)a.n &&
           epb > (uint32_t)NW && ceil_div(F, epb / 2) <= most)
      epb /= 2;
  }
  const uint32_t epw = epb / NW;
  const uint32_t nvb = ceil_div(F, epb);
  // thresholded parents listed by this workgroup
  if (tid == 0) s_ser[0] = PH == PH_SERIAL ? a.sercnt[blockIdx.x] : 0u;
  __syncthreads();

  // Fold into the copy not probed at this level: one atomic per frontier
  // entry, or, for BFS after a one-copy level or with more frontier entries
  // than bitmap words, one per non-zero word of the probed bitmap.  BFS with
  // per-XCD copies: a wide level starts by copying bitmap vc into every XCD's
  // copy (each XCD's workgroups write their own copy), before pass 1 so that
  // pass 2 mostly probes complete copies; narrow levels keep no copy up to
  // date, which is why the next wide level copies it whole.
  const bool own = P == PROB_BFS && a.hint;
  const bool word_fold =
      !own && PH != PH_SERIAL && P == PROB_BFS && split && (stale || F > (uint32_t)a.vwords);
  const bool entry_fold = P == PROB_SSSP || (!own && split && !word_fold);
  if (own && split && PH != PH_SERIAL) {
    const bool local = gridDim.x % NHINT == 0;
    const uint32_t x0 = local ? blockIdx.x % NHINT : 0u, nx = local ? 1u : (uint32_t)NHINT;
    const uint32_t k = local ? blockIdx.x / NHINT : blockIdx.x;
    const uint32_t nk = local ? gridDim.x / NHINT : gridDim.x;
    for (uint32_t w = k * PB + tid; w < (uint32_t)a.vwords; w += nk * PB) {
      const uint32_t cw = a.visit[(size_t)vc * a.vwords + w];
      if (cw)
        for (uint32_t x = x0; x < x0 + nx; ++x) a.visit[(size_t)(2 + x) * a.vwords + w] = cw;
    }
  }
  // a workgroup with at most one virtual block keeps its thresholded parents
  // in registers (narrow levels are latency-bound)
  const bool in_regs = PH == PH_BOTH && nvb <= gridDim.x;
  int32_t e = 0, end = 0;     // this lane's serial child: edges [e, end)
  Elem ctx{0, 0, 0, 0, 0u};

  // Queries that go bottom-up: their entries are not this kernel's, and only
  // noted as live.  Which of the workgroup's virtual blocks hold others is found
  // first, four at a time, because a level has most entries when most queries go
  // bottom-up (512 queries: 13 M entries in 40 rounds of dependent loads and
  // barriers otherwise).
  auto goes_up = [&](uint32_t q) {
    const bool up = s_up[q >> 5] >> (q & 31) & 1u;
    if (up && !(s_live[q >> 5] >> (q & 31) & 1u)) atomicOr(&s_live[q >> 5], 1u << (q & 31));
    return up;
  };
  if (by_query) {
    for (int i = tid; i < SOME_WORDS; i += PB) s_some[P == PROB_BFS ? i : 0] = 0;
    __syncthreads();
    const uint32_t rounds = blockIdx.x < nvb ? (nvb - 1 - blockIdx.x) / gridDim.x + 1 : 0;
    for (uint32_t r = 0; r < rounds; r += 4) {
      uint32_t bits = 0, q[4];
      int32_t slot[4];
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c) {
        const uint64_t i =
            ((uint64_t)blockIdx.x + (uint64_t)(r + c) * gridDim.x) * epb + wave * epw + lane;
        const bool in = r + c < rounds && (uint32_t)lane < epw && i < F;
        slot[c] = in ? frontier_at(a, fin, s_fpre, (uint32_t)i) : -1;
      }
      pin(slot);
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c) q[c] = slot[c] >= 0 ? (uint32_t)a.qmap[(uint32_t)slot[c] >> 5] : 0u;
      pin(q);
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c)
        if (slot[c] >= 0 && !goes_up(q[c])) bits |= 1u << c;
#pragma unroll
      for (uint32_t c = 0; c < 4; ++c)
        if (__any(bits >> c & 1u) && lane == 0)
          atomicOr(&s_some[P == PROB_BFS ? (r + c) / 32 % SOME_WORDS : 0], 1u << ((r + c) & 31));
    }
    __syncthreads();
  }

  // ---- pass 1: every frontier entry once.  Threshold, coarsened grid size,
  // aggregation and launch records; thresholded parents go to this
  // workgroup's serial list for pass 2.
  for (uint32_t vb = blockIdx.x; vb < (PH == PH_SERIAL ? 0u : nvb); vb += gridDim.x) {
    const uint32_t i = (uint32_t)lane < epw ? vb * epb + wave * epw + lane : F;
    int32_t start = 0, deg = 0, q = 0, slot = 0;
    uint32_t du = 0, cg = 0;
    bool launch = false, ser = false;
    if (by_query) {
      const uint32_t r = (vb - blockIdx.x) / gridDim.x;
      if (!(s_some[P == PROB_BFS ? r / 32 % SOME_WORDS : 0] >> (r & 31) & 1u)) {
        // nothing here for this kernel, but its group still counts the block
        if (G == AGG_MULTI && tid == 0 && group_block_done(a, vb, nvb, L))
          publish_group(a, cur, vb, epb, L, cn.desc);
        continue;
      }
    }
    const bool mine =
        i < F && !(by_query && goes_up((uint32_t)a.qmap[(uint32_t)frontier_at(a, fin, s_fpre, i) >> 5]));
    if (mine) {
      const Parent p = load_parent<P>(a, fin, s_fpre, i, L);
      start = p.start;
      deg = p.deg;
      q = (int32_t)p.q;
      slot = p.slot;
      ++cn.front;
      if (!(s_live[p.q >> 5] >> (p.q & 31) & 1u)) atomicOr(&s_live[p.q >> 5], 1u << (p.q & 31));
      if (P == PROB_SSSP) {
        du = vis.probe[slot];
        // PH_LIST runs before any relaxation of its level, so this is the
        // entry's only writer and du is never above the value it replaces
        // (the copy lacks just the frontier's improvements): a plain store
        if (PH == PH_LIST) vis.fold[slot] = du;
        else atomicMin(&vis.fold[slot], du);
        if (a.bound) a.bound[slot] = (uint8_t)bound_of(du);
      } else if (entry_fold) {
        atomicOr(&vis.fold[(uint32_t)slot >> 5], 1u << (slot & 31));
      }
      launch = G != AGG_FLAT && deg > 0 && deg >= p.T;
      ser = deg > 0 && !launch;
      if (launch) {
        // coarsened grid size (Sec. IV-B)
        cg = ceil_div(ceil_div((uint32_t)deg, (uint32_t)a.CB), (uint32_t)p.CF);
      }
      if (ser) {
        ++cn.serial;
        if (in_regs) {
          e = start;
          end = start + deg;
          ctx = p.e;
          ctx.du = du;
        }
      }
    }
    if (!in_regs) {
      // entry k of the list sits in this workgroup's own virtual blocks
      const unsigned long long m = __ballot(ser);
      uint32_t base = 0;
      if (lane == 0 && m) base = atomicAdd(&s_ser[0], (uint32_t)__popcll(m));
      base = __shfl(base, 0, 64);
      if (ser) {
        const uint32_t k = base + lane_rank(m);
        a.ser[(size_t)(blockIdx.x + (k / PB) * gridDim.x) * PB + k % PB] =
            make_int4(start, deg, slot, (int32_t)du);
      }
    }
    pc.mark(TP_PARENT);
    if (G != AGG_FLAT) {
      if (launch) ++cn.rec;

      if (G == AGG_NONE) {
        // every launching parent publishes its own grid; its record sits at
        // its frontier index
        if (TM) {
          if (launch) put_record<P>(a, i, start, deg, 0u, du, q, slot);
          pc.mark(TP_AGG);
        }
        if (launch) {
          if (!TM) put_record<P>(a, i, start, deg, 0u, du, q, slot);
          publish(a, cur, vb % NQD, i, 1u, cg);
          ++cn.desc;
        }
        pc.mark(TP_LAUNCH);
      } else if (G == AGG_WAVE) {
        const unsigned long long m = __ballot(launch);
        const uint32_t nrec = (uint32_t)__popcll(m);
        const uint32_t seg = vb * epb + wave * epw;
        if (m && nrec < (uint32_t)a.agg_threshold) {
          // too few participants (Sec. V-B): each parent launches its own grid
          if (launch) put_record<P>(a, seg + lane_rank(m), start, deg, 0u, du, q, slot);
          pc.mark(TP_AGG);
          if (launch) {
            publish(a, cur, vb % NQD, seg + lane_rank(m), 1u, cg);
            ++cn.desc;
          }
          pc.mark(TP_LAUNCH);
        } else if (m) {  // wave-uniform
          const uint32_t incl = wave_incl_scan(cg, lane);
          const uint32_t total = __shfl(incl, 63, 64);
          if (launch) {
            put_record<P>(a, seg + lane_rank(m), start, deg, incl - cg, du, q, slot);
          }
          pc.mark(TP_AGG);
          if (lane == 0) {
            publish(a, cur, vb % NQD, seg, nrec, total);
            ++cn.desc;
          }
          pc.mark(TP_LAUNCH);
        }
      } else {
        // block-level scan of (launch, cg): wave scans, then across waves in LDS
        const unsigned long long m = __ballot(launch);
        const uint32_t incl = wave_incl_scan(cg, lane);
        if (lane == 63) {
          s_scan[wave] = (uint32_t)__popcll(m);
          s_scan[NW + wave] = incl;
        }
        __syncthreads();
        uint32_t roff = 0, coff = 0, nrec_b = 0, total_b = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          if (w < wave) { roff += s_scan[w]; coff += s_scan[NW + w]; }
          nrec_b += s_scan[w];
          total_b += s_scan[NW + w];
        }
        if (G == AGG_BLOCK) {
          const uint32_t seg = vb * epb;
          if (nrec_b < (uint32_t)a.agg_threshold) {
            // too few participants (Sec. V-B): each parent launches its own grid
            const uint32_t r = seg + roff + lane_rank(m);
            if (launch) put_record<P>(a, r, start, deg, 0u, du, q, slot);
            pc.mark(TP_AGG);
            if (launch) {
              publish(a, cur, vb % NQD, r, 1u, cg);
              ++cn.desc;
            }
            pc.mark(TP_LAUNCH);
          } else {
            if (launch) {
              put_record<P>(a, seg + roff + lane_rank(m), start, deg, coff + incl - cg, du, q, slot);
            }
            pc.mark(TP_AGG);
            if (tid == 0 && nrec_b) {
              publish(a, cur, vb % NQD, seg, nrec_b, total_b);
              ++cn.desc;
            }
            pc.mark(TP_LAUNCH);
          }
          __syncthreads();  // s_scan reuse
        } else {  // AGG_MULTI: group of k consecutive virtual blocks (Sec. V-A)
          const uint32_t g = vb / (uint32_t)a.k;
          const uint32_t seg = g * (uint32_t)a.k * epb;
          unsigned long long* gp = &a.grp_packed[(L % 3) * a.ngroups_cap + g];
          if (tid == 0) {
            unsigned long long old = 0;
            if (nrec_b)
              old = atomicAdd(gp, ((unsigned long long)nrec_b << 32) | (unsigned long long)total_b);
            s_bc[0] = (uint32_t)(old >> 32);
            s_bc[1] = (uint32_t)old;
          }
          __syncthreads();
          const uint32_t slot0 = s_bc[0], off0 = s_bc[1];
          if (launch) {
            put_record<P>(a, seg + slot0 + roff + lane_rank(m), start, deg, off0 + coff + incl - cg,
                          du, q, slot);
          }
          // the group's last block to finish "launches" the aggregated grid;
          // its packed-counter add returned before this increment was issued
          bool last_block = false;
          if (tid == 0) last_block = group_block_done(a, vb, nvb, L);
          pc.mark(TP_AGG);
          if (last_block) publish_group(a, cur, vb, epb, L, cn.desc);
          pc.mark(TP_LAUNCH);
          __syncthreads();  // s_scan / s_bc reuse
        }
      }
      pc.mark(TP_AGG);
    }
  }

  // ---- pass 2: the thresholded children (Sec. III-B: no launch; the parent's
  // own threads run the child work).
  __syncthreads();
  if (PH == PH_LIST && tid == 0) a.sercnt[blockIdx.x] = s_ser[0];
  if (PH != PH_LIST) {
    const uint32_t nser = s_ser[0];
    // This workgroup's list entries [r0, r1).  PH_SERIAL: the lists are
    // complete, and the workgroups split their concatenation evenly (a block
    // scan of the list lengths), so each runs the same number of thresholded
    // parents however many its own list holds.
    uint32_t r0 = 0, r1 = nser, nl = 0;
    if (PH == PH_SERIAL && G != AGG_FLAT && a.serial_wave) {
      nl = min(gridDim.x, nvb);
      constexpr int PER = MAX_GRID / PB;
      uint32_t vals[PER], sum = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const uint32_t l = (uint32_t)tid * PER + j;
        vals[j] = l < nl ? a.sercnt[l] : 0u;
        sum += vals[j];
      }
      const uint32_t incl = wave_incl_scan(sum, lane);
      if (lane == 63) s_scan[wave] = incl;
      __syncthreads();
      uint32_t run = incl - sum, tot = 0;
#pragma unroll
      for (int w2 = 0; w2 < NW; ++w2) {
        if (w2 < wave) run += s_scan[w2];
        tot += s_scan[w2];
      }
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const uint32_t l = (uint32_t)tid * PER + j;
        if (l < nl) s_lpre[l] = run;
        run += vals[j];
      }
      if (tid == 0) s_lpre[nl] = tot;
      r0 = (uint32_t)((uint64_t)blockIdx.x * tot / gridDim.x);
      r1 = (uint32_t)((uint64_t)(blockIdx.x + 1) * tot / gridDim.x);
    }
    if (tid == 0) s_ser[1] = r0;  // next list entry
    __syncthreads();
    constexpr int U = 8;
    if (G != AGG_FLAT && a.serial_wave) {
      // The wave runs the children of up to 64 parents together: their edges
      // are concatenated (a wave scan of the degrees) and taken 64 at a time,
      // each lane finding its parent by a search of the scanned offsets, so
      // lanes read consecutive edges and none idles while a long child runs.
      uint32_t* off = s_soff[wave];
      bool first = true;
      while (true) {
        int32_t cs = 0, cd = 0;
        Elem cc{0, 0, 0, 0, 0u};
        if (in_regs) {  // the lanes' own parents from pass 1: one group
          if (!first) break;
          cs = e;
          cd = end - e;
          cc = ctx;
          cn.eser += (uint32_t)cd;
        } else {
          uint32_t base = 0, n = 64;
          int4 r = make_int4(0, 0, 0, 0);
          if (PH == PH_SERIAL) {
            // Claim the next entries of this workgroup's range whose children
            // total at most GROUP_EDGES edges (at least one entry): groups of
            // similar length, so no wave's last group holds up its workgroup.
            while (true) {
              if (lane == 0)
                base = __hip_atomic_load(&s_ser[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              base = __shfl(base, 0, 64);
              if (base >= r1) break;
              uint32_t k = base + (uint32_t)lane;
              uint32_t dg = 0;
              if (k < r1) {
                // list holding entry k of the concatenation: the last list
                // whose prefix is <= k (empty lists share their successor's)
                uint32_t lo = 0, hi = nl;
                while (hi - lo > 1) {
                  const uint32_t mid = (lo + hi) >> 1;
                  if (s_lpre[mid] <= k) lo = mid; else hi = mid;
                }
                k -= s_lpre[lo];
                r = a.ser[(size_t)(lo + (k / PB) * gridDim.x) * PB + k % PB];
                dg = (uint32_t)r.y;
              }
              const uint32_t inc = wave_incl_scan(dg, lane);
              n = (uint32_t)__popcll(__ballot(base + (uint32_t)lane < r1 && inc <= GROUP_EDGES));
              n = max(n, 1u);
              uint32_t won = 0;
              if (lane == 0) won = atomicCAS(&s_ser[1], base, base + n) == base ? 1u : 0u;
              if (__shfl(won, 0, 64)) break;
            }
          } else {
            if (lane == 0) base = atomicAdd(&s_ser[1], 64u);
            base = __shfl(base, 0, 64);
            const uint32_t k = base + (uint32_t)lane;
            if (k < r1) r = a.ser[(size_t)(blockIdx.x + (k / PB) * gridDim.x) * PB + k % PB];
            n = base < r1 ? min(64u, r1 - base) : 0u;
          }
          if (base >= r1) break;
          if ((uint32_t)lane < n) {
            const Query Q = a.q[a.qmap[(uint32_t)r.z >> 5]];
            cs = r.x;
            cd = r.y;
            cc = Elem{Q.vbase, Q.n, Q.slot0 - Q.vbase, (int32_t)(L + 1) - Q.lstart, (uint32_t)r.w};
            // SSSP: a parent lowered again during this level expands at the next
            if (P == PROB_SSSP && coherent_load(&vis.claim[r.z]) < (uint32_t)r.w) cd = 0;
            cn.eser += (uint32_t)cd;
          }
        }
        first = false;
        const uint32_t incl = wave_incl_scan((uint32_t)cd, lane);
        const uint32_t excl = incl - (uint32_t)cd;
        const uint32_t total = __shfl(incl, 63, 64);
        wave_lds_sync();
        off[lane] = excl;
        wave_lds_sync();
        for (uint32_t x0 = 0; x0 < total; x0 += 64u * U) {
          int32_t v[U], out[U];
          uint32_t w[U];
          Elem c[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const uint32_t x = x0 + (uint32_t)u * 64u + (uint32_t)lane;
            const uint32_t xs = x < total ? x : total - 1;
            // parent of edge xs: the last lane whose offset is <= xs
            uint32_t pl = 0;
#pragma unroll
            for (uint32_t st = 32; st; st >>= 1)
              if (off[pl + st] <= xs) pl += st;
            const int32_t sp = __shfl(cs, (int)pl, 64);
            const uint32_t ep = (uint32_t)__shfl((int32_t)excl, (int)pl, 64);
            c[u] = Elem{__shfl(cc.vbase, (int)pl, 64), __shfl(cc.n, (int)pl, 64),
                        __shfl(cc.sbase, (int)pl, 64), __shfl(cc.lv, (int)pl, 64),
                        (uint32_t)__shfl((int32_t)cc.du, (int)pl, 64)};
            const int32_t ei = sp + (int32_t)(xs - ep);
            v[u] = x < total ? a.col[ei] : -1;
            w[u] = (P == PROB_SSSP && x < total) ? a.w[ei] : 0u;
          }
          pin(v);
          if (P == PROB_SSSP) pin(w);
          visit_batch<P, U>(a, vis, v, w, c, L, out);
#pragma unroll
          for (int u = 0; u < U; ++u) stage_push(s, out[u] >= 0, out[u], a, cur, fout, lane);
        }
        wave_lds_sync();  // off[] is rewritten by the next group
      }
    } else {
      // Each child runs sequentially in one lane (the paper's form; always
      // used by the flat kernel).  A lane whose child is done takes the next
      // parent of the list, so lanes do not idle until the wave's largest
      // child finishes.
      uint32_t pnow = 0xFFFFFFFFu;  // SSSP: the lane's parent distance when taken
      while (true) {
        // SSSP: a parent lowered again during this level expands at the next
        // (checked one batch after the load was issued, so nothing waits)
        if (P == PROB_SSSP && pnow < ctx.du) end = e;
        const bool idle = e >= end;
        const unsigned long long m = __ballot(idle);
        uint32_t base = 0;
        if (m) {
          if (lane == __builtin_ctzll(m)) base = atomicAdd(&s_ser[1], (uint32_t)__popcll(m));
          base = __shfl(base, __builtin_ctzll(m), 64);
        }
        if (idle) {
          const uint32_t k = base + lane_rank(m);
          if (k < nser) {
            const int4 r = a.ser[(size_t)(blockIdx.x + (k / PB) * gridDim.x) * PB + k % PB];
            const Query Q = a.q[a.qmap[(uint32_t)r.z >> 5]];
            e = r.x;
            end = r.x + r.y;
            if (P == PROB_SSSP) pnow = coherent_load(&vis.claim[r.z]);
            ctx.vbase = Q.vbase;
            ctx.n = Q.n;
            ctx.sbase = Q.slot0 - Q.vbase;
            ctx.lv = (int32_t)(L + 1) - Q.lstart;
            ctx.du = (uint32_t)r.w;
          }
        }
        if (!__any(e < end)) break;
        int32_t v[U], out[U];
        uint32_t w[U];
        Elem c[U];
#pragma unroll
        for (int r = 0; r < U; ++r) {
          v[r] = (e + r < end) ? a.col[e + r] : -1;
          w[r] = (P == PROB_SSSP && e + r < end) ? a.w[e + r] : 0u;
          c[r] = ctx;
        }
        pin(v);
        if (P == PROB_SSSP) pin(w);
        visit_batch<P, U>(a, vis, v, w, c, L, out);
#pragma unroll
        for (int r = 0; r < U; ++r) stage_push(s, out[r] >= 0, out[r], a, cur, fout, lane);
        const int32_t e2 = min(e + U, end);
        cn.eser += (uint32_t)(e2 - e);
        e = e2;
      }
    }
  }
  if (word_fold) {
    for (uint32_t w = blockIdx.x * PB + tid; w < (uint32_t)a.vwords; w += gridDim.x * PB) {
      const uint32_t x = vis.probe[w];
      if (x) atomicOr(&vis.fold[w], x);
    }
  }
  block_flush(s, a, cur, fout, tid, s_bc);
  // queries with frontier entries at this level are still running
  __syncthreads();
  if (PH != PH_SERIAL)
    for (int i = tid; i < a.nq; i += PB)
      if (s_live[i >> 5] & (1u << (i & 31))) a.q[i].last = (int32_t)L;
  add_stats(a, s_stats, cn, tid);
  pc.mark(TP_PARENT);
  tm_write<TM>(a, pc, PH == PH_SERIAL ? TK_SERIAL : TK_PARENT, L, t_entry, tid);
}

// ------------------------------------------------------------ child kernel
// Largest p in [0, n) with key(p) <= t, where key(0) <= t and keys increase:
// 64-ary wave search (each round narrows the range 64-fold).
template <typename KeyFn>
__device__ __forceinline__ uint32_t wave_upper_search(uint32_t n, uint32_t t, int lane, KeyFn key) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t step = (hi - lo + 63) / 64;
    const uint32_t p = lo + (uint32_t)lane * step;
    const bool le = p < hi && key(p) <= t;
    const uint32_t k = (uint32_t)__popcll(__ballot(le));
    lo += (k - 1) * step;
    hi = min(lo + step, hi);
  }
  return lo;
}

// Lane k of a wave holds record r0 + k of the current descriptor, the fields
// of its query and its share of the wave's child blocks [t0, t1): blocks
// [lo, hi) of its coarsened grid, i.e. the edges [elo, ehi) of its row, cut
// into 64-lane slices.  Consecutive small records cost one wave-wide load.
struct Window {
  int32_t rs, elo, ehi;             // row start, edge range of the share
  uint32_t excl, nslices;           // exclusive scan of the slice counts, total
  int32_t vbase, n, sbase, lv;      // query fields (Elem)
  uint32_t du;
  int32_t ps;                       // SSSP: the parent's slot
  bool last;                        // the wave's range ends in this window
  bool bad;
};

// Window of the records base .. base + wn - 1.  SSSP: a parent whose distance
// was lowered again during this level is already queued for the next level,
// where it expands with the lower distance; every relaxation of its share here
// would be dominated then, so the share is dropped (claim: the distance copy
// this level's atomicMin updates).
template <int P>
__device__ __forceinline__ Window load_window(const Args& a, const uint32_t* claim, uint32_t base,
                                              uint32_t wn, uint32_t gbase, uint32_t t0, uint32_t t1,
                                              int lane, uint32_t L, uint32_t& blocks) {
  Window w{0, 0, 0, 0u, 0u, 0, 0, 0, 0, 0u, 0, false, false};
  uint32_t ns = 0;
  bool bad = false, ends = false;
  if ((uint32_t)lane < wn) {
    const int4 rec = a.rec[base + lane];
    const int32_t q = a.rec_q[base + lane];
    uint32_t pnow = 0xFFFFFFFFu;  // the parent's distance now (SSSP)
    if (P == PROB_SSSP) {
      w.ps = a.rec_slot[base + lane];
      if ((uint32_t)w.ps < (uint32_t)a.slots) pnow = coherent_load(&claim[w.ps]);
      else bad = true;
    }
    int32_t CF = 1;
    if ((uint32_t)q < (uint32_t)a.nq) {
      const Query Q = a.q[q];
      CF = max(Q.CF, 1);
      w.vbase = Q.vbase;
      w.n = Q.n;
      w.sbase = Q.slot0 - Q.vbase;
      w.lv = (int32_t)(L + 1) - Q.lstart;
    } else {
      bad = true;
    }
    const int32_t deg = rec.y;
    if (deg <= 0 || rec.x < 0 || (int64_t)rec.x + deg > (int64_t)a.m) bad = true;
    if (!bad) {
      // coarsened grid of the record (Sec. IV-B): ceil(ceil(deg / CB) / CF)
      // blocks of CF * CB edges, starting at global block G
      const uint32_t span = (uint32_t)CF * (uint32_t)a.CB;
      const uint32_t cgr = ceil_div((uint32_t)deg, span);
      const uint32_t G = gbase + (uint32_t)rec.z;
      const uint32_t lo = max(G, t0), hi = min(G + cgr, t1);
      ends = G + cgr >= t1;
      const bool superseded = P == PROB_SSSP && pnow < (uint32_t)rec.w;
      if (hi > lo && !superseded) {
        w.rs = rec.x;
        w.elo = (int32_t)((lo - G) * span);
        w.ehi = min(deg, (int32_t)((hi - G) * span));
        ns = ceil_div((uint32_t)(w.ehi - w.elo), 64u);
        blocks += hi - lo;
      }
      w.du = (uint32_t)rec.w;
    }
  }
  const uint32_t incl = wave_incl_scan(ns, lane);
  w.excl = incl - ns;
  w.nslices = __shfl(incl, 63, 64);
  w.last = __any(ends);
  w.bad = __any(bad);
  return w;
}

// One wave runs a contiguous share [t0, t1) of the level's aggregated child
// blocks: the parent of its first block is found by search (the
// disaggregation of Sec. V-A), then records are taken 64 at a time and their
// slices U at a time.
template <int P, bool TM, bool NT>
__global__ __launch_bounds__(PB) void child_kernel(Args a, uint32_t step) {
  __shared__ int32_t s_stage[NW][STAGE];
  __shared__ uint32_t s_bc[NW + 8];
  __shared__ uint32_t s_qpre[NQD + 1];
  __shared__ uint32_t s_qnd[NQD];
  __shared__ unsigned long long s_stats[NSTAT];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  State* st = a.st;
  uint64_t t_entry = 0;
  if (TM) t_entry = realtime();
  PhaseClock<TM> pc;
  pc.start();
  if (st->done || st->error) return;
  const uint32_t L = st->base + step;
  LevelSet* cur = &st->set[L % 3];
  int32_t* fout = (L & 1) ? a.front0 : a.front1;

  // aggregated child blocks of this level, queue by queue
  if (wave == 0) {
    const unsigned long long c = lane < NQD ? cur->qctr[lane] : 0ull;
    const uint32_t incl = wave_incl_scan((uint32_t)c, lane);
    if (lane < NQD) {
      s_qnd[lane] = (uint32_t)(c >> 32);
      s_qpre[lane + 1] = incl;
    }
    if (lane == 0) s_qpre[0] = 0;
  }
  if (tid < NSTAT) s_stats[tid] = 0;
  __syncthreads();
  const uint32_t B = s_qpre[NQD];
  if (B == 0) return;
  const uint32_t vm = cur->vmode;
  const Vis vis = vis_of<P>(a, vm & 1u, (vm & 2u) != 0);
  // Blocks of the level for this wave.  dyn_pct = 0: an even share of all B.
  // Otherwise the blocks are split into one range per XCD group (workgroups w
  // with the same w % 8, which run on the same XCD); a wave takes an even
  // share of (100 - dyn_pct)% of its group's range, then claims chunks of the
  // rest from its group's counter until none is left, as a hardware block
  // scheduler hands out the blocks of a grid.
  uint32_t t0, t1, dyn0 = 0, dyn1 = 0, csz = 1, xg = 0;
  if (a.dyn_pct == 0 || gridDim.x % NQD) {
    const uint32_t nwaves = gridDim.x * NW, gw = blockIdx.x * NW + wave;
    t0 = (uint32_t)((uint64_t)gw * B / nwaves);
    t1 = (uint32_t)((uint64_t)(gw + 1) * B / nwaves);
  } else {
    xg = blockIdx.x % NQD;
    const uint32_t nwx = (gridDim.x / NQD) * NW, k = (blockIdx.x / NQD) * NW + wave;
    const uint32_t r0 = (uint32_t)((uint64_t)xg * B / NQD);
    const uint32_t r1 = (uint32_t)((uint64_t)(xg + 1) * B / NQD);
    const uint32_t share = (uint32_t)((uint64_t)(r1 - r0) * (uint32_t)(100 - a.dyn_pct) / 100u) / nwx;
    t0 = r0 + k * share;
    t1 = t0 + share;
    dyn0 = r0 + nwx * share;
    dyn1 = r1;
    csz = max(1u, (dyn1 - dyn0) / (2u * nwx));  // about two chunks per wave
  }
  // wave-uniform by construction (scalar registers)
  t0 = __builtin_amdgcn_readfirstlane(t0);
  t1 = __builtin_amdgcn_readfirstlane(t1);
  dyn0 = __builtin_amdgcn_readfirstlane(dyn0);
  dyn1 = __builtin_amdgcn_readfirstlane(dyn1);
  csz = __builtin_amdgcn_readfirstlane(csz);
  Counters cn{0, 0, 0, 0, 0, 0, 0};
  Stage s{s_stage[wave], 0u};
  pc.mark(TP_LAUNCH);  // reading the level's published grids

  bool failed = false;
  while (true) {
    if (t0 < t1) {
      // disaggregation of the first block (Sec. V-A): queue, descriptor, record
      uint32_t q = 0;
      while (t0 >= s_qpre[q + 1]) ++q;
      const int4* dq = a.desc + (size_t)q * a.desc_cap;
      const uint32_t tq = t0 - s_qpre[q];
      uint32_t d = wave_upper_search(s_qnd[q], tq, lane, [&](uint32_t p) { return (uint32_t)dq[p].z; });
      int4 dd = dq[d];
      uint32_t r = wave_upper_search((uint32_t)dd.y, tq - (uint32_t)dd.z, lane,
                                     [&](uint32_t p) { return (uint32_t)a.rec[dd.x + p].z; });
      constexpr int U = 8;
      while (true) {
        const uint32_t wn = min(64u, (uint32_t)dd.y - r);
        const Window win = load_window<P>(a, vis.claim, (uint32_t)dd.x + r, wn,
                                          s_qpre[q] + (uint32_t)dd.z, t0, t1, lane, L, cn.child);
        pc.mark(TP_DISAGG);
        if (win.bad) {
          if (lane == 0) set_error(st, ERR_CAPACITY);
          failed = true;
          break;
        }
        // Coarsening loop (Sec. IV-B): a coarsened block covers original blocks
        // j*CF .. j*CF+CF-1 of CB lanes, the contiguous edges [j*CF*CB,
        // (j+1)*CF*CB) of its row, taken here 64 lanes at a time.
        // SSSP: the parents' distances are loaded again with each batch and
        // checked at the next one (by then the load has returned), so shares of
        // parents lowered while the wave runs them are cut short.
        uint32_t pnow = 0xFFFFFFFFu;
        for (uint32_t x0 = 0; x0 < win.nslices; x0 += U) {
          int32_t v[U], out[U];
          uint32_t w[U];
          Elem c[U];
          unsigned long long sup = 0ull;  // records whose parent was lowered
          if (P == PROB_SSSP) {
            sup = __ballot((uint32_t)lane < wn && pnow < win.du);
            if ((uint32_t)lane < wn) pnow = coherent_load(&vis.claim[win.ps]);
          }
  #pragma unroll
          for (int u = 0; u < U; ++u) {
            v[u] = -1;
            w[u] = 0u;
            c[u] = Elem{0, 0, 0, 0, 0u};
            const uint32_t x = x0 + u;
            if (x < win.nslices) {
              // record of slice x: the last lane whose scan start is <= x
              const uint32_t k =
                  (uint32_t)__popcll(__ballot((uint32_t)lane < wn && win.excl <= x)) - 1u;
              const int32_t rs = __builtin_amdgcn_readlane(win.rs, k);
              const int32_t e0 = rs + __builtin_amdgcn_readlane(win.elo, k) +
                                 (int32_t)((x - (uint32_t)__builtin_amdgcn_readlane((int32_t)win.excl, k)) * 64u);
              const int32_t e1 = rs + __builtin_amdgcn_readlane(win.ehi, k);
              c[u].vbase = __builtin_amdgcn_readlane(win.vbase, k);
              c[u].n = __builtin_amdgcn_readlane(win.n, k);
              c[u].sbase = __builtin_amdgcn_readlane(win.sbase, k);
              c[u].lv = __builtin_amdgcn_readlane(win.lv, k);
              c[u].du = (uint32_t)__builtin_amdgcn_readlane((int32_t)win.du, k);
              if (e0 + lane < e1 && !((sup >> k) & 1ull)) {
                // NT (with found bytes: single traversals, the serving
                // engine): the level's adjacency (and weights) are read once,
                // so their lines leave L2 first and the probed bitmaps or
                // distances and the found bytes stay.  A batch of many
                // traversals over few graphs reads each adjacency again.
                v[u] = NT ? __builtin_nontemporal_load(&a.col[e0 + lane]) : a.col[e0 + lane];
                if (P == PROB_SSSP)
                  w[u] = NT ? __builtin_nontemporal_load(&a.w[e0 + lane]) : a.w[e0 + lane];
              }
            }
          }
          pin(v);
          if (P == PROB_SSSP) pin(w);
          if (a.count_stats) {  // edges run (lane 0 keeps the wave's count)
  #pragma unroll
            for (int u = 0; u < U; ++u) {
              const uint32_t nv = (uint32_t)__popcll(__ballot(v[u] >= 0));
              if (lane == 0) cn.echild += nv;
            }
          }
          visit_batch<P, U>(a, vis, v, w, c, L, out);
  #pragma unroll
          for (int u = 0; u < U; ++u) stage_push(s, out[u] >= 0, out[u], a, cur, fout, lane);
        }
        pc.mark(TP_CHILD);
        if (win.last) break;
        // next window: rest of this descriptor, else the next one (next queue
        // if need be)
        r += wn;
        if (r >= (uint32_t)dd.y) {
          r = 0;
          if (++d >= s_qnd[q]) {
            d = 0;
            do { ++q; } while (q < NQD && s_qnd[q] == 0);
            if (q >= NQD) {
              if (lane == 0) set_error(st, ERR_CAPACITY);
              failed = true;
              break;
            }
            dq = a.desc + (size_t)q * a.desc_cap;
          }
          dd = dq[d];
        }
      }
    }
    // next chunk of the group's dynamic part, if any is left
    if (failed || dyn0 >= dyn1) break;
    uint32_t j = 0;
    if (lane == 0) j = atomicAdd(&cur->cclaim[xg][0], 1u);
    j = __builtin_amdgcn_readfirstlane(j);
    const uint64_t c0 = (uint64_t)dyn0 + (uint64_t)j * csz;
    if (c0 >= dyn1) break;
    t0 = (uint32_t)c0;
    t1 = min(t0 + csz, dyn1);
    pc.mark(TP_LAUNCH);
  }
  block_flush(s, a, cur, fout, tid, s_bc);
  add_stats(a, s_stats, cn, tid);
  pc.mark(TP_CHILD);
  tm_write<TM>(a, pc, TK_CHILD, L, t_entry, tid);
}

// ------------------------------------------------------------ harvest kernel
// The last kernel of a level step with found bytes (Args::hint).  SSSP: every
// found vertex was improved at this level; it joins the next frontier once and
// its byte is cleared for the next level.  BFS with per-XCD copies, after a
// wide level: a found vertex that the visited bitmap lacks was discovered at
// this level.  It gets its level, its bit there and a place in the next frontier
// (in slot order, which also makes the next level's row loads mostly
// consecutive).  A wave owns the found bytes and the bitmap bytes of 512 slots at
// a time.  Found bytes are never cleared within a traversal: one set at an
// earlier level belongs to a vertex that the harvest
// of that level put into the bitmap.  Admission clears a query's found bytes,
// and a serving engine clears all of them when it is created
// (clear_found_kernel), so slots outside every admitted query hold none.  A
// narrow level claimed and appended in place, and its harvest returns at once.
template <int P, bool TM>
__global__ __launch_bounds__(PB) void harvest_kernel(Args a, uint32_t step) {
  __shared__ int32_t s_stage[NW][STAGE];
  __shared__ uint32_t s_bc[NW + 8];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  State* st = a.st;
  uint64_t t_entry = 0;
  if (TM) t_entry = realtime();
  PhaseClock<TM> pc;
  pc.start();
  if (st->done || st->error) return;
  const uint32_t L = st->base + step;
  LevelSet* cur = &st->set[L % 3];
  if (P == PROB_BFS && !(cur->vmode & 2u)) return;
  uint32_t* seen = a.visit + (size_t)(cur->vmode & 1u) * (uint32_t)a.vwords;  // BFS
  int32_t* fout = (L & 1) ? a.front0 : a.front1;
  Stage s{s_stage[wave], 0u};
  const uint32_t n = (uint32_t)a.slots;
  // BFS: a single traversal has one level value; with several queries it is
  // looked up per found vertex
  const int32_t lv1 = P == PROB_BFS ? (int32_t)(L + 1) - a.q[0].lstart : 0;
  // A lane reads the found bytes of 8 slots and, for BFS, their byte of the
  // bitmap; the runs of 64 slots with something new are then spread over the
  // wave, a lane per slot.
  const uint8_t* seen8 = (const uint8_t*)seen;
  for (uint32_t b = (blockIdx.x * NW + wave) * 512u; b < n; b += gridDim.x * PB * 8) {
    const uint32_t v8 = b + (uint32_t)lane * 8u;
    uint32_t bits = 0;
    if (v8 < n) {  // (n is a multiple of 32)
      const unsigned long long f = *(const unsigned long long*)(a.found + v8);
      bits = (uint32_t)((f * 0x0102040810204080ull) >> 56);  // byte j (0 or 1) -> bit j
      if (P == PROB_BFS) bits &= ~(uint32_t)seen8[v8 >> 3];
      else if (f) *(unsigned long long*)(a.found + v8) = 0;
    }
    const unsigned long long some = __ballot(bits != 0);
    if (some == 0) continue;
    if (P == PROB_BFS && bits) ((uint8_t*)seen)[v8 >> 3] = (uint8_t)(seen8[v8 >> 3] | bits);
    for (uint32_t k = 0; k < 8; ++k) {
      if (!(some >> (8 * k) & 0xFFull)) continue;
      const uint32_t v = b + k * 64u + (uint32_t)lane;
      const bool nw = (uint32_t)__shfl((int)bits, (int)(8 * k) + (lane >> 3), 64) >> (lane & 7) & 1u;
      if (P == PROB_BFS && nw)
        a.level[v] = a.nq == 1 ? lv1 : (int32_t)(L + 1) - a.q[a.qmap[v >> 5]].lstart;
      stage_push(s, nw, (int32_t)v, a, cur, fout, lane);
    }
  }
  block_flush(s, a, cur, fout, tid, s_bc);
  pc.mark(TP_CHILD);
  tm_write<TM>(a, pc, TK_HARVEST, L, t_entry, tid);
}

// ------------------------------------------------------------ narrow levels
// One workgroup runs consecutive narrow levels of a single traversal in one
// launch, the frontier in LDS from level to level.  A narrow level has too few
// edges to fill the chip; as a level step of its own it costs two to four
// launches and their chains of dependent loads.  Here it is two dependent loads
// (a vertex's row, its edges) and a few barriers: BFS on a 514 x 514 road-like
// graph (about 610 levels of 430 vertices) 15.4 -> 3.9 us a level, 9.6 -> 2.4
// ms; R-MAT of 4,096 vertices 238 -> 81 us.  What is left is latency: 0.7 us
// per load and about 0.25 us per barrier.
//
// The visited bitmap is in LDS too when it fits beside the frontier, so that a
// claim is an LDS atomic; else the kernel claims the global bitmap as a one-copy
// level does.  (SSSP on small graphs: solo_kernel.)
//
// The kernel leaves what a level step expects (frontier, level sets, group
// counters, visited copies) when a level is wide: more frontier entries than
// LDS holds, or more edges than one compute unit runs in the time of a level
// step's launches (NARROW_EDGES, NARROW_FAR_EDGES).
struct NarrowLds {
  uint32_t words[NARROW_WORDS];
  uint32_t fpre[NQF + 2];
  uint32_t wsum[NARROW_BLOCK / 64], wrows[NARROW_BLOCK / 64];
  __align__(8) uint8_t heads[NARROW_BLOCK / 64][64 * NARROW_U];  // per wave: row starts in its chunk
  uint32_t cnt, bad;
};

// Tells the host how the launch ended (pinned memory; nullptr: nobody waits).
__device__ __forceinline__ void post_verdict(uint32_t* verdict, uint32_t ticket, uint32_t code,
                                             uint32_t error) {
  if (verdict)
    __hip_atomic_store(verdict, ticket << 8 | error << 4 | code, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Workgroup barrier that orders LDS only: global stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Degrees of the rows [start[j], end[j]) in the ends' place, as a level step takes
// them: a row that ends before it starts has no entries, and one that would launch
// (T) outside the adjacency is not read, but an error.  per: rows in use.
template <uint32_t PER>
__device__ __forceinline__ void row_degrees(const Args& a, const uint32_t (&start)[PER], uint32_t (&end)[PER],
                                            uint32_t per, uint32_t T, uint32_t& bad) {
  uint32_t top = 0;
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    if (j >= per) break;
    top = max(top, max(start[j], end[j]));
    end[j] = (uint32_t)max((int32_t)(end[j] - start[j]), 0);
  }
  if (top <= (uint32_t)a.m) return;
  for (uint32_t j = 0; j < PER; ++j) {
    if (end[j] == 0 || end[j] < T || max(start[j], start[j] + end[j]) <= (uint32_t)a.m) continue;
    end[j] = 0;
    bad = ERR_CAPACITY;
  }
}

// Rows of 64 * NARROW_U consecutive edges, by a wave: heads[x - 1] is set if a
// row begins at edge x > 0 of them, so that the marks below an edge's own place
// count the rows begun up to it.
__device__ __forceinline__ void clear_heads(uint8_t* heads, int lane) {
  static_assert(NARROW_U == 8, "a lane clears 8 bytes");
  ((unsigned long long*)heads)[lane] = 0;
  wave_lds_sync();
}

// Row of edge u * 64 + lane; p: row of edge u * 64, less the one beginning
// there, moved on to the next 64 edges.
__device__ __forceinline__ uint32_t row_of(const uint8_t* heads, uint32_t u, int lane, uint32_t& p) {
  const unsigned long long h = __ballot(heads[u * 64 + lane] != 0);
  const uint32_t k = __builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32),
                                               __builtin_amdgcn_mbcnt_lo((uint32_t)h, p));
  p += (uint32_t)__popcll(h);
  return k;
}

// One batch of a wave's edges (v: target, or NONE): f[u] = v[u] joins the next
// frontier.  All probes are issued before any atomic, all atomics before any
// use, so their round trips overlap.
template <bool LDS>
__device__ __forceinline__ void narrow_visit(const Args& a, uint32_t* s_bits, uint32_t* vis,
                                             const uint32_t (&v)[NARROW_U], uint32_t L,
                                             bool (&f)[NARROW_U]) {
  constexpr int U = NARROW_U;
  uint32_t x[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    x[u] = ~0u;
    if (v[u] != NONE) x[u] = LDS ? s_bits[v[u] >> 5] : vis[v[u] >> 5];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t bit = 1u << (v[u] & 31);
    if (x[u] & bit) x[u] = ~0u;
    else x[u] = LDS ? atomicOr(&s_bits[v[u] >> 5], bit) : atomicOr(&vis[v[u] >> 5], bit);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    f[u] = !(x[u] & (1u << (v[u] & 31)));
    if (f[u]) a.level[v[u]] = (int32_t)L + 1;
  }
}

// Does an entry of v's row lack its reverse?  A sample that spares a directed graph
// the symmetry check, which reads all of it: entry h modulo the degree, looked up
// if the row it would be in is short (else: not found out).  False for a vertex
// without entries.
__device__ __forceinline__ bool lacks_reverse(const Args& a, uint32_t n, uint32_t v, uint32_t h) {
  const uint32_t m = (uint32_t)a.m, first = (uint32_t)a.rp[v];
  const int32_t deg = (int32_t)((uint32_t)a.rp[v + 1] - first);
  if (deg <= 0) return false;
  const uint32_t y = first + h % (uint32_t)deg, w = y < m ? (uint32_t)a.col[y] : n;
  if (w >= n) return true;
  const uint32_t b = (uint32_t)a.rp[w], e = (uint32_t)a.rp[w + 1];
  bool missing = e - b <= SYM_SAMPLE_DEGREE && e <= m;
  for (uint32_t x = b; x < e && missing; x += 8) {
    uint32_t t[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) t[u] = (uint32_t)a.col[min(x + u, e - 1)];
    pin(t);
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) missing = missing && t[u] != v;
  }
  return missing;
}

// Entries that a bottom-up level would read of the row of a vertex drawn by h (0 if
// it is visited), and its degree if it would be found.  The first SAMPLE_ROW entries
// are looked at; a row without a visited neighbour among them counts in full.
// vbase, n: the graph's vertices; vis: their bits.
__device__ __forceinline__ void sample_row(const Args& a, uint32_t vbase, uint32_t n, const uint32_t* vis,
                                           uint32_t h, uint32_t& read, uint32_t& found) {
  constexpr uint32_t SAMPLE_ROW = 16;
  h = (h ^ h >> 15) * 0x85EBCA6Bu;
  h ^= h >> 13;
  const uint32_t v = (uint32_t)((uint64_t)h * n >> 32);
  const uint32_t b = (uint32_t)a.rp[vbase + v], e = (uint32_t)a.rp[vbase + v + 1];
  read = found = 0;
  if (vis[v >> 5] >> (v & 31) & 1u || b >= e || e > (uint32_t)a.m) return;
  uint32_t t[SAMPLE_ROW];
#pragma unroll
  for (uint32_t u = 0; u < SAMPLE_ROW; ++u) t[u] = min((uint32_t)a.col[min(b + u, e - 1)] - vbase, n - 1);
  pin(t);
#pragma unroll
  for (uint32_t u = 0; u < SAMPLE_ROW; ++u) t[u] = vis[t[u] >> 5] >> (t[u] & 31) & 1u;
  pin(t);
  const uint32_t deg = min(e - b, 1u << 20);
  read = deg;
#pragma unroll
  for (uint32_t u = SAMPLE_ROW; u-- > 0;)
    if (t[u]) {
      read = min(u + 1, deg);
      found = deg;
    }
}

// after: what ran since the last launch: so many level steps, or AFTER_BOTTOM_UP.
// LDS: the visited bits are in LDS.
template <bool LDS>
__global__ __launch_bounds__(NARROW_BLOCK) void narrow_kernel(Args a, uint32_t after, uint32_t ticket,
                                                              uint32_t* verdict) {
  __shared__ NarrowLds sh;
  constexpr uint32_t NB = NARROW_BLOCK, PER = NARROW_FRONT / NB, U = NARROW_U;
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  State* st = a.st;
  if (st->done || st->error) {
    if (tid == 0) post_verdict(verdict, ticket, st->error ? V_ERROR : V_DONE, st->error);
    return;
  }
  const bool bottom_up = goes_bottom_up(st);
  const uint32_t adv = after == AFTER_BOTTOM_UP ? bottom_up : after;
  uint32_t symmetric = st->plan == V_CHECK ? (bottom_up ? 1u : 2u) : st->symmetric;
  // (a planned level's edges count once it has run, however often it is planned,
  // and for those of the level steps behind it)
  unsigned long long run_edges = st->run_edges + adv * st->plan_edges, plan_edges = 0;
  uint32_t L = st->base + adv;
  const uint32_t n = (uint32_t)a.q[0].n, T = (uint32_t)a.q[0].T;
  if (tid == 0) sh.bad = 0;
  const LevelSet* prv = &st->set[(L + 2) % 3];
  if (wave == 0) {
    const uint32_t c = min(prv->fcnt[lane], (uint32_t)a.fcap);
    const uint32_t incl = wave_incl_scan(c, lane);
    sh.fpre[lane + 1] = incl;
    if (lane == 0) sh.fpre[0] = 0;
    if (lane == 63) sh.fpre[NQF + 1] = incl + prv->fcnt[NQF];
  }
  __syncthreads();
  uint32_t F = sh.fpre[NQF + 1];
  // LDS: the bits, then frontier arrays of FC entries each
  const uint32_t nbits = LDS ? (uint32_t)a.vwords : 0u;
  const uint32_t FC = min((uint32_t)NARROW_FRONT, (NARROW_WORDS - nbits) / 4);
  constexpr uint32_t max_edges = LDS ? NARROW_EDGES : NARROW_FAR_EDGES;
  const uint32_t max_front = min(FC, max_edges);
  uint32_t* s_bits = sh.words;
  uint32_t* s_front = sh.words + nbits;  // two of FC: this level's, the next one's
  uint32_t* s_start = s_front + 2 * FC;
  uint32_t* s_off = s_front + 3 * FC;
  uint32_t cur = 0, nxt = FC;         // offsets into s_front
  const uint32_t c = st->vsel[L & 1];
  // the copy this traversal's one-copy levels probe and update
  uint32_t* vis = a.visit + (size_t)c * (uint32_t)a.vwords;
  const uint32_t L0 = L;
  bool wide = F > max_front;
  if (F != 0 && !wide) {
    const int32_t* fin = (L & 1) ? a.front1 : a.front0;
    for (uint32_t i = tid; i < F; i += NB) s_front[i] = (uint32_t)frontier_at(a, fin, sh.fpre, i);
    for (uint32_t i = tid; i < nbits; i += NB) s_bits[i] = vis[i];
  }
  __syncthreads();
  while (F != 0 && !wide) {
    // rows of this thread's entries [tid * per, tid * per + per)
    const uint32_t per = (uint32_t)__builtin_amdgcn_readfirstlane((int)ceil_div(F, NB));
    uint32_t start[PER], deg[PER], sum = 0, rows = 0;
    bool big = F > NB;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      const uint32_t i = tid * per + j;
      start[j] = deg[j] = 0;
      if (j < per && i < F) {
        const uint32_t v = s_front[cur + i];
        start[j] = (uint32_t)a.rp[v];
        deg[j] = (uint32_t)a.rp[v + 1];
      }
    }
    if (tid == 0) sh.cnt = 0;
    row_degrees<PER>(a, start, deg, per, T, sh.bad);
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      if (j >= per) break;
      sum += deg[j];
      rows += deg[j] != 0;
      big |= deg[j] > U;
    }
    int32_t* fout = (L & 1) ? a.front0 : a.front1;
    // runs a batch of edges, and appends what joins the next frontier: to LDS,
    // what does not fit to the overflow queue
    auto edges = [&](const bool (&valid)[U], const uint32_t (&ei)[U]) {
      uint32_t v[U];
      bool f[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) v[u] = valid[u] ? (uint32_t)a.col[ei[u]] : NONE;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        if (v[u] >= n && valid[u]) {
          sh.bad = ERR_ARG;
          v[u] = NONE;
        }
      }
      narrow_visit<LDS>(a, s_bits, vis, v, L, f);
      unsigned long long m[U];
      uint32_t total = 0, base = 0;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        m[u] = __ballot(f[u]);
        total += (uint32_t)__popcll(m[u]);
      }
      if (total == 0) return;
      if (lane == 0) base = atomicAdd(&sh.cnt, total);
      base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t pos = base + lane_rank(m[u]);
        base += (uint32_t)__popcll(m[u]);
        if (!f[u]) continue;
        if (pos < FC) s_front[nxt + pos] = v[u];
        else if (pos < (uint32_t)a.slots) fout[(size_t)NQF * a.fcap + pos] = (int32_t)v[u];
      }
    };
    if (!__syncthreads_or(big)) {
      // one short row per thread: it runs the row, with no scan of the
      // degrees and no search for an edge's row
      if (__any(deg[0] != 0)) {
        bool valid[U];
        uint32_t ei[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          valid[u] = u < deg[0];
          ei[u] = start[0] + u;
        }
        edges(valid, ei);
      }
    } else {
      // the non-empty rows and their scanned degrees, in LDS
      const uint32_t incl = wave_incl_scan(sum, lane), rincl = wave_incl_scan(rows, lane);
      if (lane == 63) {
        sh.wsum[wave] = incl;
        sh.wrows[wave] = rincl;
      }
      lds_barrier();
      uint32_t run = incl - sum, E = 0, row = rincl - rows, R = 0;
#pragma unroll
      for (uint32_t w = 0; w < NB / 64; ++w) {
        if (w < (uint32_t)wave) {
          run += sh.wsum[w];
          row += sh.wrows[w];
        }
        E += sh.wsum[w];
        R += sh.wrows[w];
      }
      if (E > max_edges) {
        wide = true;
        break;
      }
      run_edges += E;
#pragma unroll
      for (uint32_t j = 0; j < PER; ++j) {
        if (deg[j] == 0) continue;
        s_start[row] = start[j] - run;  // edge x of the level is start + x
        s_off[row] = run;
        run += deg[j];
        ++row;
      }
      lds_barrier();
      // A wave runs chunks of 64 * U consecutive edges of the level.  A mark per
      // edge that begins a row gives each edge its row by a count of the marks
      // up to it: one LDS store per row instead of a search per edge.
      uint8_t* heads = sh.heads[wave];
      for (uint32_t x0 = wave * 64 * U; x0 < E; x0 += NB * U) {
        const uint32_t p0 = wave_upper_search(R, x0, lane, [&](uint32_t k) { return s_off[k]; });
        clear_heads(heads, lane);
        for (uint32_t k = p0 + 1 + lane; k < R; k += 64) {
          const uint32_t x = s_off[k] - x0;
          if (x >= 64 * U) break;
          heads[x - 1] = 1;
        }
        wave_lds_sync();
        bool valid[U];
        uint32_t ei[U], p = p0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          const uint32_t x = x0 + u * 64 + lane;
          const uint32_t k = row_of(heads, u, lane, p);
          valid[u] = x < E;
          ei[u] = s_start[k] + x;
        }
        edges(valid, ei);
        wave_lds_sync();  // heads is cleared by the next chunk
      }
    }
    lds_barrier();
    ++L;
    F = sh.cnt;
    const uint32_t t = cur;
    cur = nxt;
    nxt = t;
    if (F > max_front) wide = true;
    lds_barrier();  // F read before the next level clears the count
    if (L - L0 >= NARROW_LEVELS) break;
  }
  __syncthreads();
  if (F == 0 || sh.bad) {
    const uint32_t err = sh.bad;
    if (tid == 0) {
      st->done = 1;
      st->error = err;
      post_verdict(verdict, ticket, err ? V_ERROR : V_DONE, err);
    }
    return;
  }
  if (L != L0) {
    // what a level step finds at level L
    int32_t* fin = (L & 1) ? a.front1 : a.front0;
    for (uint32_t i = tid; i < min(F, FC); i += NB)
      fin[(size_t)NQF * a.fcap + i] = (int32_t)s_front[cur + i];
    for (uint32_t i = tid; i < nbits; i += NB) vis[i] = s_bits[i];
    for (uint32_t i = tid; i < (uint32_t)a.ngroups_cap; i += NB) {
      a.grp_packed[(L % 3) * a.ngroups_cap + i] = 0;
      a.grp_done[(L % 3) * a.ngroups_cap + i] = 0;
    }
    uint32_t* sets = (uint32_t*)&st->set[0];
    const uint32_t fill = (uint32_t)(&st->set[(L + 2) % 3].fcnt[NQF] - sets);
    for (uint32_t i = tid; i < 3 * sizeof(LevelSet) / 4; i += NB) sets[i] = i == fill ? F : 0u;
  }
  const uint32_t top_down = L == L0 ? V_STILL : V_TOP_DOWN;
  uint32_t code = wide ? top_down : V_MORE;
  if (a.bottom_up && wide) {
    // the level's edges, from the degrees of up to NB of its vertices
    const int32_t* fin = (L & 1) ? a.front1 : a.front0;
    uint32_t deg = 0, v = 0;
    if (tid < F) {
      const uint32_t i = F <= NB ? tid : (uint32_t)((uint64_t)tid * F / NB);
      v = L == L0 ? (uint32_t)frontier_at(a, fin, sh.fpre, i)
          : i < FC ? s_front[cur + i] : (uint32_t)fin[(size_t)NQF * a.fcap + i];
      deg = (uint32_t)max(a.rp[v + 1] - a.rp[v], 0);
    }
    const uint32_t incl = wave_incl_scan(deg, lane);
    if (lane == 63) sh.wsum[wave] = incl;
    __syncthreads();
    unsigned long long E = 0;
#pragma unroll
    for (uint32_t w = 0; w < NB / 64; ++w) E += sh.wsum[w];
    if (F > NB) E = E * F / NB;
    const unsigned long long left = (unsigned long long)a.m > run_edges ? a.m - run_edges : 0;
    bool pays = symmetric != 2 && E * BU_ALPHA >= left;
    if (pays && (!symmetric || E * BU_SURE < left)) {
      // what the level would read, and find, from some of its vertices
      uint32_t read = 0, found = 0;
      if (tid < BU_SAMPLES) sample_row(a, 0, n, vis, (L * NB + tid) * 0x9E3779B1u, read, found);
#pragma unroll
      for (int o = 32; o; o >>= 1) {
        read += (uint32_t)__shfl_xor((int)read, o, 64);
        found += (uint32_t)__shfl_xor((int)found, o, 64);
      }
      __syncthreads();
      if (lane == 0) {
        sh.wsum[wave] = read;
        sh.wrows[wave] = found;
      }
      __syncthreads();
      unsigned long long S = 0, H = 0;
#pragma unroll
      for (uint32_t w = 0; w < NB / 64; ++w) {
        S += sh.wsum[w];
        H += sh.wrows[w];
      }
      S = S * n / BU_SAMPLES;
      H = H * n / BU_SAMPLES;
      const bool one_copy = F < (uint32_t)a.split_min;
      pays = S * 2 <= (E + H) * (one_copy ? BU_READ_ONE_COPY : BU_READ) &&
             (symmetric || (unsigned long long)a.m <= (E + H) * (one_copy ? BU_CHECK_ONE_COPY : BU_CHECK));
    }
    if (pays) {
      code = V_BOTTOM_UP;
      if (!symmetric) {
        // (on the directed graphs one meets a few entries tell)
        const bool missing = tid < SYM_SAMPLES && deg && lacks_reverse(a, n, v, tid * 0x9E3779B1u);
        code = V_CHECK;
        if (__syncthreads_or(missing)) {
          symmetric = 2;
          code = top_down;
        }
      }
    }
    plan_edges = E;
  }
  if (tid == 0) {
    st->base = L;
    st->plan = code;
    st->symmetric = symmetric;
    st->run_edges = run_edges;
    st->plan_edges = plan_edges;
    if (L != L0) {
      st->vsel[L & 1] = c;
      st->vstale[L & 1] = 1u;
      st->levels_run = L;
    }
    post_verdict(verdict, ticket, code, 0);
  }
}

// ------------------------------------------------------------ solo traversals
// SSSP on a small graph in one workgroup, from the source to the last level,
// distances and frontier in LDS.  On such a graph a level step is four kernels
// of 5 to 25 us whose relaxations meet on a few hubs; here a level is two
// dependent loads, and then about 1.3 edges a cycle, bound by the compute unit's
// instructions (about 45 a wave and 64 edges).  Frontier entries past what LDS
// holds go to the overflow queues and are run in passes.
//
// FAR: level order relaxes a dense graph's edges two to three times.  A vertex
// improved to a distance above the bound waits instead, until no vertex below it
// is left and the bound moves to 1.5 times the least distance that waits; once
// half of the entries have been run it is lifted, as what is left is many levels
// of few edges.  8,191 vertices, 204,000 entries, weights up to 255: 14 levels and
// 2 new bounds instead of 13 levels, a third of the edges; level steps 422 us,
// level order 356, with the bound 195 (other seeds 180 to 265; never lifted 227; moved to 1.25 or 2 times
// the least distance 277 / 272).  16,383 vertices, 245,000 entries 459 -> 261.
// Equal weights gain nothing and pay for the two bit sets: 131 -> 145.
struct SoloLds {
  uint32_t words[SOLO_WORDS];
  unsigned long long rows[NARROW_BLOCK / 64][64];  // per wave: {row start, distance} of a window
  __align__(8) uint8_t heads[NARROW_BLOCK / 64][64 * NARROW_U];
  uint32_t wsum[NARROW_BLOCK / 64], wrows[NARROW_BLOCK / 64];
  uint32_t cnt, bad, low, ran;
};

// Writes its output and its verdict and needs nothing of the workspace but the
// overflow queues.
template <bool FAR>
__global__ __launch_bounds__(NARROW_BLOCK) void solo_kernel(Args a, uint32_t src, uint32_t T,
                                                            uint32_t* verdict) {
  __shared__ SoloLds sh;
  constexpr uint32_t NB = NARROW_BLOCK, PER = SOLO_FRONT / NB, U = NARROW_U;
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint32_t n = (uint32_t)a.n, nbits = (n + 31) / 32;
  const uint32_t FC = min((uint32_t)SOLO_FRONT, (SOLO_WORDS - (FAR ? 2 : 1) * nbits - n) / 5);
  uint32_t* s_dist = sh.words;
  uint32_t* s_bits = s_dist + n;       // queued for the next level
  uint32_t* s_far = s_bits + (FAR ? nbits : 0u);  // waiting for the bound to reach them
  uint32_t* s_front = s_far + nbits;  // two of FC: this level's, the next one's
  uint32_t* s_start = s_front + 2 * FC;
  uint32_t* s_off = s_front + 3 * FC;
  uint32_t* s_slot = s_front + 4 * FC;
  for (uint32_t i = tid; i < n; i += NB) s_dist[i] = i == src ? 0u : 0xFFFFFFFFu;
  for (uint32_t i = tid; i < (FAR ? 2 : 1) * nbits; i += NB) s_bits[i] = 0;
  if (tid == 0) {
    s_front[0] = src;
    sh.bad = 0;
    sh.cnt = 0;
    sh.low = 0xFFFFFFFFu;
    sh.ran = 0;
  }
  __syncthreads();
  uint32_t cur = 0, nxt = FC, F = 1, ran = 0;
  uint32_t bound = FAR ? 0u : 0xFFFFFFFFu;
  // (as many levels for a bound's vertices as there are, and one to raise it)
  for (uint32_t L = 0; F != 0 && L <= (FAR ? 2 * n + 1 : n); ++L) {
    uint32_t* spill_in = (uint32_t*)((L & 1) ? a.front1 : a.front0) + (size_t)NQF * a.fcap;
    uint32_t* spill_out = (uint32_t*)((L & 1) ? a.front0 : a.front1) + (size_t)NQF * a.fcap;
    // appends what a batch found
    auto append = [&](const bool (&f)[U], const uint32_t (&v)[U]) {
      bool any = false;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) any |= f[u];
      if (!__any(any)) return;
      unsigned long long m[U];
      uint32_t total = 0, base = 0;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        m[u] = __ballot(f[u]);
        total += (uint32_t)__popcll(m[u]);
      }
      if (lane == 0) base = atomicAdd(&sh.cnt, total);
      base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t pos = base + lane_rank(m[u]);
        base += (uint32_t)__popcll(m[u]);
        if (!f[u]) continue;
        if (pos < FC) s_front[nxt + pos] = v[u];
        else if (pos < n) spill_out[pos] = v[u];
      }
    };
    // edges ei[u] of rows at distance du[u] (all ones: none); all loads, then
    // all probes, then all atomics
    auto edges = [&](const uint32_t (&ei)[U], const uint32_t (&du)[U]) {
      uint32_t v[U], nd[U], x[U];
      bool f[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const bool on = du[u] != 0xFFFFFFFFu;
        v[u] = on ? (uint32_t)a.col[ei[u]] : 0u;
        nd[u] = on ? a.w[ei[u]] : 0u;
      }
      pin(v);
      pin(nd);
      bool bad = false;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t sum = du[u] + nd[u];  // saturating, as in visit_batch
        nd[u] = sum < du[u] ? 0xFFFFFFFFu : sum;
        bad |= v[u] >= n;
        x[u] = s_dist[min(v[u], n - 1)];
      }
      if (bad) sh.bad = ERR_ARG;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        if (nd[u] < x[u] && v[u] < n) x[u] = atomicMin(&s_dist[v[u]], nd[u]);
        else x[u] = 0;
      }
      pin(x);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t bit = 1u << (v[u] & 31);
        const bool better = nd[u] < x[u];
        if (FAR && better && nd[u] > bound) atomicOr(&s_far[v[u] >> 5], bit);
        if (better && (!FAR || nd[u] <= bound)) x[u] = atomicOr(&s_bits[v[u] >> 5], bit) & bit;
        else x[u] = 1;
      }
      pin(x);
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) f[u] = x[u] == 0;
      append(f, v);
    };
    for (uint32_t done = 0; done < F; done += FC) {
      const uint32_t count = min(F - done, FC);
      if (done) {
        for (uint32_t i = tid; i < count; i += NB) s_front[cur + i] = spill_in[done + i];
        __syncthreads();
      }
      // rows of this thread's entries [tid * per, tid * per + per)
      const uint32_t per = (uint32_t)__builtin_amdgcn_readfirstlane((int)ceil_div(count, NB));
      uint32_t start[PER], deg[PER], sum = 0, rows = 0;
      bool big = count > NB;
#pragma unroll
      for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t i = tid * per + j;
        start[j] = deg[j] = 0;
        if (j < per && i < count) {
          const uint32_t v = s_front[cur + i];
          start[j] = (uint32_t)a.rp[v];
          deg[j] = (uint32_t)a.rp[v + 1];
          atomicAnd(&s_bits[v >> 5], ~(1u << (v & 31)));  // may be queued again
        }
      }
      row_degrees<PER>(a, start, deg, per, T, sh.bad);
#pragma unroll
      for (uint32_t j = 0; j < PER; ++j) {
        if (j >= per) break;
        sum += deg[j];
        rows += deg[j] != 0;
        big |= deg[j] > U;
      }
      ran += sum;
      if (!__syncthreads_or(big)) {
        // one short row per thread, which it runs itself
        if (__any(deg[0] != 0)) {
          const uint32_t d = deg[0] ? s_dist[s_front[cur + tid]] : 0xFFFFFFFFu;
          uint32_t ei[U], du[U];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) {
            ei[u] = start[0] + u;
            du[u] = u < deg[0] ? d : 0xFFFFFFFFu;
          }
          edges(ei, du);
        }
      } else {
        // the non-empty rows and their scanned degrees
        const uint32_t incl = wave_incl_scan(sum, lane), rincl = wave_incl_scan(rows, lane);
        if (lane == 63) {
          sh.wsum[wave] = incl;
          sh.wrows[wave] = rincl;
        }
        lds_barrier();
        uint32_t run = incl - sum, E = 0, row = rincl - rows, R = 0;
#pragma unroll
        for (uint32_t w = 0; w < NB / 64; ++w) {
          if (w < (uint32_t)wave) {
            run += sh.wsum[w];
            row += sh.wrows[w];
          }
          E += sh.wsum[w];
          R += sh.wrows[w];
        }
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
          if (deg[j] == 0) continue;
          s_start[row] = start[j] - run;  // edge x of the pass is start + x
          s_off[row] = run;
          s_slot[row] = s_front[cur + tid * per + j];
          run += deg[j];
          ++row;
        }
        lds_barrier();
        // a wave runs chunks of 64 * U edges, their rows in windows of 64
        uint8_t* heads = sh.heads[wave];
        unsigned long long* info = sh.rows[wave];
        for (uint32_t x0 = wave * 64 * U; x0 < E; x0 += NB * U) {
          const uint32_t hi = min(x0 + 64 * U, E);
          uint32_t p0 = wave_upper_search(R, x0, lane, [&](uint32_t k) { return s_off[k]; });
          for (uint32_t lo = x0; lo < hi; p0 += 64) {
            const uint32_t k = p0 + (uint32_t)lane;
            const uint32_t off = k < R ? s_off[k] : E;
            const uint32_t end = min(hi, p0 + 64 < R ? s_off[p0 + 64] : E);
            clear_heads(heads, lane);
            if (off < end) {
              // a parent improved (and queued) again meanwhile does no work now
              const uint32_t v = s_slot[k];
              const uint32_t d = s_bits[v >> 5] >> (v & 31) & 1u ? 0xFFFFFFFFu : s_dist[v];
              info[lane] = (unsigned long long)d << 32 | s_start[k];
              if (off > lo) heads[off - lo - 1] = 1;
            }
            wave_lds_sync();
            uint32_t ei[U], du[U], p = 0;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
              const uint32_t x = lo + u * 64 + lane;
              const unsigned long long r = info[row_of(heads, u, lane, p)];
              ei[u] = (uint32_t)r + x;
              du[u] = x < end ? (uint32_t)(r >> 32) : 0xFFFFFFFFu;
            }
            edges(ei, du);
            wave_lds_sync();  // heads and rows are rewritten by the next window
            lo = end;
          }
        }
      }
      // (with a spilled frontier the next pass or level reads what this one
      // stored globally)
      __syncthreads();
    }
    if (FAR && sh.cnt == 0 && bound != 0xFFFFFFFFu) {
      // The least distance that waits, and the new bound's vertices.  One that
      // waits below the old bound was improved again and has been queued since.
      uint32_t low = 0xFFFFFFFFu;
      for (uint32_t v = tid; v < n; v += NB) {
        const uint32_t d = s_dist[v];
        if ((s_far[v >> 5] >> (v & 31) & 1u) && d > bound) low = min(low, d);
      }
      if (__any(low != 0xFFFFFFFFu)) {
#pragma unroll
        for (int o = 32; o; o >>= 1) low = min(low, (uint32_t)__shfl_xor((int)low, o, 64));
        if (lane == 0) atomicMin(&sh.low, low);
      }
#pragma unroll
      for (int o = 32; o; o >>= 1) ran += (uint32_t)__shfl_xor((int)ran, o, 64);
      if (lane == 0) atomicAdd(&sh.ran, ran);
      ran = 0;
      lds_barrier();
      low = sh.low;
      const uint32_t old = bound;
      bound = low + low / 2 < low || sh.ran >= (uint32_t)a.m / 2 ? 0xFFFFFFFFu : low + low / 2;
      if (low != 0xFFFFFFFFu) {
        for (uint32_t v0 = wave * 64; v0 < n; v0 += NB) {
          const uint32_t v = v0 + (uint32_t)lane;
          const bool far = v < n && (s_far[v >> 5] >> (v & 31) & 1u);
          const uint32_t d = far ? s_dist[v] : 0xFFFFFFFFu;
          const unsigned long long off = __ballot(far && d <= bound);
          if (off == 0) continue;
          const bool take = far && d <= bound && d > old;
          const unsigned long long m = __ballot(take);
          const uint32_t half = (uint32_t)(off >> (lane & 32)), mine = (uint32_t)(m >> (lane & 32));
          if ((lane & 31) == 0 && half) {  // the wave's own words
            s_far[v >> 5] &= ~half;
            s_bits[v >> 5] |= mine;
          }
          uint32_t base = 0;
          if (lane == 0 && m) base = atomicAdd(&sh.cnt, (uint32_t)__popcll(m));
          const uint32_t pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + lane_rank(m);
          if (take) {
            if (pos < FC) s_front[nxt + pos] = v;
            else if (pos < n) spill_out[pos] = v;
          }
        }
      }
      __syncthreads();
      if (tid == 0) sh.low = 0xFFFFFFFFu;
    }
    F = sh.cnt;
    const uint32_t t = cur;
    cur = nxt;
    nxt = t;
    lds_barrier();
    if (tid == 0) sh.cnt = 0;
    lds_barrier();
  }
  for (uint32_t i = tid; i < n; i += NB) a.dist[i] = s_dist[i];
  if (tid == 0) {
    const uint32_t err = sh.bad ? sh.bad : F ? (uint32_t)ERR_TIMEOUT : 0u;
    post_verdict(verdict, 0, err ? V_ERROR : V_DONE, err);
  }
}

// ------------------------------------------------- near-far on sparse graphs
// SSSP on a sparse graph of long paths (a road network), in one workgroup.
// Frontier Bellman-Ford relaxes such a graph's entries again and again (a
// 301 x 257 road-like graph: 37 times, 608 levels of 2,900 vertices, 16 us a
// level step).  Here a vertex improved to a distance below the bound joins the
// next frontier, any other waits in the far list until the frontier is empty
// and the bound moves on; a round is then a few hundred vertices, small enough
// for one compute unit, and three dependent round trips (row and distance,
// entries, atomicMin) of about 0.8 us.  The order of relaxations does not change
// the distances.  That graph: 9.3 -> 3.7 ms; 490 x 480: 24.9 -> 9.3.
//
// A frontier too wide for that (NEAR_EDGES) means that the graph is not of this
// kind: everything that waits becomes frontier 0 of the level steps, which the
// start kernel's state is ready for.
struct NearLds {
  uint32_t words[NEAR_WORDS];
  __align__(8) uint8_t heads[NARROW_BLOCK / 64][64 * NARROW_U];
  uint32_t wsum[NARROW_BLOCK / 64], wrows[NARROW_BLOCK / 64];
  uint32_t cnt, far, low, bad;  // next frontier, far list: entries, its least distance
};

__global__ __launch_bounds__(NARROW_BLOCK) void near_kernel(Args a, uint32_t src, uint32_t* verdict) {
  __shared__ NearLds sh;
  constexpr uint32_t NB = NARROW_BLOCK, FC = NEAR_FRONT, PER = FC / NB, U = NARROW_U;
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint32_t n = (uint32_t)a.n, m = (uint32_t)a.m, nbits = (n + 31) / 32, T = (uint32_t)a.q[0].T;
  uint32_t* s_near = sh.words;  // in the next frontier
  uint32_t* s_wait = s_near + nbits;  // in the far list
  uint32_t* s_front = s_wait + nbits;
  uint32_t* s_start = s_front + 2 * FC;
  uint32_t* s_off = s_front + 3 * FC;
  uint32_t* s_du = s_front + 4 * FC;
  uint32_t* dist = a.dist;
  uint32_t* out = (uint32_t*)a.front0 + (size_t)NQF * a.fcap;  // frontier 0 of the level steps
  uint32_t* far[2] = {(uint32_t*)a.front1, (uint32_t*)a.front1 + a.slots};
  for (uint32_t i = tid; i < 2 * nbits; i += NB) sh.words[i] = 0;
  // the bound moves by NEAR_STEP average weights
  unsigned long long wsum = m ? a.w[(uint32_t)((uint64_t)tid * m / NB)] : 0u;
#pragma unroll
  for (int d = 32; d; d >>= 1) wsum += __shfl_xor(wsum, d, 64);
  if (lane == 0) sh.wsum[wave] = (uint32_t)min(wsum / 64, (unsigned long long)0xFFFFFFFFu);
  if (tid == 0) {
    s_front[0] = src;
    sh.cnt = sh.far = sh.bad = 0;
    sh.low = 0xFFFFFFFFu;
  }
  __syncthreads();
  unsigned long long mean = 0;
  for (uint32_t w = 0; w < NB / 64; ++w) mean += sh.wsum[w];
  const unsigned long long step = max(mean * NEAR_STEP / (NB / 64), 1ull);
  unsigned long long bound = step;
  uint32_t cur = 0, nxt = FC, F = 1, side = 0;
  bool wide = false;
  // f[u]: v[u] was improved to nd[u]; into the next frontier or the far list
  auto append = [&](bool (&f)[U], const uint32_t (&v)[U], const uint32_t (&nd)[U]) {
    bool any = false;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) any |= f[u];
    if (!__any(any)) return;
    uint32_t old[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      uint32_t* bits = nd[u] < bound ? s_near : s_wait;
      old[u] = ~0u;
      if (f[u]) old[u] = atomicOr(&bits[v[u] >> 5], 1u << (v[u] & 31));
    }
    pin(old);
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      f[u] = !(old[u] >> (v[u] & 31) & 1u);
      const bool close = nd[u] < bound;
      const unsigned long long m0 = __ballot(f[u] && close), m1 = __ballot(f[u] && !close);
      if ((m0 | m1) == 0) continue;
      uint32_t b0 = 0, b1 = 0;
      if (lane == 0 && m0) b0 = atomicAdd(&sh.cnt, (uint32_t)__popcll(m0));
      if (lane == 0 && m1) b1 = atomicAdd(&sh.far, (uint32_t)__popcll(m1));
      b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0) + lane_rank(m0);
      b1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b1) + lane_rank(m1);
      if (f[u] && close) {
        if (b0 < FC) s_front[nxt + b0] = v[u];
        else if (b0 < n) out[b0] = v[u];
      }
      if (f[u] && !close) {
        if (b1 < n) far[side][b1] = v[u];
        atomicMin(&sh.low, nd[u]);
      }
    }
  };
  auto edges = [&](const uint32_t (&ei)[U], const uint32_t (&du)[U]) {
    uint32_t v[U], nd[U], x[U];
    bool f[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const bool on = du[u] != 0xFFFFFFFFu;
      v[u] = on ? (uint32_t)a.col[ei[u]] : 0u;
      nd[u] = on ? a.w[ei[u]] : 0u;
    }
    pin(v);
    pin(nd);
    bool bad = false;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t sum = du[u] + nd[u];  // saturating, as in visit_batch
      nd[u] = sum < du[u] || v[u] >= n ? 0xFFFFFFFFu : sum;
      bad |= v[u] >= n;
      // no probe first: it would be one more round trip, for as many accesses
      x[u] = nd[u] != 0xFFFFFFFFu ? atomicMin(&dist[v[u]], nd[u]) : 0u;
    }
    if (bad) sh.bad = ERR_ARG;
    pin(x);
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) f[u] = nd[u] < x[u];
    append(f, v, nd);
  };
  for (unsigned long long round = 0; F != 0 && !wide && !sh.bad; ++round) {
    const uint32_t per = (uint32_t)__builtin_amdgcn_readfirstlane((int)ceil_div(F, NB));
    uint32_t start[PER], deg[PER], du[PER], sum = 0, rows = 0;
    bool big = F > NB;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      const uint32_t i = tid * per + j;
      start[j] = deg[j] = 0;
      du[j] = 0xFFFFFFFFu;
      if (j < per && i < F) {
        const uint32_t v = s_front[cur + i];
        start[j] = (uint32_t)a.rp[v];
        deg[j] = (uint32_t)a.rp[v + 1];
        du[j] = coherent_load(&dist[v]);  // atomics of earlier rounds wrote it
        atomicAnd(&s_near[v >> 5], ~(1u << (v & 31)));
      }
    }
    pin(start);
    pin(deg);
    pin(du);
    if (tid == 0) sh.cnt = 0;
    row_degrees<PER>(a, start, deg, per, T, sh.bad);
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      if (j >= per) break;
      const uint32_t i = tid * per + j;
      if (i < F) a.dist2[s_front[cur + i]] = du[j];  // as a level step folds
      sum += deg[j];
      rows += deg[j] != 0;
      big |= deg[j] > U;
    }
    if (!__syncthreads_or(big)) {
      if (__any(deg[0] != 0)) {
        uint32_t ei[U], dd[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          ei[u] = start[0] + u;
          dd[u] = u < deg[0] ? du[0] : 0xFFFFFFFFu;
        }
        edges(ei, dd);
      }
    } else {
      const uint32_t incl = wave_incl_scan(sum, lane), rincl = wave_incl_scan(rows, lane);
      if (lane == 63) {
        sh.wsum[wave] = incl;
        sh.wrows[wave] = rincl;
      }
      lds_barrier();
      uint32_t run = incl - sum, E = 0, row = rincl - rows, R = 0;
#pragma unroll
      for (uint32_t w = 0; w < NB / 64; ++w) {
        if (w < (uint32_t)wave) {
          run += sh.wsum[w];
          row += sh.wrows[w];
        }
        E += sh.wsum[w];
        R += sh.wrows[w];
      }
      if (E > NEAR_EDGES) {  // (their bits in s_near do not matter any more)
        for (uint32_t i = tid; i < F; i += NB) s_front[nxt + i] = s_front[cur + i];
        if (tid == 0) sh.cnt = F;
        wide = true;
      } else {
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
          if (deg[j] == 0) continue;
          s_start[row] = start[j] - run;
          s_off[row] = run;
          s_du[row] = du[j];
          run += deg[j];
          ++row;
        }
        lds_barrier();
        uint8_t* heads = sh.heads[wave];
        for (uint32_t x0 = wave * 64 * U; x0 < E; x0 += NB * U) {
          const uint32_t p0 = wave_upper_search(R, x0, lane, [&](uint32_t k) { return s_off[k]; });
          clear_heads(heads, lane);
          for (uint32_t k = p0 + 1 + lane; k < R; k += 64) {
            const uint32_t x = s_off[k] - x0;
            if (x >= 64 * U) break;
            heads[x - 1] = 1;
          }
          wave_lds_sync();
          uint32_t ei[U], dd[U], p = p0;
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) {
            const uint32_t x = x0 + u * 64 + lane;
            const uint32_t k = row_of(heads, u, lane, p);
            ei[u] = s_start[k] + x;
            dd[u] = x < E ? s_du[k] : 0xFFFFFFFFu;
          }
          edges(ei, dd);
          wave_lds_sync();
        }
      }
    }
    __syncthreads();  // (far list and spilled frontier are global)
    F = sh.cnt;
    uint32_t K = sh.far;
    if (F > FC) wide = true;
    while (F == 0 && K != 0 && !wide) {
      // the bound moves past the least distance that waits; what was improved
      // below the old bound since it was listed has been run already
      const unsigned long long was = bound;
      bound = max(bound, (unsigned long long)sh.low) + step;
      const uint32_t* list = far[side];
      __syncthreads();
      side ^= 1;
      if (tid == 0) {
        sh.far = 0;
        sh.low = 0xFFFFFFFFu;
      }
      __syncthreads();
      for (uint32_t i0 = 0; i0 < K; i0 += NB * U) {
        uint32_t v[U], d[U];
        bool f[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          const uint32_t i = i0 + u * NB + tid;
          v[u] = i < K ? list[i] : NONE;
        }
        pin(v);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) d[u] = v[u] != NONE ? coherent_load(&dist[v[u]]) : 0u;
        pin(d);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          f[u] = v[u] != NONE && d[u] >= was;
          if (v[u] != NONE) atomicAnd(&s_wait[v[u] >> 5], ~(1u << (v[u] & 31)));
          if (!f[u]) v[u] = 0;
        }
        append(f, v, d);
      }
      __syncthreads();
      F = sh.cnt;
      K = sh.far;
      if (F > FC) wide = true;
    }
    const uint32_t t = cur;
    cur = nxt;
    nxt = t;
    if (round > (unsigned long long)n * 64) sh.bad = ERR_TIMEOUT;
    __syncthreads();
  }
  __syncthreads();
  uint32_t code = V_DONE, err = sh.bad;
  if (err) code = V_ERROR;
  if (wide && !err) {
    code = V_TOP_DOWN;
    // the frontier, then what waits and is not in it
    for (uint32_t i = tid; i < min(F, FC); i += NB) out[i] = s_front[cur + i];
    if (tid == 0) sh.cnt = F;
    __syncthreads();
    for (uint32_t i = tid; i < sh.far; i += NB) {
      const uint32_t v = far[side][i];
      if (coherent_load(&dist[v]) < bound) continue;
      const uint32_t at = atomicAdd(&sh.cnt, 1u);
      if (at < n) out[at] = v;
    }
    __syncthreads();
    if (tid == 0) a.st->set[2].fcnt[NQF] = sh.cnt;
  }
  if (tid == 0) post_verdict(verdict, 0, code, err);
}

// ------------------------------------------------------------ bottom-up levels
// Is the graph symmetric (every entry (u, v) as often as (v, u))?  A bottom-up
// level looks for a parent of v along v's own row, which finds the edges into v
// only then.  Nothing promises it, so the first level that would go bottom-up
// is preceded by this pass over the adjacency: the sum over all entries of
// h(u, v) where u < v and -h(v, u) where u > v, h a keyed mix (add_pair), is zero
// modulo 2^64 if the graph is symmetric, and otherwise for few keys: for none if
// one entry lacks its reverse, for some 2^-47 of them or fewer for the worst small
// sets that were looked for.  The key is drawn anew for each check.  An id out of
// range counts as asymmetric, and so does a row that ends before it starts or rows
// that are not those of a.m entries: what a level step reports of them, a bottom-up
// level would not.  Bound by its instructions (three quarter-rate multiply-adds an
// entry among them) and the adjacency stream together: scale 22, 513 MB in 157 us,
// 3.3 TB/s.
//
// A wave runs an even share of the entries in slices of 64 * U, the next slice's
// loads issued before a slice is summed; the rows come in windows of 64.
// ARENA: `vbase` holds the first vertex of each of `ngraphs` graphs (and n after
// them), and an entry that leaves its row's graph counts as asymmetric too: a
// bottom-up level might pass it by, where a top-down one reports it.  A single
// traversal asks for the check only after a sample (lacks_reverse).  Here each
// workgroup takes SYM_BLOCK_SAMPLES entries of its own first, and ends if one lacks
// its reverse, as on a directed arena nearly all do: the check of 10 directed
// graphs takes 12 us, of 10 symmetric ones 48, as without the sample.
template <bool ARENA>
__global__ __launch_bounds__(PB) void symmetry_kernel(Args a, uint32_t n, const PairKey key,
                                                      const uint32_t* vbase, uint32_t ngraphs) {
  constexpr uint32_t U = NARROW_U;
  __shared__ uint32_t s_row[NW][64];  // its vertex, with the key's first word added
  __shared__ uint32_t s_lo[ARENA ? NW : 1][64], s_n[ARENA ? NW : 1][64];  // its graph's vertices
  __shared__ __align__(8) uint8_t s_heads[NW][64 * U];
  __shared__ unsigned long long s_sum[NW];
  State* st = a.st;
  if (st->done || st->error || (st->plan != V_CHECK && a.bottom_up != BU_QUERIES)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t m = (uint32_t)a.m;
  const uint32_t nw = gridDim.x * NW, gw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * NW + wave));
  uint32_t x0 = (uint32_t)((uint64_t)gw * m / nw);
  const uint32_t x1 = (uint32_t)((uint64_t)(gw + 1) * m / nw);
  unsigned long long sum = 0;
  if (ARENA) {
    bool missing = false;
    if (tid < SYM_BLOCK_SAMPLES) {
      uint32_t h = (blockIdx.x * SYM_BLOCK_SAMPLES + (uint32_t)tid + 1) * 0x9E3779B1u ^ key.k[1];
      h = (h ^ h >> 15) * (key.k[2] | 1u);
      h = (h ^ h >> 13) * 0x85EBCA6Bu;
      missing = lacks_reverse(a, n, (uint32_t)((uint64_t)h * n >> 32), h ^ key.k[3]);
    }
    if (__syncthreads_or(missing)) {
      if (tid == 0) st->asymmetric = 1;
      return;
    }
  }
  if (x0 < x1) {
    uint32_t r = wave_upper_search(n, x0, lane, [&](uint32_t p) { return (uint32_t)a.rp[p]; });
    r = (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
    uint32_t top = 0;     // largest id
    bool leaves = false;  // an entry leaves its graph
    uint32_t g0 = 0, g1 = 0;  // vertices of the lane's row's graph, as of the last window
    bool one = true;          // the window's rows are of one graph,
    uint32_t u0 = 0, un = 0;  // with these vertices
    uint32_t v[U], ahead[U];
    auto fetch = [&](uint32_t at, uint32_t (&t)[U]) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t x = at + u * 64u + (uint32_t)lane;
        t[u] = x < x1 ? (uint32_t)__builtin_nontemporal_load(&a.col[x]) : 0u;
      }
    };
    fetch(x0, ahead);
    uint32_t b = (uint32_t)a.rp[min(r + lane, n)], e = (uint32_t)a.rp[min(r + lane + 1, n)];
    bool fresh = true;  // the window is not in LDS yet
    bool some = false;
    uint32_t wend = 0;
    while (x0 < x1 && r < n) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) v[u] = ahead[u];
      const uint32_t send = min(x1 - x0, 64u * U) + x0;
      fetch(send, ahead);
      uint32_t lo = x0;
      while (true) {
        if (fresh) {
          wend = (uint32_t)__builtin_amdgcn_readlane((int)e, 63);
          some = e > b && e > lo;
          top = e < b ? ~0u : top;
          const unsigned long long rows = __ballot(some);
          if (some) s_row[wave][lane_rank(rows)] = r + lane + key.k[0];
          if (ARENA && some) {
            if (r + lane >= g1) {
              uint32_t g = 0, end = ngraphs;
              while (end - g > 1) {
                const uint32_t mid = (g + end) >> 1;
                if (vbase[mid] <= r + lane) g = mid; else end = mid;
              }
              g0 = vbase[g];
              g1 = vbase[g + 1];
            }
            s_lo[wave][lane_rank(rows)] = g0;
            s_n[wave][lane_rank(rows)] = g1 - g0;
          }
          if (ARENA && rows) {
            const int l = __builtin_ctzll(rows);
            u0 = (uint32_t)__builtin_amdgcn_readlane((int)g0, l);
            un = (uint32_t)__builtin_amdgcn_readlane((int)g1, l) - u0;
            one = __all(!some || g0 == u0);
          }
          wave_lds_sync();
          fresh = false;
        }
        // the window's entries of the slice: [lo, hi)
        const uint32_t hi = min(send, wend);
        if (lo < hi) {
          const uint32_t first = (uint32_t)__popcll(__ballot(some && b <= lo)) - 1u;
          const bool begins = some && b > lo && b < hi;
          const bool whole = lo == x0 && hi == x0 + 64u * U;
          if (__any(begins)) {
            clear_heads(s_heads[wave], lane);
            if (begins) s_heads[wave][b - x0 - 1] = 1;
            wave_lds_sync();
            uint32_t p = first;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
              const uint32_t k = row_of(s_heads[wave], u, lane, p);
              uint32_t w = s_row[wave][k];
              const bool in = whole || x0 + u * 64u + (uint32_t)lane - lo < hi - lo;
              if (!in) w = v[u] + key.k[0];
              if (ARENA && !one) leaves |= in && v[u] - s_lo[wave][k] >= s_n[wave][k];
              sum = add_pair(sum, w, v[u] + key.k[0], key.k);
            }
            wave_lds_sync();
          } else {  // within one row
            const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_row[wave][first]);
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
              const bool in = whole || x0 + u * 64u + (uint32_t)lane - lo < hi - lo;
              if (ARENA && !one) leaves |= in && v[u] - s_lo[wave][first] >= s_n[wave][first];
              sum = add_pair(sum, in ? row : v[u] + key.k[0], v[u] + key.k[0], key.k);
            }
          }
          if (ARENA && one) {  // the usual case, without the lookups
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
              const bool in = whole || x0 + u * 64u + (uint32_t)lane - lo < hi - lo;
              leaves |= in && v[u] - u0 >= un;
            }
          }
          lo = hi;
        }
        if (wend >= send || r >= n) break;
        r += 64;
        b = (uint32_t)a.rp[min(r + lane, n)];
        e = (uint32_t)a.rp[min(r + lane + 1, n)];
        fresh = true;
        wave_lds_sync();
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) top = max(top, v[u]);
      if (lo < send) break;  // rows that end before the entries do
      x0 = send;
    }
    const bool bad = __any(top >= n || leaves) || x0 < x1 || (uint32_t)a.rp[n] != m;
    if (bad && lane == 0) st->asymmetric = 1;
  }
#pragma unroll
  for (int d = 32; d; d >>= 1) sum += __shfl_down(sum, d, 64);
  if (lane == 0) s_sum[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    unsigned long long all = 0;
    for (int w = 0; w < NW; ++w) all += s_sum[w];
    if (all) atomicAdd(&st->sym_sum[blockIdx.x & 7], all);
  }
}

// A wide BFS level of a symmetric graph, bottom-up: a lane per vertex not yet
// visited, which looks along its row for a visited neighbour; on a symmetric
// graph that one is in the frontier (had it been visited earlier, so would the
// vertex have been).  Where the frontier has a good part of the edges left the
// first few entries of a row decide, and nothing is written but what is found:
// no atomic, no found byte.  Reads one bitmap and writes the other, whole words
// by the wave that owns them.  A vertex without edges counts as visited from
// then on (no row names it).  Rows are read by their lane up to BU_LANE
// entries, then by the wave together.  Bound by the lines its row heads lie in:
// scale 22's growing, widest and next level take 59, 23 and 11 us where a level
// step takes 270 (growing) and 540 (widest), so that with the check, once per
// traversal, the traversal goes from 1083 to 484 us (454 since).
__global__ __launch_bounds__(PB) void bottom_up_kernel(Args a) {
  __shared__ int32_t s_stage[NW][STAGE];
  __shared__ uint32_t s_bc[NW + 8];
  constexpr int U = 4;
  State* st = a.st;
  if (st->done || st->error || !goes_bottom_up(st)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t L = st->base, n = (uint32_t)a.q[0].n;
  LevelSet* cur = &st->set[L % 3];
  int32_t* fout = (L & 1) ? a.front0 : a.front1;
  const uint32_t c = st->vsel[L & 1];
  const uint32_t* seen = a.visit + (size_t)c * (uint32_t)a.vwords;
  uint32_t* next = a.visit + (size_t)(c ^ 1u) * (uint32_t)a.vwords;
  // what the parent kernel does for the level after
  if (blockIdx.x == 0) {
    LevelSet* z = &st->set[(L + 1) % 3];
    if (tid <= NQF) z->fcnt[tid] = 0;
    if (tid < NQD) z->qctr[tid] = 0;
    if (tid < NQD) z->cclaim[tid][0] = 0;
    if (tid == 0) {
      st->levels_run = L + 1;
      st->vsel[(L + 1) & 1] = c ^ 1u;
      st->vstale[(L + 1) & 1] = 1u;
    }
  }
  for (int i = blockIdx.x * PB + tid; i < a.ngroups_cap; i += gridDim.x * PB) {
    a.grp_packed[(L + 1) % 3 * a.ngroups_cap + i] = 0;
    a.grp_done[(L + 1) % 3 * a.ngroups_cap + i] = 0;
  }
  Stage s{s_stage[wave], 0u};
  for (uint32_t b = (blockIdx.x * NW + wave) * 64u; b < (uint32_t)a.slots; b += gridDim.x * PB) {
    const uint32_t v = b + (uint32_t)lane;
    const uint32_t word = v < (uint32_t)a.slots ? seen[v >> 5] : ~0u;
    bool need = v < n && !(word >> (v & 31) & 1u);
    uint32_t x = 0, e = 0;
    if (need) {
      x = (uint32_t)a.rp[v];
      e = (uint32_t)a.rp[v + 1];
    }
    const bool alone = need && x == e;
    bool found = false;
    need = x < e;
    for (uint32_t it = 0; it < BU_LANE / U && __any(need); ++it) {
      uint32_t w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) w[u] = need ? (uint32_t)a.col[min(x + u, e - 1)] : 0u;
      pin(w);
      uint32_t words[U];
#pragma unroll
      for (int u = 0; u < U; ++u) words[u] = need ? seen[w[u] >> 5] : 0u;
      pin(words);
#pragma unroll
      for (int u = 0; u < U; ++u) found |= (words[u] >> (w[u] & 31) & 1u) != 0;
      x += U;
      need = need && !found && x < e;
    }
    for (unsigned long long rest = __ballot(need); rest; rest &= rest - 1) {
      const int k = __builtin_ctzll(rest);
      const uint32_t y1 = (uint32_t)__builtin_amdgcn_readlane((int)e, k);
      bool hit = false;
      for (uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, k); y < y1 && !hit; y += 64 * U) {
        uint32_t w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = (uint32_t)a.col[min(y + (uint32_t)(u * 64 + lane), y1 - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) hit |= seen[w[u] >> 5] >> (w[u] & 31) & 1u;
        hit = __any(hit);
      }
      found |= hit && lane == k;
    }
    const unsigned long long add = __ballot(found || alone);
    if ((lane & 31) == 0 && v < (uint32_t)a.slots) next[v >> 5] = word | (uint32_t)(add >> (lane & 32));
    if (found) a.level[v] = (int32_t)L + 1;
    stage_push(s, found, (int32_t)v, a, cur, fout, lane);
  }
  block_flush(s, a, cur, fout, tid, s_bc);
}


// ------------------------------------------------- bottom-up levels, by query
// Several queries (a batch, a serving engine) are at different points of their
// traversals, so each goes bottom-up or top-down by itself: the tally kernel
// adds up the edges of each query's frontier, the bottom-up kernel runs the
// queries that qualify and leaves what it finds as found bytes, the parent
// kernel passes over their entries, and the level's harvest takes the found
// bytes of both.
//
// Tally: the degrees of a sample of the frontier, 64 consecutive entries of
// every `stride` * 64 so that about TALLY_SAMPLE are read.  The entries of a
// wave are mostly one query's (the harvest appends in slot order): they are
// summed by the wave, else in LDS.  Then a wave per running query samples the rows
// that a bottom-up level would read.
__global__ __launch_bounds__(PB) void tally_kernel(Args a, uint32_t step) {
  __shared__ uint32_t s_fpre[NQF + 2];
  __shared__ uint32_t s_edges[MAX_QUERIES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const State* st = a.st;
  if (st->done || st->error || st->symmetric != 1) return;
  const uint32_t L = st->base + step;
  const LevelSet* prv = &st->set[(L + 2) % 3];
  if (tid < 64) {
    const uint32_t incl = wave_incl_scan(min(prv->fcnt[lane], (uint32_t)a.fcap), lane);
    s_fpre[lane + 1] = incl;
    if (lane == 0) s_fpre[0] = 0;
    if (lane == 63) s_fpre[NQF + 1] = incl + prv->fcnt[NQF];
  }
  for (int i = tid; i < a.nq; i += PB) s_edges[i] = 0;
  __syncthreads();
  const uint32_t F = s_fpre[NQF + 1];
  if (F < TALLY_MIN || F > (uint32_t)a.slots) return;
  for (uint32_t q = blockIdx.x * NW + wave; q < (uint32_t)a.nq; q += gridDim.x * NW) {
    const Query Q = a.q[q];
    if (Q.n <= 0 || Q.last + 1 < (int32_t)L) continue;
    uint32_t read, found;
    sample_row(a, (uint32_t)Q.vbase, (uint32_t)Q.n, a.visit + ((uint32_t)Q.slot0 >> 5),
               (L * 64u + (uint32_t)lane + 1) * 0x9E3779B1u, read, found);
#pragma unroll
    for (int o = 32; o; o >>= 1) {
      read += (uint32_t)__shfl_xor((int)read, o, 64);
      found += (uint32_t)__shfl_xor((int)found, o, 64);
    }
    if (lane == 0) {
      a.tally[4 * a.nq + q] = (uint32_t)min((uint64_t)read * (uint32_t)Q.n / 64u, (uint64_t)0xFFFFFFFFu);
      a.tally[5 * a.nq + q] = (uint32_t)min((uint64_t)found * (uint32_t)Q.n / 64u, (uint64_t)0xFFFFFFFFu);
    }
  }
  const int32_t* fin = (L & 1) ? a.front1 : a.front0;
  const uint32_t stride = ceil_div(F, TALLY_SAMPLE);
  for (uint32_t c = blockIdx.x * NW + wave; c * stride * 64u < F; c += gridDim.x * NW) {
    const uint32_t i = c * stride * 64u + (uint32_t)lane;
    uint32_t q = NONE, deg = 0;
    if (i < F) {
      const uint32_t slot = (uint32_t)frontier_at(a, fin, s_fpre, i);
      q = (uint32_t)a.qmap[slot >> 5];
      const int32_t v = a.q[q].vbase + ((int32_t)slot - a.q[q].slot0);
      deg = (uint32_t)(a.rp[v + 1] - a.rp[v]) * stride;
    }
    const uint32_t q0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
    if (__all(q == q0 || q == NONE)) {
      const uint32_t sum = __shfl(wave_incl_scan(deg, lane), 63, 64);
      if (lane == 0) atomicAdd(&s_edges[q0], sum);
    } else if (q != NONE) {
      atomicAdd(&s_edges[q], deg);
    }
  }
  __syncthreads();
  for (int i = tid; i < a.nq; i += PB)
    if (s_edges[i]) {
      atomicAdd(&a.tally[(L & 1) * a.nq + i], s_edges[i]);
      atomicAdd(&a.tally[2 * a.nq + i], s_edges[i]);
    }
}

// The bottom-up level of the queries that qualify runs queries of one graph
// together, up to BU_GROUP of them: per vertex a word with a bit per query of
// the group, set if that query has visited it, so that one load of a
// neighbour's word answers for all of them and a row is read once.  With one
// bitmap per query, 512 queries over 64 graphs made 100 M random probes on the
// growing level, 490 us at the chip's rate for random loads; now that level
// takes 41 us for the words and 253 for the rows, 1.5 ms top-down (2.6 for the
// widest, now 146), and the batch 5.93 -> 2.00 ms.
//
// The first of its two kernels lists the qualifying queries by graph, then
// their groups with their runs of 64 vertices (scanned; every workgroup for
// itself, the first one for the second kernel), and writes the words.  Lists
// and words lie where the parent kernel will put the level's records.
struct UpLists {
  const uint16_t* query;  // qualifying queries
  const uint16_t* first;  // first of them of each group, and their number
  const uint32_t* run;    // first run of each group, and the number of runs
  const uint32_t* count;  // groups
};

__device__ __forceinline__ UpLists up_lists(const Args& a) {
  uint32_t* t = (uint32_t*)a.rec_q;  // (a query has at least 32 slots)
  return UpLists{(const uint16_t*)(t + 1 + a.nq + 1), (const uint16_t*)(t + 1 + a.nq + 1) + a.nq + 1,
                 t + 1, t};
}

// Words of a group, by vertex of its graph; slot0: of its first query.
__device__ __forceinline__ uint16_t* up_words(const Args& a, uint32_t slot0) {
  return (uint16_t*)(a.rec + slot0);
}

__global__ __launch_bounds__(QB) void bottom_up_words_kernel(Args a, uint32_t step) {
  __shared__ uint16_t s_list[MAX_QUERIES + 1], s_first[MAX_QUERIES + 1];
  __shared__ uint32_t s_pre[MAX_QUERIES + 1];
  constexpr int NW = QB / 64;
  __shared__ uint32_t s_sum[3][NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const State* st = a.st;
  if (st->done || st->error || st->symmetric != 1) return;
  const uint32_t L = st->base + step;
  uint32_t count = 0;
  for (int q0 = 0; q0 < a.nq; q0 += QB) {
    const int q = q0 + tid;
    const bool on = q < a.nq && query_goes_bottom_up(a, (uint32_t)q, L);
    const unsigned long long m = __ballot(on);
    if (lane == 0) s_sum[0][wave] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t c = count + lane_rank(m);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) c += s_sum[0][w];
      count += s_sum[0][w];
    }
    if (on) {
      s_list[c] = (uint16_t)q;
      s_pre[c] = (uint32_t)a.q[q].vbase;
    }
    __syncthreads();
  }
  const UpLists up = up_lists(a);
  if (count == 0) {
    if (blockIdx.x == 0 && tid == 0) *(uint32_t*)up.count = 0;
    return;
  }
  if (count <= BU_SORT) {  // a batch has a graph's queries together, an engine does not
    uint32_t rank = 0, q = 0;
    if ((uint32_t)tid < count) {
      const uint32_t vb = s_pre[tid];
      q = s_list[tid];
      for (uint32_t k = 0; k < count; ++k) rank += s_pre[k] < vb || (s_pre[k] == vb && k < (uint32_t)tid);
    }
    __syncthreads();
    if ((uint32_t)tid < count) s_list[rank] = (uint16_t)q;
    __syncthreads();
  }
  uint32_t groups = 0, runs = 0, since = 0;  // since: where the graph's queries begin in the list
  for (uint32_t k0 = 0; k0 < count; k0 += QB) {
    const uint32_t k = k0 + (uint32_t)tid;
    int32_t vb = 0, n = 0;
    bool other = false;
    if (k < count) {
      vb = a.q[s_list[k]].vbase;
      n = a.q[s_list[k]].n;
      other = k == 0 || vb != a.q[s_list[k - 1]].vbase;
    }
    uint32_t from = other ? k : 0u;  // max-scanned
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(from, d, 64);
      if (lane >= d) from = max(from, y);
    }
    if (lane == 63) s_sum[0][wave] = from;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) from = max(from, s_sum[0][w]);
    }
    from = max(from, since);
#pragma unroll
    for (int w = 0; w < NW; ++w) since = max(since, s_sum[0][w]);
    const bool begins = k < count && (k - from) % BU_GROUP == 0;
    const uint32_t r = begins ? ceil_div((uint32_t)n, 64u) : 0u;
    const unsigned long long m = __ballot(begins);
    const uint32_t incl = wave_incl_scan(r, lane);
    if (lane == 63) {
      s_sum[1][wave] = (uint32_t)__popcll(m);
      s_sum[2][wave] = incl;
    }
    __syncthreads();
    uint32_t g = groups + lane_rank(m), x = runs + incl - r;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) {
        g += s_sum[1][w];
        x += s_sum[2][w];
      }
      groups += s_sum[1][w];
      runs += s_sum[2][w];
    }
    if (begins) {
      s_first[g] = (uint16_t)k;
      s_pre[g] = x;
    }
    __syncthreads();
  }
  if (tid == 0) {
    s_first[groups] = (uint16_t)count;
    s_pre[groups] = runs;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (uint32_t k = tid; k < count; k += QB) ((uint16_t*)up.query)[k] = s_list[k];
    for (uint32_t g = tid; g <= groups; g += QB) {
      ((uint16_t*)up.first)[g] = s_first[g];
      ((uint32_t*)up.run)[g] = s_pre[g];
    }
    if (tid == 0) *(uint32_t*)up.count = groups;
  }
  const uint32_t nw = gridDim.x * NW, gw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * NW + wave));
  uint32_t t = (uint32_t)((uint64_t)gw * runs / nw);
  const uint32_t t1 = (uint32_t)((uint64_t)(gw + 1) * runs / nw);
  if (t >= t1) return;
  uint32_t g = wave_upper_search(groups, t, lane, [&](uint32_t p) { return s_pre[p]; });
  for (; t < t1; ++g) {
    const uint32_t k0 = s_first[g], nk = s_first[g + 1] - k0, tg = s_pre[g], te = min(t1, s_pre[g + 1]);
    const uint32_t slot0 = (uint32_t)lane < nk ? (uint32_t)a.q[s_list[k0 + lane]].slot0 : 0u;
    const uint32_t n = (uint32_t)a.q[s_list[k0]].n;
    uint16_t* words = up_words(a, (uint32_t)__builtin_amdgcn_readlane((int)slot0, 0));
    for (; t < te; ++t) {
      const uint32_t v = (t - tg) * 64u + (uint32_t)lane;
      uint32_t w = 0;
      for (uint32_t j = 0; j < nk; ++j) {
        const uint32_t* seen = a.visit + ((uint32_t)__builtin_amdgcn_readlane((int)slot0, j) >> 5);
        if (v < n) w |= (seen[v >> 5] >> (v & 31) & 1u) << j;
      }
      if (v < n) words[v] = (uint16_t)w;
    }
  }
}

// The second: as bottom_up_kernel, but the visited bitmaps stay as they are and
// what is found goes to the found bytes.
__global__ __launch_bounds__(PB) void bottom_up_queries_kernel(Args a, uint32_t step) {
  constexpr int U = 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const State* st = a.st;
  if (st->done || st->error || st->symmetric != 1) return;
  const UpLists up = up_lists(a);
  const uint32_t groups = *up.count;
  if (groups == 0) return;
  const uint32_t runs = up.run[groups];
  const uint32_t nw = gridDim.x * NW, gw = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * NW + wave));
  uint32_t t = (uint32_t)((uint64_t)gw * runs / nw);
  const uint32_t t1 = (uint32_t)((uint64_t)(gw + 1) * runs / nw);
  if (t >= t1) return;
  uint32_t g = wave_upper_search(groups, t, lane, [&](uint32_t p) { return up.run[p]; });
  for (; t < t1; ++g) {
    g = (uint32_t)__builtin_amdgcn_readfirstlane((int)g);
    const uint32_t k0 = up.first[g], nk = up.first[g + 1] - k0, tg = up.run[g], te = min(t1, up.run[g + 1]);
    const Query Q = a.q[up.query[k0]];
    const uint32_t n = (uint32_t)Q.n;
    // first slot of the group's queries, a lane each
    const uint32_t slot0 = (uint32_t)lane < nk ? (uint32_t)a.q[up.query[k0 + lane]].slot0 : 0u;
    const uint16_t* words = up_words(a, (uint32_t)Q.slot0);
    const uint32_t all = (1u << nk) - 1u;
    for (; t < te; ++t) {
      const uint32_t v = (t - tg) * 64u + (uint32_t)lane;  // vertex of the graph
      uint32_t need = v < n ? all & ~(uint32_t)words[v] : 0u, found = 0;  // a bit per query
      uint32_t x = 0, e = 0;
      if (need) {
        x = (uint32_t)a.rp[Q.vbase + v];
        e = (uint32_t)a.rp[Q.vbase + v + 1];
      }
      // a vertex without edges counts as visited from now on (no row names it)
      const unsigned long long alone = __ballot(need && x == e);
      if (alone) {
        const uint32_t bits = (uint32_t)(alone >> (lane & 32));
        for (uint32_t j = 0; j < nk; ++j) {
          uint32_t* seen = a.visit + ((uint32_t)__builtin_amdgcn_readlane((int)slot0, j) >> 5);
          if ((lane & 31) == 0 && bits) seen[v >> 5] |= bits;
        }
      }
      if (x >= e) need = 0;
      for (uint32_t it = 0; it < BU_LANE / U && __any(need != 0); ++it) {
        uint32_t w[U], hit = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
          w[u] = need ? (uint32_t)a.col[min(x + u, e - 1)] : (uint32_t)Q.vbase;
        pin(w);
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = need ? words[min(w[u] - (uint32_t)Q.vbase, n - 1)] : 0u;
        pin(w);
#pragma unroll
        for (int u = 0; u < U; ++u) hit |= w[u];
        found |= hit & need;
        need &= ~found;
        x += U;
        if (x >= e) need = 0;
      }
      for (unsigned long long rest = __ballot(need != 0); rest; rest &= rest - 1) {
        const int l = __builtin_ctzll(rest);
        const uint32_t y1 = (uint32_t)__builtin_amdgcn_readlane((int)e, l);
        const uint32_t asked = (uint32_t)__builtin_amdgcn_readlane((int)need, l);
        uint32_t want = asked;
        for (uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, l); y < y1 && want; y += 64 * U) {
          uint32_t w[U], hit = 0;
#pragma unroll
          for (int u = 0; u < U; ++u)
            w[u] = min((uint32_t)(a.col[min(y + (uint32_t)(u * 64 + lane), y1 - 1)] - Q.vbase), n - 1);
#pragma unroll
          for (int u = 0; u < U; ++u) hit |= (uint32_t)words[w[u]];
#pragma unroll
          for (int d = 1; d < 64; d <<= 1) hit |= (uint32_t)__shfl_xor((int)hit, d, 64);
          want &= ~(uint32_t)__builtin_amdgcn_readfirstlane((int)hit);
        }
        if (lane == l) found |= asked & ~want;
      }
      if (__any(found != 0))
        for (uint32_t j = 0; j < nk; ++j)
          if (found >> j & 1u) a.found[(uint32_t)__builtin_amdgcn_readlane((int)slot0, j) + v] = 1;
    }
  }
}

// After a symmetry check that the host asked for (several queries).
__global__ void settle_symmetry_kernel(State* st, uint32_t ticket, uint32_t* verdict) {
  if (threadIdx.x || blockIdx.x) return;
  const bool symmetric = found_symmetric(st);
  st->symmetric = symmetric ? 1u : 2u;
  st->plan = 0;
  post_verdict(verdict, ticket, symmetric ? V_BOTTOM_UP : V_TOP_DOWN, 0);
}

// Before the first level that tallies after some that did not.
__global__ __launch_bounds__(PB) void clear_tally_kernel(Args a) {
  for (int i = blockIdx.x * PB + threadIdx.x; i < 2 * a.nq; i += gridDim.x * PB) a.tally[i] = 0;
}

// ------------------------------------------------------------ init / admit / advance
// Traversal-set start: level sets and counters cleared.  Queries are
// started by admit_kernel.
__global__ __launch_bounds__(PB) void init_kernel(Args a) {
  const uint32_t gsz = gridDim.x * PB;
  const uint32_t gid = blockIdx.x * PB + threadIdx.x;
  for (uint32_t i = gid; i < 3u * (uint32_t)a.ngroups_cap; i += gsz) {
    a.grp_packed[i] = 0;
    a.grp_done[i] = 0;
  }
  for (uint32_t i = gid; i < (uint32_t)(MAX_GRID * NSTAT); i += gsz) a.stats[i] = 0;
  uint32_t* stw = (uint32_t*)a.st;
  for (uint32_t i = gid; i < sizeof(State) / 4; i += gsz) stw[i] = 0;
}

// Start of a single traversal in one launch: level sets, counters, outputs and
// visited state, the query's record and its source as frontier 0.  No
// workgroup reads what another writes, so what the batch and serving paths do
// with an init kernel, two uploads and two admit kernels needs no order here;
// the query travels by value.  Bound by its stores (s22: 26 MB); on small
// graphs by the launch itself, which is why it is one.
template <int P>
__global__ __launch_bounds__(PB) void start_kernel(Args a, Query Q) {
  const uint32_t gsz = gridDim.x * PB;
  const uint32_t gid = blockIdx.x * PB + threadIdx.x;
  const uint32_t src = (uint32_t)Q.src, n = (uint32_t)Q.n;
  for (uint32_t v = gid; v < n; v += gsz) {
    if (P == PROB_BFS) {
      a.level[v] = (v == src) ? 0 : -1;
    } else {
      const uint32_t d = (v == src) ? 0u : 0xFFFFFFFFu;
      a.dist[v] = d;
      a.dist2[v] = d;
      if (!a.hint) a.visit[v] = 0u;  // iteration stamps
    }
  }
  for (uint32_t i = gid; i < (uint32_t)a.vwords; i += gsz) {
    a.qmap[i] = 0;
    if (P == PROB_BFS) {  // every bitmap in use holds the source
      const uint32_t x = (i == src >> 5) ? (1u << (src & 31)) : 0u;
      for (uint32_t h = 0; h < (a.hint ? 2u + NHINT : 2u); ++h) a.visit[(size_t)h * a.vwords + i] = x;
    }
  }
  if (a.hint) {  // nothing found yet
    uint32_t* f = (uint32_t*)a.found;
    for (uint32_t i = gid; i < (uint32_t)a.vwords * 8u; i += gsz) f[i] = 0u;
  }
  if (P == PROB_SSSP && a.bound)
    for (uint32_t i = gid; i < (uint32_t)a.vwords * 8u; i += gsz) ((uint32_t*)a.bound)[i] = ~0u;
  for (uint32_t i = gid; i < 3u * (uint32_t)a.ngroups_cap; i += gsz) {
    a.grp_packed[i] = 0;
    a.grp_done[i] = 0;
  }
  if (a.count_stats)
    for (uint32_t i = gid; i < (uint32_t)(MAX_GRID * NSTAT); i += gsz) a.stats[i] = 0;
  // frontier 0 is the source alone, in the overflow queue: the fills of
  // frontier L are in set (L + 2) % 3
  uint32_t* stw = (uint32_t*)a.st;
  const uint32_t fill = (uint32_t)(&a.st->set[2].fcnt[NQF] - stw);
  for (uint32_t i = gid; i < sizeof(State) / 4; i += gsz) stw[i] = i == fill ? 1u : 0u;
  if (gid == 0) {
    a.q[0] = Q;
    a.front0[(size_t)NQF * a.fcap] = Q.src;
  }
}

// Starts the queries list[0 .. count) at level index L = st->base: their
// outputs set to "unreached" except the source, their visit state cleared and
// their 32-slot chunks mapped to them.  Query list[k] is served by the
// workgroups [pre[k], pre[k + 1]) (pre = list + count, a host-built prefix of
// per-query workgroup counts proportional to n), so a batch of many small
// queries does not leave most of the grid idle.
template <int P>
__global__ __launch_bounds__(PB) void admit_kernel(Args a, const int32_t* list, int32_t count) {
  const int32_t* pre = list + count;
  // query of this workgroup: largest k with pre[k] <= blockIdx.x
  int32_t lo = 0, hi = count;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (pre[mid] <= (int32_t)blockIdx.x) lo = mid; else hi = mid;
  }
  const int32_t qi = list[lo];
  const uint32_t j = blockIdx.x - (uint32_t)pre[lo];
  const uint32_t stride = (uint32_t)(pre[lo + 1] - pre[lo]) * PB;
  const Query Q = a.q[qi];
  const uint32_t s0 = (uint32_t)Q.slot0, src = (uint32_t)Q.src;
  for (uint32_t v = j * PB + threadIdx.x; v < (uint32_t)Q.n; v += stride) {
    if (P == PROB_BFS) {
      a.level[s0 + v] = (v == src) ? 0 : -1;
    } else {
      const uint32_t d = (v == src) ? 0u : 0xFFFFFFFFu;
      a.dist[s0 + v] = d;
      a.dist2[s0 + v] = d;
      if (!a.hint) a.visit[s0 + v] = 0u;  // iteration stamps
    }
  }
  const uint32_t words = ((uint32_t)Q.n + 31) / 32;
  for (uint32_t i = j * PB + threadIdx.x; i < words; i += stride) {
    a.qmap[s0 / 32 + i] = qi;
    if (P == PROB_BFS) {
      const uint32_t x = (i == src >> 5) ? (1u << (src & 31)) : 0u;
      a.visit[s0 / 32 + i] = x;  // both bitmaps hold the source
      a.visit[(size_t)a.vwords + s0 / 32 + i] = x;
      if (a.hint) {  // the per-XCD copies hold the source too; nothing found yet
        for (uint32_t h = 0; h < (uint32_t)NHINT; ++h) a.visit[(size_t)(2 + h) * a.vwords + s0 / 32 + i] = x;
        uint32_t* f = (uint32_t*)(a.found + (size_t)(s0 / 32 + i) * 32);
        for (int k = 0; k < 8; ++k) f[k] = 0u;
      }
    } else if (a.hint) {  // SSSP: nothing found yet
      uint32_t* f = (uint32_t*)(a.found + (size_t)(s0 / 32 + i) * 32);
      for (int k = 0; k < 8; ++k) f[k] = 0u;
      if (a.bound)
        for (int k = 0; k < 8; ++k) ((uint32_t*)a.bound)[(size_t)(s0 / 32 + i) * 8 + k] = ~0u;
    }
  }
}

// Results of finished queries to their callers' arrays: entry k of the list is
// {output address (two words), first slot, vertices}, and it is copied by the
// workgroups [pre[k], pre[k + 1]), ADMIT_CHUNK slots each.  One launch for all:
// as a copy command each, 48 results took 0.4 ms of commands.
__global__ __launch_bounds__(PB) void retire_kernel(const uint32_t* slots, const uint4* list,
                                                    const int32_t* pre, int32_t count) {
  int32_t lo = 0, hi = count;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (pre[mid] <= (int32_t)blockIdx.x) lo = mid; else hi = mid;
  }
  const uint4 e = list[lo];
  uint32_t* out = (uint32_t*)((uint64_t)e.y << 32 | e.x);
  const uint32_t v0 = (blockIdx.x - (uint32_t)pre[lo]) * ADMIT_CHUNK;
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < ADMIT_CHUNK; i += PB)
    if (v0 + i < e.w) out[v0 + i] = slots[e.z + v0 + i];
}

// BFS with per-XCD copies: every found byte of the workspace cleared (a
// serving engine's output arena has slots that no query has been admitted to
// yet; the harvest kernel must see no found vertex there).
__global__ __launch_bounds__(PB) void clear_found_kernel(Args a) {
  uint32_t* f = (uint32_t*)a.found;
  const uint32_t nw = (uint32_t)a.vwords * 8u;
  for (uint32_t i = blockIdx.x * PB + threadIdx.x; i < nw; i += gridDim.x * PB) f[i] = 0u;
}

// Second half of admission (after admit_kernel): sources into frontier L.
__global__ void admit_sources_kernel(Args a, const int32_t* list, int32_t count) {
  State* st = a.st;
  const uint32_t L = st->base;
  LevelSet* ls = &st->set[(L + 2) % 3];  // fills of frontier L
  int32_t* fin = (L & 1) ? a.front1 : a.front0;
  const int32_t k = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k < count) {
    Query* Q = &a.q[list[k]];
    Q->lstart = (int32_t)L;
    Q->last = (int32_t)L;
    if (a.bottom_up == BU_QUERIES) {
      const int32_t q = list[k];
      for (int i = 0; i < 3; ++i) a.tally[i * a.nq + q] = 0;
      a.tally[3 * a.nq + q] = (uint32_t)(a.rp[Q->vbase + Q->n] - a.rp[Q->vbase]);
    }
    const uint32_t pos = atomicAdd(&ls->fcnt[NQF], 1u);
    if (pos < (uint32_t)a.slots) fin[(size_t)NQF * a.fcap + pos] = Q->slot0 + Q->src;
    else set_error(st, ERR_CAPACITY);
  }
  if (k == 0) st->done = 0;
}

// End of a replay (one wave): the level base moves on, an empty frontier ends
// the traversals without another replay to find it empty, and base, done, error
// and levels_run go to the host's flags (pinned memory), so that no copy has to
// follow the replay.
__global__ void advance_kernel(State* st, uint32_t steps, uint32_t* flags) {
  const int lane = threadIdx.x;
  const uint32_t base = st->base + steps;
  const LevelSet* prv = &st->set[(base + 2) % 3];
  const bool some = prv->fcnt[lane] != 0 || prv->fcnt[NQF] != 0;
  const bool empty = !__any(some);
  if (lane != 0) return;
  st->base = base;
  if (empty) st->done = 1;
  if (!flags) return;
  const uint32_t v[4] = {base, st->done, st->error, st->levels_run};
  for (int i = 0; i < 4; ++i)
    __hip_atomic_store(&flags[i], v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------- tables
template <int P, int PH, bool TM>
static const void* parent_for(int g) {
  switch (g) {
    case AGG_NONE: return (const void*)parent_kernel<P, AGG_NONE, PH, TM>;
    case AGG_WAVE: return (const void*)parent_kernel<P, AGG_WAVE, PH, TM>;
    case AGG_BLOCK: return (const void*)parent_kernel<P, AGG_BLOCK, PH, TM>;
    case AGG_MULTI: return (const void*)parent_kernel<P, AGG_MULTI, PH, TM>;
    default: return nullptr;
  }
}

template <bool TM>
static const void* parent_ptr(int problem, int gran) {
  if (gran == AGG_FLAT)
    return problem == PROB_BFS ? (const void*)parent_kernel<PROB_BFS, AGG_FLAT, PH_BOTH, TM>
                               : (const void*)parent_kernel<PROB_SSSP, AGG_FLAT, PH_BOTH, TM>;
  return problem == PROB_BFS ? parent_for<PROB_BFS, PH_BOTH, TM>(gran)
                             : parent_for<PROB_SSSP, PH_LIST, TM>(gran);
}

// BFS, and the flat kernel: both passes in one kernel.  SSSP with child
// kernels: pass 1, the child kernel, then pass 2 (serial_kernel_ptr).
const void* parent_kernel_ptr(int problem, int gran, bool timed) {
  return timed ? parent_ptr<true>(problem, gran) : parent_ptr<false>(problem, gran);
}

const void* serial_kernel_ptr(int problem, int gran, bool timed) {
  if (problem == PROB_BFS || gran == AGG_FLAT) return nullptr;
  return timed ? parent_for<PROB_SSSP, PH_SERIAL, true>(gran)
               : parent_for<PROB_SSSP, PH_SERIAL, false>(gran);
}

const void* harvest_kernel_ptr(int problem, bool timed) {
  if (problem == PROB_BFS)
    return timed ? (const void*)harvest_kernel<PROB_BFS, true>
                 : (const void*)harvest_kernel<PROB_BFS, false>;
  return timed ? (const void*)harvest_kernel<PROB_SSSP, true>
               : (const void*)harvest_kernel<PROB_SSSP, false>;
}

template <bool TM>
static const void* child_ptr(int problem, bool nt) {
  if (problem == PROB_BFS)
    return nt ? (const void*)child_kernel<PROB_BFS, TM, true>
              : (const void*)child_kernel<PROB_BFS, TM, false>;
  return nt ? (const void*)child_kernel<PROB_SSSP, TM, true>
            : (const void*)child_kernel<PROB_SSSP, TM, false>;
}

const void* child_kernel_ptr(int problem, bool timed, bool nt) {
  return timed ? child_ptr<true>(problem, nt) : child_ptr<false>(problem, nt);
}

const void* init_kernel_ptr(int) { return (const void*)init_kernel; }

const void* narrow_kernel_ptr(int32_t slots) {
  return slots / 32 <= NARROW_BITS ? (const void*)narrow_kernel<true> : (const void*)narrow_kernel<false>;
}

const void* near_kernel_ptr() { return (const void*)near_kernel; }

const void* solo_kernel_ptr(bool far) {
  return far ? (const void*)solo_kernel<true> : (const void*)solo_kernel<false>;
}

const void* symmetry_kernel_ptr(bool arena) {
  return arena ? (const void*)symmetry_kernel<true> : (const void*)symmetry_kernel<false>;
}

const void* bottom_up_kernel_ptr() { return (const void*)bottom_up_kernel; }

const void* tally_kernel_ptr() { return (const void*)tally_kernel; }

const void* bottom_up_words_kernel_ptr() { return (const void*)bottom_up_words_kernel; }

const void* bottom_up_queries_kernel_ptr() { return (const void*)bottom_up_queries_kernel; }

const void* clear_tally_kernel_ptr() { return (const void*)clear_tally_kernel; }

const void* settle_symmetry_kernel_ptr() { return (const void*)settle_symmetry_kernel; }

const void* start_kernel_ptr(int problem) {
  return problem == PROB_BFS ? (const void*)start_kernel<PROB_BFS>
                             : (const void*)start_kernel<PROB_SSSP>;
}

const void* admit_kernel_ptr(int problem) {
  return problem == PROB_BFS ? (const void*)admit_kernel<PROB_BFS>
                             : (const void*)admit_kernel<PROB_SSSP>;
}

const void* admit_sources_kernel_ptr() { return (const void*)admit_sources_kernel; }

const void* retire_kernel_ptr() { return (const void*)retire_kernel; }

const void* clear_found_kernel_ptr() { return (const void*)clear_found_kernel; }

const void* advance_kernel_ptr() { return (const void*)advance_kernel; }

}  // namespace dpo
