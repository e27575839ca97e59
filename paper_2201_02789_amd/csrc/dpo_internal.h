// Shared declarations of the HIP library (device kernels and host driver).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace dpo {

constexpr int PB = 256;          // parent workgroup: 256 frontier entries per virtual block
constexpr int NW = PB / 64;      // wave64s per workgroup
// A parent wave has as many frontier entries as have this many edges on the
// graph's average, if there are workgroups for it.  A wave runs the thresholded
// children of its entries 512 edges at a time, one batch after another, so a
// frontier of a few hundred entries in blocks of PB is a handful of waves with
// 2,000 edges each while the rest of the chip has none.  Whole BFS calls (us;
// Erdos-Renyi, vertices/average degree), full blocks -> at 384: 2 M/30 432 -> 386,
// 1 M/16 322 -> 307, 100 K/64 205 -> 159, 250 K/8 257 -> 262; R-MAT of 1 M, degree 32,
// 248 -> 240.  At 768 2 M/30 takes 390 and 100 K/64 174; at 192 250 K/8 takes 292:
// blocks of few edges cost more than they spread.
constexpr int SPREAD_EDGES = 384;
// A single traversal's level that probes and claims one bitmap spreads over so many
// blocks at most: where neighbours have ids close together its claims meet on few lines, the more
// waves the worse (us, at 32 / 64 / without a limit; level steps of full blocks in
// brackets: 300 layers of 3,000 vertices, degree 24, 9,980 / 11,390 / 11,990
// [9,310], 100 layers of 20,000 3,840 / 3,840 / 5,080 [3,810], a 100^3 grid of 26
// neighbours 3,950 / 3,910 / 4,430 [4,040]; ids at random: the same grid 3,040 /
// 2,940 / 2,650 [3,170], Erdos-Renyi of 1 M, degree 16, 322 / 312 / 308 [331]).
// Several queries' claims meet less: 300 queries served four at a time take 21.1 ms
// with the limit, 19.8 without.
constexpr uint32_t ONE_COPY_BLOCKS = 32;
constexpr int STAGE = 512;       // LDS slots per wave for next-frontier staging
constexpr int NQD = 8;           // descriptor queues (one per XCD: queue = virtual block % 8)
constexpr int NQF = 64;          // frontier queues (queue = workgroup % 64), plus one overflow
constexpr int MAX_GRID = 4096;   // persistent grid cap (rows of the per-workgroup counters)
constexpr int NSTAT = 8;
// parent kernel phases
constexpr int PH_BOTH = 0;    // pass 1 and pass 2
constexpr int PH_LIST = 1;    // pass 1; thresholded parents listed for PH_SERIAL
constexpr int PH_SERIAL = 2;  // pass 2 of the listed parents (after the child kernel)
constexpr uint32_t GROUP_EDGES = 1024;  // wave-run serial children: edges per group (about)
constexpr int MAX_QUERIES = 4096;  // per-query tables are staged in LDS
constexpr int ADMIT_CHUNK = 4096;  // output slots initialised per admit workgroup
// SSSP bounds are kept from this many slots on: more distances than an XCD's L2
// holds (4 MiB), while their bytes fit, so that fewer reads miss it (scale 21, the
// widest level's child grids: 11.0 M -> 6.5 M misses).  Off / on (us; R-MAT of degree
// 32 and 16, Erdos-Renyi of degree 16): 1 M vertices 1,330 / 1,315, 1,255 / 1,255,
// 1,850 / 2,020; 1.25 M 1,430 / 1,405, 1,310 / 1,320, 2,080 / 2,190; 1.5 M 1,620 /
// 1,580, 1,295 / 1,285, 2,670 / 2,680; 2 M 2,120 / 2,040, 1,665 / 1,635, 3,760 /
// 3,655; 4 M 3,620 / 3,315, 2,930 / 2,805, 7,320 / 6,885.  An engine goes by its pool,
// of which few slots may be in use: with one of 16 M, 24 queries of scales 11 to 13
// take 871 / 857, of 13 to 16 1,230 / 1,257, of 13 to 18 2,325 / 2,165.
constexpr int64_t BOUND_MIN_SLOTS = 3 << 19;
constexpr int PRECHECK_MIN = 32;   // claim candidates per 512-lane batch above which
                                   // a coherent load precedes the atomics
constexpr int NHINT = 8;           // BFS per-XCD visited copies (Args::hint), one per XCD
constexpr int HARVEST_RUNS = 8;    // harvest kernel: 64-slot runs per wave and round
constexpr int HINT_AUTO_MIN_DEGREE = 8;  // DPO_HINT_AUTO: per-XCD copies from this average
                                         // degree (m / n) up
// narrow levels (one workgroup, frontier in LDS)
constexpr int NARROW_BLOCK = 1024;
constexpr uint32_t NARROW_U = 8;              // edges per lane and batch
constexpr uint32_t NARROW_WORDS = 36 * 1024;  // LDS words: bits, distances, frontier arrays
constexpr uint32_t NARROW_FRONT = 8192;       // most frontier entries
// Most edges of a narrow level.  One compute unit runs about 2.4 edges per
// nanosecond when the visited bits (distances) are in its LDS, but makes only
// about one random access per nanosecond to global ones, while a level step
// takes 30 to 50 us (16 us on a road-like graph) however few its edges are
// (global bits, 4,096 / 8,192 / 32,768 edges: a 1400 x 1300 road-like graph 28.7
// / 19.5 / 19.7 ms, an Erdos-Renyi graph of 2 M 381 / 377 / 440 us).
constexpr uint32_t NARROW_EDGES = 1 << 17;
constexpr uint32_t NARROW_FAR_EDGES = 1 << 13;
// Bitmap words that go to LDS, beside half of NARROW_FRONT frontier entries or
// more.
constexpr int32_t NARROW_BITS = NARROW_WORDS - 4 * (NARROW_FRONT / 2);
// Solo SSSP: vertices whose distances fit LDS beside 3,400 frontier entries or
// more (3,481, with the two bit sets of the form with a bound), and entries up to which one compute unit is faster than level steps on
// any graph (us, solo / level steps, 16,383 vertices and about 450,000 entries:
// R-MAT 631 / 531, Erdos-Renyi 454 / 633).
constexpr int32_t SOLO_VERTICES = 16384;
constexpr int32_t SOLO_EDGES = 1 << 18;
// Entries from which solo SSSP keeps a bound: below, a level takes as long
// whatever its edges, and the bound's levels are more (us, without / with: 64,000
// entries 272 / 294, 80,000 207 / 202, 93,000 277 / 243, 104,000 201 / 165).
constexpr int32_t SOLO_FAR_EDGES = 88 << 10;
constexpr uint32_t SOLO_WORDS = 34 * 1024;
constexpr uint32_t SOLO_FRONT = 4096;
static_assert((SOLO_WORDS - 2 * (SOLO_VERTICES / 32) - SOLO_VERTICES) / 5 >= 3400, "solo frontier in LDS");
// near-far SSSP: frontier entries, vertices (two bits each in LDS), edges of a
// round, average weights by which the bound moves (a 301 x 257 road-like graph
// takes 4.15 / 3.73 / 3.85 / 4.69 / 7.5 ms at 4 / 8 / 16 / 32 / 64)
constexpr uint32_t NEAR_WORDS = 36 * 1024;
constexpr uint32_t NEAR_FRONT = 4096;
constexpr int32_t NEAR_VERTICES = (NEAR_WORDS - 5 * NEAR_FRONT) / 2 * 32;
constexpr uint32_t NEAR_EDGES = 1 << 14;
constexpr uint32_t NEAR_STEP = 8;
constexpr uint32_t NONE = 0xFFFFFFFFu;        // no vertex
constexpr uint32_t NARROW_LEVELS = 4096;      // most levels per launch (a few ms)
// How a narrow launch ended: the traversal done or failed, more narrow levels,
// or a wide level, which goes top-down (a level step; V_STILL: and the launch ran
// no level before it), bottom-up, or bottom-up if the graph turns out symmetric.
enum { V_DONE = 1, V_ERROR, V_MORE, V_TOP_DOWN, V_BOTTOM_UP, V_CHECK, V_STILL };
// What a narrow launch follows: a bottom-up level if one was due, or so many
// level steps.
constexpr uint32_t AFTER_BOTTOM_UP = ~0u;

// bottom-up levels (BFS)
// A level goes bottom-up if its frontier has at least 1 / BU_ALPHA of the edges
// not yet run, so that a vertex looks at about BU_ALPHA entries at most.
// Measured (us, worst of three seeds) at 8 / 16 / 32 / 64: Erdos-Renyi of 2 M
// 386 / 382 / 382 / 584, a batch of 512 1,860 / 1,824 / 1,903 / 2,085; R-MAT of
// scale 22 618 / 472 / 472.
constexpr uint32_t BU_ALPHA = 16;
// The edges left count what the search never reaches, and rows that end without a
// visited neighbour are read whole.  So before the symmetry check, and when the
// frontier has less than 1 / BU_SURE of the edges left, a sample of the unvisited
// vertices (sample_row) says how many entries the level would read, and how many
// edges those have that it finds: twice the entries read are to be at most BU_READ
// times the frontier's edges and the found vertices' together, and all entries, which
// the check reads, at most BU_CHECK times.  One-copy levels are slow enough for the
// larger factors.  Us, top-down only / without the sample / with it: R-MAT of scale
// 20 beside another, beside 3, beside 7 445 / 655 / 420, 450 / 1,235 / 420, 470 /
// 1,690 / 425; 30 layers of 100,000 vertices 975 / 1,200 / 1,000, a 100^3 grid of 26
// neighbours 2,650 / 2,025 / 1,950; R-MAT of scale 20 450 / 245 / 245, Erdos-Renyi of
// 1 M, degree 24, 408 / 275 / 280 (BU_READ 2 / 3 / 5 of the entries against the
// frontier's edges alone: 340 / 300 / 280, but two R-MAT graphs 412 / 473 / 641); a
// band of 1 M vertices in one-copy levels 1,400 / 1,065 / 1,120.
// Vertices in it, 34 random accesses each, of which a compute unit makes about one a
// ns: of 1,024 the launch takes 13 us longer on an Erdos-Renyi graph of 2 M vertices, of
// 256 4; of 128 an R-MAT of scale 20 beside another takes 560 us instead of 405.
constexpr uint32_t BU_SAMPLES = 256;
constexpr uint32_t BU_SURE = 8, BU_READ = 1, BU_READ_ONE_COPY = 16, BU_CHECK = 5, BU_CHECK_ONE_COPY = 40;
// For a query of several, whose rows are read for up to BU_GROUP queries at once (us,
// top-down only / without the sample / with it at 1 / 3 / 10: 64 over 8 graphs of 8
// R-MAT graphs each 528 / 822 / 569 / 569 / 701, served 854 / 900 / 640 / 641 / 792; 48
// over 6 of 4 631 / 738 / 597 / 677 / 732; 24 served over 40 layers of 8,000 vertices
// 2,412 / 4,570 / 2,925 / 3,165 / 4,365; 512 over R-MAT graphs 5,905 / 1,795 / 1,785 /
// 1,790 / 1,820; 32 over 4 of 2 1,088 / 901 / 999 / 1,011 / 938).
constexpr uint32_t BU_QUERY_READ = 1;
// Queries go bottom-up if they have this many entries together.  Measured (us, top-down /
// bottom-up): batches of 2.4 M entries 228 / 280, 12 M 420 / 465, 19 M 390 / 390 and 449 /
// 456, 30 M 676 / 602, 50 M 700 / 618; served queries of 13 M 333 / 412, 15 M 365 / 447,
// 46 M 525 / 484, 57 M 656 / 618, 180 M 1,441 / 847.
constexpr int64_t BU_QUERIES_EDGES = 20 << 20;
// Several queries: frontier entries from which a level's edges are tallied, and
// edges from which a query may go bottom-up (fewer are run top-down in less
// time than the tally and the bottom-up kernel take).
constexpr uint32_t TALLY_MIN = 8192;
constexpr uint32_t TALLY_SAMPLE = 1 << 17;  // of them read, about
constexpr uint32_t BU_QUERY_EDGES = 1 << 14;
constexpr uint32_t BU_GROUP = 16;  // queries of one graph run together (bits of a word)
constexpr int QB = 1024;           // workgroup that lists them
constexpr uint32_t BU_SORT = QB;   // queries it puts in order of their graphs
constexpr uint32_t BU_LANE = 32;    // edges a lane looks at before the wave shares its row
constexpr uint32_t SYM_EDGES = 1024;  // symmetry check: least edges per wave
constexpr uint32_t SYM_SAMPLES = 128;  // entries whose reverse is looked up first, if
constexpr int SYM_BLOCK_SAMPLES = 64;  // (an arena's check: per workgroup)
constexpr uint32_t SYM_SAMPLE_DEGREE = 32;  // the row it would be in is this short

enum { PROB_BFS = 0, PROB_SSSP = 1 };
enum { AGG_NONE = 0, AGG_WAVE = 1, AGG_BLOCK = 2, AGG_MULTI = 3, AGG_FLAT = 4 };
// device error codes (stored as the negated dpo_status)
enum { ERR_ARG = 1, ERR_CAPACITY = 4, ERR_TIMEOUT = 5 };
enum { S_FRONT = 0, S_SERIAL, S_REC, S_CHILD, S_ESER, S_ECHILD, S_DESC };

// Phase timing (the timed instantiations of the level kernels only).  Each
// workgroup of each level kernel writes one row of TM_ROW words at
// tm[((level * TM_KINDS + kind) * MAX_GRID + workgroup) * TM_ROW]:
//   [0] realtime clock at entry, [1] at exit (constant-rate counter),
//   [2 + p] shader-clock cycles its waves spent in phase p (summed over the
//   workgroup's waves), [7] the largest total of one wave.
// Rows of levels >= TM_LEVELS are not written.
constexpr int TM_LEVELS = 64;
constexpr int TM_KINDS = 4;  // parent kernel, child kernel, thresholded children, harvest
constexpr int TM_ROW = 8;
enum { TK_PARENT = 0, TK_CHILD = 1, TK_SERIAL = 2, TK_HARVEST = 3 };
enum { TP_PARENT = 0, TP_AGG, TP_LAUNCH, TP_DISAGG, TP_CHILD, TP_N };

// Counters of one level; three sets rotate by level % 3 so that the parent
// kernel of level L can clear the set of level L + 1 while nobody uses it.
struct LevelSet {
  uint32_t fcnt[NQF + 1];              // next-frontier queue fills (+ overflow)
  uint32_t vmode;                      // visited copies of this level: bit 0 probed
                                       // buffer, bit 1 split (claims in the other one)
  uint32_t pad0[14];
  unsigned long long qctr[NQD];        // descriptor queues: hi32 count, lo32 child blocks
  uint32_t cclaim[NQD][32];            // child kernel: chunks claimed per XCD group (one
                                       // 128-byte line each)
};

struct State {
  uint32_t base;        // level index of step 0 of the current graph replay
  uint32_t done;        // set when a level starts with an empty frontier
  uint32_t error;       // first device error code, 0 = none
  uint32_t levels_run;  // index of the last non-empty level + 1
  uint32_t vsel[2];     // probed visited buffer of levels with parity 0 / 1
  uint32_t vstale[2];   // BFS: the other bitmap missed folds (a one-copy level ran)
  uint32_t plan;        // single traversals: verdict of the last narrow launch
  uint32_t symmetric;   // 0 not checked, 1 yes, 2 no
  unsigned long long run_edges;  // edges of the levels so far (about)
  unsigned long long sym_sum[8];  // symmetry check: shares of the signed sum
  unsigned long long plan_edges;  // edges of the level planned last, not in run_edges yet
  uint32_t asymmetric;  // symmetry check: met an id out of range
  uint32_t pad[31];
  LevelSet set[3];
};

// One traversal ("query") of a batch.  Its outputs occupy the slots
// [slot0, slot0 + n) of the output arena; slot s is vertex s - slot0 + vbase of
// the CSR arena.
struct Query {
  int32_t slot0;   // first output slot
  int32_t n;       // vertices of its graph
  int32_t vbase;   // global id of its graph's vertex 0 in the CSR arena
  int32_t lstart;  // level index at which it started (its source is at level lstart)
  int32_t T;       // threshold of its size bucket
  int32_t CF;      // coarsening factor of its size bucket
  int32_t last;    // last level index with frontier entries (written by the kernels)
  int32_t src;     // source (local id)
};

// Kernel arguments (by value).  All pointers are device pointers.
struct Args {
  const int32_t* rp;
  const int32_t* col;
  const uint32_t* w;
  int32_t* level;                  // [slots] BFS output
  uint32_t* dist;                  // [slots] SSSP output (distance array 0)
  uint32_t* dist2;                 // [slots] SSSP distance array 1 (equal to dist at the end)
  State* st;
  Query* q;                        // [nq]
  unsigned long long* grp_packed;  // [3][ngroups_cap]: hi32 records, lo32 child blocks
  uint32_t* grp_done;              // [3][ngroups_cap]: blocks of the group finished
  int32_t* front0;                 // [NQF * fcap + slots]
  int32_t* front1;
  uint32_t* visit;                 // BFS: two bitmaps of vwords words, then NHINT per-XCD
                                   // copies; SSSP: stamps [slots]
  uint8_t* found;                  // [vwords * 32] bytes (Args::hint), set for the vertices
                                   // a level's child bodies find (BFS: wide levels) or
                                   // improve (SSSP); read by the harvest kernel
  uint8_t* bound;                  // SSSP with found bytes on many slots: [vwords * 32] a byte
                                   // above which no sum improves the vertex; else null
  int4* rec;                       // [slots] launch records {row start, deg, offset, parent dist}
  int32_t* rec_q;                  // [slots] query of each record
  int32_t* rec_slot;               // [slots] SSSP: slot of each record's parent
  int4* ser;                       // [slots rounded up to PB] thresholded parents
                                   // {row start, deg, slot, parent distance}
  int32_t* qmap;                   // [slots / 32] query owning each 32-slot chunk
  int4* desc;                      // [NQD][desc_cap] {record base, records, block base, -}
  unsigned long long* stats;       // [MAX_GRID][NSTAT], one row per workgroup
  uint32_t* sercnt;                // [MAX_GRID] listed thresholded parents per workgroup
  unsigned long long* tm;          // phase-timing rows (timed kernels only)
  int32_t slots;                   // total output slots (sum of the queries' n)
  int32_t n;                       // CSR arena vertices
  int32_t m;                       // CSR arena entries
  int32_t nq;
  int32_t CB;
  int32_t k;
  int32_t ngroups_cap;
  int32_t desc_cap;                // per descriptor queue
  int32_t fcap;                    // per frontier queue
  int32_t count_stats;
  int32_t agg_threshold;           // wave / block granularity: fewer launching parents
                                   // than this launch individually (Sec. V-B)
  int32_t vwords;                  // words of one BFS bitmap (slots / 32)
  int32_t split_min;               // frontier size from which a level probes one
                                   // visited copy and updates the other
  int32_t serial_wave;             // thresholded children: run by the wave together
                                   // (1) or each in its parent's lane (0)
  int32_t dyn_pct;                 // child kernel: percent of each XCD group's blocks
                                   // that its waves claim in chunks (0 = even split)
  int32_t hint;                    // found bytes and the harvest kernel in use.  BFS:
                                   // per-XCD visited copies on wide levels (probed by the
                                   // XCD's workgroups, at visit + (2 + x) * vwords, x =
                                   // XCD), discoveries taken into bitmap 0 by the harvest;
                                   // SSSP: improvements queued by the harvest instead of
                                   // iteration stamps
  int32_t bottom_up;               // wide BFS levels may go bottom-up (with Args::hint):
                                   // BU_SINGLE as the narrow kernel plans, BU_QUERIES each
                                   // query's by its tallied edges
  uint32_t* tally;                 // BU_QUERIES: [nq] each (TALLIES): edges of the frontier at an
                                   // even level, at an odd one, of all levels tallied, of the
                                   // graph; entries a bottom-up level would read, edges it would
                                   // find; then the arena's graph_vbase for the symmetry check (all
                                   // in the place of Args::stats, whose counters are off)
};

constexpr int TALLIES = 6;

enum { BU_OFF = 0, BU_SINGLE = 1, BU_QUERIES = 2 };

// timed: the instantiation that stamps its phases into Args::tm
const void* parent_kernel_ptr(int problem, int gran, bool timed = false);
// nt: the child kernel's adjacency (and weight) loads are non-temporal (used
// with found bytes, Args::hint)
const void* child_kernel_ptr(int problem, bool timed = false, bool nt = false);
const void* serial_kernel_ptr(int problem, int gran, bool timed = false);
const void* harvest_kernel_ptr(int problem, bool timed = false);
const void* init_kernel_ptr(int problem);
const void* narrow_kernel_ptr(int32_t slots);
const void* near_kernel_ptr();
const void* solo_kernel_ptr(bool far);
const void* symmetry_kernel_ptr(bool arena);
const void* bottom_up_kernel_ptr();
const void* tally_kernel_ptr();
const void* bottom_up_words_kernel_ptr();
const void* bottom_up_queries_kernel_ptr();
const void* settle_symmetry_kernel_ptr();
const void* clear_tally_kernel_ptr();
const void* start_kernel_ptr(int problem);
const void* admit_kernel_ptr(int problem);
const void* admit_sources_kernel_ptr();
const void* retire_kernel_ptr();
const void* clear_found_kernel_ptr();
const void* advance_kernel_ptr();

}  // namespace dpo
