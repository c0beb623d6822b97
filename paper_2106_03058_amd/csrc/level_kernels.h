// One level of the randomized residue push (Algorithm 2 of "Approximate
// Graph Propagation", Section 4) for many columns at once, shared by the
// batched entry points (agp_propagate*) and the query server.
//
// A column is one signal (a feature column or one query).  Every column
// carries its own level parameters (ColParams), so columns at different
// levels, with different weights, exponents a/b, thresholds and random keys
// advance together in one launch.
//
// Cells: the residue of node u in column c lives at cell u * su + c * sc
// (row-major n x C for agp_propagate; a served query's residues live at
// positions of its own table instead).  Next-level residues are exact
// integers of a per-column unit
// (int64 cells for binary32, 128-bit cells for binary64), so the integer
// atomics that add contributions commute and the result does not depend on
// the order in which pushes land.
//
// A wave takes batches of up to 64 frontier entries (u, c) (from a list, or,
// at level 0 of a mostly non-zero signal, every cell in order): each lane
// converts one entry's residue, updates the reserve (pi(u) += kappa_i r(u)),
// finds the deterministic prefix J of the degree-sorted row (increment >=
// theta, by binary search) and counts the work items of its sampled suffix;
// the wave then makes the batch's deterministic pushes with all lanes (a
// wave-wide scan spreads them) and lanes draw sampled work items (runs of
// 64-position windows) from a per-wave queue, walking their Philox /
// geometric-skip chains.  Rows with long deterministic prefixes and entries
// with many sampled work items are deferred to grid-wide kernels
// (k_det_big, k_samp_big) that run right after the level.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "agp_device.h"

namespace agp {
namespace lvl {

constexpr int kThreads = 256;
constexpr int kLevelBlocks = 4096;
constexpr int kNumCounters = 6;   // frontier, hash, det, cand, acc, runs
// Batched calls: each level's counters and contribution mass are kept as
// kCountShards rows of one 64-byte line (the six counters, the mass, a pad);
// block b adds the sums of its waves to row b mod kCountShards, and
// k_fold_counts adds the rows up at the end of the call.  Atomics on one
// address serialise at 12 ns, and with one row per level that every wave of
// the grid added seven values to, these additions were most of a small
// level (10^4 entries on 16384 waves: 0.38 ms): a PPR query of 21 levels on a
// 10^4-node graph took 8.96 ms, 4.58 ms with the rows; with three binary64
// columns 14.5 and 4.63 ms.
constexpr int kCountShards = 64;
constexpr int kCountStride = 8;   // words of a row
constexpr int kCountMass = 6;     // the mass (binary64) after the counters
// The server keeps the same rows per slot (counters accumulate over a
// query's levels; word 7 stays free for its error flags): kServeShards sets
// of one row per slot (one set from kServeShardSlots slots on, whose rows are
// shared by fewer blocks), block b adding to set b mod kServeShards.
constexpr int kServeShards = 16;
constexpr int kServeShardSlots = 8192;
constexpr size_t kCountLevelBytes = sizeof(unsigned long long) * kCountShards * kCountStride;
constexpr int kThetaRows = 4096;  // rows per partial sum of ||x||_1
constexpr int kServeLdsSlots = 128;  // server columns whose counters a block sums in LDS

enum : int { kLastLevel = 1, kAZero = 2, kDrop = 4 };

// How the next frontier of a level is formed (written by k_level):
enum : int {
  kModeSparse = 0,    // first contributions appended directly
  kModeCompact = 1,   // fire-and-forget atomics, then a compaction scan
  kModeBinned = 2,    // records binned by destination and summed in LDS
  kModeOverflow = 3,  // record buffer overflowed: atomics, then compaction
};

// Binned aggregation: a record is (cell | sign << 31) of a sampled push;
// cells are grouped into at most 1024 buckets of 2^shift cells (shift
// chosen per call from n * C, at least kBinLog2) and every bucket into bins
// of 8192 cells (32-bit counts in 32 KiB of LDS), so n * C must stay below
// 2^31.
constexpr int kBinLog2 = 13;
constexpr int kMaxBinsPerBucket = 1024;
constexpr int kBuckets = 1024;

// Rows with many deterministic pushes (a hub with a large residue) would
// keep one wave busy while the rest of the grid idles; a level
// defers rows of at least big_row (default kBigRow) deterministic pushes to a
// list that k_det_big then spreads over the whole grid, and, when a batch
// makes more than kBatchDet pushes in all (64 columns of one hub are one
// batch), its rows of kBatchDetRow and more.
constexpr uint32_t kBigRow = 4096;
constexpr uint32_t kBatchDet = 2048, kBatchDetRow = 128;
constexpr unsigned long long kBigChunk = 4096;  // pushes per wave of k_det_big at most
constexpr int kBigShift = 40;    // list counter: deferred rows << 40 | their pushes (a level's pushes < 2^40)

struct BigRow {
  unsigned long long off;  // deterministic pushes of the rows deferred before this one
  int64_t rp;              // first arc of the row
  double cv;               // c = rho |r| d_u^-b
  uint32_t c, J;           // c: with the flags of BatchLds
};

// Likewise an entry whose sampled suffix makes samp_items (64 by default)
// or more work items (a hub holding a small residue in some column), or
// kBatchItemRow or more in a batch of more than kBatchItems: its items go to
// a second list that k_samp_big spreads evenly over the whole grid.
constexpr long long kBigItems = 64;
constexpr uint32_t kBatchItems = 512, kBatchItemRow = 8;

struct BigSamp {
  unsigned long long off;  // work items of the entries deferred before this one
  int64_t rp;              // first arc of the row
  double cv;               // c = rho |r| d_u^-b
  double p0;               // as in BatchLds
  uint32_t u, c, J, d;     // c: with the flags of BatchLds
  uint32_t items, pad;
};

// How a launch takes its columns' level parameters: a batched call's levels
// are the same for every column and sit in scalar registers, with a = 0 and
// a > 0 as kernels of their own (each holds only its own lane state: with one
// kernel for all, the parameters of every entry were loads and lane
// registers); the server's columns are each at a level of their own.
enum : int { kBatchAZ = 0, kBatchAP = 1, kPerColumn = 2 };

// One level of a batched call (device memory, so that a captured level loop
// serves every call with the same buffers).
struct LevelParams {
  double rho, kappa;    // Y_{i+1} / Y_i and S w_i / Y_i
  int flags;            // kLastLevel
  uint32_t key0, key1;  // 64-bit seed
  int pad;
};

// rho to out_stride, key0 to flags: the server's columns only.
struct ColParams {
  double theta;          // eps * ||x_c||_1
  double scale;          // 2^-ue (binary32 units)
  long long dtheta;      // fl(theta) in units
  double rho;            // Y_{i+1} / Y_i at the column's current level
  double kappa;          // S w_i / Y_i at the column's current level
  const double* da;      // d^-a, d = 0..max degree
  const double* db;      // d^-b
  void* out;             // reserve of node u at out + u * out_stride
  long long out_stride;
  int ue;                // exponent of the unit
  uint32_t qid;          // query id of the column's random streams
  uint32_t key0, key1;   // 64-bit seed
  int level;
  int flags;             // kLastLevel | kAZero | kDrop
  float theta_w;         // fl(theta) in binary32
};

struct LevelArgs {
  const int64_t* rp;
  const uint32_t* col;
  const uint32_t* nd;
  const uint32_t* gend;  // row-relative end of each arc's degree group
  const int32_t* deg;   // row lengths (neighbours to push to)
  const int32_t* fdeg;  // degrees in the factors d^-a, d^-b
  const ColParams* cp;
  // batched calls: the level's parameters, the degree-power tables and the
  // reserve of node u, column c at out[u * out_stride + c]
  const LevelParams* lp;
  const double *da, *db;
  void* out;
  long long out_stride;
  // batched calls (one a and b for every column): per node u, d_u^-b and the
  // d^-a of its first neighbour (2 doubles; 0 for a node without arcs), or
  // null (the setup then reads them through the degree tables)
  const double* nodefac;
  // batched calls: d^-a of every arc's neighbour (arc order), or null
  const double* arcfac;
  long long su, sc;  // cell = u * su + c * sc
  long long xld;     // level 0 of a batched call: x[u * xld + c]
  int level;         // batched calls: counter row
  const uint64_t* fin;
  const unsigned long long* cnt_in;
  uint64_t* fout;
  unsigned long long* cnt_out;
  unsigned long long* counters;  // batched: per level and shard (kCountShards rows); server: per shard and slot
  int slots;                     // server: rows per shard
  int shard_mask;                // server: shards - 1 (a power of two of them)
  int* err;                      // batched: one flag; server: one per column
  // batched calls: the next residues are kept rep_mask + 1 times, rep_stride
  // words apart; block b adds to copy b mod (rep_mask + 1), k_merge adds them up
  uint32_t rep_mask;
  long long rep_stride;
  int positive;                  // non-negative signals: sparse levels allowed
  unsigned long long dense_cut;  // frontier size from which a level is dense
  int* mode_out;                 // how the next frontier is formed (kMode*)
  // binned aggregation (binary32 batched calls; rec == nullptr: disabled);
  // records are kept per column group (rec_groups groups of rec_gw columns,
  // 1 group: the whole row) and there in kRecSegs segments, segment k of
  // group g at rec + (g * kRecSegs + k) * rec_cap
  uint32_t* rec;
  unsigned long long* rec_count;  // this level's record count of each segment, kRecStride apart
  unsigned long long rec_cap;     // records per segment
  int rec_groups;
  uint32_t rec_gw;
  unsigned int* bucket_count;    // records per bucket of this level (kBuckets, kBuckets / 2 per group with two)
  int bucket_shift;              // cells per bucket = 2^bucket_shift
  const double* bin_est;         // non-null: bin only if *bin_est >= bin_pushes (estimated pushes)
  double bin_pushes;
  // deferred rows (nullptr: every row is pushed by its wave)
  uint32_t big_row;              // deterministic pushes from which an entry's row is deferred
  unsigned long long* big_ctr;   // this level's list counter, zero at the start
  BigRow* big;
  unsigned long long big_cap;
  unsigned long long* samp_ctr;  // the same for deferred sampled suffixes (entries << 40 | items)
  BigSamp* samp;
  long long samp_items;          // work items from which an entry's sampled suffix is deferred
  // binned levels: deterministic pushes mark their destination bin (nullptr:
  // no marks); group g's bins at det_bins + g * det_bins_g
  uint8_t* det_bins;
  unsigned long long det_bins_g;
  // served queries: each query's residues live in an open-addressing table
  // of one pool (query c owns positions tab_off[c] .. tab_off[c] + tab_mask[c];
  // a key is node + 1, 0 when free); frontier entries are (position, c)
  uint32_t* keys_cur;
  uint32_t* keys_nxt;
  const uint32_t* tab_off;   // the next level's tables
  const uint32_t* tab_mask;
  const uint32_t* tab_cur;   // this level's tables
};

// The arguments of the running kernel (whose first parameter is a LevelArgs),
// read from its argument segment again: the value hidden in the empty asm
// keeps the compiler from holding every argument of a batch's setup or of a
// flush in scalar registers across the draw loop, where more than fit became
// a lane read (a vector instruction) at each use: 231 of them in the a > 0
// kernel, 45 this way.  With the kernels split by kBatchAZ / kBatchAP, 128
// columns of features on 2.4M nodes took 101 -> 90 ms, 32 columns on 8M nodes
// 42.7 -> 37.5, 64 transition columns on 2^22 nodes 129 -> 121.
__device__ __forceinline__ const LevelArgs& args_again() {
  using KernArg = const LevelArgs __attribute__((address_space(4)));
  KernArg* p = (KernArg*)__builtin_amdgcn_kernarg_segment_ptr();
  __asm__ volatile("" : "+s"(p));
  return *(const LevelArgs*)p;
}

// An argument that the draw loop reads in every step, kept in scalar registers
// (read again from the argument segment, each use is a scalar load that the
// wave waits for).
template <typename V>
__device__ __forceinline__ V pinned(V v) {
  __asm__ volatile("" : "+s"(v));
  return v;
}

template <typename V>
__device__ __forceinline__ const V* pinned(const V* p) {  // (device memory, so that its loads stay global ones)
  using Global = const V __attribute__((address_space(1)));
  Global* g = (Global*)p;
  __asm__ volatile("" : "+s"(g));
  return (const V*)g;
}

// Position of node v in a query's table, claiming it if v is not there yet
// (*first: v was not there); ~0u when the table is too full.  mask == ~0u:
// a direct table of n entries (position base + v); else 2^k = mask + 1
// entries probed linearly from a multiplicative hash of v, at most
// kMaxProbes of them (a table at most half full needs a few; more means
// that the query outgrew its table).
constexpr uint32_t kDirectTable = ~0u;
// mask == kDirectPlain: a direct table of a query whose residues cannot
// cancel (a non-negative signal): no keys (the node is the position's
// offset), plain atomic adds, and the next frontier is formed by a scan of
// the table's non-zero positions after the level
constexpr uint32_t kDirectPlain = ~1u;
constexpr uint32_t kMaxProbes = 128;
__device__ __forceinline__ uint32_t table_find_or_insert(uint32_t* keys, uint32_t base, uint32_t mask, uint32_t v,
                                                         bool* first) {
  // a key changes only once per level (0 -> node + 1), so a coherent read
  // that already shows v spares the compare-and-swap
  if (mask == kDirectTable) {
    const uint32_t pos = base + v;
    uint32_t old = __hip_atomic_load(keys + pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 0u) old = atomicCAS(keys + pos, 0u, v + 1u);
    *first = old == 0u;
    return pos;
  }
  const uint32_t h = static_cast<uint32_t>((static_cast<unsigned long long>(v) * 0x9E3779B97F4A7C15ull) >> 32);
  const uint32_t probes = mask < kMaxProbes ? mask + 1u : kMaxProbes;
  for (uint32_t k = 0; k < probes; ++k) {
    const uint32_t pos = base + ((h + k) & mask);
    uint32_t old = __hip_atomic_load(keys + pos, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 0u) old = atomicCAS(keys + pos, 0u, v + 1u);
    if (old == 0u || old == v + 1u) {
      *first = old == 0u;
      return pos;
    }
  }
  *first = false;
  return ~0u;
}
constexpr int kErrTableFull = 2;  // server: a query's table had no free position

// ----------------------------------------------------- working precision
template <typename T>
struct Prec;

__device__ __forceinline__ void atomic_add_relaxed(unsigned long long* p, unsigned long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long atomic_add_ret(unsigned long long* p, unsigned long long v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <>
struct Prec<float> {
  using Cell = long long;
  using Delta = long long;
  static constexpr int kWords = 1;
  static __device__ __forceinline__ float take(Cell* acc, size_t cell, const ColParams& p) {
    const long long K = acc[cell];
    acc[cell] = 0;
    return units_to_f32(K, p.ue);
  }
  static __device__ __forceinline__ bool to_units(float v, const ColParams& p, Delta* d) {
    return f32_to_units(v, p.scale, d);
  }
  static __device__ __forceinline__ Delta theta_units(const ColParams& p, bool neg) {
    return neg ? -p.dtheta : p.dtheta;
  }
  static __device__ __forceinline__ double mag_units(float v, const ColParams& p) {
    return fabs(static_cast<double>(v)) * p.scale;
  }
  // true if the cell held zero before (first contribution of the level)
  static __device__ __forceinline__ bool add_ret(Cell* acc, size_t cell, Delta d) {
    return atomic_add_ret(reinterpret_cast<unsigned long long*>(acc + cell),
                          static_cast<unsigned long long>(d)) == 0ull;
  }
  static __device__ __forceinline__ void add(Cell* acc, size_t cell, Delta d) {
    atomic_add_relaxed(reinterpret_cast<unsigned long long*>(acc + cell), static_cast<unsigned long long>(d));
  }
  static __device__ __forceinline__ bool nonzero(const Cell* acc, size_t cell) { return acc[cell] != 0; }
  // whole cells (k_merge)
  static __device__ __forceinline__ Delta load(const Cell* acc, size_t cell) { return acc[cell]; }
  static __device__ __forceinline__ void store(Cell* acc, size_t cell, Delta v) { acc[cell] = v; }
  static __device__ __forceinline__ bool is_zero(Delta v) { return v == 0; }
  static __device__ __forceinline__ Delta sum(Delta a, Delta b) { return a + b; }
  static __device__ __forceinline__ void set_units(Cell* acc, size_t cell, long long v) { acc[cell] = v; }
};

template <>
struct Prec<double> {
  using Cell = unsigned long long;  // two words per cell
  using Delta = U128;
  static constexpr int kWords = 2;
  static __device__ __forceinline__ double take(Cell* acc, size_t cell, const ColParams& p) {
    U128 K{acc[2 * cell], static_cast<long long>(acc[2 * cell + 1])};
    acc[2 * cell] = 0;
    acc[2 * cell + 1] = 0;
    return units_to_f64(K, p.ue);
  }
  static __device__ __forceinline__ bool to_units(double v, const ColParams& p, Delta* d) {
    return f64_to_units(v, p.ue, d);
  }
  static __device__ __forceinline__ Delta theta_units(const ColParams& p, bool neg) {
    const long long d = neg ? -p.dtheta : p.dtheta;
    return U128{static_cast<unsigned long long>(d), d < 0 ? -1ll : 0ll};
  }
  static __device__ __forceinline__ double mag_units(double v, const ColParams& p) {
    return ldexp(fabs(v), -p.ue);
  }
  // the carry out of the low word needs the old value
  static __device__ __forceinline__ void add(Cell* acc, size_t cell, Delta d) {
    const unsigned long long old = atomic_add_ret(acc + 2 * cell, d.lo);
    const unsigned long long carry = (old + d.lo < old) ? 1ull : 0ull;
    const unsigned long long h = static_cast<unsigned long long>(d.hi) + carry;
    if (h != 0ull) atomic_add_relaxed(acc + 2 * cell + 1, h);
  }
  static __device__ __forceinline__ bool add_ret(Cell* acc, size_t cell, Delta d) {
    add(acc, cell, d);
    return false;  // binary64 calls always compact the next frontier
  }
  static __device__ __forceinline__ Delta load(const Cell* acc, size_t cell) {
    return U128{acc[2 * cell], static_cast<long long>(acc[2 * cell + 1])};
  }
  static __device__ __forceinline__ void store(Cell* acc, size_t cell, Delta v) {
    acc[2 * cell] = v.lo;
    acc[2 * cell + 1] = static_cast<unsigned long long>(v.hi);
  }
  static __device__ __forceinline__ bool is_zero(Delta v) { return (v.lo | static_cast<unsigned long long>(v.hi)) == 0ull; }
  static __device__ __forceinline__ Delta sum(Delta a, Delta b) {
    const unsigned long long lo = a.lo + b.lo;
    return U128{lo, static_cast<long long>(static_cast<unsigned long long>(a.hi) + static_cast<unsigned long long>(b.hi) +
                                           (lo < a.lo ? 1ull : 0ull))};
  }
  static __device__ __forceinline__ bool nonzero(const Cell* acc, size_t cell) {
    return (acc[2 * cell] | acc[2 * cell + 1]) != 0ull;
  }
  static __device__ __forceinline__ void set_units(Cell* acc, size_t cell, long long v) {
    acc[2 * cell] = static_cast<unsigned long long>(v);
    acc[2 * cell + 1] = v < 0 ? ~0ull : 0ull;
  }
};

__device__ __forceinline__ float to_w(double v, float) { return static_cast<float>(v); }
__device__ __forceinline__ double to_w(double v, double) { return v; }

// ------------------------------------------------- record staging
// On binned levels a sampled push becomes a 4-byte record, cell | sign << 31
// (its value is -/+ fl(theta_c) of the cell's column c); deterministic pushes
// still use atomics.  Records go to their group's buffer in chunks (one
// atomic per chunk).  Records beyond the buffer capacity are added to the
// accumulator directly; the level then ends in kModeOverflow (the buffered
// records are applied with atomics too).
//
// The cell of a record is local to a column group, so that it stays below
// 2^31 when n C does not: with one group it is u * su + c * sc; with two
// (row-major cells only) group g = [c >= rec_gw] holds the columns from
// g rec_gw on and the local cell is u * rec_gw + (c - g rec_gw).
constexpr int kRecStage = 2 * kStage;  // 4-byte records per wave stage (both groups)
constexpr uint32_t kRecCellMask = 0x7FFFFFFFu;
// A group's records go to kRecSegs segments in turn, each with a counter on a
// line of its own: returning atomics on one address serialise at 12 ns, and
// the 622 thousand flushes of a dense transition level (637M records, 64
// columns of 2^22 nodes) took 7.5 of its 9.5 ms on one counter.
constexpr int kRecSegs = 16;
constexpr int kRecStride = 16;  // words between counters (128 bytes)
constexpr int kMaxRecGroups = 2;

// kG: the groups of the launch (A.rec_groups of a binned level), a template
// argument so that one-group levels keep the plain single-group code.
struct RecCell {
  uint32_t g, cell;
};
// What the cell of a record is made from: the row stride (one group; records
// are kept on row-major cells only) or the columns of a group, and the
// buckets' size.
struct RecShape {
  uint32_t width;
  int shift;
};
template <int kG>
__device__ __forceinline__ RecShape rec_shape(const LevelArgs& A) {
  return RecShape{kG > 1 ? A.rec_gw : static_cast<uint32_t>(A.su), A.bucket_shift};
}
template <int kG>
__device__ __forceinline__ RecCell rec_cell(const RecShape& R, uint32_t u, uint32_t c) {
  if constexpr (kG > 1) {
    const uint32_t g = c >= R.width ? 1u : 0u;
    return RecCell{g, u * R.width + (c - g * R.width)};
  } else {
    return RecCell{0u, u * R.width + c};
  }
}

// (kG = 0: the groups of A at run time)
template <int kG>
__device__ __forceinline__ void apply_record(const LevelArgs& A, long long* acc, uint32_t rec, uint32_t g) {
  const uint32_t cell = rec & kRecCellMask;
  uint32_t c;
  size_t at = cell;
  if (kG > 1 || (kG == 0 && A.rec_groups > 1)) {
    const uint32_t u = cell / A.rec_gw;
    c = g * A.rec_gw + (cell - u * A.rec_gw);
    at = static_cast<size_t>(u) * static_cast<size_t>(A.su) + c;
  } else {
    c = A.sc == 1 ? cell % static_cast<uint32_t>(A.su) : cell / static_cast<uint32_t>(A.sc);
  }
  const long long d = (rec >> 31) ? -A.cp[c].dtheta : A.cp[c].dtheta;
  atomic_add_relaxed(reinterpret_cast<unsigned long long*>(acc + at), static_cast<unsigned long long>(d));
}

template <int kG>
__device__ __forceinline__ void apply_record(const LevelArgs&, unsigned long long*, uint32_t, uint32_t) {}

// The column word of a batch's entry: the column, the residue's sign, and (a
// batch's own) whether a = 0 and the log2 of the windows per work item.
constexpr uint32_t kBatchNeg = 1u << 31, kBatchAZero = 1u << 30;
constexpr int kBatchShiftBit = 27;  // three bits
constexpr uint32_t kBatchCol = (1u << kBatchShiftBit) - 1u;

// Staged record counts of a wave: the count (one group), or group 0's in the
// low 16 bits and group 1's in the high 16 bits of one wave-uniform int.
//
// The staged records out: group 0's from the front of the stage, group 1's
// from its back (one atomic on each group's count; records beyond a group's
// buffer are added with atomics).  Wave-uniform.
template <int kG, typename Cell>
__device__ __forceinline__ void stage_flush_records(uint32_t* stage, int& staged, int& seg, Cell* acc) {
  const LevelArgs& A = args_again();
  if constexpr (kG == 1) {
    if (staged == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    unsigned long long base = 0;
    if (lane_id() == 0) base = atomicAdd(A.rec_count + seg * kRecStride, static_cast<unsigned long long>(staged));
    base = uniform(base);
    uint32_t* const rec = A.rec + static_cast<size_t>(seg) * A.rec_cap;
    for (int i = lane_id(); i < staged; i += kWave) {
      if (base + i < A.rec_cap)
        rec[base + i] = stage[i];
      else
        apply_record<kG>(A, acc, stage[i], 0u);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    staged = 0;
    seg = (seg + 1) & (kRecSegs - 1);
    return;
  }
  const int n0 = staged & 0xFFFF, n1 = staged >> 16;
  const int total = n0 + n1;
  if (total == 0) return;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const int lane = lane_id();
  unsigned long long base = 0;
  if (lane < 2) {
    const int k = lane == 0 ? n0 : n1;
    if (k > 0) base = atomicAdd(A.rec_count + (lane * kRecSegs + seg) * kRecStride, static_cast<unsigned long long>(k));
  }
  const unsigned long long base0 = uniform(base), base1 = uniform(__shfl(base, 1));
  for (int i = lane; i < total; i += kWave) {
    const uint32_t g = i < n0 ? 0u : 1u;
    const int j = i - (g ? n0 : 0);
    const uint32_t r = g ? stage[kRecStage - 1 - j] : stage[j];
    const unsigned long long at = (g ? base1 : base0) + static_cast<unsigned long long>(j);
    if (at < A.rec_cap)
      A.rec[static_cast<size_t>(g * kRecSegs + seg) * A.rec_cap + at] = r;
    else
      apply_record<kG>(A, acc, r, g);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  staged = 0;
  seg = (seg + 1) & (kRecSegs - 1);
}

// One sampled push of every lane that emits (a wave-uniform call) as a
// record of its group: its bucket counted in s_hist (kBuckets buckets, or
// kBuckets / 2 per group with two groups), the record staged (group 0 from
// the front of the stage, group 1 from its back); the stage goes out when it
// is nearly full.
template <int kG, typename Cell>
__device__ __forceinline__ void emit_record(const RecShape& R, unsigned int* s_hist, uint32_t* stage, int& staged,
                                            int& seg, bool emit, uint32_t v, uint32_t cw, Cell* acc) {
  uint32_t rec = 0, g = 0;
  if (emit) {
    const RecCell rc = rec_cell<kG>(R, v, cw & kBatchCol);
    g = rc.g;
    rec = rc.cell | (cw & kBatchNeg);
    atomicAdd(&s_hist[g * (kBuckets / kMaxRecGroups) + (rc.cell >> R.shift)], 1u);
  }
  if constexpr (kG > 1) {
    const int n0 = staged & 0xFFFF, n1 = staged >> 16;
    const unsigned long long m1 = wave_ballot(emit && g != 0);
    const unsigned long long m0 = wave_ballot(emit) & ~m1;
    if (emit) stage[g ? kRecStage - 1 - static_cast<int>(lanes_below(m1, n1)) : static_cast<int>(lanes_below(m0, n0))] = rec;
    const int k0 = n0 + __popcll(m0), k1 = n1 + __popcll(m1);
    staged = static_cast<int>(uniform(static_cast<uint32_t>(k0 | (k1 << 16))));
    if (k0 + k1 > kRecStage - kWave) stage_flush_records<kG>(stage, staged, seg, acc);
  } else {
    const unsigned long long m0 = wave_ballot(emit);
    if (emit) stage[lanes_below(m0, staged)] = rec;
    staged = static_cast<int>(uniform(static_cast<uint32_t>(staged + __popcll(m0))));
    if (staged > kRecStage - kWave) stage_flush_records<kG>(stage, staged, seg, acc);
  }
}

// The end of a binned launch: the staged records out, then (after a block
// barrier) the block's bucket counts added to the level's.
template <int kG, typename Cell>
__device__ __forceinline__ void finish_records(const LevelArgs& A, unsigned int* s_hist, uint32_t* stage, int& staged,
                                               int& seg, Cell* acc) {
  stage_flush_records<kG>(stage, staged, seg, acc);
  __syncthreads();
  for (int i = threadIdx.x; i < kBuckets; i += blockDim.x)
    if (s_hist[i]) atomicAdd(A.bucket_count + i, s_hist[i]);
}

// a deterministic push's mark on its destination bin (binned levels)
template <int kG>
__device__ __forceinline__ void mark_det_bin(const LevelArgs& A, uint8_t* det_bins, uint32_t v, uint32_t c) {
  const RecCell rc = rec_cell<kG>(rec_shape<kG>(A), v, c);
  det_bins[rc.g * A.det_bins_g + (rc.cell >> kBinLog2)] = 1;
}

// Server counters: LDS sums for the first kServeLdsSlots columns (one block's
// share of a step), atomics on the block's row of the column beyond.
struct ServeSums {
  uint32_t front, cand, acc, runs;
  unsigned long long det;
  double mass;
};
__device__ __forceinline__ unsigned long long* serve_row(const LevelArgs& A, uint32_t c) {
  return A.counters + (static_cast<size_t>(blockIdx.x & A.shard_mask) * A.slots + c) * kCountStride;
}
__device__ __forceinline__ void serve_flush(unsigned long long* row, const ServeSums& v) {
  if (v.front) atomic_add_relaxed(row + 0, v.front);
  if (v.det) atomic_add_relaxed(row + 2, v.det);
  if (v.cand) atomic_add_relaxed(row + 3, v.cand);
  if (v.acc) atomic_add_relaxed(row + 4, v.acc);
  if (v.runs) atomic_add_relaxed(row + 5, v.runs);
  if (v.mass != 0.0) atomicAdd(reinterpret_cast<double*>(row + kCountMass), v.mass);
}
__device__ __forceinline__ void serve_entry(const LevelArgs& A, ServeSums* lds, uint32_t c, uint32_t det, double mass) {
  if (c < kServeLdsSlots) {
    atomicAdd(&lds[c].front, 1u);
    if (det) atomicAdd(&lds[c].det, static_cast<unsigned long long>(det));
    if (mass != 0.0) atomicAdd(&lds[c].mass, mass);
  } else {
    serve_flush(serve_row(A, c), ServeSums{1u, 0u, 0u, 0u, det, mass});
  }
}
__device__ __forceinline__ void serve_item(const LevelArgs& A, ServeSums* lds, uint32_t c, uint32_t cand, uint32_t acc,
                                           uint32_t runs) {
  if (c < kServeLdsSlots) {
    if (cand) atomicAdd(&lds[c].cand, cand);
    if (acc) atomicAdd(&lds[c].acc, acc);
    if (runs) atomicAdd(&lds[c].runs, runs);
  } else {
    serve_flush(serve_row(A, c), ServeSums{0u, cand, acc, runs, 0ull, 0.0});
  }
}

// The block's counter row of the level (batched calls).
__device__ __forceinline__ unsigned long long* count_row(const LevelArgs& A) {
  return A.counters +
         (static_cast<size_t>(A.level) * kCountShards + (blockIdx.x & (kCountShards - 1))) * kCountStride;
}

// ------------------------------------------------------------ the level
// Work is organised per wave.  A wave takes batches of up to 64 frontier
// entries (batch b of the level goes to wave b mod #waves); for each batch a lane
// sets up one entry (reserve update, c, the deterministic prefix J, the
// number of sampled work items), the wave then makes the batch's
// deterministic pushes with all lanes, one push per lane and step, and puts
// the sampled work items in a queue that idle lanes draw from.  A sampled
// work item is a run of 1 to 16 consecutive 64-position windows of one
// entry's suffix, as many as are expected to take about 64 draws (so
// that no lane is left with a long chain while the others idle); a lane walks
// their Philox / geometric-skip chains one draw per step and takes the next
// item from the queue in the step after its last draw, so lanes stay busy
// across entries and batches.  All loops run in lockstep per wave so that
// staging can use wave-wide ballots.
//
// What bounds it: the draw loop's own steps (taking items, runs and emits
// beside the draw) with lanes that wait for their wave: dense transition
// levels make 129 Gdraw/s (runs and candidates) of the 460 that draws alone
// make at a = 0, the first level of a feature matrix 99 of the 421 at a > 0
// (draw-only loops of 84 and 92 vector instructions); copies of such a level
// without the record writes, the neighbour loads or the Philox rounds take 7,
// 9 and 7% less.  The a = 0 kernels of levels 1 on hold five waves per SIMD (90
// registers, 94 with two record groups or binary64, of the 96 that five allow;
// 29 KB of LDS per block); level 0 in binary32 (98 and 101), a > 0 (104 to 113)
// and the server's (114) four.  On levels with hubs the longest lane used to be the bound: items of 16 windows are up to 1024
// draws for one lane, and the 64 columns of a hub are one batch.  Items of
// even draws and batch-wise deferral took a level of 64 Katz columns on a
// 2^20-node R-MAT graph (47M draws) from 6.3 to 1.2 ms, the call from 148 to
// 41 ms, and 64 ten-step transition columns on 2^22 nodes from 155 to 129 ms
// (90 with all that followed).
constexpr int kBatch = kWave;
constexpr int kMaxItemShift = 4;  // at most 16 windows per item
constexpr int kItemMap = 128;
// A level with at most kFewEntries entries (one batch per resident wave) is
// bound by the longest chain of a lane, not by issue: its batches hold
// entries / kResidentWaves entries and its items aim at a quarter of the draws.
constexpr unsigned long long kResidentWaves = 4096;  // four blocks of four waves on each of 256 CUs
constexpr unsigned long long kFewEntries = kResidentWaves * kWave;

// log2 of the windows of an entry's work items, given an upper bound p on its
// sampling probability: a window takes about 1 + 64 p draws, an item about
// 64 (16 with few entries).
__device__ __forceinline__ uint32_t item_shift(double p, bool few) {
  const float f = 1.0f + 64.0f * static_cast<float>(p);
  uint32_t s = f <= 4.0f ? 4u : f <= 8.0f ? 3u : f <= 16.0f ? 2u : f <= 32.0f ? 1u : 0u;
  if (few) s = s > 2u ? s - 2u : 0u;
  return s;
}

struct BatchLds {
  int64_t rp[kBatch];
  double cv[kBatch];
  double p0[kBatch];           // a = 0: sampling probability of every run of the entry;
                               // a > 0: the first arc's factor when the entry has no
                               // deterministic push (its first run starts there), else 0
  long long doff[kBatch];      // deterministic pushes before each entry (exclusive scan)
  uint32_t ioff[kBatch];       // sampled work items before each entry
  // the entry's column parameters that its work items need (theta, the
  // random stream's counter word), so that taking an item reads LDS
  double th[kBatch];
  uint32_t ctr3[kBatch];
  // c: column | kBatchNeg (negative residue) | kBatchAZero (server: a = 0) |
  // log2 of the windows per work item << kBatchShiftBit
  uint32_t u[kBatch], c[kBatch], d[kBatch], J[kBatch];
  uint8_t item_entry[kItemMap];  // the entry of each of the batch's first kItemMap work items
};
static_assert(kMaxItemShift < 8, "three bits hold the shift");
// columns of one level launch at most (the column index leaves those bits free)
constexpr int32_t kMaxTileColumns = static_cast<int32_t>(kBatchCol);

// floor(a / C) and a mod C for a < 2^22, from rc = 1 / C rounded to binary32:
// the product is within one of the quotient, and one correction makes it exact
__device__ __forceinline__ uint32_t div_small(uint32_t a, uint32_t C, float rc, uint32_t* rem) {
  uint32_t q = static_cast<uint32_t>(static_cast<float>(a) * rc);
  int32_t r = static_cast<int32_t>(a) - static_cast<int32_t>(q * C);
  if (r < 0) {
    --q;
    r += static_cast<int32_t>(C);
  } else if (r >= static_cast<int32_t>(C)) {
    ++q;
    r -= static_cast<int32_t>(C);
  }
  *rem = static_cast<uint32_t>(r);
  return q;
}

// Level 0 of a batched call whose signal is mostly non-zero: the frontier is
// every cell in order, entry e = (e / C, e mod C), and no list is formed
// (A.fin == nullptr; C = A.su <= kVirtualMaxC); its zero cells are skipped
// by the level kernel as if they were not listed.
constexpr long long kVirtualMaxC = 1 << 21;

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// largest e in [0, 64) with off[e] <= k (off non-decreasing, off[0] <= k)
template <typename I>
__device__ __forceinline__ int batch_find(const I* off, I k) {
  int e = 0;
#pragma unroll
  for (int step = kBatch / 2; step > 0; step >>= 1)
    if (off[e + step] <= k) e += step;
  return e;
}

// One push of every lane that emits (all lanes together), added to the
// accumulators with atomics: on sparse levels the first contribution to a
// cell appends it to the next frontier; a served query's push goes to its
// table, first touches to the next frontier.
template <typename T, int kMode>
__device__ __forceinline__ void push_atomic(const LevelArgs& A, uint64_t* stage, int& staged, bool sparse, bool emit,
                                            uint32_t v, uint32_t c, const typename Prec<T>::Delta& delta,
                                            typename Prec<T>::Cell* acc_next) {
  using P = Prec<T>;
  bool first = false;
  if constexpr (kMode == kPerColumn) {
    uint32_t pos = 0;
    if (emit) {
      const uint32_t mask = A.tab_mask[c];
      if (mask == kDirectPlain) {  // the next frontier comes from a scan of the table
        pos = A.tab_off[c] + v;
        P::add(acc_next, pos, delta);
      } else {
        pos = table_find_or_insert(A.keys_nxt, A.tab_off[c], mask, v, &first);
        if (pos == ~0u)
          atomicOr(A.err + c, kErrTableFull);
        else
          P::add(acc_next, pos, delta);
      }
    }
    stage_push(stage, staged, (static_cast<uint64_t>(pos) << 32) | c, first, A.fout, A.cnt_out);
  } else {
    const size_t vcell = static_cast<size_t>(v) * A.su + static_cast<size_t>(c) * A.sc;
    if (emit) {
      if (sparse)
        first = P::add_ret(acc_next, vcell, delta);
      else
        P::add(acc_next, vcell, delta);
    }
    if (sparse)  // stage first-touched cells, flush in chunks
      stage_push(stage, staged, (static_cast<uint64_t>(v) << 32) | c, first, A.fout, A.cnt_out);
  }
}

// Exclusive scans of the batch's work items into B.ioff, and the entry of each
// of the first kItemMap items; returns the items of the whole batch.
__device__ __forceinline__ uint32_t queue_items(BatchLds& B, uint32_t iwork) {
  const int lane = lane_id();
  const uint32_t iinc = wave_scan(iwork);
  B.ioff[lane] = iinc - iwork;
  const int j1 = static_cast<int>(iinc < kItemMap ? iinc : kItemMap);
  for (int j = static_cast<int>(iinc - iwork < kItemMap ? iinc - iwork : kItemMap); j < j1; ++j)
    B.item_entry[j] = static_cast<uint8_t>(lane);
  return last_lane(iinc);
}

// v < fl(p / q) for v in [0, 1) and factors p, q > 0: fl(p / q) is p / q and
// fl(v q) is v q to 2^-53 each, so a product off p by more than 2^-50 decides;
// the division is left for the others (one in about 2^48).
__device__ __forceinline__ bool below_ratio(double v, double p, double q) {
  const double vq = v * q;
  if (vq < p * (1.0 - 0x1p-50)) return true;
  if (vq > p * (1.0 + 0x1p-50)) return false;
  return v < p / q;
}

// Sum of v over the lanes before this one in its group of eight.
__device__ __forceinline__ uint32_t group_scan_before(uint32_t v) {
  const uint32_t sub = lane_id() & 7;
  // (moves outside the selections: under one, its lanes alone would take part)
  uint32_t m = lane_move<0x111, 0xf>(v);
  uint32_t x = sub >= 1 ? m : 0u;  // v of the lane before
  m = lane_move<0x111, 0xf>(x);
  x += sub >= 1 ? m : 0u;
  m = lane_move<0x112, 0xf>(x);
  x += sub >= 2 ? m : 0u;
  m = lane_move<0x114, 0xf>(x);
  x += sub >= 4 ? m : 0u;
  return x;
}

// Draws the queued work items of the batches that refill sets up:
// refill(it_next, it_total) puts the next batch in B and its queue of items
// [it_next, it_total), or returns false when none is left; emit(pushed, v, cw)
// makes a sampled push of every lane that has one to node v in the column of
// word cw (all lanes together); served(c, candidates, accepted, runs) gets a
// finished item's counts (server).  w_*: wave-uniform counts (batched calls).
//
// A lane's state is a few integers, compared where a step needs to know it
// (kept as flags, every one of them was a handful of lane-mask operations per
// step): the item's windows [s, rend), the run in progress from s up to run_end
// with its next position pos.  A lane is idle when s >= rend and between runs
// when run_end == s; the lanes all draw in every step, an idle one with pos =
// run_end, past which no skip is a candidate.
//
// group (levels with few entries): the eight lanes of a group take one item
// together and make eight draws of its run in a step.  Draw t of a run is a
// function of the run and t alone, so only the positions chain: a scan of the
// skips over the group.  A lane's chain of up to 64 draws, a memory round trip
// each, had been the length of a small level.  (refill may set it with a wave's
// first batch, when every lane is idle.)
constexpr int kGroup = 8;
constexpr unsigned long long kGroupItems = 16;  // k_samp_big: items per wave up to which groups draw
// Idle lanes from which items are taken on large levels with a = 0: fewer steps
// read the queue (8 against 1: transition block 96.8 and 98.0 ms, Katz block
// 44.0 and 44.7; for a > 0 and on small levels every idle lane is worth the
// read: 128 feature columns on 2.4M nodes 83.8 and 82.1).
constexpr int kRefillIdle = 8;
template <int kMode, typename Refill, typename Emit, typename Served>
__device__ __forceinline__ void sample_loop(const LevelArgs& A, BatchLds& B, Refill&& refill, Emit&& emit_sampled,
                                            Served&& served, int refill_idle, bool& group, uint32_t& w_cand, uint32_t& w_acc,
                                            uint32_t& w_runs) {
  constexpr bool kServe = kMode == kPerColumn;
  constexpr uint32_t kFirstRun = ~0u;  // in t: the item has no run yet
  uint32_t it_next = 0, it_total = 0;  // wave-uniform: queue of the loaded batch
  bool more = true;                    // wave-uniform: refill may have another batch

  uint32_t u = 0, cw = 0, s = 0, rend = 0, run_end = 0, pos = 0, t = 0, ctr3 = 0;
  uint32_t key0 = kServe ? 0u : uniform(A.lp->key0);
  uint32_t key1 = kServe ? 0u : uniform(A.lp->key1);
  uint32_t it_cand = 0, it_acc = 0, it_runs = 0;
  int64_t rpu = 0;
  double cv = 0.0, dstart = 1.0, th = 0.0;
  const uint32_t* const col = pinned(A.col);
  const double* const arcfac = kMode == kBatchAP ? pinned(A.arcfac) : nullptr;
  const double* da = A.da;
  SkipTable tab{};
  constexpr unsigned long long kGroupFirst = 0x0101010101010101ull;  // the groups' first lanes
  // a = 0 (a constant but for the server)
  auto azero = [&]() { return kServe ? (cw & kBatchAZero) != 0 : kMode == kBatchAZ; };

  for (;;) {
    unsigned long long idle = wave_ballot(s >= rend);
    if (__popcll(idle) >= refill_idle) {
      // the queue is empty: set up the next batch
      if (more && it_next >= it_total) more = refill(it_next, it_total);
      const uint32_t sub = group ? lane_id() & (kGroup - 1) : 0u;
      if (it_next < it_total) {  // idle lanes take work items
        // (a group's lanes share the item of its first lane)
        const unsigned long long takers = group ? idle & kGroupFirst : idle;
        const uint32_t it = group ? lanes_below(takers, it_next) - (sub != 0u && s >= rend ? 1u : 0u)
                                  : lanes_below(takers, it_next);
        if (s >= rend && it < it_total) {
          const int e = it < kItemMap ? B.item_entry[it] : batch_find<uint32_t>(B.ioff, it);
          const uint32_t il = it - B.ioff[e];
          u = B.u[e];
          cw = B.c[e];
          rpu = B.rp[e];
          const uint32_t J = B.J[e], d = B.d[e];
          ctr3 = B.ctr3[e];
          if (kServe) {
            const ColParams& cp = A.cp[cw & kBatchCol];
            key0 = cp.key0;
            key1 = cp.key1;
            da = cp.da;
          }
          const uint32_t shift = (cw >> kBatchShiftBit) & 7u;
          const uint32_t w0 = (J >> kSegLog2) + (il << shift);
          const uint32_t ws = w0 << kSegLog2, we = (w0 + (1u << shift)) << kSegLog2;
          s = ws > J ? ws : J;
          rend = we < d ? we : d;
          run_end = pos = s;
          t = kFirstRun;
          if (azero()) {
            tab = make_skip_table(B.p0[e]);
          } else {
            cv = B.cv[e];
            th = B.th[e];
            dstart = il == 0 ? B.p0[e] : 0.0;  // the first run's factor when the entry's setup has it (else 0)
          }
          if (kServe) it_cand = it_acc = it_runs = 0;
        }
        it_next = uniform(it_next + static_cast<uint32_t>(__popcll(takers)));
        if (it_next > it_total) it_next = it_total;
        idle = wave_ballot(s >= rend);
      }
      if (idle == ~0ull) {
        if (!more && it_next >= it_total) break;  // nothing queued, no batch left
        continue;
      }
    }
    // a run: the rest of the current window, or (a > 0) of its degree group
    // unless few candidates are expected over the rest of the window
    const bool fresh = run_end == s;  // (an idle lane's run stays empty)
    const uint32_t wnext = (s | (kSeg - 1u)) + 1u;
    const uint32_t wend = wnext < rend ? wnext : rend;
    if constexpr (kMode == kBatchAZ) {
      const uint32_t end = wend > s ? wend : s;
      run_end = fresh ? end : run_end;
      t = fresh ? 0u : t;
    } else if (fresh && s < rend) {
      run_end = wend;
      if (kServe) it_runs += !group || (lane_id() & (kGroup - 1)) == 0 ? 1u : 0u;
      if (!azero()) {
        // the factor of the run's first arc (for an item's first run at the
        // row start, from the entry's setup); the group end only when the
        // run stops there
        if (!(t == kFirstRun && dstart > 0.0))
          dstart = arcfac != nullptr ? arcfac[rpu + s] : da[A.nd[rpu + s]];
        const double num = cv * dstart;
        const double pr = num / th;
        if (!(pr * static_cast<double>(wend - s) <= kMergeCandidates)) {
          const uint32_t ge = A.gend[rpu + s];
          if (ge < wend) run_end = ge;
        }
        tab = make_skip_table(pr);
      }
      t = 0;
    }
    // one draw of the run's chain (a group: draws t to t + 7)
    const uint32_t sub = group ? lane_id() & (kGroup - 1) : 0u;
    const uint32_t draw = t + sub;
    const U4 o = kServe ? philox4x32_10(draw, s, u, ctr3, key0, key1)
                        : philox4x32_10_skey(draw, s, u, ctr3, key0, key1);
    uint32_t cand = geometric_skip64(tab, unit_double(o.x, o.y));
    if (group) cand += group_scan_before(cand + 1u);
    cand += pos;
    const bool hit = cand < run_end;  // (the draws of a group after its first miss miss too)
    bool emit = hit;
    uint32_t v = 0;
    if (hit) {
      const int64_t arc = rpu + cand;
      // the neighbour is loaded beside its factor degree, before the
      // acceptance test needs it (one round trip instead of two)
      v = col[arc];
      if (!azero())  // (a = 0: the ratio is 1 and every uniform is below it)
        emit = below_ratio(unit_double(o.z, o.w), arcfac != nullptr ? arcfac[arc] : da[A.nd[arc]], dstart);
    }
    const unsigned long long hit_mask = wave_ballot(hit);
    // whether the run goes on (a group: all eight draws hit), and its next position
    bool on = hit;
    uint32_t next = cand + 1u;
    unsigned long long ended = ~idle & ~hit_mask;  // active lanes whose run ended
    if (group) {
      next = __shfl(next, lane_id() | (kGroup - 1));
      on = ((hit_mask >> (lane_id() & ~(kGroup - 1))) & 0xffull) == 0xffull;
      ended = ~idle & ~wave_ballot(on) & kGroupFirst;
    }
    if (!kServe) {
      w_cand += static_cast<uint32_t>(__popcll(hit_mask));
      w_runs += static_cast<uint32_t>(__popcll(ended));
      w_acc += static_cast<uint32_t>(__popcll(kMode == kBatchAZ ? hit_mask : wave_ballot(emit)));
    } else {
      it_cand += hit ? 1u : 0u;
      it_acc += emit ? 1u : 0u;
      if (!on && s < rend && run_end >= rend) served(cw & kBatchCol, it_cand, it_acc, it_runs);  // the item's end
    }
    s = on ? s : run_end;
    pos = on ? next : run_end;
    t = on ? t + (group ? kGroup : 1u) : t;
    emit_sampled(emit, v, cw);
  }
}

// Reserves list slots for the lanes that defer (wave-uniform call): the list
// counter takes one atomic for all of them, which returns the slot and the
// work before it; false where the list is full (or the lane does not defer).
// The counter is read first, so that it never wraps.
__device__ __forceinline__ bool defer_slots(unsigned long long* ctr, unsigned long long cap, bool want,
                                            unsigned long long work, unsigned long long* slot,
                                            unsigned long long* off) {
  const unsigned long long mask = wave_ballot(want);
  if (mask == 0ull) return false;
  // (one value for the wave: other waves add to the counter, and the lanes scan together below)
  const unsigned long long seen = uniform(__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if ((seen >> kBigShift) >= cap) return false;
  const int lane = lane_id();
  const unsigned long long inc = wave_scan(want ? work : 0ull);
  const unsigned long long total = last_lane(inc);
  unsigned long long old = 0;
  if (lane == 0) old = atomic_add_ret(ctr, (static_cast<unsigned long long>(__popcll(mask)) << kBigShift) | total);
  old = uniform(old);
  *slot = (old >> kBigShift) + static_cast<unsigned long long>(__popcll(mask & ((1ull << lane) - 1ull)));
  *off = (old & ((1ull << kBigShift) - 1ull)) + inc - work;
  return want && *slot < cap;
}

// kFirst: the residues are the signal x (level 0 of a batched call).
// kMode: kBatchAZ, kBatchAP or kPerColumn (the server: counters and overflow
// mass are kept per column instead of per level).
// kG: column groups of the records on binned levels (1 or 2).
template <typename T, bool kFirst, int kMode, int kG = 1>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_level(LevelArgs A, const T* __restrict__ x,
                                                    typename Prec<T>::Cell* __restrict__ acc_cur,
                                                    typename Prec<T>::Cell* __restrict__ acc_next) {
  using P = Prec<T>;
  using Delta = typename P::Delta;
  constexpr bool kServe = kMode == kPerColumn;
  constexpr int kWaves = kThreads / kWave;
  __shared__ BatchLds s_batch[kWaves];
  __shared__ uint64_t s_stage[kWaves][kStage];
  __shared__ unsigned int s_hist[kServe ? 1 : kBuckets];
  // server: per-column counters summed in LDS, flushed once per block
  __shared__ ServeSums s_serve[kServe ? kServeLdsSlots : 1];

  const unsigned long long count = *A.cnt_in;
  if (!kServe) acc_next += (blockIdx.x & A.rep_mask) * A.rep_stride;
  // Binned levels write (cell, value) records that later kernels group by
  // destination and sum in LDS.  Without binning, sparse levels detect the
  // first contribution to a cell from the atomic's old value and append the
  // cell to the next frontier; dense levels use fire-and-forget atomics and a
  // compaction pass builds the next frontier.
  const bool binned = A.rec != nullptr && (A.bin_est == nullptr || *A.bin_est >= A.bin_pushes);
  const bool sparse = kServe || (!binned && A.positive && count < A.dense_cut);
  if (blockIdx.x == 0 && threadIdx.x == 0)
    *A.mode_out = binned ? kModeBinned : (sparse ? kModeSparse : kModeCompact);
  // up to 64 entries per batch; fewer when the level has fewer entries than
  // 64 per resident wave, so that small frontiers spread over the whole chip
  // (but no wider: spread over four generations of waves, a level of 10^5
  // entries paid four times for the setup's chain of loads with a third of
  // the lanes busy; nine queries on a 30011-node graph: 4.07 -> 1.95 ms)
  const unsigned long long nwaves = static_cast<unsigned long long>(gridDim.x) * kWaves;
  const unsigned long long want = (count + kResidentWaves - 1) / kResidentWaves;
  const unsigned long long eb = want < 1ull ? 1ull : (want > (unsigned long long)kBatch ? kBatch : want);
  const bool few = count <= kFewEntries;
  const unsigned long long nbatch = (count + eb - 1) / eb;
  if (static_cast<unsigned long long>(blockIdx.x) * kWaves >= nbatch) return;  // the whole block: no batch
  if (binned) {
    for (int i = threadIdx.x; i < kBuckets; i += blockDim.x) s_hist[i] = 0;
    __syncthreads();
  }
  if (kServe) {
    for (int i = threadIdx.x; i < kServeLdsSlots; i += blockDim.x) s_serve[i] = ServeSums{};
    __syncthreads();
  }
  const int lane = lane_id();
  const int wave = static_cast<int>(uniform(threadIdx.x / kWave));
  BatchLds& B = s_batch[wave];
  uint64_t* stage = s_stage[wave];
  int staged = 0;  // wave-uniform
  int seg = (blockIdx.x * kWaves + wave) & (kRecSegs - 1);  // wave-uniform: the next flush's record segment

  // 32 bits hold a launch's counts: 2^32 candidates of one wave are minutes of
  // draws (a wave makes some 3e7 a second), and a lane's deterministic pushes
  // are the prefixes (below 2^31) of the entries it sets up, one on levels of
  // at most 2^18 entries and on larger ones one a batch of its wave, so that
  // rows of 2^32 arcs in all would have to meet in one lane; the hash wraps
  // mod 2^64
  uint32_t n_det = 0;
  uint32_t w_front = 0, w_cand = 0, w_acc = 0, w_runs = 0;  // wave-uniform (ballot counts)
  unsigned long long n_hash = 0;
  double mass = 0.0;

  // One contribution per lane (or none), in exact units of the next
  // residue.  Wave-uniform calls.  emit_det: a deterministic push (atomics
  // on every level); emit_sampled: a sampled push of -/+ fl(theta) (a
  // 4-byte record on binned levels).
  auto emit_atomic = [&](bool emit, uint32_t v, uint32_t ec, const Delta& delta) {
    push_atomic<T, kMode>(A, stage, staged, sparse, emit, v, ec, delta, acc_next);
  };
  const RecShape shape{pinned(rec_shape<kG>(A).width), pinned(A.bucket_shift)};
  auto emit_sampled = [&](bool emit, uint32_t v, uint32_t cw) {
    if (binned) {
      emit_record<kG>(shape, s_hist, reinterpret_cast<uint32_t*>(stage), staged, seg, emit, v, cw, acc_next);
    } else {
      const uint32_t ec = cw & kBatchCol;
      Delta delta{};
      if (emit) delta = P::theta_units(A.cp[ec], (cw & kBatchNeg) != 0);
      emit_atomic(emit, v, ec, delta);
    }
  };

  unsigned long long bnext = static_cast<unsigned long long>(blockIdx.x) * kWaves + wave;
  // the frontier items of this wave's next batch, loaded one batch ahead so
  // that a batch's setup starts from its items.  Listed levels of few entries
  // deal them out to the batches: the lists are in node order, and the hubs of
  // a power-law graph, neighbours by id, would be one wave's batch (one PPR
  // query on 10^4 nodes 0.58 ms, 0.51 dealt out; three in binary64 0.95 and
  // 0.66; a cluster's estimate and sweep on 4e5 nodes 1.74 and 1.37)
  constexpr uint64_t kNoItem = ~0ull;
  auto load_items = [&](unsigned long long b) -> uint64_t {
    if (b >= nbatch || static_cast<unsigned long long>(lane) >= eb) return kNoItem;
    if (!kFirst) {
      const uint32_t step = few ? static_cast<uint32_t>(nbatch) : 1u;
      const unsigned long long e = b * (few ? 1ull : eb) + static_cast<uint32_t>(lane) * step;
      return e < count ? A.fin[e] : kNoItem;
    }
    const unsigned long long e = b * eb;
    if (e + lane >= count) return kNoItem;
    if (A.fin == nullptr) {  // every cell: (e / C, e mod C)
      const uint32_t C = static_cast<uint32_t>(A.su);
      const unsigned long long u0 = e / C;
      uint32_t c = 0;
      const uint32_t q = div_small(static_cast<uint32_t>(e - u0 * C) + static_cast<uint32_t>(lane), C,
                                   1.0f / static_cast<float>(C), &c);
      return ((u0 + q) << 32) | c;
    }
    return A.fin[e + lane];
  };
  uint64_t next_items = load_items(bnext);

  bool group = false, first_batch = true;
  auto refill = [&](uint32_t& it_next, uint32_t& it_total) -> bool {
    if (bnext >= nbatch) return false;
    const LevelArgs& A = args_again();
    wave_sync();  // every lane has read the previous batch
    bnext += nwaves;
    const uint64_t batch_item = next_items;
    next_items = load_items(bnext);
    long long dwork = 0;
    uint32_t iwork = 0;
    uint32_t eu = 0, ec = 0, ed = 0, eJ = 0, ecw = 0;
    int64_t erp = 0;
    double ecv = 0.0, ep0 = 0.0;
    bool eneg = false;
    bool front_live = false, serve_live = false;
    double emass = 0.0;  // server: the entry's share of its column's mass
    if (batch_item != kNoItem) {
      const uint64_t item = batch_item;
      eu = static_cast<uint32_t>(item >> 32);
      ec = static_cast<uint32_t>(item);
      size_t cell = static_cast<size_t>(eu) * A.su + static_cast<size_t>(ec) * A.sc;
      if constexpr (kServe) {  // (table position, query): the node is the key (or the offset); free it
        cell = eu;
        if (A.tab_mask[ec] == kDirectPlain) {
          eu = static_cast<uint32_t>(cell) - A.tab_cur[ec];
        } else {
          eu = A.keys_cur[cell] - 1u;
          A.keys_cur[cell] = 0u;
        }
      }
      // The loads that need only the entry go out together (a batched
      // entry always names a node of the graph and a live column: its row
      // bounds and factor degree beside its residue and column parameters),
      // then the ones that need their results (the reserve's old value, the
      // first neighbour's factor degree, d_u^-b).
      uint32_t deg_u = 0;
      int32_t fdeg_u = 0;
      int64_t rp_u = 0;
      const bool pre = !kServe && A.nodefac != nullptr;  // the node's two factors in one load
      const bool pre_arc = !kServe && A.arcfac != nullptr;  // each arc's neighbour factor in one load
      double2 nf = make_double2(0.0, 0.0);
      if (!kServe) {
        deg_u = static_cast<uint32_t>(A.deg[eu]);
        if (pre)
          nf = reinterpret_cast<const double2*>(A.nodefac)[eu];
        else
          fdeg_u = A.fdeg[eu];
        rp_u = A.rp[eu];
      }
      const ColParams& cp = A.cp[ec];
      const double rho = kServe ? cp.rho : A.lp->rho, kappa = kServe ? cp.kappa : A.lp->kappa;
      const int lflags = kServe ? cp.flags : A.lp->flags;
      const bool azero = kServe ? (lflags & kAZero) != 0 : kMode == kBatchAZ;
      const double* const da = kServe ? cp.da : A.da;
      const double* const db = kServe ? cp.db : A.db;
      T r;
      if (kFirst)
        r = x[static_cast<size_t>(eu) * static_cast<size_t>(A.xld) + ec];
      else
        r = P::take(acc_cur, cell, cp);
      // (a served query's table also holds nodes whose sum cancelled to zero,
      // and level 0 over every cell holds the zero cells of x: they are not
      // in the frontier)
      const bool live = !(kServe && (lflags & kDrop)) && !((kServe || (kFirst && A.fin == nullptr)) && r == T(0));
      if (kServe && live) {
        deg_u = static_cast<uint32_t>(A.deg[eu]);
        fdeg_u = A.fdeg[eu];
        rp_u = A.rp[eu];
      }
      T* const o = kServe ? static_cast<T*>(cp.out) + static_cast<size_t>(eu) * static_cast<size_t>(cp.out_stride)
                          : static_cast<T*>(A.out) + static_cast<size_t>(eu) * static_cast<size_t>(A.out_stride) + ec;
      const T o_old = (live && kappa != 0.0) ? *o : T(0);
      // (a = 0: every factor d^-a is 1, no degree is read)
      const uint32_t nd_first = (!pre && live && deg_u > 0 && !azero) ? A.nd[rp_u] : 0u;
      const double db_u = live ? (pre ? nf.x : db[fdeg_u]) : 0.0;
      eneg = r < T(0);
      ecw = ec | (eneg ? kBatchNeg : 0u) | (kServe && azero ? kBatchAZero : 0u);
      // (the previous batch is no longer read: these slots are free; the
      // lanes without an entry get no work items)
      B.th[lane] = cp.theta;
      B.ctr3[lane] = (cp.qid << 8) | static_cast<uint32_t>(kServe ? cp.level : A.level);
      if (live) {
        if (kServe) {
          serve_live = true;
        } else {
          front_live = true;
          n_hash += splitmix64(eu);
        }
        // reserve: pi(u) += (S w_i / Y_i) r(u), rounded to the working precision
        if (kappa != 0.0) {
          const T q = to_w(kappa * static_cast<double>(r), T());
          *o = o_old + q;
        }
        if (!(lflags & kLastLevel) && rho != 0.0) {
          ed = deg_u;
          if (ed > 0) {
            const double absr = fabs(static_cast<double>(r));
            const double t0 = rho * absr;
            ecv = t0 * db_u;
            const double eth = cp.theta;
            erp = rp_u;
            double inc0 = ecv;
            if (azero) {
              eJ = (ecv >= eth) ? ed : 0u;
              const double num = ecv * 1.0;  // every neighbour's factor d^-0 is 1
              ep0 = num / eth;
            } else {  // increments fall along the degree-sorted row: binary search
              const double da0 = pre ? nf.y : da[nd_first];
              inc0 = ecv * da0;
              uint32_t lo = 0, hi = ed;
              if (!(inc0 >= eth))
                hi = 0;  // no deterministic push
              else if (ecv * (pre_arc ? A.arcfac[erp + ed - 1] : da[A.nd[erp + ed - 1]]) >= eth)
                lo = ed;  // every push is deterministic
              while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                const double inc = ecv * (pre_arc ? A.arcfac[erp + mid] : da[A.nd[erp + mid]]);
                if (inc >= eth)
                  lo = mid + 1;
                else
                  hi = mid;
              }
              eJ = lo;
              // without deterministic pushes the first sampled run starts at
              // the row's first arc: its factor goes with the entry
              ep0 = eJ == 0 ? da0 : 0.0;
            }
            const long long windows =
                (eJ < ed) ? static_cast<long long>(((ed - 1) >> kSegLog2) - (eJ >> kSegLog2) + 1) : 0;
            dwork = eJ;
            // (past a deterministic prefix the probability starts below 1)
            const uint32_t shift = item_shift(eJ == 0 ? inc0 / eth : 1.0, few);
            ecw |= shift << kBatchShiftBit;
            iwork = static_cast<uint32_t>((windows + (1ll << shift) - 1) >> shift);
            // bound on the magnitude this entry can add (every contribution
            // is at most max(inc_0, theta)), for the overflow check
            const T big = to_w(inc0 > eth ? inc0 : eth, T());
            const double m = static_cast<double>(ed) * P::mag_units(big, cp);
            if (kServe) {
              emass = m;
            } else {
              n_det += eJ;
              mass += m;
            }
          }
        }
      }
    }
    if (!kServe) w_front += static_cast<uint32_t>(__popcll(wave_ballot(front_live)));
    if (kServe && serve_live) serve_entry(A, s_serve, ec, eJ, emass);
    // long deterministic prefixes and entries with many work items leave for
    // the deferred lists
    if (A.big_ctr != nullptr && wave_any(eJ >= kBatchDetRow || eJ >= A.big_row)) {
      const bool full = wave_sum_all(eJ < (1u << 20) ? eJ : (1u << 20)) > kBatchDet;
      unsigned long long slot = 0, off = 0;
      if (defer_slots(A.big_ctr, A.big_cap, eJ >= A.big_row || (full && eJ >= kBatchDetRow), eJ, &slot, &off)) {
        BigRow br;
        br.off = off;
        br.rp = erp;
        br.cv = ecv;
        br.c = ecw;
        br.J = eJ;
        A.big[slot] = br;
        dwork = 0;
      }
    }
    const uint32_t big_items = static_cast<uint32_t>(A.samp_items);
    if (A.samp_ctr != nullptr && wave_any(iwork >= kBatchItemRow || iwork >= big_items)) {
      const bool full = wave_sum_all(iwork < (1u << 20) ? iwork : (1u << 20)) > kBatchItems;
      unsigned long long slot = 0, off = 0;
      if (defer_slots(A.samp_ctr, A.big_cap, iwork >= big_items || (full && iwork >= kBatchItemRow), iwork, &slot,
                      &off)) {
        BigSamp bs;
        bs.off = off;
        bs.rp = erp;
        bs.cv = ecv;
        bs.p0 = ep0;
        bs.u = eu;
        bs.c = ecw;
        bs.J = eJ;
        bs.d = ed;
        bs.items = iwork;
        bs.pad = 0;
        A.samp[slot] = bs;
        iwork = 0;
      }
    }
    long long dtot = 0;  // deterministic pushes of the batch
    if (wave_any(dwork != 0)) {
      const unsigned long long dinc = wave_scan(static_cast<unsigned long long>(dwork));
      B.doff[lane] = static_cast<long long>(dinc) - dwork;
      dtot = static_cast<long long>(last_lane(dinc));
    }
    B.rp[lane] = erp;
    B.cv[lane] = ecv;
    B.p0[lane] = ep0;
    B.u[lane] = eu;
    B.c[lane] = ecw;
    B.d[lane] = ed;
    B.J[lane] = eJ;
    it_next = 0;
    it_total = queue_items(B, iwork);
    // groups where the items' chains are long (single windows of 8 expected
    // draws or more) and at most one per lane, or where there is one per group
    // at most; rows of small probabilities are better off with a lane each (a
    // cluster's estimate on 4e5 nodes 1.82 ms, 3.1 with groups throughout)
    if (few && first_batch) {
      const uint32_t chains = wave_sum_all(((ecw >> kBatchShiftBit) & 7u) == 0u ? iwork : 0u);
      group = it_total <= static_cast<uint32_t>(kWave / kGroup) ||
              (it_total <= static_cast<uint32_t>(kWave) && 2u * chains > it_total);
    }
    first_batch = false;
    wave_sync();
    // deterministic pushes of the batch: the increment reaches theta
    for (long long kb = 0; kb < dtot; kb += kWave) {
      const long long k = kb + lane;
      bool emit = false;
      uint32_t v = 0, vc = 0;
      Delta delta{};
      if (k < dtot) {
        const int e = batch_find<long long>(B.doff, k);
        const int64_t arc = B.rp[e] + (k - B.doff[e]);
        const uint32_t cw = B.c[e];
        vc = cw & kBatchCol;
        const ColParams* cpd = A.cp + vc;
        v = A.col[arc];
        double inc = B.cv[e];
        if (kServe ? !(cw & kBatchAZero) : kMode == kBatchAP)
          inc = inc * (A.arcfac != nullptr ? A.arcfac[arc] : (kServe ? cpd->da : A.da)[A.nd[arc]]);
        T val = to_w(inc, T());
        if (cw & kBatchNeg) val = -val;
        emit = P::to_units(val, *cpd, &delta);
        if (!emit) atomicOr(A.err + (kServe ? vc : 0u), 1);
        if (binned && A.det_bins != nullptr) mark_det_bin<kG>(A, A.det_bins, v, vc);
      }
      emit_atomic(emit, v, vc, delta);
    }
    return true;
  };
  auto served = [&](uint32_t c, uint32_t cand, uint32_t acc, uint32_t runs) {
    if (kServe) serve_item(A, s_serve, c, cand, acc, runs);
  };
  sample_loop<kMode>(A, B, refill, emit_sampled, served, kMode == kBatchAZ && !few ? kRefillIdle : 1, group, w_cand, w_acc,
                     w_runs);
  if (sparse) stage_flush(stage, staged, A.fout, A.cnt_out);
  if (binned) finish_records<kG>(A, s_hist, reinterpret_cast<uint32_t*>(stage), staged, seg, acc_next);
  if (kServe) {  // flush the block's per-column sums
    __syncthreads();
    for (int i = threadIdx.x; i < kServeLdsSlots && i < A.slots; i += blockDim.x) serve_flush(serve_row(A, i), s_serve[i]);
  }
  if (!kServe) {  // per-level counters: the block's sums, one row of atomics
    const unsigned long long v1 = wave_sum_u64(n_hash);
    const unsigned long long v2 = wave_sum_u64(n_det);
    double m = mass;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m += __shfl_down(m, off);
    // (a wave's batch is no longer read: its row starts go to the other waves)
    unsigned long long* mine = reinterpret_cast<unsigned long long*>(B.rp);
    if (lane == 0) {
      mine[0] = w_front;
      mine[1] = v1;
      mine[2] = v2;
      mine[3] = w_cand;
      mine[4] = w_acc;
      mine[5] = w_runs;
      mine[kCountMass] = static_cast<unsigned long long>(__double_as_longlong(m));
    }
    __syncthreads();
    if (threadIdx.x <= kCountMass) {
      unsigned long long* row = count_row(A);
      const int k = threadIdx.x;
      if (k == kCountMass) {
        double sum = 0.0;
        for (int w = 0; w < kWaves; ++w)
          sum += __longlong_as_double(reinterpret_cast<const long long*>(s_batch[w].rp)[k]);
        if (sum != 0.0) atomicAdd(reinterpret_cast<double*>(row + k), sum);
      } else {
        unsigned long long sum = 0;
        for (int w = 0; w < kWaves; ++w) sum += reinterpret_cast<const unsigned long long*>(s_batch[w].rp)[k];
        if (sum) atomic_add_relaxed(row + k, sum);
      }
    }
  }
}

// ------------------------------------------------- deferred rows
// The deterministic pushes of the rows a level deferred, after its k_level
// launch: a wave takes a chunk of consecutive pushes of the concatenated rows
// (lane l pushes l, l + 64, ...), finds its row once by binary search over
// the rows' offsets and moves to the next row when it crosses its end.  The
// pushes are computed and accumulated as in k_level (first contributions of
// a sparse level appended to the next frontier).
template <typename T, int kMode, int kG = 1>
__global__ __launch_bounds__(kThreads) void k_det_big(LevelArgs A, typename Prec<T>::Cell* __restrict__ acc_next) {
  using P = Prec<T>;
  using Delta = typename P::Delta;
  constexpr bool kServe = kMode == kPerColumn;
  constexpr int kWaves = kThreads / kWave;
  __shared__ uint64_t s_stage[kWaves][kStage];
  const unsigned long long ctr = *A.big_ctr;
  unsigned long long nb = ctr >> kBigShift;
  if (nb == 0) return;
  if (nb > A.big_cap) nb = A.big_cap;  // rows beyond the list were pushed by their waves
  const BigRow* R = A.big;
  const unsigned long long total = R[nb - 1].off + R[nb - 1].J;
  if (!kServe) acc_next += (blockIdx.x & A.rep_mask) * A.rep_stride;
  const bool sparse = *A.mode_out == kModeSparse;
  uint8_t* const det_bins = *A.mode_out == kModeBinned ? A.det_bins : nullptr;
  const int lane = lane_id();
  const int wave = static_cast<int>(uniform(threadIdx.x / kWave));
  uint64_t* stage = s_stage[wave];
  int staged = 0;  // wave-uniform
  // a chunk of pushes per wave: as many as give every wave one, in whole
  // steps of 64, at most kBigChunk
  const unsigned long long nw = static_cast<unsigned long long>(gridDim.x) * kWaves;
  unsigned long long chunk = ((total + nw - 1) / nw + kWave - 1) & ~static_cast<unsigned long long>(kWave - 1);
  if (chunk > kBigChunk) chunk = kBigChunk;
  const unsigned long long nchunks = (total + chunk - 1) / chunk;
  for (unsigned long long ch = static_cast<unsigned long long>(blockIdx.x) * kWaves + wave; ch < nchunks; ch += nw) {
    unsigned long long k = ch * chunk + lane;
    unsigned long long e = 0, hi = nb;  // last row with off <= k
    while (hi - e > 1) {
      const unsigned long long mid = (e + hi) >> 1;
      if (R[mid].off <= k)
        e = mid;
      else
        hi = mid;
    }
    unsigned long long off = R[e].off, next = e + 1 < nb ? R[e + 1].off : total;
    for (unsigned long long j = 0; j < chunk; j += kWave, k += kWave) {
      bool emit = false;
      uint32_t v = 0, vc = 0;
      Delta delta{};
      if (k < total) {
        while (k >= next) {
          ++e;
          off = next;
          next = e + 1 < nb ? R[e + 1].off : total;
        }
        const BigRow& br = R[e];
        vc = br.c & kBatchCol;
        const ColParams* cpd = A.cp + vc;
        const int64_t arc = br.rp + static_cast<int64_t>(k - off);
        v = A.col[arc];
        double inc = br.cv;
        if (kServe ? !(br.c & kBatchAZero) : kMode == kBatchAP)
          inc = inc * (A.arcfac != nullptr ? A.arcfac[arc] : (kServe ? cpd->da : A.da)[A.nd[arc]]);
        T val = to_w(inc, T());
        if (br.c & kBatchNeg) val = -val;
        emit = P::to_units(val, *cpd, &delta);
        if (!emit) atomicOr(A.err + (kServe ? vc : 0u), 1);
      }
      if (emit && det_bins != nullptr) mark_det_bin<kG>(A, det_bins, v, vc);
      push_atomic<T, kMode>(A, stage, staged, sparse, emit, v, vc, delta, acc_next);
    }
  }
  if (sparse) stage_flush(stage, staged, A.fout, A.cnt_out);
}

// The sampled work items of the entries a level deferred, after its k_level
// launch: every wave takes the same number of consecutive items (an item is
// about the same number of draws whatever its entry), finds its first entry
// by binary search over the entries' item offsets, loads up to 64 entries at
// a time into its batch and draws their items exactly as k_level does (the
// same runs, draws and acceptance tests, so the same pushes); the pushes are
// emitted as in k_level's mode for the level (records, first-touch appends or
// plain atomics), and the level's candidate and acceptance counters get this
// kernel's counts.
template <typename T, int kMode, int kG = 1>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_samp_big(
    LevelArgs A, typename Prec<T>::Cell* __restrict__ acc_next) {
  using P = Prec<T>;
  using Delta = typename P::Delta;
  constexpr bool kServe = kMode == kPerColumn;
  constexpr int kWaves = kThreads / kWave;
  __shared__ BatchLds s_batch[kWaves];
  __shared__ uint64_t s_stage[kWaves][kStage];
  __shared__ unsigned int s_hist[kServe ? 1 : kBuckets];
  __shared__ ServeSums s_serve[kServe ? kServeLdsSlots : 1];
  const unsigned long long ctr = *A.samp_ctr;
  unsigned long long nb = ctr >> kBigShift;
  if (nb == 0) return;  // the whole grid
  if (nb > A.big_cap) nb = A.big_cap;  // entries beyond the list kept their items
  const BigSamp* R = A.samp;
  const unsigned long long total = R[nb - 1].off + R[nb - 1].items;
  if (!kServe) acc_next += (blockIdx.x & A.rep_mask) * A.rep_stride;
  const int mode = *A.mode_out;
  const bool binned = mode == kModeBinned;
  const bool sparse = mode == kModeSparse;
  if (binned) {
    for (int i = threadIdx.x; i < kBuckets; i += blockDim.x) s_hist[i] = 0;
    __syncthreads();
  }
  if (kServe) {
    for (int i = threadIdx.x; i < kServeLdsSlots; i += blockDim.x) s_serve[i] = ServeSums{};
    __syncthreads();
  }
  const int lane = lane_id();
  const int wave = static_cast<int>(uniform(threadIdx.x / kWave));
  BatchLds& B = s_batch[wave];
  uint64_t* stage = s_stage[wave];
  int staged = 0;  // wave-uniform
  int seg = (blockIdx.x * kWaves + wave) & (kRecSegs - 1);  // wave-uniform: the next flush's record segment
  uint32_t w_cand = 0, w_acc = 0, w_runs = 0;

  // items [i0, i1) of this wave, from entry e on
  const unsigned long long nw = static_cast<unsigned long long>(gridDim.x) * kWaves;
  const unsigned long long per = (total + nw - 1) / nw;
  unsigned long long i0 = (static_cast<unsigned long long>(blockIdx.x) * kWaves + wave) * per;
  const unsigned long long i1 = i0 + per < total ? i0 + per : total;
  unsigned long long e = 0;
  if (i0 < i1) {
    unsigned long long hi = nb;  // last entry with off <= i0
    while (hi - e > 1) {
      const unsigned long long mid = (e + hi) >> 1;
      if (R[mid].off <= i0)
        e = mid;
      else
        hi = mid;
    }
  }
  auto refill = [&](uint32_t& it_next, uint32_t& it_total) -> bool {
    if (i0 >= i1) return false;
    const LevelArgs& A = args_again();
    const BigSamp* const R = A.samp;
    wave_sync();  // every lane has read the previous batch
    const int k = static_cast<int>(nb - e < (unsigned long long)kBatch ? nb - e : kBatch);
    BigSamp bs{};
    if (lane < k) bs = R[e + lane];
    const ColParams& cp = A.cp[bs.c & kBatchCol];
    B.rp[lane] = bs.rp;
    B.cv[lane] = bs.cv;
    B.p0[lane] = bs.p0;
    B.th[lane] = cp.theta;
    B.ctr3[lane] = (cp.qid << 8) | static_cast<uint32_t>(kServe ? cp.level : A.level);
    B.u[lane] = bs.u;
    B.c[lane] = bs.c;
    B.d[lane] = bs.d;
    B.J[lane] = bs.J;
    const uint32_t items = queue_items(B, bs.items);
    wave_sync();
    const unsigned long long first = R[e].off;  // the offsets of consecutive entries are contiguous
    const unsigned long long end = first + items;
    it_next = static_cast<uint32_t>(i0 - first);
    it_total = static_cast<uint32_t>((end < i1 ? end : i1) - first);
    i0 = end < i1 ? end : i1;
    e += static_cast<unsigned long long>(k);
    return true;
  };
  const RecShape shape{pinned(rec_shape<kG>(A).width), pinned(A.bucket_shift)};
  auto emit_sampled = [&](bool emit, uint32_t v, uint32_t cw) {
    if (binned) {
      emit_record<kG>(shape, s_hist, reinterpret_cast<uint32_t*>(stage), staged, seg, emit, v, cw, acc_next);
      return;
    }
    const uint32_t c = cw & kBatchCol;
    Delta delta{};
    if (emit) delta = P::theta_units(A.cp[c], (cw & kBatchNeg) != 0);
    push_atomic<T, kMode>(A, stage, staged, sparse, emit, v, c, delta, acc_next);
  };
  auto served = [&](uint32_t c, uint32_t cand, uint32_t acc, uint32_t runs) {
    if (kServe) serve_item(A, s_serve, c, cand, acc, runs);
  };
  bool group = per <= kGroupItems;
  sample_loop<kMode>(A, B, refill, emit_sampled, served, kMode == kBatchAZ ? kRefillIdle : 1, group, w_cand, w_acc,
                     w_runs);
  if (sparse) stage_flush(stage, staged, A.fout, A.cnt_out);
  if (binned) finish_records<kG>(A, s_hist, reinterpret_cast<uint32_t*>(stage), staged, seg, acc_next);
  if (kServe) {  // flush the block's per-column sums
    __syncthreads();
    for (int i = threadIdx.x; i < kServeLdsSlots && i < A.slots; i += blockDim.x) serve_flush(serve_row(A, i), s_serve[i]);
  } else if (lane == 0) {
    unsigned long long* cnt = count_row(A);
    if (w_cand) atomicAdd(cnt + 3, static_cast<unsigned long long>(w_cand));
    if (w_acc) atomicAdd(cnt + 4, static_cast<unsigned long long>(w_acc));
    if (w_runs) atomicAdd(cnt + 5, static_cast<unsigned long long>(w_runs));
  }
}

// ------------------------------------------------- push estimate
// An upper bound on the pushes of a level (deterministic rows count d_u,
// sampled rows their expected d_u c / theta with c = rho |r| d_u^-b), summed
// over the frontier (over a sample of it when it is large): decides whether
// the level is worth binning.
// One atomic a block on one address, about 10 ns each: few, large blocks.
constexpr int kEstimateThreads = 1024;
constexpr int kEstimateBlocks = 256;

template <typename T, bool kFirst>
__global__ __launch_bounds__(kEstimateThreads) void k_estimate(LevelArgs A, const T* __restrict__ x,
                                                       const typename Prec<T>::Cell* __restrict__ acc_cur,
                                                       double* __restrict__ est) {
  __shared__ double s_part[kEstimateThreads / kWave];
  const unsigned long long count = *A.cnt_in;
  // large frontiers: an evenly spaced sample of 2^20 to 2^21 entries, scaled
  // up (the estimate only chooses between interchangeable aggregation modes)
  const unsigned long long stride = count >= (1ull << 21) ? count >> 20 : 1ull;
  const double rho = A.lp->rho;
  if ((A.lp->flags & kLastLevel) || rho == 0.0) return;
  double sum = 0.0;
  for (unsigned long long j = blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x; j * stride < count;
       j += (unsigned long long)gridDim.x * blockDim.x) {
    uint32_t u, c;
    if (kFirst && A.fin == nullptr) {  // every cell (see kVirtualMaxC)
      const unsigned long long e = j * stride;
      u = static_cast<uint32_t>(e / static_cast<unsigned long long>(A.su));
      c = static_cast<uint32_t>(e - static_cast<unsigned long long>(u) * static_cast<unsigned long long>(A.su));
    } else {
      const uint64_t item = A.fin[j * stride];
      u = static_cast<uint32_t>(item >> 32);
      c = static_cast<uint32_t>(item);
    }
    const ColParams& cp = A.cp[c];
    const uint32_t d = static_cast<uint32_t>(A.deg[u]);
    if (d == 0) continue;
    const size_t cell = static_cast<size_t>(u) * A.su + static_cast<size_t>(c) * A.sc;
    double absr;
    if (kFirst) {
      absr = fabs(static_cast<double>(x[static_cast<size_t>(u) * static_cast<size_t>(A.xld) + c]));
    } else if (sizeof(T) == 4) {
      const long long K = reinterpret_cast<const long long*>(acc_cur)[cell];
      absr = fabs(static_cast<double>(K)) / cp.scale;
    } else {
      absr = 0.0;  // binary64 calls are never binned
    }
    const double cv = rho * absr * A.db[A.fdeg[u]];
    sum += cv >= cp.theta ? static_cast<double>(d) : static_cast<double>(d) * (cv / cp.theta);
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_down(sum, off);
  if (lane_id() == 0) s_part[threadIdx.x / kWave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {  // one atomic per block
    double b = 0.0;
    for (int w = 0; w < kEstimateThreads / kWave; ++w) b += s_part[w];
    if (b != 0.0) atomicAdd(est, b * static_cast<double>(stride));
  }
}

// ------------------------------------------------- frontier compaction
// (u << 32 | c) of every cell u * C + c of a row-major n x C array whose
// predicate holds.  Every chunk that goes out costs one atomic on the list
// counter, a round trip to one shared address that all waves contend for,
// so chunks are made large: a wave takes segments of seg consecutive cells
// (a multiple of kCompactUnroll x 64, at most kCompactSeg: large arrays take
// the largest, small ones smaller segments so that every CU has waves),
// issues kCompactUnroll loads of 64 cells together, and stages the passing
// cells as 2-byte offsets into its segment (up to kCompactCap of them, 8 KiB
// of LDS per wave); a chunk goes out when the stage is nearly full and at the
// end of each segment, in cell order.  Rows and columns of the staged cells
// are formed when they go out, from one 64-bit division per segment and a
// float-reciprocal division corrected to the exact quotient per entry.
constexpr int kCompactUnroll = 16;
constexpr int kCompactCap = 4096;
constexpr long long kCompactSeg = 1ll << 16;  // the largest segment: offsets fit in 16 bits
static_assert(kCompactSeg % (kCompactUnroll * kWave) == 0, "segments hold whole load groups");

// The staged offsets of a segment that starts at row u0, column r0: one
// atomic for the chunk, then the items in staging order.  Wave-uniform.
__device__ __forceinline__ void compact_flush(const uint16_t* stage, int& staged, long long u0, uint32_t r0,
                                              uint32_t C, float rc, bool small, uint64_t* __restrict__ F,
                                              unsigned long long* __restrict__ cnt) {
  if (staged == 0) return;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  unsigned long long base = 0;
  if (lane_id() == 0) base = atomicAdd(cnt, static_cast<unsigned long long>(staged));
  base = uniform(base);
  for (int i = lane_id(); i < staged; i += kWave) {
    const uint32_t a = r0 + stage[i];  // < C + kCompactSeg
    uint32_t c = 0, q = 0;
    if (small) {
      q = div_small(a, C, rc, &c);
    } else {
      q = a / C;
      c = a - q * C;
    }
    F[base + i] = (static_cast<uint64_t>(u0 + q) << 32) | c;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  staged = 0;
}

template <typename Pred>
__global__ __launch_bounds__(kThreads) void k_compact(Pred pred, int64_t n, int C, long long seg,
                                                      uint64_t* __restrict__ F, unsigned long long* __restrict__ cnt,
                                                      const int* __restrict__ mode) {
  if (mode && *mode != kModeCompact && *mode != kModeOverflow) return;  // formed elsewhere
  constexpr int kWaves = kThreads / kWave;
  __shared__ uint16_t s_stage[kWaves][kCompactCap];
  const int lane = lane_id();
  uint16_t* stage = s_stage[threadIdx.x / kWave];
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  const long long total = static_cast<long long>(n) * C;
  const float rc = 1.0f / static_cast<float>(C);
  const bool small = C <= (1 << 21);  // div_small's range: C + kCompactSeg < 2^22
  const long long wave = static_cast<long long>(blockIdx.x) * kWaves + threadIdx.x / kWave;
  const long long nwaves = static_cast<long long>(gridDim.x) * kWaves;
  for (long long base = wave * seg; base < total; base += nwaves * seg) {
    const long long u0 = base / C;
    const uint32_t r0 = static_cast<uint32_t>(base - u0 * C);
    int staged = 0;  // wave-uniform
    for (int j = 0; j < seg && base + j < total; j += kCompactUnroll * kWave) {
      // the index is clamped instead of guarded, so that the loads carry no
      // branch and go out together
      bool p[kCompactUnroll];
#pragma unroll
      for (int k = 0; k < kCompactUnroll; ++k) {
        const long long i = base + j + k * kWave + lane;
        const bool in = i < total;
        p[k] = pred(0, 0, static_cast<size_t>(in ? i : total - 1)) && in;
      }
#pragma unroll
      for (int k = 0; k < kCompactUnroll; ++k) {
        const unsigned long long m = wave_ballot(p[k]);
        if (p[k]) stage[staged + __popcll(m & lt_mask)] = static_cast<uint16_t>(j + k * kWave + lane);
        staged += __popcll(m);
        if (staged > kCompactCap - kWave) compact_flush(stage, staged, u0, r0, C, rc, small, F, cnt);
      }
    }
    compact_flush(stage, staged, u0, r0, C, rc, small, F, cnt);
  }
}

template <typename T>
struct NonZeroCell {
  const typename Prec<T>::Cell* acc;
  __device__ bool operator()(int64_t, int64_t, size_t cell) const { return Prec<T>::nonzero(acc, cell); }
};

inline unsigned grid_for(int64_t items, int threads, int64_t cap = 65536) {
  int64_t b = (items + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return static_cast<unsigned>(b);
}

}  // namespace lvl
}  // namespace agp
