// devtab.h -- device-side problem table and launch arguments (internal).
//
// One table per problem (or per replica in a batch) is a flat array of
// 32-bit words, written by the host into the caller's workspace and read by
// the kernels with uniform (scalar) loads, except the duration table which
// each block stages in LDS because its index depends on the lane.
//
// Tools are stored under internal labels 0..N-1 that follow a topological
// order of the DAG (every predecessor has a smaller label), so one ascending
// sweep over the labels sees each tool after all of its predecessors.  The
// mapping index keeps the caller's tool numbering: it is mixed radix, digit v
// being the rank of original tool v's mode among the r_v modes allowed to it
// (r_v = 3 when all are), with weight W_v = r_0 r_1 ... r_(v-1).  Tools with a
// single allowed mode take no digit: their mode is fixed in the header.
#pragma once
#include <stdint.h>

namespace devmap {

constexpr int kMaxTools = 40;
constexpr int kMaxLevels = 64;
constexpr uint32_t kInf = 0xFFFFFFFFu;  // "never": unknown ready time, infeasible
constexpr int kBlock = 256;             // threads per search block (4 waves)
constexpr int kMaxInnerDigits = 6;      // inner (wave-uniform) digits per lane
#ifndef DEVMAP_SHARED_INNER
#define DEVMAP_SHARED_INNER 2
#endif
constexpr uint32_t kSharedInner = DEVMAP_SHARED_INNER;  // inner digits of a shared-prefix search
// Variants of the fixed-at-start shared-prefix search for spaces without
// gpu_queue (the GPU/CPU spaces): a pass then has no queue to look after, and
// (kVarFree: the budget holds every footprint together) no VRAM to sum.  Built
// from kVarMinN tools: below, such a space has too few mappings for shared
// prefixes to fill the GPU.  Mixed DAGs of 22, 26 and 32 tools (2^21 to 2^30
// mappings) without a budget: 152 us, 2.35 ms, 76.1 ms, against 190 us, 2.86
// ms, 88.5 ms.  Three inner digits, to share a prefix among 8 combinations in
// place of 4, helped some DAGs (26 tools 2.16 ms) and cost others more (22
// tools 314 us, 32 tools 99.6 ms).
enum : int { kVarAll = 0, kVarNoQueue = 1, kVarFree = 2 };
constexpr int kVarMinN = 21;
constexpr int kPrefixMaxN = 32;         // tool counts served by shared prefixes (fixed at start:
                                        // N LDS words per lane)
constexpr int kPrefixMaxNShare = 24;    // the same under processor sharing (1.5N words per lane)
// From this many tools a fixed-at-start shared-prefix search needs its inner
// tools on the last kSharedInner labels: their words (0 whenever a prefix
// saves its state) are left out of the LDS column, so that N - kSharedInner
// words per lane leave room for 5 blocks per CU up to kPrefixMaxN tools.
constexpr int kCompactSnapN = 27;
static_assert(kCompactSnapN > kPrefixMaxNShare, "the compact column is fixed-at-start only");

// Header words.
enum : uint32_t {
  kHdrN = 0,          // number of tools
  kHdrLevels = 1,     // contention levels stored = min(K, N)
  kHdrBudget = 2,     // VRAM budget, clamped to the summed footprint
  kHdrBigLo = 3,      // tools whose footprint exceeds the budget (bits 0..31)
  kHdrBigHi = 4,      //                                           (bits 32..63)
  kHdrDurOff = 5,     // word offset of the duration table
  kHdrPositions = 6,  // P: tools with more than one allowed mode (digit positions)
  kHdrFixGnLo = 7,    // labels of tools fixed on gpu_now (bits 0..31)
  kHdrFixGnHi = 8,    //                                   (bits 32..63)
  kHdrFixGqLo = 9,    // labels of tools fixed on gpu_queue
  kHdrFixGqHi = 10,
  kHdrBoundOff = 11,  // word offset of the bound table
  kHdrShareOff = 12,  // word offset of the processor-sharing table
  kHdrFlags = 13,     // kFlag* bits
  kHdrDeferLo = 14,   // inner tools of a shared-prefix search that are sinks with
  kHdrDeferHi = 15,   // predecessors: the search defers them (bits 0..31, 32..63)
  // The walk of a full-order search over this table: which outer combinations
  // it covers and how (see SearchArgs, whose fields of the same names these
  // are).  In the table, so that one launch can serve tables of different sizes.
  kHdrOuterLoLo = 16,
  kHdrOuterLoHi = 17,
  kHdrNOuterLo = 18,
  kHdrNOuterHi = 19,
  kHdrInnerDigits = 20,
  kHdrInnerCount = 21,
  kHdrPrefix = 22,
  // The outer combinations of a walk may come from a list of (bound, y) pairs
  // (its device address; 0: none): the outer combination numbered k then has
  // the digits of k mod kHdrListRest, and above them those of y of entry
  // k / kHdrListRest.
  kHdrListLo = 23,
  kHdrListHi = 24,
  kHdrListRest = 25,
  // Bounds of the children of listed assignments (device address; 0: of all
  // assignments): the one numbered k extends y of entry k / kHdrChildren by the
  // digits of k mod kHdrChildren, above the kHdrParents assignments there are.
  kHdrParentLo = 26,
  kHdrParentHi = 27,
  kHdrParents = 28,
  kHdrChildren = 29,
  kHdrLanes = 30,     // lanes per wave that take an outer combination (SearchArgs::lanes)
  kHdrWords = 32,     // (one to spare: the tool records start on a 128-byte line)
};

// A fan-out (no edges) whose footprints all fit the budget together, scored
// with fixed-at-start contention: every tool is ready at 0, no start can run
// out of memory and no queued tool waits for VRAM, so a mapping's schedule
// follows in closed form (evaluate_fanout).  Its internal labels are the
// original tool numbers.
constexpr uint32_t kFlagFreeFanout = 1u;

// Full-order searches in closed form (closed.hip), by the kind of problem: a
// fan-out as above with at most four contention levels, or a serial chain (the
// tool with label i depends on the tool with label i - 1 alone) scored with
// fixed-at-start contention.  The combinations of the last kClosedInner labels
// (or fewer) are walked per lane.
enum : uint32_t { kClosedNone = 0, kClosedChain = 1, kClosedFanout = 2 };
constexpr uint32_t kClosedInner = 5;
constexpr uint32_t kClosedInnerMost = 243;  // 3^kClosedInner
constexpr int kClosedFanoutTools = 32;
constexpr uint32_t kClosedFanoutLevels = 4;

// Record of the tool with internal label i at kHdrWords + kToolWords * i.
enum : uint32_t {
  kToolCpu = 0,       // cpu_us
  kToolMem = 1,       // footprint, clamped to budget + 1
  kToolXfer = 2,      // input transfer across devices
  kToolPredLo = 3,    // predecessor mask bits 0..31
  kToolPredHi = 4,    // predecessor mask bits 32..63
  kToolOrig = 5,      // (original tool number << kOrigLabelBits) | label
  kToolWords = 6,
};

// kToolOrig holds the original number above the label, so that the lowest
// word among candidate tools names both the first in the queue's tie order and
// its label.
constexpr uint32_t kOrigLabelBits = 6;
constexpr uint32_t kOrigLabelMask = (1u << kOrigLabelBits) - 1u;
static_assert(kMaxTools <= (1 << kOrigLabelBits), "labels must fit below the original number");

// A table is laid out for n tools: those of its problem, or more where
// problems of several sizes share one launch (a kernel for n tools then runs
// a smaller problem with tools n_tools..n-1 on the CPU, of no length).  The
// layout is as short as the problem allows, so that one table travels in a
// kernel's arguments (TableArg).
//
// pos[v]: internal label of original tool v.
constexpr uint32_t pos_base(uint32_t n) { return kHdrWords + kToolWords * n; }
// Enumeration order of a search over positions 0..P-1: position p holds the
// digit of the tool with internal label elab[p], whose weight in the mapping
// index is ew[p] = W_v of its original number v (two words, low first), and
// whose options eo[p] give its radix (bits 0-1, 2 or 3) and the mode of
// digit d in bits 2+2d..3+2d.  Positions 0..J-1 are the inner digits, J.. the
// outer ones.
constexpr uint32_t enum_lab_base(uint32_t n) { return pos_base(n) + n; }
constexpr uint32_t enum_weight_base(uint32_t n) { return enum_lab_base(n) + n; }
constexpr uint32_t enum_opt_base(uint32_t n) { return enum_weight_base(n) + 2u * n; }
// The duration table follows.
constexpr uint32_t dur_base(uint32_t n) { return enum_opt_base(n) + n; }

// Radix and digit -> mode of an enumeration position's options word.
inline constexpr uint32_t opt_radix(uint32_t o) { return o & 3u; }
inline constexpr uint32_t opt_mode(uint32_t o, uint32_t d) { return (o >> (2u + 2u * d)) & 3u; }

// Duration table: dur[(i * 2 + q) * levels + (level - 1)] for internal label
// i, q = 0 for gpu_now (base gpu_us), q = 1 for gpu_queue (gpu_us + load_us).
//
// Processor-sharing table (after the duration table): for internal label i,
// b[2i] = gpu_us and b[2i + 1] = gpu_us + load_us (isolated latencies), then
// for each contention level the work rate w = round(2^32 / F) in 2^-16 us of
// isolated work per us, then for each level floor(2^48 / w) (two words, low
// first), the reciprocal the device divides by.
//
// Bound table (last; only the bound kernel and the host read it): for internal
// label i, four words bt[4i + m] = the shortest duration tool i can have in
// mode m (cpu, gpu_now, gpu_queue: the least over contention levels), and
// bt[4i + 3] = the least of those over the modes the problem allows it; kInf
// for a GPU mode of a tool whose footprint exceeds the budget (it can never
// run there).
constexpr uint32_t kBoundWords = 4;

constexpr uint32_t share_base(uint32_t n, uint32_t levels) {
  return dur_base(n) + n * 2u * levels;
}
constexpr uint32_t bound_base(uint32_t n, uint32_t levels) {
  return share_base(n, levels) + 2u * n + 3u * levels;
}
constexpr uint32_t table_words(uint32_t n, uint32_t levels) {
  return bound_base(n, levels) + kBoundWords * n;
}

// One table (without its bound table) in a kernel's arguments, which saves a
// small call its copy to the device.
constexpr uint32_t kArgWords = 960;
struct TableArg {
  uint32_t w[kArgWords];
};

struct Partial {
  uint64_t index;
  uint32_t makespan;
  uint32_t pad;
};

struct DevResult {
  uint64_t index;
  int64_t makespan;
};

struct SearchArgs {
  const uint32_t* tables;     // n_tables tables, table_stride words apart; null: one table,
                              // in the kernel's arguments
  const uint32_t* host_table; // that table on the host, host_words of it
  Partial* partials;          // one per block
  DevResult* results;         // one per table, or one for all of them (one_result); null:
                              // the caller reduces the partials
  const uint32_t* block_first;  // n_tables + 1 entries: the first block of each table, then
                              // the number of blocks; null: blocks_per_table each
  uint64_t lo, hi;            // index range searched in every table
  uint64_t outer_lo;          // first outer combination
  uint64_t n_outer;           // outer combinations covering [lo, hi)
  uint32_t table_stride;
  uint32_t host_words;
  uint32_t n_tables;
  uint32_t inner_digits;      // J: enumeration positions 0..J-1 are walked per lane
  uint32_t inner_count;       // product of the radices of positions 0..J-1
  uint64_t items_per_table;   // ceil(n_outer / kBlock)
  uint32_t blocks_per_table;
  uint32_t full_range;        // 1: the tables' own walks, any enumeration order (lo and hi
                              //    are not read)
  uint32_t sharing;           // 1: processor-sharing contention
  uint32_t prefix;            // 1: shared prefixes (kSharedInner inner digits on the
                              //    deepest tools, full range, fixed at start)
  uint32_t lds_levels;        // the most contention levels any of the tables stores
  uint32_t n_blocks;          // blocks of the launch
  uint32_t closed;            // kClosed*: all tables are of this kind; inner_digits is then the
                              // number of last labels walked per lane
  int32_t variant;            // kVar*
  uint32_t lanes;             // lanes per wave that take an outer combination: all 64, or fewer
                              // where the GPU has waves to spare
  uint32_t thin;              // 1: shared prefixes as with prefix, but in such waves
  uint32_t one_result;        // 1: the tables are parts of one search, results has one entry
  uint32_t* record;           // full range, one table: every scored mapping's makespan
                              // (kInf if infeasible) goes to record[index]; null: none
};

// Scoring of explicit indices.
struct EvalArgs {
  const uint32_t* tab;        // null: the table in the kernel's arguments
  const uint64_t* idx;
  int64_t n;
  uint64_t n_mappings;
  int64_t* out;
};
enum : uint32_t {
  kEvalSharing = 1u,          // processor sharing
  kEvalHostTable = 2u,        // tab is the host's table, to go into the kernel's arguments
};

}  // namespace devmap
