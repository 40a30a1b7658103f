// api.cpp -- the C ABI of include/sched_search.h: validation, topological checks,
// device problem tables, work planning, launches and result copies.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <numeric>
#include <optional>
#include <vector>

#include "sched_search.h"
#include "devtab.h"
#include "launch.h"

using namespace devmap;

struct sched_problem {
  int32_t n = 0;
  std::vector<sched_tool> tools;
  std::vector<std::vector<int32_t>> preds;  // ascending, deduplicated
  std::vector<int32_t> order;               // order[i]: original tool with internal label i
  std::vector<int32_t> late;                // tools from the deepest in the DAG to the shallowest
  std::vector<uint32_t> contention;         // F[k-1]
  std::vector<uint8_t> allowed;             // per tool: bit m set if mode m is allowed
  std::vector<uint8_t> radix;               // number of allowed modes
  std::vector<uint64_t> weight;             // W_v: product of the radices of tools < v
  std::vector<int32_t> enum_tools;          // tools with radix > 1, ascending
  int64_t budget = 0;
  int32_t sharing = 0;                      // 1: processor-sharing contention
  bool free_fanout = false;                 // no edges, all footprints fit (kFlagFreeFanout)
  uint32_t closed = kClosedNone;            // kind of closed form, if any
  int32_t variant = kVarAll;                // of a shared-prefix search (kVar*)
  uint64_t n_mappings = 0;
  uint32_t table_words = 0;
  std::vector<uint32_t> table;       // device image with the problem's own latencies
  std::vector<uint32_t> table_full;  // the same, ordered for a one-table full-range search
};

namespace {

constexpr uint32_t kMaxBlocks = 65536;       // cap on search blocks per call
constexpr uint64_t kTargetLanes = 1ull << 19;  // lanes that fill an MI355X
constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) & ~(kAlign - 1); }

// Mode of digit d of tool v (the d-th allowed mode, ascending).
int mode_of_digit(const sched_problem& p, int v, int d) {
  for (int m = 0; m < 3; ++m)
    if ((p.allowed[v] >> m) & 1) {
      if (d == 0) return m;
      --d;
    }
  return -1;
}

// Digit of mode m of tool v, or -1 if m is not allowed.
int digit_of_mode(const sched_problem& p, int v, int m) {
  if (m < 0 || m > 2 || !((p.allowed[v] >> m) & 1)) return -1;
  int d = 0;
  for (int k = 0; k < m; ++k) d += (p.allowed[v] >> k) & 1;
  return d;
}

// Options word of tool v's enumeration position: radix, then the mode of
// each digit.
uint32_t options_word(const sched_problem& p, int v) {
  uint32_t o = p.radix[v];
  for (int d = 0; d < p.radix[v]; ++d) o |= uint32_t(mode_of_digit(p, v, d)) << (2 + 2 * d);
  return o;
}

// round(b * f / 2^16), halves up, in 128-bit arithmetic where 64 bits do not
// hold the product (f <= 2^24).
uint64_t scale_q16(uint64_t b, uint32_t f) {
  if (b < (1ull << 39)) return (b * f + 32768u) >> 16;
  unsigned __int128 p = (unsigned __int128)b * f + 32768u;
  unsigned __int128 r = p >> 16;
  return r > ~0ull ? ~0ull : uint64_t(r);
}

int check_latencies(int64_t gpu, int64_t cpu, int64_t load, int64_t xfer) {
  if (gpu < 1 || cpu < 1 || load < 0 || xfer < 0) return SCHED_E_VALUE;
  return SCHED_OK;
}

// The tools a shared-prefix search defers (header words kHdrDefer*): those
// of its inner positions 0..kSharedInner-1 that are sinks with predecessors.
// Reads the predecessor masks, the tool count and the enumeration already in
// the table.
static void write_deferred(uint32_t* table) {
  const int n = int(table[kHdrN]);
  uint64_t has_succ = 0, has_pred = 0;
  for (int i = 0; i < n; ++i) {
    const uint32_t* rec = table + kHdrWords + kToolWords * uint32_t(i);
    const uint64_t pm = uint64_t(rec[kToolPredLo]) | (uint64_t(rec[kToolPredHi]) << 32);
    has_succ |= pm;
    if (pm) has_pred |= 1ull << i;
  }
  uint64_t inner = 0;
  for (uint32_t j = 0; j < kSharedInner; ++j)
    inner |= 1ull << table[enum_lab_base(uint32_t(n)) + j];
  const uint64_t d = inner & ~has_succ & has_pred;
  table[kHdrDeferLo] = uint32_t(d);
  table[kHdrDeferHi] = uint32_t(d >> 32);
}

// A sequence of tools (an enumeration order) held without heap memory, so
// that planning a search allocates nothing.
struct Seq {
  int32_t v[kMaxTools];
  int n = 0;
  void push_back(int32_t x) { v[n++] = x; }
  int size() const { return n; }
  int32_t operator[](int k) const { return v[k]; }
};

// Write the enumeration order seq[0..n) into a table whose tools are in place.
void set_enumeration(const sched_problem& p, const int32_t* seq, int n, uint32_t* table) {
  const uint32_t lay = table[kHdrN];
  for (int k = 0; k < n; ++k) {
    const int v = seq[k];
    table[enum_lab_base(lay) + k] = table[pos_base(lay) + v];
    table[enum_weight_base(lay) + 2 * k] = uint32_t(p.weight[v]);
    table[enum_weight_base(lay) + 2 * k + 1] = uint32_t(p.weight[v] >> 32);
    table[enum_opt_base(lay) + k] = options_word(p, v);
  }
  write_deferred(table);
}

void set_enumeration(const sched_problem& p, const Seq& seq, uint32_t* table) {
  set_enumeration(p, seq.v, seq.n, table);
}

void set_enumeration(const sched_problem& p, const std::vector<int32_t>& seq, uint32_t* table) {
  set_enumeration(p, seq.data(), int(seq.size()), table);
}

// Contention levels stored in a problem's table.
uint32_t table_levels(const sched_problem& p) {
  return uint32_t(std::min<int>(int(p.contention.size()), p.n));
}

// The words of a table that depend on latencies (lat; nullptr: the problem's
// own): cpu_us and xfer_us, the duration and processor-sharing tables, and the
// bound table if asked for.  The rest of the table is in place (lay_table).
// Returns SCHED_E_VALUE, or SCHED_E_OVERFLOW when the 32-bit guards fail.
int fill_latencies(const sched_problem& p, const sched_lat* lat, uint32_t* out, bool bounds) {
  const int n = p.n;
  const uint32_t lay = out[kHdrN], levels = out[kHdrLevels];
  const uint32_t dur_off = out[kHdrDurOff], share_off = out[kHdrShareOff];
  const uint64_t big = uint64_t(out[kHdrBigLo]) | (uint64_t(out[kHdrBigHi]) << 32);
  unsigned __int128 bound = 0;  // worst-case makespan: sum of longest durations + transfers
  for (int i = 0; i < n; ++i) {
    const int v = p.order[i];
    const sched_tool& tl = p.tools[v];
    const int64_t gpu = lat ? lat[v].gpu_us : tl.gpu_us;
    const int64_t cpu = lat ? lat[v].cpu_us : tl.cpu_us;
    const int64_t load = lat ? lat[v].load_us : tl.load_us;
    const int64_t xfer = lat ? lat[v].xfer_us : tl.xfer_us;
    if (check_latencies(gpu, cpu, load, xfer) != SCHED_OK) return SCHED_E_VALUE;

    uint64_t longest = uint64_t(cpu);
    for (int q = 0; q < 2; ++q) {
      const uint64_t base = q == 0 ? uint64_t(gpu) : uint64_t(gpu) + uint64_t(load);
      for (uint32_t l = 0; l < levels; ++l) {
        const uint64_t d = scale_q16(base, p.contention[l]);
        longest = std::max(longest, d);
        out[dur_off + (uint32_t(i) * 2u + uint32_t(q)) * levels + l] =
            d < (1ull << 31) ? uint32_t(d) : 0u;
      }
    }
    bound += (unsigned __int128)longest + (unsigned __int128)uint64_t(xfer);
    if (bound >= ((unsigned __int128)1 << 30)) return SCHED_E_OVERFLOW;
    uint32_t* rec = out + kHdrWords + kToolWords * uint32_t(i);
    rec[kToolCpu] = uint32_t(cpu);
    rec[kToolXfer] = uint32_t(xfer);
    out[share_off + 2 * uint32_t(i)] = uint32_t(gpu);
    out[share_off + 2 * uint32_t(i) + 1] = uint32_t(gpu + load);
  }
  if (!bounds) return SCHED_OK;
  // Bound table: shortest durations per mode and over the allowed modes.
  // Fixed at start, a GPU task lasts one of its scaled durations; under
  // processor sharing at least its work over the fastest rate.
  const uint32_t bound_off = out[kHdrBoundOff];
  for (int i = 0; i < n; ++i) {
    const int v = p.order[i];
    uint32_t best[3] = {out[kHdrWords + kToolWords * uint32_t(i) + kToolCpu], kInf, kInf};
    if (!((big >> i) & 1))
      for (int q = 0; q < 2; ++q)
        for (uint32_t l = 0; l < levels; ++l) {
          uint32_t d = out[dur_off + (uint32_t(i) * 2u + uint32_t(q)) * levels + l];
          if (p.sharing) {
            const uint64_t work = uint64_t(out[share_off + 2 * uint32_t(i) + uint32_t(q)]) << 16;
            const uint64_t w = out[share_off + 2 * lay + l];
            d = uint32_t((work + w - 1) / w);
          }
          best[1 + q] = std::min(best[1 + q], d);
        }
    uint32_t any = kInf;
    for (int m = 0; m < 3; ++m) {
      out[bound_off + kBoundWords * uint32_t(i) + m] = best[m];
      if ((p.allowed[v] >> m) & 1) any = std::min(any, best[m]);
    }
    out[bound_off + kBoundWords * uint32_t(i) + 3] = any;
  }
  return SCHED_OK;
}

// The words of problem p's table, laid out for `lay` tools (at least its own),
// that do not depend on latencies; the others are 0.  Returns
// SCHED_E_OVERFLOW when the 32-bit guard of VRAM sums fails.
int lay_table(const sched_problem& p, uint32_t lay, uint32_t* out) {
  const int n = p.n;
  const uint32_t levels = table_levels(p);
  std::memset(out, 0, sizeof(uint32_t) * table_words(lay, levels));

  int64_t sum_mem = 0;
  for (const auto& t : p.tools) sum_mem += t.mem_mib;
  const int64_t budget = std::min<int64_t>(p.budget, sum_mem);
  // VRAM sums of up to N footprints (each clamped to budget+1) plus the
  // budget must stay below 2^32.
  if ((unsigned __int128)(n + 1) * (unsigned __int128)(budget + 1) >= ((unsigned __int128)1 << 32))
    return SCHED_E_OVERFLOW;

  int32_t label[kMaxTools];
  for (int i = 0; i < n; ++i) label[p.order[i]] = i;
  uint64_t big = 0;
  for (int i = 0; i < n; ++i) {
    const int v = p.order[i];
    const sched_tool& tl = p.tools[v];
    uint32_t* rec = out + kHdrWords + kToolWords * uint32_t(i);
    rec[kToolMem] = uint32_t(std::min<int64_t>(tl.mem_mib, budget + 1));
    uint64_t pm = 0;
    for (int32_t u : p.preds[v]) pm |= 1ull << label[u];
    rec[kToolPredLo] = uint32_t(pm);
    rec[kToolPredHi] = uint32_t(pm >> 32);
    rec[kToolOrig] = (uint32_t(v) << kOrigLabelBits) | uint32_t(i);
    out[pos_base(lay) + uint32_t(v)] = uint32_t(i);
    if (tl.mem_mib > budget) big |= 1ull << i;
  }
  // Index order: position k holds the k-th tool with a choice; the others
  // are fixed in the header.
  uint64_t fix_gn = 0, fix_gq = 0;
  for (int v = 0; v < n; ++v)
    if (p.radix[v] == 1) {
      const int m = mode_of_digit(p, v, 0);
      if (m == 1) fix_gn |= 1ull << label[v];
      if (m == 2) fix_gq |= 1ull << label[v];
    }
  out[kHdrN] = lay;
  out[kHdrLevels] = levels;
  out[kHdrBudget] = uint32_t(budget);
  out[kHdrBigLo] = uint32_t(big);
  out[kHdrBigHi] = uint32_t(big >> 32);
  out[kHdrDurOff] = dur_base(lay);
  out[kHdrPositions] = uint32_t(p.enum_tools.size());
  out[kHdrFixGnLo] = uint32_t(fix_gn);
  out[kHdrFixGnHi] = uint32_t(fix_gn >> 32);
  out[kHdrFixGqLo] = uint32_t(fix_gq);
  out[kHdrFixGqHi] = uint32_t(fix_gq >> 32);
  out[kHdrShareOff] = share_base(lay, levels);
  out[kHdrBoundOff] = bound_base(lay, levels);
  out[kHdrFlags] = p.free_fanout ? kFlagFreeFanout : 0u;
  set_enumeration(p, p.enum_tools, out);
  // Processor sharing: the work rate of each contention level, round(2^32 / F)
  // halves up, and floor(2^48 / w): the device divides by w through this
  // reciprocal.
  uint32_t* const rates = out + share_base(lay, levels) + 2 * lay;
  for (uint32_t l = 0; l < levels; ++l) {
    const uint64_t f = p.contention[l];
    const uint64_t w = ((1ull << 33) + f) / (2 * f);
    rates[l] = uint32_t(w);
    const uint64_t winv = (1ull << 48) / w;
    rates[levels + 2 * l] = uint32_t(winv);
    rates[levels + 2 * l + 1] = uint32_t(winv >> 32);
  }
  return SCHED_OK;
}

// The table of problem p with latencies lat (nullptr: the problem's own).
int build_table(const sched_problem& p, const sched_lat* lat, uint32_t* out) {
  const int rc = lay_table(p, uint32_t(p.n), out);
  return rc != SCHED_OK ? rc : fill_latencies(p, lat, out, true);
}

// Relabel p so that the first kSharedInner tools with a choice in p.late
// (a shared-prefix search's inner digits) take the last labels, when no other
// tool depends on them: Kahn's algorithm over the other tools, lowest number
// first, then the inner tools in topological order among themselves.
// Otherwise p.order stays as it is.
static void label_inner_last(sched_problem& p) {
  const int n = p.n;
  std::vector<char> inner(n, 0);
  int taken = 0;
  for (int32_t v : p.late)
    if (p.radix[v] > 1 && taken < int(kSharedInner)) {
      inner[v] = 1;
      ++taken;
    }
  if (taken < int(kSharedInner)) return;
  std::vector<int32_t> indeg(n, 0);
  for (int32_t v = 0; v < n; ++v) indeg[v] = int32_t(p.preds[v].size());
  std::vector<int32_t> order;
  std::vector<char> done(n, 0);
  for (int pass = 0; pass < 2; ++pass) {  // the other tools, then the inner ones
    for (;;) {
      int32_t u = -1;
      for (int32_t v = 0; v < n && u < 0; ++v)
        if (!done[v] && indeg[v] == 0 && (inner[v] != 0) == (pass == 1)) u = v;
      if (u < 0) break;
      done[u] = 1;
      order.push_back(u);
      for (int32_t v = 0; v < n; ++v)
        for (int32_t x : p.preds[v])
          if (x == u) --indeg[v];
    }
    // a tool left after the first pass depends on an inner tool
    if (pass == 0 && int(order.size()) != n - int(kSharedInner)) return;
  }
  if (int(order.size()) == n) p.order = order;
}

// The first kSharedInner tools with a choice in p.late (a shared-prefix
// search's inner digits) hold the last labels.
static bool inner_last(const sched_problem& p) {
  int taken = 0;
  for (int32_t v : p.late) {
    if (p.radix[v] <= 1) continue;
    if (taken == int(kSharedInner)) break;
    ++taken;
    int32_t label = 0;
    while (p.order[label] != v) ++label;
    if (label < p.n - int(kSharedInner)) return false;
  }
  return taken == int(kSharedInner);
}

// Enumeration order (tools, inner positions first) of a search with J inner
// digits.  Index order (a partial range): the tools with a choice in
// ascending number, so that the walk follows the index.  A full range: the
// four tools deepest in the DAG take the positions right above the J inner
// digits, so that the lanes of a wave (consecutive outer combinations) differ
// in tools that act late in every schedule and step through their passes
// together; the other tools follow from deepest to shallowest.  Any order
// visits every mapping once.
// Full-range searches of problems the shared-prefix kernel serves use
// kSharedInner inner digits on the deepest tools (the kernel then computes
// each lane's schedule prefix once for all of their modes) and the next four
// deepest on the lanes: the plain deepest-first order.
// prefix_able: the kernel for `lay` tools has shared prefixes for the problem.
bool prefix_able(const sched_problem& p, int lay) {
  if (lay > (p.sharing ? kPrefixMaxNShare : kPrefixMaxN) || p.enum_tools.size() < kSharedInner)
    return false;
  // from kCompactSnapN tools the kernel's LDS column leaves out the last labels
  if (lay >= kCompactSnapN && (p.n != lay || !inner_last(p))) return false;
  return !p.free_fanout;  // scored in closed form, nothing to share
}

// Combinations of a shared-prefix search's inner digits.
uint64_t shared_inner_count(const sched_problem& p) {
  uint64_t inner = 1;
  int taken = 0;
  for (int32_t t : p.late)
    if (p.radix[t] > 1 && taken < int(kSharedInner)) {
      inner *= p.radix[t];
      ++taken;
    }
  return inner;
}

bool prefix_plan(const sched_problem& p, uint64_t n_tables) {
  // enough lanes left to fill the GPU with kSharedInner inner digits
  return prefix_able(p, p.n) &&
         (unsigned __int128)(p.n_mappings / shared_inner_count(p)) * n_tables >= kTargetLanes;
}

Seq enumeration(const sched_problem& p, bool full, int J, bool prefix) {
  Seq seq;
  if (!full) {
    for (int32_t v : p.enum_tools) seq.push_back(v);
    return seq;
  }
  Seq late;
  for (int32_t v : p.late)
    if (p.radix[v] > 1) late.push_back(v);
  if (prefix) return late;
  const int P = late.size();
  const int lanes = std::min(4, P - J);
  for (int k = 0; k < J; ++k) seq.push_back(late[lanes + k]);
  for (int k = 0; k < lanes; ++k) seq.push_back(late[k]);
  for (int k = lanes + J; k < P; ++k) seq.push_back(late[k]);
  return seq;
}

uint64_t inner_count(const sched_problem& p, const Seq& seq, int J) {
  uint64_t c = 1;
  for (int k = 0; k < J; ++k) c *= p.radix[seq[k]];
  return c;
}

// Lanes per wave of a shared-prefix search over a space too small to fill the
// GPU with full waves of prefixes (0: one mapping per lane in place of it).
// With as many prefixes as make four rounds of combinations, 2^17 prefixes
// still give the GPU 4,681 waves: 13 tools, 177,147 prefixes, whole calls
// 102 us layered and 126 tight, 152 and 147 with a mapping per lane (full
// waves: 133 and 190; two rounds per wave 117 and 128).  At 12 tools a mapping
// per lane is the shorter way (68 us; two rounds 71, four 83).
uint32_t thin_lanes(const sched_problem& p) {
  const uint64_t inner = shared_inner_count(p);
  return prefix_able(p, p.n) && inner >= 6 && p.n_mappings / inner >= (1ull << 17)
             ? uint32_t(256u / inner) : 0u;
}

// Split [lo, hi) x n_tables into blocks of kBlock lanes; each lane owns one
// outer combination and enumerates the inner ones.  J grows while the lanes
// still number about kTargetLanes.
void plan_search(const sched_problem& p, uint64_t lo, uint64_t hi, uint32_t n_tables,
                 SearchArgs& a) {
  const bool full = lo == 0 && hi == p.n_mappings;
  const int P = int(p.enum_tools.size());
  const unsigned __int128 work = (unsigned __int128)(hi - lo) * n_tables;
  int J = 0;
  const bool prefix = full && prefix_plan(p, n_tables);
  a.lanes = 64;
  a.thin = 0;
  if (prefix) {
    J = int(kSharedInner);
    a.variant = p.variant;
  } else if (const uint32_t lanes = n_tables == 1 && full ? thin_lanes(p) : 0u) {
    a.thin = 1;
    J = int(kSharedInner);
    a.lanes = lanes;
  } else {
    while (J < kMaxInnerDigits && J < P) {
      const uint64_t next = inner_count(p, enumeration(p, full, J + 1, false), J + 1);
      if ((unsigned __int128)next * kTargetLanes > work) break;
      ++J;
    }
  }
  const uint64_t inner = inner_count(p, enumeration(p, full, J, prefix || a.thin), J);
  a.lo = lo;
  a.hi = hi;
  a.inner_digits = uint32_t(J);
  a.inner_count = uint32_t(inner);
  a.outer_lo = lo / inner;
  const uint64_t outer_hi = hi / inner + (hi % inner ? 1 : 0);
  a.n_outer = outer_hi - a.outer_lo;
  const uint64_t per_item = uint64_t(a.lanes) * (kBlock / 64);
  a.items_per_table = (a.n_outer + per_item - 1) / per_item;
  const uint64_t cap = std::max<uint64_t>(1, kMaxBlocks / n_tables);
  a.blocks_per_table = uint32_t(std::min<uint64_t>(a.items_per_table, cap));
  a.n_tables = n_tables;
  a.n_blocks = a.blocks_per_table * n_tables;
  a.full_range = full ? 1u : 0u;
  a.sharing = uint32_t(p.sharing);
  a.prefix = prefix ? 1u : 0u;
  a.lds_levels = table_levels(p);
}

// The walk of plan a in a table's header, where the full-order kernel reads it.
void write_walk(const SearchArgs& a, uint32_t* table) {
  table[kHdrOuterLoLo] = uint32_t(a.outer_lo);
  table[kHdrOuterLoHi] = uint32_t(a.outer_lo >> 32);
  table[kHdrNOuterLo] = uint32_t(a.n_outer);
  table[kHdrNOuterHi] = uint32_t(a.n_outer >> 32);
  table[kHdrInnerDigits] = a.inner_digits;
  table[kHdrInnerCount] = a.inner_count;
  table[kHdrPrefix] = a.prefix | a.thin;
  table[kHdrLanes] = a.lanes ? a.lanes : 64u;
}

// Labels walked per lane by a closed-form launch over `work` mappings (0: the
// general kernel, one mapping per lane).  A lane's walk is a series of up to
// 243 dependent steps, so labels are added while 2^16 outer combinations are
// left to hide it behind: a 14-tool chain took 29.2 us with 3 labels, 48.4
// with 5, a 14-tool fan-out 42.9 with 3 and 58.9 with 4.  A chain is worth it
// at any size (8 tools: 23 us, event loop 36), a fan-out from 2^15 lanes of 9
// (12 tools: 29.7 us, one by one 41.9; 11 tools 28.9 either way).
uint32_t closed_inner(uint32_t closed, unsigned __int128 work) {
  uint32_t j = closed == kClosedChain ? 1 : 0;
  if (closed == kClosedFanout && work / 9 >= (1ull << 15)) j = 2;
  if (j == 0) return 0;
  for (uint64_t c = j == 1 ? 9 : 27; j < kClosedInner && work / c >= (1ull << 16); c *= 3) ++j;
  return j;
}

// Combinations of the last j labels of problem p, and the outer ones of a
// closed-form walk over them.
uint64_t closed_combos(const sched_problem& p, uint32_t j) {
  uint64_t inner = 1;
  for (uint32_t k = 0; k < j; ++k) inner *= p.radix[p.order[p.n - 1 - int(k)]];
  return inner;
}

uint64_t closed_outer(const sched_problem& p, uint32_t j) {
  return p.n_mappings / closed_combos(p, j);
}

// Whether problem p gains from its closed form over its last j labels, in a
// launch whose problems of this kind have `work` mappings.  A fan-out's lane
// runs the outer tools' queue for every set of inner tools on gpu_now, which has
// to serve more than a mapping or two: where the labels hold fewer than three
// combinations (tools of one mode), one by one is the shorter way but for small
// searches (30 tools with five such labels, 6.7e7 mappings: 1.27 ms, in closed
// form 2.69; with three combinations 172 us against 260).  Work for two labels
// (up to 1.8e6 mappings) is mostly launch and wait: two combinations take 0.54
// to 0.80 times as long as one by one (0.79 to 1.23 with work for three labels),
// one 0.82 to 0.88 times up to 1e6 mappings and 1.09 beyond.
bool closed_pays(const sched_problem& p, uint32_t j, unsigned __int128 work) {
  if (j == 0 || p.closed != kClosedFanout) return j > 0;
  const uint64_t combos = closed_combos(p, j);
  return combos >= 3 || (j == 2 && closed_inner(kClosedFanout, work) == 2 &&
                         (combos == 2 || work < (1u << 20)));
}

// Turns the plan of a one-table full-range search into a closed-form one where
// the problem has one.
void plan_closed(const sched_problem& p, SearchArgs& a) {
  const uint32_t j = closed_inner(p.closed, p.n_mappings);
  if (!closed_pays(p, j, p.n_mappings)) return;
  a.closed = p.closed;
  a.inner_digits = j;
  const uint64_t items = (closed_outer(p, j) + kBlock - 1) / kBlock;
  a.n_blocks = a.blocks_per_table = uint32_t(std::min<uint64_t>(items, kMaxBlocks));
}

// The plan of a one-table full-range search.
void plan_full(const sched_problem& p, SearchArgs& a) {
  plan_search(p, 0, p.n_mappings, 1, a);
  plan_closed(p, a);
}

// Whether a plan's launch shares schedule prefixes (a closed-form one does not).
int32_t shares_prefixes(const SearchArgs& a) {
  return a.closed == kClosedNone && (a.prefix | a.thin) != 0 ? 1 : 0;
}

// A partial range [lo, hi) as parts of a full-order search.  A part of level k
// is a run of aligned blocks of W_k mappings (W_k: the product of the radices
// of the first k tools with a choice): the modes of those k tools are free in
// it, so they can be enumerated deepest first with shared prefixes as in a
// full search, and the tools above them count through the run.  The largest
// level that has a whole block in [lo, hi) takes the middle; each smaller
// level takes what it can of the two ends, down to kPartMin mappings, and
// what is left at the ends is walked in index order, one mapping per lane.
// Two parts a level: kMaxParts reaches ten levels below the middle, so an end
// left over by that limit is shorter than the block of the tenth, W_k over the
// product of ten radices (2^-10 to 3^-10 of the middle's blocks).
struct Part {
  uint64_t lo, hi;
  int level;  // k; 0: index order
};
constexpr uint64_t kPartMin = 19683;
constexpr int kMaxParts = 24;

// Words that the tables of a launch over parts and their first blocks take.
size_t parts_words(const sched_problem& p) {
  return size_t(kMaxParts) * p.table_words + kMaxParts + 1;
}

int split_range(const sched_problem& p, uint64_t lo, uint64_t hi, Part* out) {
  const int P = int(p.enum_tools.size());
  uint64_t w[kMaxTools + 1];
  w[0] = 1;
  for (int k = 0; k < P; ++k) w[k + 1] = w[k] * p.radix[p.enum_tools[k]];
  int n = 0, k = P;
  uint64_t left = 0, right = 0;  // the middle covers [left, right)
  for (; k >= int(kSharedInner) && w[k] >= kPartMin; --k) {
    const uint64_t a = lo / w[k] + (lo % w[k] != 0), b = hi / w[k];
    if (a < b) {
      left = a * w[k];
      right = b * w[k];
      break;
    }
  }
  if (left >= right) return 0;
  out[n++] = {left, right, k};
  for (--k; k >= int(kSharedInner) && w[k] >= kPartMin; --k) {
    const uint64_t a = (lo / w[k] + (lo % w[k] != 0)) * w[k], b = hi / w[k] * w[k];
    if (n + 4 > kMaxParts) break;
    if (a < left) {
      out[n++] = {a, left, k};
      left = a;
    }
    if (b > right) {
      out[n++] = {right, b, k};
      right = b;
    }
  }
  if (lo < left) out[n++] = {lo, left, 0};
  if (right < hi) out[n++] = {right, hi, 0};
  return n;
}

// Whether a partial range is searched in parts: the kernel has shared
// prefixes for the problem whatever its inner tools' labels are, and the
// range has lanes enough left to fill the GPU with kSharedInner inner digits
// (the rule of a full search).  Below that, one mapping per lane in index
// order is the shorter chain.  145 M of 3^19 mappings (mixed DAG): 3.97 ms in parts,
// 19.9 ms in index order.  Without edges every tool is read in the first pass:
// a prefix then shares next to nothing, and parts gain only by their rounds,
// from three times as many lanes on (16 tools: 5e6 to 1.2e7 mappings take up to
// 1.2 times as long in parts, 1.5e7 0.78 times), and with two modes per tool never
// (24 tools, 1.4e7 mappings: 771 us in parts, 605 in index order).
bool range_in_parts(const sched_problem& p, uint64_t lo, uint64_t hi) {
  if (p.n >= kCompactSnapN || !prefix_able(p, p.n)) return false;
  uint64_t inner = 1;
  for (uint32_t j = 0; j < kSharedInner; ++j) inner *= 3;
  bool edges = false, three = false;
  for (const auto& pl : p.preds) edges = edges || !pl.empty();
  for (uint8_t r : p.radix) three = three || r == 3;
  if (!edges && !three) return false;
  return (hi - lo) / inner >= (edges ? 1 : 3) * kTargetLanes && parts_words(p) <= kStageWords;
}

// Enumeration order of a part: its free tools deepest first, then the tools
// that count through the run.
Seq part_enumeration(const sched_problem& p, int level) {
  Seq seq;
  bool low[kMaxTools] = {};
  for (int k = 0; k < level; ++k) low[p.enum_tools[k]] = true;
  for (int32_t v : p.late)
    if (low[v]) seq.push_back(v);
  for (size_t k = size_t(level); k < p.enum_tools.size(); ++k) seq.push_back(p.enum_tools[k]);
  return seq;
}

size_t partial_capacity(uint64_t n_tables) {
  return size_t(std::max<uint64_t>(n_tables, kMaxBlocks));
}

struct Layout {
  size_t tables, partials, results, total;
};

Layout layout_for(size_t table_bytes_total, size_t n_partials, size_t n_results) {
  Layout l;
  l.tables = 0;
  l.partials = align_up(table_bytes_total);
  l.results = l.partials + align_up(n_partials * sizeof(Partial));
  l.total = l.results + align_up(n_results * sizeof(DevResult));
  return l;
}

int check_workspace(void* ws, size_t ws_bytes, size_t need) {
  if (ws == nullptr) return SCHED_E_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) % kAlign != 0) return SCHED_E_WORKSPACE;
  if (ws_bytes < need) return SCHED_E_WORKSPACE;
  return SCHED_OK;
}

int create_problem(const sched_tool* tools, int32_t n_tools, const sched_edge* edges,
                   int32_t n_edges, const uint32_t* contention_q16, int32_t n_levels,
                   int64_t vram_budget_mib, const uint8_t* allowed, int32_t sharing,
                   sched_problem** out) {
  if (out == nullptr || tools == nullptr || contention_q16 == nullptr) return SCHED_E_NULL;
  if (n_edges > 0 && edges == nullptr) return SCHED_E_NULL;
  if (n_tools < 1 || n_tools > kMaxTools || n_edges < 0 || n_levels < 1 || n_levels > kMaxLevels)
    return SCHED_E_SIZE;
  if (vram_budget_mib < 0) return SCHED_E_VALUE;
  for (int32_t v = 0; v < n_tools; ++v) {
    const sched_tool& t = tools[v];
    if (check_latencies(t.gpu_us, t.cpu_us, t.load_us, t.xfer_us) != SCHED_OK || t.mem_mib < 0)
      return SCHED_E_VALUE;
  }
  for (int32_t l = 0; l < n_levels; ++l)
    if (contention_q16[l] < 65536u || contention_q16[l] > (1u << 24)) return SCHED_E_VALUE;
  if (allowed != nullptr)
    for (int32_t v = 0; v < n_tools; ++v)
      if (allowed[v] < 1 || allowed[v] > 7) return SCHED_E_VALUE;
  if (sharing != 0 && sharing != 1) return SCHED_E_VALUE;

  sched_problem* p = new (std::nothrow) sched_problem;
  if (p == nullptr) return SCHED_E_NOMEM;
  try {
    p->n = n_tools;
    p->sharing = sharing;
    p->tools.assign(tools, tools + n_tools);
    p->contention.assign(contention_q16, contention_q16 + n_levels);
    p->budget = vram_budget_mib;
    p->preds.assign(n_tools, {});
    for (int32_t e = 0; e < n_edges; ++e) {
      const int32_t u = edges[e].src, v = edges[e].dst;
      if (u < 0 || u >= n_tools || v < 0 || v >= n_tools || u == v) {
        delete p;
        return SCHED_E_EDGE;
      }
      p->preds[v].push_back(u);
    }
    int32_t total = 0;
    for (auto& pl : p->preds) {
      std::sort(pl.begin(), pl.end());
      pl.erase(std::unique(pl.begin(), pl.end()), pl.end());
      total += int32_t(pl.size());
    }
    // Kahn's algorithm: every tool must be reachable in a topological order.
    std::vector<int32_t> indeg(n_tools, 0);
    std::vector<std::vector<int32_t>> succ(n_tools);
    for (int32_t v = 0; v < n_tools; ++v)
      for (int32_t u : p->preds[v]) {
        succ[u].push_back(v);
        indeg[v]++;
      }
    // Kahn's algorithm, always taking the lowest-numbered ready tool: the
    // internal labels of the device tables (a cycle leaves tools unlabelled).
    std::vector<char> done(n_tools, 0);
    for (int32_t step = 0; step < n_tools; ++step) {
      int32_t u = -1;
      for (int32_t v = 0; v < n_tools && u < 0; ++v)
        if (!done[v] && indeg[v] == 0) u = v;
      if (u < 0) break;
      done[u] = 1;
      p->order.push_back(u);
      for (int32_t v : succ[u]) --indeg[v];
    }
    if (int32_t(p->order.size()) != n_tools) {
      delete p;
      return SCHED_E_CYCLE;
    }
    // Depth of every tool (longest chain from a source, in tools) and its
    // number of ancestors, in topological order; deepest first, ties to
    // more ancestors, then to the lower tool number.
    std::vector<int32_t> depth(n_tools, 1);
    std::vector<std::vector<char>> anc(n_tools, std::vector<char>(n_tools, 0));
    for (int32_t v : p->order)
      for (int32_t u : p->preds[v]) {
        depth[v] = std::max(depth[v], depth[u] + 1);
        anc[v][u] = 1;
        for (int32_t w = 0; w < n_tools; ++w)
          if (anc[u][w]) anc[v][w] = 1;
      }
    std::vector<int32_t> n_anc(n_tools, 0);
    for (int32_t v = 0; v < n_tools; ++v)
      for (int32_t w = 0; w < n_tools; ++w) n_anc[v] += anc[v][w];
    p->late.resize(n_tools);
    std::iota(p->late.begin(), p->late.end(), 0);
    std::stable_sort(p->late.begin(), p->late.end(), [&](int32_t a, int32_t b) {
      if (depth[a] != depth[b]) return depth[a] > depth[b];
      return n_anc[a] > n_anc[b];
    });
    // Decision space: allowed modes, radices and mixed-radix weights.
    p->allowed.assign(n_tools, uint8_t(7));
    if (allowed != nullptr) p->allowed.assign(allowed, allowed + n_tools);
    p->radix.resize(n_tools);
    p->weight.resize(n_tools);
    uint64_t w = 1;
    for (int32_t v = 0; v < n_tools; ++v) {
      const uint8_t a = p->allowed[v];
      p->radix[v] = uint8_t((a & 1) + ((a >> 1) & 1) + ((a >> 2) & 1));
      p->weight[v] = w;
      w *= p->radix[v];
      if (p->radix[v] > 1) p->enum_tools.push_back(v);
    }
    p->n_mappings = w;
    int64_t sum_mem = 0;
    for (const sched_tool& t : p->tools) sum_mem += t.mem_mib;
    const bool fanout_fits = total == 0 && sharing == 0 && p->budget >= sum_mem;
    if (n_tools >= kCompactSnapN && n_tools <= kPrefixMaxN && sharing == 0 && !fanout_fits)
      label_inner_last(*p);
    bool identity = true;
    for (int32_t i = 0; i < n_tools; ++i) identity = identity && p->order[i] == i;
    p->free_fanout = fanout_fits && identity;
    bool chain = n_tools >= 2 && sharing == 0;
    for (int32_t i = 0; i < n_tools && chain; ++i) {
      const auto& pl = p->preds[p->order[i]];
      chain = i == 0 ? pl.empty() : pl.size() == 1 && pl[0] == p->order[i - 1];
    }
    bool queue = false;
    for (uint8_t m : p->allowed) queue = queue || (m & 4);
    if (!queue && sharing == 0 && n_tools >= kVarMinN && n_tools <= kPrefixMaxN)
      p->variant = p->budget >= sum_mem ? kVarFree : kVarNoQueue;
    if (n_tools >= int32_t(kClosedInner)) {
      if (chain) p->closed = kClosedChain;
      if (p->free_fanout && n_tools <= kClosedFanoutTools &&
          table_levels(*p) <= kClosedFanoutLevels)
        p->closed = kClosedFanout;
    }
    p->table_words = table_words(uint32_t(n_tools), table_levels(*p));
    p->table.assign(p->table_words, 0u);
    const int rc = build_table(*p, nullptr, p->table.data());
    if (rc != SCHED_OK) {
      delete p;
      return rc;
    }
    // the table of a one-table full-range search, in its enumeration order
    SearchArgs a{};
    plan_search(*p, 0, p->n_mappings, 1, a);
    p->table_full = p->table;
    set_enumeration(*p, enumeration(*p, true, int(a.inner_digits), a.prefix != 0 || a.thin != 0),
                    p->table_full.data());
    write_walk(a, p->table_full.data());
  } catch (const std::bad_alloc&) {
    delete p;
    return SCHED_E_NOMEM;
  }
  *out = p;
  return SCHED_OK;
}

#define HIP_TRY(expr)                                  \
  do {                                                 \
    if ((expr) != hipSuccess) return SCHED_E_DEVICE;   \
  } while (0)

// Waits for a call's stream where an error leaves the call before its own wait:
// what the stream has been given may still read host memory of the call.
class StreamWait {
 public:
  explicit StreamWait(hipStream_t s) : stream_(s) {}
  StreamWait(const StreamWait&) = delete;
  StreamWait& operator=(const StreamWait&) = delete;
  ~StreamWait() {
    if (!waited_) (void)hipStreamSynchronize(stream_);
  }
  // The stream has been waited for, or has been given nothing.
  void waited() { waited_ = true; }

 private:
  hipStream_t stream_;
  bool waited_ = false;
};

// Page-locked host memory that kernels read and write directly, so that a
// small call needs no copies: its indices and its results (or its blocks'
// partial minima) cross the link as part of the kernel.  One allocation of
// kSlots slots for the process, made at the first call that wants one; a call
// holds one slot from before its launch until its stream is done with it, and
// gives it back.  With every slot taken a call copies through its workspace
// instead, and so does one whose allocation fails (it may while another thread
// captures a graph); the next call tries again.  A 16-byte result and its copy back measured
// 26.4 us from launch to host, written straight to the host 17.6 us.
constexpr int kSlots = 8;
constexpr size_t kSlotBytes = size_t(32) << 10;
std::mutex g_slot_mutex;
char* g_slots = nullptr;
uint32_t g_slots_taken = 0;

class Slot {
 public:
  explicit Slot(hipStream_t s) : stream_(s) {
    std::lock_guard<std::mutex> lock(g_slot_mutex);
    if (g_slots == nullptr) {
      void* p = nullptr;
      if (hipHostMalloc(&p, kSlots * kSlotBytes, hipHostMallocPortable) == hipSuccess)
        g_slots = static_cast<char*>(p);
      else
        (void)hipGetLastError();
    }
    for (int k = 0; g_slots != nullptr && k < kSlots; ++k)
      if (!((g_slots_taken >> k) & 1u)) {
        g_slots_taken |= 1u << k;
        at_ = k;
        break;
      }
  }
  Slot(const Slot&) = delete;
  Slot& operator=(const Slot&) = delete;
  ~Slot() {
    if (at_ < 0) return;
    if (launched_) (void)hipStreamSynchronize(stream_);  // an error left the call early
    std::lock_guard<std::mutex> lock(g_slot_mutex);
    g_slots_taken &= ~(1u << at_);
  }
  char* data() const { return at_ < 0 ? nullptr : g_slots + size_t(at_) * kSlotBytes; }
  // Between launched() and waited() the stream may still write the slot.
  void launched() { launched_ = true; }
  void waited() { launched_ = false; }

 private:
  hipStream_t stream_;
  int at_ = -1;
  bool launched_ = false;
};

// Whether a table (up to its bound table) fits a kernel's arguments.
bool fits_arguments(const uint32_t* table) {
  return bound_base(table[kHdrN], table[kHdrLevels]) <= kArgWords;
}

// Makespans of m mapping indices of problem p with the host table `table`
// (INT64_MAX: infeasible), through a slot, or through device memory: d_tab
// (the table), d_idx and d_ms (m entries each).  Waits for the stream.
int score(const sched_problem& p, const uint32_t* table, const uint64_t* idx, size_t m,
          int64_t* ms, uint32_t* d_tab, uint64_t* d_idx, int64_t* d_ms, hipStream_t s) {
  uint32_t flags = p.sharing ? kEvalSharing : 0u;
  const uint32_t* tab = table;
  StreamWait wait(s);
  if (fits_arguments(table)) {
    flags |= kEvalHostTable;
  } else {
    HIP_TRY(hipMemcpyAsync(d_tab, table, size_t(p.table_words) * 4, hipMemcpyHostToDevice, s));
    tab = d_tab;
  }
  if (m * 16 <= kSlotBytes) {
    Slot slot(s);
    if (char* h = slot.data()) {
      std::memcpy(h, idx, m * 8);
      int64_t* const h_ms = reinterpret_cast<int64_t*>(h) + m;
      slot.launched();
      HIP_TRY(launch_eval(p.n, tab, reinterpret_cast<const uint64_t*>(h), int64_t(m), p.n_mappings,
                          h_ms, flags, s));
      HIP_TRY(hipStreamSynchronize(s));
      slot.waited();
      wait.waited();
      std::memcpy(ms, h_ms, m * 8);
      return SCHED_OK;
    }
  }
  HIP_TRY(hipMemcpyAsync(d_idx, idx, m * 8, hipMemcpyHostToDevice, s));
  HIP_TRY(launch_eval(p.n, tab, d_idx, int64_t(m), p.n_mappings, d_ms, flags, s));
  HIP_TRY(hipMemcpyAsync(ms, d_ms, m * 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  wait.waited();
  return SCHED_OK;
}

// One what-if candidate around a base mapping.
struct Cand {
  int kind, tool, mode, swap_tool;  // kind 0 base, 1 single-tool move, 2 swap
};

// The base mapping and its neighbourhood in the order of Algorithm 1: for
// each tool i and each other allowed mode a, the move i -> a, followed, when
// a is gpu_now, by one swap per tool j on gpu_now that may use gpu_queue
// (i -> gpu_now, j -> gpu_queue).  Every swap is listed; callers decide
// which to keep.
void neighbourhood(const sched_problem& p, uint64_t base, std::vector<uint64_t>& idx,
                   std::vector<Cand>& cands) {
  const int n = p.n;
  std::vector<int32_t> d(n);
  sched_mapping_modes(&p, base, d.data());
  // Moving tool v from mode d[v] to mode a changes its digit, weighted by W_v.
  auto with = [&](uint64_t x, int v, int a) {
    return x - uint64_t(digit_of_mode(p, v, d[v])) * p.weight[v] +
           uint64_t(digit_of_mode(p, v, a)) * p.weight[v];
  };
  auto ok = [&](int v, int a) { return ((p.allowed[v] >> a) & 1) != 0; };
  idx.clear();
  cands.clear();
  idx.push_back(base);
  cands.push_back({0, -1, -1, -1});
  for (int i = 0; i < n; ++i)
    for (int a = 0; a < 3; ++a) {
      if (a == d[i] || !ok(i, a)) continue;
      idx.push_back(with(base, i, a));
      cands.push_back({1, i, a, -1});
      if (a == 1)
        for (int j = 0; j < n; ++j)
          if (j != i && d[j] == 1 && ok(j, 2)) {
            idx.push_back(with(with(base, i, 1), j, 2));
            cands.push_back({2, i, 1, j});
          }
    }
}

// ---------------------------------------------------------------------------
// Exact search with pruning.

constexpr uint64_t kPruneMinSpace = 1ull << 22;  // smaller spaces: one exhaustive search
constexpr uint64_t kMaxPrefixes = 1ull << 24;    // bounded prefix assignments per call
constexpr uint64_t kMinSubspace = 1ull << 12;    // mappings per searched subspace, at least
// Prefixes searched together, in the first chunk of several and in the others:
// the first mostly lowers the bound for all that follow, so it is kept short
// (two modes, 34 tools: 6.9 ms with a first chunk of 2,048, 14.9 with 8,192
// prefixes; 19 tools, 8,019 survivors: 1.1 and 2.4 ms).  A chunk more costs 90
// us, so twice as many are still searched at once.
#ifndef DEVMAP_CHUNK_PREFIXES
#define DEVMAP_CHUNK_PREFIXES 8192
#endif
constexpr uint32_t kChunkPrefixes = DEVMAP_CHUNK_PREFIXES;
constexpr uint32_t kFirstPrefixes = std::min<uint32_t>(2048, kChunkPrefixes);
constexpr uint64_t kMaxChildren = 243;           // assignments of the extension tools
constexpr uint64_t kMinRest = 81;                // mappings left per extended prefix, at least

// The prefix: tools with a choice whose shortest durations differ most
// between their modes come first (their choice moves the bound most), then
// as many as fit kMaxPrefixes while the subspaces keep kMinSubspace mappings.
// A prefix that survives its bound is extended by the next tools of that order
// and its children bounded again, with more modes known, before what is left
// of them is searched: a bound costs about a tenth of a mapping's score, and
// most of a surviving prefix does not survive its own children.  Tight 24-tool
// DAG, whole calls: 6.8 ms without the second bounds (2,048 tables of 19,683
// mappings per launch), 2.5 ms with them; 18 tools 469 us and 431 us.
struct PrunePlan {
  std::vector<int32_t> prefix;  // prefix tools, digit order of the prefix index
  uint64_t n_prefixes = 1;
  uint64_t subspace = 1;        // mappings per prefix
  std::vector<int32_t> ext;     // extension tools, their digits above the prefix's
  uint64_t n_children = 1;
  uint64_t rest = 1;            // mappings per child
};

PrunePlan plan_prune(const sched_problem& p) {
  PrunePlan pl;
  const uint32_t* bt = p.table.data() + p.table[kHdrBoundOff];
  std::vector<std::pair<uint64_t, int32_t>> spread;
  for (int32_t v : p.enum_tools) {
    const uint32_t i = p.table[pos_base(uint32_t(p.n)) + uint32_t(v)];
    uint32_t lo = kInf, hi = 0;
    for (int m = 0; m < 3; ++m) {
      if (!((p.allowed[v] >> m) & 1)) continue;
      const uint32_t d = bt[kBoundWords * i + m];
      lo = std::min(lo, d);
      hi = std::max(hi, d == kInf ? (1u << 30) : d);
    }
    spread.push_back({uint64_t(hi - lo), v});
  }
  std::stable_sort(spread.begin(), spread.end(),
                   [](const auto& a, const auto& b) { return a.first > b.first; });
  pl.subspace = p.n_mappings;
  for (const auto& sv : spread) {
    const uint64_t r = p.radix[sv.second];
    if (pl.n_prefixes * r > kMaxPrefixes || pl.subspace / r < kMinSubspace) break;
    pl.prefix.push_back(sv.second);
    pl.n_prefixes *= r;
    pl.subspace /= r;
  }
  pl.rest = pl.subspace;
  for (size_t k = pl.prefix.size(); k < spread.size(); ++k) {
    const uint64_t r = p.radix[spread[k].second];
    if (pl.n_children * r > kMaxChildren || pl.rest / r < kMinRest) break;
    pl.ext.push_back(spread[k].second);
    pl.n_children *= r;
    pl.rest /= r;
  }
  return pl;
}

struct PruneLayout {
  size_t tables, partials, results, bounds, probe_idx, probe_ms, total;
  size_t chunk;  // prefixes searched together
};

PruneLayout prune_layout(const sched_problem& p, const PrunePlan& pl) {
  PruneLayout l;
  const size_t probes = size_t(1 + 2 * p.n + p.n * (p.n - 1));
  l.tables = 0;
  l.partials = align_up(size_t(p.table_words) * 4);
  l.results = l.partials + align_up(partial_capacity(1) * sizeof(Partial));
  l.bounds = l.results + align_up(sizeof(DevResult));
  // Survivor count (one word, padded) and then (bound, y) pairs: first up to
  // n_prefixes of the prefixes, then a chunk of them and its children.
  l.chunk = size_t(std::min<uint64_t>(kChunkPrefixes, pl.n_prefixes));
  const size_t pairs = std::max<size_t>(size_t(pl.n_prefixes), l.chunk * size_t(1 + pl.n_children));
  l.probe_idx = l.bounds + align_up(4) + align_up(pairs * 8);
  l.probe_ms = l.probe_idx + align_up(probes * 8);
  l.total = l.probe_ms + align_up(probes * 8);
  return l;
}

// Workspace of a search over one table, which is the least that a call takes,
// and of one over a range's parts (their tables and first blocks).
Layout one_table_layout(const sched_problem& p) {
  return layout_for(4 * size_t(p.table_words), partial_capacity(1), 1);
}

Layout parts_layout(const sched_problem& p) {
  return layout_for(4 * parts_words(p), partial_capacity(1), 1);
}

// Workspace bytes with which any search of the problem goes its best way.
size_t one_search_bytes(const sched_problem& p) {
  return (range_in_parts(p, 0, p.n_mappings) ? parts_layout(p) : one_table_layout(p)).total;
}

// Plan and tables of a search over the parts of [lo, hi), staged in `stage`
// (parts_words): n_tables tables, then their first blocks.  Returns the number
// of staged words.
size_t stage_parts(const sched_problem& p, uint64_t lo, uint64_t hi, SearchArgs& a,
                   uint32_t* stage) {
  Part parts[kMaxParts];
  const int n = split_range(p, lo, hi, parts);
  a.lo = lo;
  a.hi = hi;
  a.full_range = 1;
  a.one_result = 1;
  a.sharing = uint32_t(p.sharing);
  a.lds_levels = table_levels(p);
  a.n_tables = uint32_t(n);
  uint32_t* const first = stage + size_t(n) * p.table_words;
  // The middle (part 0) comes last: the short parts are then done when its
  // last blocks are.
  uint32_t blocks = 0;
  for (int i = 0; i < n; ++i) {
    const int at = n - 1 - i;
    const Part& part = parts[at];
    uint32_t* const tb = stage + size_t(i) * p.table_words;
    std::copy(p.table.begin(), p.table.end(), tb);
    const Seq seq = part_enumeration(p, part.level);
    set_enumeration(p, seq, tb);
    SearchArgs w{};
    w.prefix = part.level > 0 ? 1u : 0u;
    w.inner_digits = w.prefix ? kSharedInner : 0u;
    const uint64_t inner = inner_count(p, seq, int(w.inner_digits));
    w.inner_count = uint32_t(inner);
    w.outer_lo = part.lo / inner;
    w.n_outer = (part.hi - part.lo) / inner;
    write_walk(w, tb);
    first[i] = blocks;
    const uint64_t items = (w.n_outer + kBlock - 1) / kBlock;
    const uint64_t cap = at == 0 ? kMaxBlocks - blocks : kMaxBlocks / (2 * kMaxParts);
    blocks += uint32_t(std::min(items, cap));
  }
  first[n] = blocks;
  a.n_blocks = blocks;
  return size_t(n) * p.table_words + size_t(n) + 1;
}

// A partial range searched in parts, in workspace ws (parts_layout), its tables staged in
// `stage` (kStageWords; null: heap memory of this call's, for the tables of 24
// parts are more than a small thread stack holds).
int search_parts(const sched_problem& p, uint64_t lo, uint64_t hi, char* ws, hipStream_t s,
                 uint32_t* stage, sched_result* h_out) {
  const Layout L = parts_layout(p);
  SearchArgs a{};
  std::unique_ptr<uint32_t[]> heap;
  if (stage == nullptr) {
    heap.reset(new (std::nothrow) uint32_t[parts_words(p)]);
    if (heap == nullptr) return SCHED_E_NOMEM;
    stage = heap.get();
  }
  const size_t words = stage_parts(p, lo, hi, a, stage);
  a.tables = reinterpret_cast<const uint32_t*>(ws + L.tables);
  a.table_stride = p.table_words;
  a.block_first = a.tables + size_t(a.n_tables) * p.table_words;
  a.partials = reinterpret_cast<Partial*>(ws + L.partials);
  a.results = reinterpret_cast<DevResult*>(ws + L.results);
  DevResult r;
  StreamWait wait(s);
  HIP_TRY(hipMemcpyAsync(ws + L.tables, stage, words * 4, hipMemcpyHostToDevice, s));
  HIP_TRY(launch_search(p.n, a, s));
  HIP_TRY(hipMemcpyAsync(&r, a.results, sizeof(r), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  wait.waited();
  h_out->best_index = r.index;
  h_out->makespan_us = r.makespan;
  return SCHED_OK;
}

// One launch of a batch: replicas [first, last) of the launch order, on the
// kernel for `lay` tools.
struct Launch {
  size_t first, last;
  int lay;
  unsigned __int128 work;  // mappings of its replicas (two of 3^40 pass 64 bits)
  SearchArgs a;
};

// Words between the tables of a batch of these problems: any of them may be
// laid out for the most tools among them.
size_t batch_stride(const sched_problem* const* problems, int32_t n_problems) {
  uint32_t lay = 1, levels = 1;
  for (int32_t i = 0; i < n_problems; ++i) {
    lay = std::max(lay, uint32_t(problems[i]->n));
    levels = std::max(levels, table_levels(*problems[i]));
  }
  return bound_base(lay, levels);
}

// Bytes of a batch's tables and of its launches' first blocks (one more entry
// than tables per launch, at most one launch per table).
size_t batch_table_bytes(size_t stride, size_t n_replicas) {
  return (n_replicas * stride + 2 * n_replicas) * 4;
}

// Launches of a batch.  Replicas of one tool count and contention reading
// share a launch, whatever their shapes, masks and sizes, but that serial
// chains and free fan-outs, where they are enough and gain from it, have a
// launch of their own kind (of any tool counts).  A launch that would
// leave the GPU partly idle (fewer mappings than kTargetLanes lanes) joins the
// next larger tool count: its tables are laid out for more tools, at the cost
// of one more resolution per added tool, instead of a launch in series.  13
// scenarios of 4 to 9 tools, 8 replicas each: 108 us in one launch, 320 us in
// eleven.
void plan_batch(const sched_problem* const* problems, int32_t n_problems,
                const int32_t* replica_problem, size_t R, std::vector<Launch>& launches,
                std::vector<int32_t>& order) {
  order.resize(R);
  std::iota(order.begin(), order.end(), 0);
  // Labels walked by the launch of each closed form: the most for which the
  // problems that gain from it have work enough (0: none).
  std::vector<uint32_t> replicas(size_t(n_problems), 0u), kind(size_t(n_problems), kClosedNone);
  for (size_t r = 0; r < R; ++r) ++replicas[size_t(replica_problem[r])];
  unsigned __int128 all[3] = {};  // mappings of each kind
  for (int32_t i = 0; i < n_problems; ++i)
    all[problems[i]->closed] += (unsigned __int128)problems[i]->n_mappings * replicas[size_t(i)];
  uint32_t walked[3] = {};
  for (uint32_t c : {uint32_t(kClosedChain), uint32_t(kClosedFanout)})
    for (uint32_t j = kClosedInner; j > 0 && walked[c] == 0; --j) {
      unsigned __int128 work = 0;
      for (int32_t i = 0; i < n_problems; ++i)
        if (problems[i]->closed == c && closed_pays(*problems[i], j, all[c]))
          work += (unsigned __int128)problems[i]->n_mappings * replicas[size_t(i)];
      if (work > 0 && closed_inner(c, work) >= j) walked[c] = j;
    }
  for (int32_t i = 0; i < n_problems; ++i) {
    const uint32_t c = problems[i]->closed;
    if (c != kClosedNone && closed_pays(*problems[i], walked[c], all[c])) kind[size_t(i)] = c;
  }
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
    const int32_t a = replica_problem[x], b = replica_problem[y];
    if (kind[size_t(a)] != kind[size_t(b)]) return kind[size_t(a)] < kind[size_t(b)];
    if (problems[a]->sharing != problems[b]->sharing)
      return problems[a]->sharing < problems[b]->sharing;
    if (problems[a]->n != problems[b]->n) return problems[a]->n < problems[b]->n;
    return a < b;
  });
  for (size_t i = 0; i < R; ++i) {
    const sched_problem& p = *problems[replica_problem[order[i]]];
    const uint32_t closed = kind[size_t(replica_problem[order[i]])];
    Launch* const g = launches.empty() ? nullptr : &launches.back();
    if (g == nullptr || g->a.closed != closed || g->a.sharing != uint32_t(p.sharing) ||
        (closed == kClosedNone && g->lay != p.n && g->work >= kTargetLanes)) {
      Launch n{i, i, p.n, 0, SearchArgs{}};
      n.a.full_range = 1;
      n.a.closed = closed;
      n.a.inner_digits = walked[closed];
      n.a.sharing = uint32_t(p.sharing);
      launches.push_back(n);
    }
    Launch& l = launches.back();
    l.lay = p.n;
    l.last = i + 1;
    l.work += p.n_mappings;
    l.a.n_tables = uint32_t(l.last - l.first);
  }
}

// The table of problem p in a launch, without latencies: laid out for the
// launch's tools, enumerated and walked for its work in all.
int lay_replica(const sched_problem& p, const Launch& g, uint32_t* table) {
  SearchArgs w{};
  if (g.a.closed != kClosedNone) {  // (closed.hip's kernels serve any tool count)
    const int rc = lay_table(p, uint32_t(p.n), table);
    w.n_outer = closed_outer(p, g.a.inner_digits);
    write_walk(w, table);
    return rc;
  }
  const int rc = lay_table(p, uint32_t(g.lay), table);
  if (rc != SCHED_OK) return rc;
  const uint64_t shared = shared_inner_count(p);
  // (a problem smaller than one wave of prefixes has nothing to gain)
  w.prefix = prefix_able(p, g.lay) && g.work / shared >= kTargetLanes &&
             p.n_mappings / shared >= 64u;
  int J = 0;
  if (w.prefix) {
    J = int(kSharedInner);
  } else {
    while (J < kMaxInnerDigits && J < int(p.enum_tools.size())) {
      const uint64_t next = inner_count(p, enumeration(p, true, J + 1, false), J + 1);
      if ((unsigned __int128)next * kTargetLanes > g.work) break;
      ++J;
    }
  }
  const Seq seq = enumeration(p, true, J, w.prefix != 0);
  const uint64_t inner = inner_count(p, seq, J);
  w.inner_digits = uint32_t(J);
  w.inner_count = uint32_t(inner);
  w.n_outer = p.n_mappings / inner;
  set_enumeration(p, seq, table);
  write_walk(w, table);
  return SCHED_OK;
}

// Work items (kBlock outer combinations) of a table's walk.
uint64_t table_items(const uint32_t* table) {
  const uint64_t n = uint64_t(table[kHdrNOuterLo]) | (uint64_t(table[kHdrNOuterHi]) << 32);
  return (n + kBlock - 1) / kBlock;
}

// Blocks up to which the host takes the minimum of a search's partials
// itself: they are written to the call's slot, 16 B each, and no reduction is
// launched.  As many as fit a slot: whole calls on 8 to 11 tools (26 to 692
// blocks) took 35.5, 36.8, 41.0 and 46.2 us, against 39.2, 40.4, 44.2 and 48.8
// with the reduction.
constexpr uint32_t kHostPartials = 2048;
static_assert(kHostPartials * sizeof(Partial) <= kSlotBytes, "partials of a small search");

// One search of [lo, hi) in workspace ws of ws_bytes (at least those of
// one_table_layout; with fewer than parts_layout has, every partial range is
// walked in index order) on stream s, then the result.  record: every
// mapping's makespan (full ranges only; null: none).  stage: null, or kStageWords of host memory for the tables of a
// range's parts: the call then allocates nothing, page-locked slots (which the
// first call that wants one allocates) included.
int search_one(const sched_problem& p, uint64_t lo, uint64_t hi, char* ws, size_t ws_bytes,
               hipStream_t s, uint32_t* record, uint32_t* stage, sched_result* h_out) {
  const Layout L = one_table_layout(p);
  SearchArgs a{};
  if ((lo > 0 || hi < p.n_mappings) && range_in_parts(p, lo, hi) &&
      ws_bytes >= parts_layout(p).total)
    return search_parts(p, lo, hi, ws, s, stage, h_out);
  if (lo == 0 && hi == p.n_mappings)
    plan_full(p, a);
  else
    plan_search(p, lo, hi, 1, a);
  const std::vector<uint32_t>& table = a.full_range ? p.table_full : p.table;
  a.table_stride = p.table_words;
  a.partials = reinterpret_cast<Partial*>(ws + L.partials);
  a.results = reinterpret_cast<DevResult*>(ws + L.results);
  a.record = record;
  DevResult r;
  StreamWait wait(s);
  if (fits_arguments(table.data())) {
    a.host_table = table.data();
    a.host_words = bound_base(uint32_t(p.n), a.lds_levels);
  } else {
    a.tables = reinterpret_cast<const uint32_t*>(ws + L.tables);
    HIP_TRY(hipMemcpyAsync(ws + L.tables, table.data(), size_t(p.table_words) * 4,
                           hipMemcpyHostToDevice, s));
  }
  std::optional<Slot> slot;
  if (stage == nullptr) slot.emplace(s);
  char* const h = slot ? slot->data() : nullptr;
  if (h != nullptr) {
    const bool small = a.n_blocks <= kHostPartials;
    if (small) {
      a.partials = reinterpret_cast<Partial*>(h);
      a.results = nullptr;
    } else {
      a.results = reinterpret_cast<DevResult*>(h);
    }
    slot->launched();
    HIP_TRY(launch_search(p.n, a, s));
    HIP_TRY(hipStreamSynchronize(s));
    slot->waited();
    wait.waited();
    if (small) {
      const Partial* const part = reinterpret_cast<const Partial*>(h);
      uint32_t ms = kInf;
      uint64_t x = ~0ull;
      for (uint32_t k = 0; k < a.n_blocks; ++k)
        if (part[k].makespan < ms || (part[k].makespan == ms && part[k].index < x)) {
          ms = part[k].makespan;
          x = part[k].index;
        }
      r.index = ms == kInf ? ~0ull : x;
      r.makespan = ms == kInf ? INT64_MAX : int64_t(ms);
    } else {
      std::memcpy(&r, h, sizeof(r));
    }
  } else {
    HIP_TRY(launch_search(p.n, a, s));
    HIP_TRY(hipMemcpyAsync(&r, a.results, sizeof(r), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    wait.waited();
  }
  h_out->best_index = r.index;
  h_out->makespan_us = r.makespan;
  return SCHED_OK;
}

}  // namespace

extern "C" {

int sched_problem_create(const sched_tool* tools, int32_t n_tools, const sched_edge* edges,
                         int32_t n_edges, const uint32_t* contention_q16, int32_t n_levels,
                         int64_t vram_budget_mib, sched_problem** out) {
  return create_problem(tools, n_tools, edges, n_edges, contention_q16, n_levels,
                        vram_budget_mib, nullptr, 0, out);
}

int sched_problem_create_desc(const sched_problem_desc* d, sched_problem** out) {
  if (d == nullptr) return SCHED_E_NULL;
  return create_problem(d->tools, d->n_tools, d->edges, d->n_edges, d->contention_q16,
                        d->n_levels, d->vram_budget_mib, d->allowed, d->contention_mode, out);
}

int sched_problem_create_masked(const sched_tool* tools, int32_t n_tools,
                                const sched_edge* edges, int32_t n_edges,
                                const uint32_t* contention_q16, int32_t n_levels,
                                int64_t vram_budget_mib, const uint8_t* allowed,
                                sched_problem** out) {
  if (allowed == nullptr) return SCHED_E_NULL;
  return create_problem(tools, n_tools, edges, n_edges, contention_q16, n_levels,
                        vram_budget_mib, allowed, 0, out);
}

void sched_problem_destroy(sched_problem* p) { delete p; }

int sched_mapping_modes(const sched_problem* p, uint64_t index, int32_t* modes) {
  if (p == nullptr || modes == nullptr) return SCHED_E_NULL;
  if (index >= p->n_mappings) return SCHED_E_RANGE;
  for (int v = 0; v < p->n; ++v) {
    const int d = int(index % p->radix[v]);
    index /= p->radix[v];
    modes[v] = mode_of_digit(*p, v, d);
  }
  return SCHED_OK;
}

int sched_mapping_index(const sched_problem* p, const int32_t* modes, uint64_t* index) {
  if (p == nullptr || modes == nullptr || index == nullptr) return SCHED_E_NULL;
  uint64_t x = 0;
  for (int v = 0; v < p->n; ++v) {
    const int d = digit_of_mode(*p, v, modes[v]);
    if (d < 0) return SCHED_E_VALUE;
    x += uint64_t(d) * p->weight[v];
  }
  *index = x;
  return SCHED_OK;
}

int sched_num_tools(const sched_problem* p, int32_t* out) {
  if (p == nullptr || out == nullptr) return SCHED_E_NULL;
  *out = p->n;
  return SCHED_OK;
}

int sched_num_mappings(const sched_problem* p, uint64_t* out) {
  if (p == nullptr || out == nullptr) return SCHED_E_NULL;
  *out = p->n_mappings;
  return SCHED_OK;
}

int sched_workspace_bytes(const sched_problem* const* problems, int32_t n_problems,
                          int32_t n_replicas, size_t* out) {
  if (problems == nullptr || out == nullptr) return SCHED_E_NULL;
  if (n_problems < 1 || n_replicas < 0) return SCHED_E_SIZE;
  size_t need = 0;
  for (int32_t i = 0; i < n_problems; ++i) {
    if (problems[i] == nullptr) return SCHED_E_NULL;
    need = std::max(need, one_search_bytes(*problems[i]));  // single-problem calls
  }
  if (n_replicas > 0) {
    const size_t r = size_t(n_replicas);
    need = std::max(need, layout_for(batch_table_bytes(batch_stride(problems, n_problems), r),
                                     partial_capacity(r), r).total);
  }
  *out = need;
  return SCHED_OK;
}

int sched_bruteforce_argmin(const sched_problem* p, uint64_t lo, uint64_t hi, void* d_workspace,
                            size_t ws_bytes, void* hip_stream, sched_result* h_out) {
  if (p == nullptr || h_out == nullptr) return SCHED_E_NULL;
  if (lo >= hi || hi > p->n_mappings) return SCHED_E_RANGE;
  const int rc = check_workspace(d_workspace, ws_bytes, one_table_layout(*p).total);
  if (rc != SCHED_OK) return rc;
  return search_one(*p, lo, hi, static_cast<char*>(d_workspace), ws_bytes,
                    reinterpret_cast<hipStream_t>(hip_stream), nullptr, nullptr, h_out);
}

int sched_bruteforce_argmin_noalloc(const sched_problem* p, uint64_t lo, uint64_t hi,
                                    void* hip_stream, sched_result* h_out) {
  if (p == nullptr || h_out == nullptr) return SCHED_E_NULL;
  if (lo >= hi || hi > p->n_mappings) return SCHED_E_RANGE;
  if (one_search_bytes(*p) > kScratchBytes) return SCHED_E_WORKSPACE;
  void* ws = nullptr;
  uint32_t* stage = nullptr;
  HIP_TRY(scratch_buffer(&ws, &stage));
  return search_one(*p, lo, hi, static_cast<char*>(ws), kScratchBytes,
                    reinterpret_cast<hipStream_t>(hip_stream), nullptr, stage, h_out);
}

int sched_bruteforce_record(const sched_problem* p, void* d_workspace, size_t ws_bytes,
                            void* hip_stream, uint32_t* d_makespan, uint64_t capacity,
                            sched_result* h_out) {
  if (p == nullptr || h_out == nullptr || d_makespan == nullptr) return SCHED_E_NULL;
  if (capacity < p->n_mappings) return SCHED_E_WORKSPACE;
  const int rc = check_workspace(d_workspace, ws_bytes, one_table_layout(*p).total);
  if (rc != SCHED_OK) return rc;
  return search_one(*p, 0, p->n_mappings, static_cast<char*>(d_workspace), ws_bytes,
                    reinterpret_cast<hipStream_t>(hip_stream), d_makespan, nullptr, h_out);
}

int sched_eval_batch(const sched_problem* const* problems, int32_t n_problems,
                     const int32_t* replica_problem, const sched_lat* replica_lat,
                     int32_t n_replicas, void* d_workspace, size_t ws_bytes, void* hip_stream,
                     sched_result* h_out) {
  if (problems == nullptr || replica_problem == nullptr || replica_lat == nullptr ||
      h_out == nullptr)
    return SCHED_E_NULL;
  if (n_problems < 1 || n_replicas < 1) return SCHED_E_SIZE;
  for (int32_t i = 0; i < n_problems; ++i)
    if (problems[i] == nullptr) return SCHED_E_NULL;
  const size_t R = size_t(n_replicas);
  for (size_t r = 0; r < R; ++r)
    if (replica_problem[r] < 0 || replica_problem[r] >= n_problems) return SCHED_E_RANGE;
  const size_t stride = batch_stride(problems, n_problems);
  const Layout L = layout_for(batch_table_bytes(stride, R), partial_capacity(R), R);
  int rc = check_workspace(d_workspace, ws_bytes, L.total);
  if (rc != SCHED_OK) return rc;

  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  char* const ws = static_cast<char*>(d_workspace);
  uint32_t* const d_tables = reinterpret_cast<uint32_t*>(ws + L.tables);
  try {
    std::vector<size_t> lat_off(R);
    size_t off = 0;
    for (size_t r = 0; r < R; ++r) {
      lat_off[r] = off;
      off += size_t(problems[replica_problem[r]]->n);
    }
    std::vector<Launch> launches;
    std::vector<int32_t> order;  // replicas in launch order
    plan_batch(problems, n_problems, replica_problem, R, launches, order);

    // The tables: what does not depend on latencies once per problem, then
    // each replica's latencies; behind them each launch's first blocks.
    std::vector<uint32_t> host(batch_table_bytes(stride, R) / 4);
    std::vector<uint32_t> laid(stride + kBoundWords * kMaxTools);  // (with room for a bound table)
    uint32_t* first = host.data() + R * stride;
    for (Launch& g : launches) {
      const sched_problem* built = nullptr;
      for (size_t i = g.first; i < g.last; ++i) {
        const int32_t r = order[i];
        const sched_problem& p = *problems[replica_problem[r]];
        uint32_t* const tb = host.data() + i * stride;
        if (&p != built) {
          rc = lay_replica(p, g, laid.data());
          if (rc != SCHED_OK) return rc;
          built = &p;
        }
        std::copy_n(laid.data(), bound_base(laid[kHdrN], laid[kHdrLevels]), tb);
        rc = fill_latencies(p, replica_lat + lat_off[r], tb, false);
        if (rc != SCHED_OK) return rc;
        g.a.lds_levels = std::max(g.a.lds_levels, table_levels(p));
      }
      // Blocks in proportion to the tables' mappings, one per work item at
      // most and at least one each.
      const uint64_t most = partial_capacity(R), count = g.last - g.first;
      uint32_t blocks = 0;
      for (size_t i = g.first; i < g.last; ++i) {
        const unsigned __int128 m = problems[replica_problem[order[i]]]->n_mappings;
        const uint64_t share = uint64_t(m * (most - count) / g.work) + 1;
        *first++ = blocks;
        blocks += uint32_t(std::min(table_items(host.data() + i * stride), share));
      }
      *first++ = blocks;
      g.a.n_blocks = blocks;
    }

    std::vector<DevResult> res(R);  // (nothing is allocated from the copy to the wait)
    StreamWait wait(s);
    HIP_TRY(hipMemcpyAsync(d_tables, host.data(), host.size() * 4, hipMemcpyHostToDevice, s));
    std::optional<Slot> slot;
    if (R * sizeof(DevResult) <= kSlotBytes) slot.emplace(s);
    char* const h = slot ? slot->data() : nullptr;
    DevResult* const results = reinterpret_cast<DevResult*>(h ? h : ws + L.results);
    const uint32_t* d_first = d_tables + R * stride;
    if (h) slot->launched();
    for (Launch& g : launches) {
      SearchArgs& a = g.a;
      a.tables = d_tables + g.first * stride;
      a.table_stride = uint32_t(stride);
      a.block_first = d_first;
      a.partials = reinterpret_cast<Partial*>(ws + L.partials);
      a.results = results + g.first;
      HIP_TRY(launch_search(g.lay, a, s));
      d_first += g.last - g.first + 1;
    }
    if (!h)
      HIP_TRY(hipMemcpyAsync(res.data(), results, R * sizeof(DevResult), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    wait.waited();
    if (h) {
      slot->waited();
      std::memcpy(res.data(), h, R * sizeof(DevResult));
    }
    for (size_t i = 0; i < R; ++i) {
      h_out[order[i]].best_index = res[i].index;
      h_out[order[i]].makespan_us = res[i].makespan;
    }
  } catch (const std::bad_alloc&) {
    return SCHED_E_NOMEM;
  }
  return SCHED_OK;
}

int sched_eval_mappings_device(const sched_problem* p, const uint64_t* d_idx, int64_t n,
                               int64_t* d_makespan, void* d_workspace, size_t ws_bytes,
                               void* hip_stream) {
  if (p == nullptr) return SCHED_E_NULL;
  if (n < 0) return SCHED_E_SIZE;
  if (n == 0) return SCHED_OK;
  if (d_idx == nullptr || d_makespan == nullptr) return SCHED_E_NULL;
  const size_t need = align_up(size_t(p->table_words) * 4);
  int rc = check_workspace(d_workspace, ws_bytes, need);
  if (rc != SCHED_OK) return rc;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  uint32_t flags = p->sharing ? kEvalSharing : 0u;
  const uint32_t* tab = p->table.data();
  StreamWait wait(s);
  if (fits_arguments(tab)) {
    flags |= kEvalHostTable;
  } else {
    HIP_TRY(hipMemcpyAsync(d_workspace, tab, size_t(p->table_words) * 4, hipMemcpyHostToDevice, s));
    tab = static_cast<const uint32_t*>(d_workspace);
  }
  HIP_TRY(launch_eval(p->n, tab, d_idx, n, p->n_mappings, d_makespan, flags, s));
  HIP_TRY(hipStreamSynchronize(s));
  wait.waited();
  return SCHED_OK;
}

int sched_eval_mappings(const sched_problem* p, const uint64_t* h_idx, int64_t n,
                        void* d_workspace, size_t ws_bytes, void* hip_stream,
                        int64_t* h_makespan) {
  if (p == nullptr) return SCHED_E_NULL;
  if (n < 0) return SCHED_E_SIZE;
  if (n == 0) return SCHED_OK;
  if (h_idx == nullptr || h_makespan == nullptr) return SCHED_E_NULL;
  for (int64_t i = 0; i < n; ++i)
    if (h_idx[i] >= p->n_mappings) return SCHED_E_RANGE;
  // the table, then chunks of indices in the rest of the workspace, overwritten
  // by their makespans
  const size_t head = align_up(size_t(p->table_words) * 4);
  int rc = check_workspace(d_workspace, ws_bytes, head + kAlign + 16);
  if (rc != SCHED_OK) return rc;
  const int64_t chunk = int64_t(std::min<size_t>((ws_bytes - head - kAlign) / 8, size_t(1) << 24));
  char* ws = static_cast<char*>(d_workspace);
  uint64_t* d_idx = reinterpret_cast<uint64_t*>(ws + head);
  int64_t* d_out = reinterpret_cast<int64_t*>(d_idx);  // (each index read before it is overwritten)
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  for (int64_t at = 0; at < n; at += chunk) {
    const int64_t m = std::min(chunk, n - at);
    rc = score(*p, p->table.data(), h_idx + at, size_t(m), h_makespan + at,
               reinterpret_cast<uint32_t*>(ws), d_idx, d_out, s);
    if (rc != SCHED_OK) return rc;
  }
  return SCHED_OK;
}

int sched_eval_reprobes(const sched_problem* p, uint64_t base_index, const sched_lat* lat,
                        void* d_workspace, size_t ws_bytes, void* hip_stream,
                        sched_probe* h_out, int32_t capacity, int32_t* n_out) {
  if (p == nullptr || h_out == nullptr || n_out == nullptr) return SCHED_E_NULL;
  if (base_index >= p->n_mappings) return SCHED_E_RANGE;
  const int n = p->n;
  const int64_t worst = 1 + 2 * int64_t(n) + int64_t(n) * (n - 1);
  if (capacity < worst) return SCHED_E_SIZE;
  const Layout L = one_table_layout(*p);
  int rc = check_workspace(d_workspace, ws_bytes, L.total);
  if (rc != SCHED_OK) return rc;

  std::vector<uint32_t> table;
  std::vector<uint64_t> idx;
  std::vector<int64_t> ms;
  std::vector<Cand> cands;
  try {
    table = p->table;
    idx.reserve(size_t(worst));
    neighbourhood(*p, base_index, idx, cands);
    ms.assign(idx.size(), 0);
  } catch (const std::bad_alloc&) {
    return SCHED_E_NOMEM;
  }
  if (lat != nullptr) {
    rc = fill_latencies(*p, lat, table.data(), false);
    if (rc != SCHED_OK) return rc;
  }
  const size_t m = idx.size();
  // Scratch for the index list and the makespans: the partials region.
  if (m * 16 > partial_capacity(1) * sizeof(Partial)) return SCHED_E_WORKSPACE;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(d_workspace);
  uint64_t* d_idx = reinterpret_cast<uint64_t*>(ws + L.partials);
  int64_t* d_ms = reinterpret_cast<int64_t*>(ws + L.partials + m * 8);
  rc = score(*p, table.data(), idx.data(), m, ms.data(), reinterpret_cast<uint32_t*>(ws + L.tables),
             d_idx, d_ms, s);
  if (rc != SCHED_OK) return rc;
  // Keep a swap only when its move to gpu_now was infeasible.
  int32_t out = 0;
  int64_t move_ms = 0;
  for (size_t k = 0; k < m; ++k) {
    const Cand& c = cands[k];
    if (c.kind == 1) move_ms = ms[k];
    if (c.kind == 2 && move_ms != INT64_MAX) continue;
    sched_probe& pr = h_out[out++];
    pr.index = idx[k];
    pr.makespan_us = ms[k];
    pr.kind = c.kind;
    pr.tool = c.tool;
    pr.mode = c.mode;
    pr.swap_tool = c.swap_tool;
  }
  *n_out = out;
  return SCHED_OK;
}

int sched_pruned_workspace_bytes(const sched_problem* p, size_t* out) {
  if (p == nullptr || out == nullptr) return SCHED_E_NULL;
  size_t need = one_search_bytes(*p);
  try {
    if (p->n_mappings >= kPruneMinSpace)
      need = std::max(need, prune_layout(*p, plan_prune(*p)).total);
  } catch (const std::bad_alloc&) {
    return SCHED_E_NOMEM;
  }
  *out = need;
  return SCHED_OK;
}

int sched_pruned_argmin(const sched_problem* p, void* d_workspace, size_t ws_bytes,
                        void* hip_stream, sched_result* h_out, sched_prune_stats* stats) {
  if (p == nullptr || h_out == nullptr) return SCHED_E_NULL;
  sched_prune_stats st{};
  if (p->n_mappings < kPruneMinSpace) {  // not worth bounding: one exhaustive search
    const int rc = sched_bruteforce_argmin(p, 0, p->n_mappings, d_workspace, ws_bytes, hip_stream,
                                           h_out);
    if (rc == SCHED_OK && stats != nullptr) {
      st.prefixes = 1;
      st.prefixes_searched = 1;
      st.mappings_searched = p->n_mappings;
      st.launches = 1;
      SearchArgs a{};
      plan_full(*p, a);
      st.shared_prefix_launches = shares_prefixes(a);
      st.initial_bound_us = INT64_MAX;
      *stats = st;
    }
    return rc;
  }
  const int n = p->n;
  PrunePlan pl;
  try {
    pl = plan_prune(*p);
  } catch (const std::bad_alloc&) {
    return SCHED_E_NOMEM;
  }
  const PruneLayout L = prune_layout(*p, pl);
  int rc = check_workspace(d_workspace, ws_bytes, L.total);
  if (rc != SCHED_OK) return rc;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(d_workspace);
  const uint32_t* d_tab = reinterpret_cast<const uint32_t*>(ws + L.tables);
  const uint32_t stride = p->table_words;

  try {
    // 1. Upper bound: steepest descent over the what-if neighbourhood of
    // Algorithm 1 (every single-tool move and swap), from index 0.
    uint64_t ub_x = 0;
    int64_t ub_ms = INT64_MAX;
    {
      std::vector<uint64_t> idx;
      std::vector<Cand> cands;
      std::vector<int64_t> ms;
      uint64_t x = 0;
      for (int round = 0; round < 4 * n + 4; ++round) {
        neighbourhood(*p, x, idx, cands);
        ms.assign(idx.size(), 0);
        uint64_t* d_idx = reinterpret_cast<uint64_t*>(ws + L.probe_idx);
        int64_t* d_ms = reinterpret_cast<int64_t*>(ws + L.probe_ms);
        rc = score(*p, p->table.data(), idx.data(), idx.size(), ms.data(),
                   reinterpret_cast<uint32_t*>(ws + L.tables), d_idx, d_ms, s);
        if (rc != SCHED_OK) return rc;
        ++st.descent_rounds;
        size_t best = 0;
        for (size_t k = 1; k < idx.size(); ++k)
          if (ms[k] < ms[best] || (ms[k] == ms[best] && idx[k] < idx[best])) best = k;
        if (ms[best] < ub_ms || (ms[best] == ub_ms && idx[best] < ub_x)) {
          ub_ms = ms[best];
          ub_x = idx[best];
        }
        if (best == 0) break;  // no neighbour improves on x
        x = idx[best];
      }
    }
    st.initial_bound_us = ub_ms;

    // 2. Bounds of every prefix assignment.
    std::vector<uint32_t> btab(p->table);
    std::vector<int32_t> seq(pl.prefix);
    for (int32_t v : p->enum_tools)
      if (std::find(pl.prefix.begin(), pl.prefix.end(), v) == pl.prefix.end()) seq.push_back(v);
    set_enumeration(*p, seq, btab.data());
    uint64_t known = 0;
    for (int32_t v : pl.prefix) known |= 1ull << p->table[pos_base(uint32_t(n)) + uint32_t(v)];
    for (int v = 0; v < n; ++v)
      if (p->radix[v] == 1) known |= 1ull << p->table[pos_base(uint32_t(n)) + uint32_t(v)];
    uint32_t* d_count = reinterpret_cast<uint32_t*>(ws + L.bounds);
    uint2* d_live = reinterpret_cast<uint2*>(ws + L.bounds + align_up(4));
    const uint32_t ub32 = ub_ms == INT64_MAX ? kInf - 1 : uint32_t(ub_ms);
    // Bounds of m assignments by btab, of at most `bound`, to out; *live: how many.
    const auto bounds = [&](size_t tools, int64_t m, uint32_t bound, uint2* out, uint32_t* live) {
      StreamWait wait(s);
      HIP_TRY(hipMemcpyAsync(ws + L.tables, btab.data(), size_t(stride) * 4, hipMemcpyHostToDevice,
                             s));
      HIP_TRY(hipMemsetAsync(d_count, 0, 4, s));
      HIP_TRY(launch_bound(n, d_tab, uint32_t(tools), known, m, bound, d_count, out, s));
      HIP_TRY(hipMemcpyAsync(live, d_count, 4, hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));
      wait.waited();
      return int64_t(*live) > m ? SCHED_E_DEVICE : SCHED_OK;
    };
    uint32_t n_live = 0;
    rc = bounds(pl.prefix.size(), int64_t(pl.n_prefixes), ub32, d_live, &n_live);
    if (rc != SCHED_OK) return rc;
    std::vector<uint2> raw(n_live);
    if (n_live) {
      StreamWait wait(s);
      HIP_TRY(hipMemcpyAsync(raw.data(), d_live, size_t(n_live) * 8, hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));
      wait.waited();
    }
    st.prefixes = pl.n_prefixes;
    st.prefix_tools = int32_t(pl.prefix.size());

    // Survivors: bound <= upper bound (equal bounds may hide a lower index),
    // most promising first; the kernel appends them in no fixed order.
    std::vector<std::pair<uint32_t, uint64_t>> live(n_live);
    for (uint32_t i = 0; i < n_live; ++i) live[i] = {raw[i].x, raw[i].y};
    std::sort(live.begin(), live.end());

    // 3. Chunks of survivors, most promising first: their children's bounds,
    // then a search over the rest of the children that survive, or of the
    // chunk (one table; the list of either gives the outer combinations their
    // upper digits).  rest_of: what the tools in `fixed` leave free.
    const auto rest_of = [&](const std::vector<int32_t>& fixed) {
      sched_problem r = *p;
      for (int32_t v : fixed) r.allowed[v] = uint8_t(1u << mode_of_digit(*p, v, 0));
      r.enum_tools.clear();
      r.n_mappings = 1;
      for (int v = 0; v < n; ++v) {
        const uint8_t a = r.allowed[v];
        r.radix[v] = uint8_t((a & 1) + ((a >> 1) & 1) + ((a >> 2) & 1));
        if (r.radix[v] > 1) r.enum_tools.push_back(v);
        r.n_mappings *= r.radix[v];
      }
      return r;
    };
    std::vector<int32_t> both(pl.prefix);
    both.insert(both.end(), pl.ext.begin(), pl.ext.end());
    const sched_problem child_rest = rest_of(both);
    std::optional<sched_problem> prefix_rest;
    // (a table counts the outer combinations of a listed assignment in a word)
    const bool prefix_outer_fits = pl.subspace <= 0xFFFFFFFFull;
    seq = both;
    for (int32_t v : child_rest.enum_tools) seq.push_back(v);
    set_enumeration(*p, seq, btab.data());
    for (int32_t v : pl.ext) known |= 1ull << p->table[pos_base(uint32_t(n)) + uint32_t(v)];
    uint2* const d_chunk = d_live;
    uint2* const d_children = d_live + L.chunk;
    const auto put_address = [](uint32_t* table, uint32_t word, const void* at) {
      table[word] = uint32_t(reinterpret_cast<uintptr_t>(at));
      table[word + 1] = uint32_t(uint64_t(reinterpret_cast<uintptr_t>(at)) >> 32);
    };
    put_address(btab.data(), kHdrParentLo, d_chunk);
    btab[kHdrParents] = uint32_t(pl.n_prefixes);
    btab[kHdrChildren] = uint32_t(pl.n_children);
    std::vector<uint32_t> stab(p->table);

    uint64_t best_x = ub_ms == INT64_MAX ? ~0ull : ub_x;
    int64_t best_ms = ub_ms;
    std::vector<uint2> chunk;
    size_t next = 0;
    while (next < live.size()) {
      if (best_ms != INT64_MAX && int64_t(live[next].first) > best_ms) break;
      chunk.clear();
      const size_t most = next == 0 && live.size() > 2 * kFirstPrefixes
                              ? std::min<size_t>(L.chunk, kFirstPrefixes) : L.chunk;
      while (next < live.size() && chunk.size() < most &&
             (best_ms == INT64_MAX || int64_t(live[next].first) <= best_ms)) {
        chunk.push_back(make_uint2(live[next].first, uint32_t(live[next].second)));
        ++next;
      }
      st.prefixes_searched += chunk.size();
      const int64_t candidates = int64_t(chunk.size() * pl.n_children);
      uint32_t n_rest = 0;
      DevResult r;
      StreamWait wait(s);
      HIP_TRY(hipMemcpyAsync(d_chunk, chunk.data(), chunk.size() * 8, hipMemcpyHostToDevice, s));
      rc = bounds(both.size(), candidates, best_ms == INT64_MAX ? kInf - 1 : uint32_t(best_ms),
                  d_children, &n_rest);
      if (rc != SCHED_OK) return rc;
      if (n_rest == 0) {
        wait.waited();
        continue;
      }
      // Where their bounds rule out less than a quarter of the children, the
      // prefixes are searched themselves: a wave's lanes then share a prefix in
      // place of holding several children, which differ in tools that act
      // early.  30 tools, 76 % left: 39.2 ms by child, 25.0 by prefix; between
      // a half and three quarters left the children are mostly the shorter way
      // (32 tools, 52 %: 3.9 and 6.3 ms).
      const bool whole = 4 * int64_t(n_rest) > 3 * candidates && prefix_outer_fits;
      if (whole && !prefix_rest) prefix_rest.emplace(rest_of(pl.prefix));
      const sched_problem& sub = whole ? *prefix_rest : child_rest;
      const std::vector<int32_t>& upper = whole ? pl.prefix : both;
      if (whole) n_rest = uint32_t(chunk.size());
      SearchArgs a{};
      plan_search(sub, 0, sub.n_mappings, n_rest, a);
      // One table over all of the children.
      const uint64_t rest = sub.n_mappings / a.inner_count;  // outer combinations of a child
      const Seq low = enumeration(sub, true, int(a.inner_digits), (a.prefix | a.thin) != 0);
      seq.assign(low.v, low.v + low.n);
      seq.insert(seq.end(), upper.begin(), upper.end());
      set_enumeration(*p, seq, stab.data());
      a.outer_lo = 0;
      a.n_outer = rest * n_rest;
      a.n_tables = 1;
      a.lanes = 64;
      a.items_per_table = (a.n_outer + kBlock - 1) / kBlock;
      a.blocks_per_table = a.n_blocks =
          uint32_t(std::min<uint64_t>(a.items_per_table, kMaxBlocks));
      write_walk(a, stab.data());
      put_address(stab.data(), kHdrListLo, whole ? d_chunk : d_children);
      stab[kHdrListRest] = uint32_t(rest);
      if (fits_arguments(stab.data())) {
        a.host_table = stab.data();
        a.host_words = bound_base(uint32_t(n), a.lds_levels);
      } else {
        a.tables = d_tab;
        HIP_TRY(hipMemcpyAsync(ws + L.tables, stab.data(), size_t(stride) * 4,
                               hipMemcpyHostToDevice, s));
      }
      a.table_stride = stride;
      a.partials = reinterpret_cast<Partial*>(ws + L.partials);
      a.results = reinterpret_cast<DevResult*>(ws + L.results);
      HIP_TRY(launch_search(n, a, s));
      HIP_TRY(hipMemcpyAsync(&r, a.results, sizeof(r), hipMemcpyDeviceToHost, s));
      HIP_TRY(hipStreamSynchronize(s));
      wait.waited();
      if (r.makespan < best_ms || (r.makespan == best_ms && r.index < best_x)) {
        best_ms = r.makespan;
        best_x = r.index;
      }
      st.mappings_searched += uint64_t(n_rest) * sub.n_mappings;
      st.launches += 1;
      st.shared_prefix_launches += shares_prefixes(a);
    }
    h_out->best_index = best_ms == INT64_MAX ? ~0ull : best_x;
    h_out->makespan_us = best_ms;
  } catch (const std::bad_alloc&) {
    return SCHED_E_NOMEM;
  }
  if (stats != nullptr) *stats = st;
  return SCHED_OK;
}

int sched_valu_probe(uint32_t blocks, uint32_t iters, uint32_t* d_out, void* hip_stream,
                     double* lane_ops) {
  if (d_out == nullptr || lane_ops == nullptr) return SCHED_E_NULL;
  if (blocks == 0 || iters == 0 || blocks > (1u << 24)) return SCHED_E_SIZE;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  double ops = 0;
  HIP_TRY(launch_valu_probe(blocks, iters, d_out, s, &ops));
  HIP_TRY(hipStreamSynchronize(s));
  *lane_ops = ops;
  return SCHED_OK;
}

int sched_wave_or_probe(const uint64_t* d_in, const uint8_t* d_active, uint32_t blocks,
                        uint64_t* d_out64, uint32_t* d_out32, void* hip_stream) {
  if (d_in == nullptr || d_active == nullptr || d_out64 == nullptr || d_out32 == nullptr)
    return SCHED_E_NULL;
  if (blocks == 0 || blocks > (1u << 16)) return SCHED_E_SIZE;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  HIP_TRY(launch_wave_or_probe(d_in, d_active, blocks, d_out64, d_out32, s));
  HIP_TRY(hipStreamSynchronize(s));
  return SCHED_OK;
}

const char* sched_strerror(int code) {
  switch (code) {
    case SCHED_OK: return "ok";
    case SCHED_E_NULL: return "null pointer argument";
    case SCHED_E_SIZE: return "size out of range";
    case SCHED_E_VALUE: return "value out of range";
    case SCHED_E_EDGE: return "edge endpoint out of range or self-loop";
    case SCHED_E_CYCLE: return "edges contain a cycle";
    case SCHED_E_RANGE: return "index range or replica map out of range";
    case SCHED_E_OVERFLOW: return "times or VRAM sums would not fit the 32-bit device path";
    case SCHED_E_WORKSPACE: return "workspace null, misaligned or too small";
    case SCHED_E_DEVICE: return "HIP runtime error";
    case SCHED_E_NOMEM: return "host allocation failed";
    default: return "unknown error";
  }
}

}  // extern "C"
