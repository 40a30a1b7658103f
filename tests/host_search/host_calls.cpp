// host_calls.cpp -- test harness: the library's calls (api.cpp) on a stand-in
// for the HIP runtime, so that their host side can be checked on the CPU.
// Copies and launches wait in their stream's list, each with the arguments it
// was given, and run when the stream is waited for; "device" memory is host
// memory.  A launch over tables of HOST_CALLS_N tools (macro, a list) runs the
// kernels' per-lane code, one lane per wave, block by block; a closed-form
// launch scores the table's mappings one by one.
//
// argv[1] is the check to run; problems come on stdin, each as: n_tools share
// n_edges n_levels budget, then n_tools lines "gpu cpu load xfer mem allowed",
// n_edges lines "src dst", then the n_levels Q16 contention factors.
#include "../../paper_2607_22242_amd/csrc/api.cpp"
#include "../../paper_2607_22242_amd/csrc/kernels.h"

#include <pthread.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <string>

#ifndef HOST_CALLS_N
#define HOST_CALLS_N 6, 10, 15, 34
#endif

// ---------------------------------------------------------------------------
// The runtime.

static std::mutex g_mutex;
static std::map<hipStream_t, std::vector<std::function<void()>>> g_work;
static std::atomic<int> g_page_locked{0};     // successful hipHostMalloc calls
static std::atomic<int> g_fail_page_locked{0};  // calls that will fail
static bool g_plan_only = false;              // launches score nothing
static uint32_t g_most_blocks = 65536;        // partials that a workspace has room for
static thread_local long t_news = 0;          // heap allocations of this thread
static thread_local long t_last_news = -1;    // those after this number fail (-1: none)

static long g_calls = 0;                      // copies, fills and launches asked for
static long g_last_call = -1;                 // those after this number fail (-1: none)

static bool refused() { return ++g_calls > g_last_call && g_last_call >= 0; }

static void enqueue(hipStream_t s, std::function<void()> f) {
  std::lock_guard<std::mutex> lock(g_mutex);
  g_work[s].push_back(std::move(f));
}

static void* allocate(size_t n) {
  return ++t_news > t_last_news && t_last_news >= 0 ? nullptr : malloc(n);
}
void* operator new(size_t n) {
  if (void* p = allocate(n)) return p;
  throw std::bad_alloc();
}
void* operator new[](size_t n) { return operator new(n); }
void* operator new(size_t n, const std::nothrow_t&) noexcept { return allocate(n); }
void* operator new[](size_t n, const std::nothrow_t&) noexcept { return allocate(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete[](void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
void operator delete[](void* p, size_t) noexcept { free(p); }

// The stand-in's own allocations are not the library's.
struct Uncounted {
  long at = t_news, last = t_last_news;
  Uncounted() { t_last_news = -1; }
  ~Uncounted() {
    t_news = at;
    t_last_news = last;
  }
};

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (g_fail_page_locked > 0) {
    --g_fail_page_locked;
    return hipErrorOutOfMemory;
  }
  ++g_page_locked;
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  Uncounted u;
  if (refused()) return hipErrorUnknown;
  enqueue(st, [=] { memcpy(d, s, n); });
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  Uncounted u;
  if (refused()) return hipErrorUnknown;
  enqueue(st, [=] { memset(d, v, n); });
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
  Uncounted u;
  std::vector<std::function<void()>> w;
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    w.swap(g_work[st]);
  }
  for (auto& f : w) f();
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
}

// ---------------------------------------------------------------------------
// The kernels.

// What the launches did.
static std::atomic<int> g_launches{0}, g_shared{0}, g_max_tables{0};
static std::atomic<uint32_t> g_slots_held{0};  // by the calls of the launches

// Observer of a full-order launch: as RecordTo, and how often each mapping was
// scored by the launches over lists, if that is kept.
static std::vector<uint8_t>* g_times = nullptr;
struct Watch {
  uint32_t* out;
  std::vector<uint8_t>* times;
  bool on() const { return out != nullptr || times != nullptr; }
  void operator()(uint64_t x, uint32_t ms) const {
    if (out != nullptr) out[x] = ms;
    if (times != nullptr) ++times->at(x);
  }
};
// The y of the pairs of the lists that were walked, by the mappings that each
// entry stands for.
static std::map<uint64_t, std::vector<uint32_t>> g_listed;

namespace devmap {

template <int N, bool SHARE>
static uint32_t score_y(const uint32_t* tab, const uint32_t* lds, uint64_t y, uint64_t& x) {
  MaskT<N> gn, gq, slot = 0;
  decode_positions<N>(tab, y, 0, tab[kHdrPositions], gn, gq, x);
  if constexpr (SHARE)
    return evaluate_sharing<N>(tab, lds, tab[kHdrLevels], tab[kHdrBudget], gn, gq, &slot);
  else
    return evaluate<N>(tab, lds, tab[kHdrLevels], tab[kHdrBudget], gn, gq, &slot);
}

static void take_min(uint32_t& ms, uint64_t& x, uint32_t m, uint64_t y) {
  if (m < ms || (m == ms && y < x)) {
    ms = m;
    x = y;
  }
}

// One search launch, its table (if it came with the arguments) in `own`.
template <int N, bool SHARE>
static void search(const SearchArgs& a, const uint32_t* own) {
  std::vector<uint32_t> snap(snap_words<N, SHARE>() * kBlock);
  uint64_t word = 0;
  MaskT<N>* slot = reinterpret_cast<MaskT<N>*>(&word);
  uint32_t table = 0;
  for (uint32_t b = 0; b < a.n_blocks; ++b) {
    uint32_t bb, nb;
    if (a.block_first != nullptr) {
      while (a.block_first[table + 1] <= b) ++table;
      bb = b - a.block_first[table];
      nb = a.block_first[table + 1] - a.block_first[table];
    } else {
      nb = a.blocks_per_table;
      table = b / nb;
      bb = b % nb;
    }
    const uint32_t* tab = a.tables != nullptr ? a.tables + size_t(table) * a.table_stride : own;
    std::vector<uint32_t> lds(lds_words_for(N, tab[kHdrLevels]));
    stage_image<N>(tab, lds.data(), 0, 1);
    uint32_t ms = kInf;
    uint64_t x = ~0ull;
    if (a.closed != kClosedNone) {
      uint64_t total = 1;
      for (uint32_t k = 0; k < tab[kHdrPositions]; ++k)
        total *= opt_radix(tab[enum_opt_base(tab[kHdrN]) + k]);
      for (uint64_t y = bb; y < total; y += nb) {
        uint64_t yx;
        const uint32_t m = score_y<N, SHARE>(tab, lds.data(), y, yx);
        if (a.record) a.record[yx] = m;
        take_min(ms, x, m, m == kInf ? ~0ull : yx);
      }
    } else if (a.full_range) {
      const TabWalk walk{Tab{tab}};
      const bool listed = tab[kHdrListRest] != 0;
      const Watch rec{a.record, listed ? g_times : nullptr};
      if (listed && b == 0) {
        const uint2* const list = list_at(Tab{tab}, kHdrListLo);
        for (uint64_t k = 0; k < walk_n_outer(walk) / tab[kHdrListRest]; ++k)
          g_listed[uint64_t(tab[kHdrListRest]) * tab[kHdrInnerCount]].push_back(list[k].y);
      }
      const uint64_t items = (walk_n_outer(walk) + kBlock - 1) / kBlock;
      for (uint64_t item = bb; item < items; item += nb)
        for (uint32_t lane = 0; lane < uint32_t(kBlock); ++lane)
          if (tab[kHdrPrefix])
            lane_search_prefix<N, SHARE>(walk, tab, lds.data(), item, lane, slot,
                                         snap.data() + lane, ms, x, rec);
          else
            lane_search<N, true, SHARE>(walk, tab, lds.data(), item, lane, slot, ms, x, rec);
    } else {
      for (uint64_t item = bb; item < a.items_per_table; item += nb)
        for (uint32_t lane = 0; lane < uint32_t(kBlock); ++lane)
          lane_search<N, false, SHARE>(a, tab, lds.data(), item, lane, slot, ms, x);
    }
    a.partials[b] = Partial{x, ms, 0};
  }
}

template <int N>
static void eval(const EvalArgs& e, const uint32_t* tab, bool share) {
  std::vector<uint32_t> lds(lds_words<N>());
  stage_image<N>(tab, lds.data(), 0, 1);
  for (int64_t i = 0; i < e.n; ++i) {
    uint64_t x;
    const uint64_t y = e.idx[i];
    uint32_t ms = kInf;
    if (y < e.n_mappings)
      ms = share ? score_y<N, true>(tab, lds.data(), y, x) : score_y<N, false>(tab, lds.data(), y, x);
    e.out[i] = ms == kInf ? INT64_MAX : int64_t(ms);
  }
}

// Calls f with the integral constant of n among the tool counts built.
template <class F, int... NS>
static void on_tools(int n, F f, std::integer_sequence<int, NS...>) {
  const bool found = ((n == NS ? (f(std::integral_constant<int, NS>{}), true) : false) || ...);
  if (!found) {
    fprintf(stderr, "no kernel for %d tools\n", n);
    abort();
  }
}
using Built = std::integer_sequence<int, HOST_CALLS_N>;

hipError_t launch_search(int n, const SearchArgs& args, hipStream_t s) {
  Uncounted u;
  if (refused()) return hipErrorUnknown;
  std::vector<uint32_t> own;
  if (args.tables == nullptr) own.assign(args.host_table, args.host_table + args.host_words);
  ++g_launches;
  if (int(args.n_tables) > g_max_tables) g_max_tables = int(args.n_tables);
  {
    std::lock_guard<std::mutex> lock(g_slot_mutex);
    g_slots_held |= g_slots_taken;
  }
  enqueue(s, [=] {
    SearchArgs a = args;
    const uint32_t* tab = own.empty() ? a.tables : own.data();
    if (a.closed == kClosedNone && a.full_range && tab[kHdrPrefix]) ++g_shared;
    if (a.n_blocks > g_most_blocks) {
      fprintf(stderr, "a launch of %u blocks\n", a.n_blocks);
      exit(1);
    }
    if (g_plan_only)
      for (uint32_t b = 0; b < a.n_blocks; ++b) a.partials[b] = Partial{a.n_tables, a.n_blocks, 0};
    else
      on_tools(n, [&](auto N) {
        a.sharing ? search<N(), true>(a, own.data()) : search<N(), false>(a, own.data());
      }, Built{});
    if (a.results == nullptr) return;
    const uint32_t results = a.one_result ? 1u : a.n_tables;
    for (uint32_t r = 0; r < results; ++r) {
      const bool listed = !a.one_result && a.block_first != nullptr;
      const uint32_t per = a.n_blocks / results;
      const uint32_t lo = listed ? a.block_first[r] : r * per;
      const uint32_t hi = listed ? a.block_first[r + 1] : lo + per;
      uint32_t ms = kInf;
      uint64_t x = ~0ull;
      for (uint32_t b = lo; b < hi; ++b) take_min(ms, x, a.partials[b].makespan, a.partials[b].index);
      a.results[r] = DevResult{ms == kInf ? ~0ull : x, ms == kInf ? INT64_MAX : int64_t(ms)};
    }
  });
  return hipSuccess;
}

hipError_t launch_eval(int n, const uint32_t* tab, const uint64_t* idx, int64_t m,
                       uint64_t n_mappings, int64_t* out, uint32_t flags, hipStream_t s) {
  Uncounted u;
  if (refused()) return hipErrorUnknown;
  std::vector<uint32_t> own;
  if (flags & kEvalHostTable) own.assign(tab, tab + bound_base(uint32_t(n), tab[kHdrLevels]));
  enqueue(s, [=] {
    const uint32_t* t = own.empty() ? tab : own.data();
    const EvalArgs e{t, idx, m, n_mappings, out};
    on_tools(n, [&](auto N) { eval<N()>(e, t, (flags & kEvalSharing) != 0); }, Built{});
  });
  return hipSuccess;
}

hipError_t launch_bound(int n, const uint32_t* tab, uint32_t K, uint64_t known, int64_t m,
                        uint32_t ub, uint32_t* count, uint2* out, hipStream_t s) {
  Uncounted u;
  if (refused()) return hipErrorUnknown;
  enqueue(s, [=] {
    const uint2* const parents = list_at(Tab{tab}, kHdrParentLo);
    on_tools(n, [&](auto N) {
      for (int64_t k = 0; k < m; ++k) {
        const uint64_t y =
            bound_assignment(parents, tab[kHdrChildren], tab[kHdrParents], uint64_t(k));
        MaskT<N()> gn, gq;
        uint64_t x;
        decode_positions<N()>(tab, y, 0, K, gn, gq, x);
        const uint32_t lb = prefix_bound<N()>(tab, gn, gq, MaskT<N()>(known));
        if (lb != kInf && lb <= ub) out[(*count)++] = make_uint2(lb, uint32_t(y));
      }
    }, Built{});
  });
  return hipSuccess;
}
hipError_t launch_valu_probe(uint32_t, uint32_t, uint32_t*, hipStream_t, double*) {
  return hipErrorUnknown;
}
hipError_t launch_wave_or_probe(const uint64_t*, const uint8_t*, uint32_t, uint64_t*, uint32_t*,
                                hipStream_t) {
  return hipErrorUnknown;
}
hipError_t scratch_buffer(void** ptr, uint32_t** stage) {
  static char* const buf = static_cast<char*>(aligned_alloc(256, kScratchBytes));
  static uint32_t words[kStageWords];
  *ptr = buf;
  *stage = words;
  return hipSuccess;
}
}  // namespace devmap

using namespace devmap;

// ---------------------------------------------------------------------------
// Problems and workspaces.

static sched_problem* read_problem() {
  int n, share, ne, nl;
  long long budget;
  if (scanf("%d %d %d %d %lld", &n, &share, &ne, &nl, &budget) != 5) return nullptr;
  std::vector<sched_tool> tools(n);
  std::vector<uint8_t> allowed(n);
  for (int v = 0; v < n; ++v) {
    long long g, c, l, x, m;
    int al;
    if (scanf("%lld %lld %lld %lld %lld %d", &g, &c, &l, &x, &m, &al) != 6) return nullptr;
    tools[v] = sched_tool{g, c, l, x, m};
    allowed[v] = uint8_t(al);
  }
  std::vector<sched_edge> e(ne);
  for (auto& x : e)
    if (scanf("%d %d", &x.src, &x.dst) != 2) return nullptr;
  std::vector<uint32_t> f(nl);
  for (auto& x : f)
    if (scanf("%u", &x) != 1) return nullptr;
  sched_problem* p = nullptr;
  sched_problem_desc d{tools.data(), n, e.data(), ne, f.data(), nl, budget, allowed.data(), share};
  return sched_problem_create_desc(&d, &p) == SCHED_OK ? p : nullptr;
}

#define CHECK(cond)                                                   \
  do {                                                                \
    if (!(cond)) {                                                    \
      fprintf(stderr, "%s:%d: not %s\n", __FILE__, __LINE__, #cond);  \
      exit(1);                                                        \
    }                                                                 \
  } while (0)

struct Workspace {
  size_t bytes;
  void* p;
  explicit Workspace(size_t n) : bytes(n), p(aligned_alloc(256, (n + 255) / 256 * 256)) {}
  ~Workspace() { free(p); }
};

static size_t bytes_for(const std::vector<sched_problem*>& ps, int replicas) {
  size_t n = 0;
  CHECK(sched_workspace_bytes(ps.data(), int(ps.size()), replicas, &n) == SCHED_OK);
  return n;
}

// ---------------------------------------------------------------------------
// Checks.

// A range in parts, called with little stack: both entry points, and no heap
// allocation in the one that promises none.
static sched_problem* g_problem;
static void* range_call(void*) {
  sched_problem* const p = g_problem;
  Workspace ws(bytes_for({p}, 0));
  sched_result a{}, b{};
  const uint64_t lo = 1, hi = p->n_mappings - 1;
  CHECK(sched_bruteforce_argmin(p, lo, hi, ws.p, ws.bytes, nullptr, &a) == SCHED_OK);
  CHECK(a.best_index > 1);  // (the tables of the launch)
  const long news = t_news;
  CHECK(sched_bruteforce_argmin_noalloc(p, lo, hi, nullptr, &b) == SCHED_OK);
  CHECK(t_news == news);
  CHECK(a.best_index == b.best_index && a.makespan_us == b.makespan_us);
  return nullptr;
}
static void check_stack() {
  g_plan_only = true;
  CHECK((g_problem = read_problem()) != nullptr);
  CHECK(range_in_parts(*g_problem, 1, g_problem->n_mappings - 1));
  pthread_attr_t attr;
  pthread_attr_init(&attr);
  CHECK(pthread_attr_setstacksize(&attr, 64 << 10) == 0);
  pthread_t t;
  CHECK(pthread_create(&t, &attr, range_call, nullptr) == 0);
  pthread_join(t, nullptr);
}

// The counters of a pruned search over a space that is searched whole, against
// what was launched; prints the launches that shared prefixes.
static void check_stats() {
  g_plan_only = true;
  sched_problem* const p = read_problem();
  CHECK(p != nullptr);
  size_t n = 0;
  CHECK(sched_pruned_workspace_bytes(p, &n) == SCHED_OK);
  Workspace ws(n);
  sched_result r;
  sched_prune_stats st;
  CHECK(sched_pruned_argmin(p, ws.p, ws.bytes, nullptr, &r, &st) == SCHED_OK);
  CHECK(st.launches == g_launches && st.shared_prefix_launches == g_shared);
  printf("%d\n", st.shared_prefix_launches);
}

// The calls that use slots, against each other's answers: with slots, with none
// to be had, and with all of them taken.  A failed allocation is tried again.
struct Answers {
  std::vector<sched_result> search;
  std::vector<int64_t> scores;
  std::vector<sched_probe> probes;
  std::vector<sched_result> batch;
  bool operator==(const Answers& o) const {
    const auto same = [](const auto& a, const auto& b, auto eq) {
      return a.size() == b.size() && std::equal(a.begin(), a.end(), b.begin(), eq);
    };
    const auto res = [](const sched_result& a, const sched_result& b) {
      return a.best_index == b.best_index && a.makespan_us == b.makespan_us;
    };
    const auto probe = [](const sched_probe& a, const sched_probe& b) {
      return a.index == b.index && a.makespan_us == b.makespan_us && a.kind == b.kind &&
             a.tool == b.tool && a.mode == b.mode && a.swap_tool == b.swap_tool;
    };
    return same(search, o.search, res) && scores == o.scores && same(probes, o.probes, probe) &&
           same(batch, o.batch, res);
  }
};

static Answers call_all(const std::vector<sched_problem*>& ps, int replicas, hipStream_t s) {
  Answers out;
  Workspace ws(bytes_for(ps, replicas));
  for (sched_problem* p : ps) {
    sched_result r{};
    CHECK(sched_bruteforce_argmin(p, 0, p->n_mappings, ws.p, ws.bytes, s, &r) == SCHED_OK);
    out.search.push_back(r);
    CHECK(sched_bruteforce_argmin(p, 1, p->n_mappings, ws.p, ws.bytes, s, &r) == SCHED_OK);
    out.search.push_back(r);
    for (size_t m : {size_t(700), size_t(2048), size_t(2049)}) {
      std::vector<uint64_t> idx(m);
      for (size_t k = 0; k < m; ++k) idx[k] = (k * 7919) % p->n_mappings;
      std::vector<int64_t> ms(m, -1);
      CHECK(sched_eval_mappings(p, idx.data(), int64_t(m), ws.p, ws.bytes, s, ms.data()) == SCHED_OK);
      out.scores.insert(out.scores.end(), ms.begin(), ms.end());
    }
    std::vector<sched_probe> pr(size_t(1 + 2 * p->n + p->n * (p->n - 1)));
    int32_t n = 0;
    CHECK(sched_eval_reprobes(p, p->n_mappings / 2, nullptr, ws.p, ws.bytes, s, pr.data(),
                              int32_t(pr.size()), &n) == SCHED_OK);
    out.probes.insert(out.probes.end(), pr.begin(), pr.begin() + n);
  }
  std::vector<int32_t> of;
  std::vector<sched_lat> lat;
  for (int r = 0; r < replicas; ++r) {
    const sched_problem* const p = ps[size_t(r) % ps.size()];
    of.push_back(int32_t(size_t(r) % ps.size()));
    for (const sched_tool& t : p->tools)
      lat.push_back({t.gpu_us + r, t.cpu_us + 3 * r, t.load_us + 2 * r, t.xfer_us + r});
  }
  out.batch.resize(size_t(replicas));
  CHECK(sched_eval_batch(ps.data(), int(ps.size()), of.data(), lat.data(), replicas, ws.p, ws.bytes, s,
                         out.batch.data()) == SCHED_OK);
  return out;
}

// Every allocation of every call fails in turn (or every copy, fill and launch):
// the call says so, and nothing is left in its stream (which would go on in
// memory that is no longer there).
static void check_failures(bool runtime) {
  std::vector<sched_problem*> ps;
  while (sched_problem* p = read_problem()) ps.push_back(p);
  CHECK(ps.size() >= 2);
  sched_problem* const wide = ps.back();  // (a table too large for a kernel's arguments)
  ps.pop_back();
  sched_problem* const big = ps.back();  // (the others are small)
  ps.pop_back();
  CHECK(!fits_arguments(wide->table.data()));
  g_plan_only = true;
  const int R = 2100;  // (more results than a slot holds)
  size_t pruned = 0;
  CHECK(sched_pruned_workspace_bytes(big, &pruned) == SCHED_OK);
  Workspace ws(std::max({bytes_for(ps, R), bytes_for({big}, 0), bytes_for({wide}, 0), pruned}));
  std::vector<int32_t> of;
  std::vector<sched_lat> lat;
  for (int r = 0; r < R; ++r) {
    of.push_back(int32_t(size_t(r) % ps.size()));
    for (const sched_tool& t : ps[size_t(r) % ps.size()]->tools)
      lat.push_back({t.gpu_us, t.cpu_us, t.load_us, t.xfer_us});
  }
  std::vector<sched_result> res(size_t(R), sched_result{7, 7});
  std::vector<sched_probe> pr(size_t(1 + 2 * big->n + big->n * (big->n - 1)));
  std::vector<uint64_t> idx(3000, 1);
  std::vector<int64_t> ms(3000);
  int32_t n = 0;
  const std::vector<std::function<int()>> calls = {
      [&] { return sched_bruteforce_argmin(big, 0, big->n_mappings, ws.p, ws.bytes, nullptr, res.data()); },
      [&] { return sched_bruteforce_argmin(big, 1, big->n_mappings, ws.p, ws.bytes, nullptr, res.data()); },
      [&] { return sched_eval_mappings(big, idx.data(), 3000, ws.p, ws.bytes, nullptr, ms.data()); },
      [&] { return sched_eval_reprobes(big, 0, nullptr, ws.p, ws.bytes, nullptr, pr.data(),
                                       int32_t(pr.size()), &n); },
      [&] { return sched_eval_batch(ps.data(), int(ps.size()), of.data(), lat.data(), 3, ws.p, ws.bytes,
                                    nullptr, res.data()); },
      [&] { return sched_eval_batch(ps.data(), int(ps.size()), of.data(), lat.data(), R, ws.p, ws.bytes,
                                    nullptr, res.data()); },
      [&] { return sched_pruned_argmin(big, ws.p, ws.bytes, nullptr, res.data(), nullptr); },
      [&] { return sched_pruned_workspace_bytes(big, &pruned); },
      [&] { return sched_bruteforce_argmin(wide, 0, 8, ws.p, ws.bytes, nullptr, res.data()); },
      [&] { return sched_eval_mappings(wide, idx.data(), 3000, ws.p, ws.bytes, nullptr, ms.data()); },
      [&] { return sched_eval_mappings_device(wide, idx.data(), 3000, ms.data(), ws.p, ws.bytes, nullptr); }};
  const int failed = runtime ? SCHED_E_DEVICE : SCHED_E_NOMEM;
  for (const auto& call : calls) {
    int rc = failed;
    for (long k = 0; rc != SCHED_OK; ++k) {
      res[0] = sched_result{7, 7};
      if (runtime) g_last_call = g_calls + k;
      else t_last_news = t_news + k;
      rc = call();
      t_last_news = g_last_call = -1;
      CHECK(rc == SCHED_OK || (rc == failed && res[0].best_index == 7));
      CHECK(g_work[nullptr].empty());
      CHECK(g_slots_taken == 0);
    }
  }
}

static void check_slots() {
  std::vector<sched_problem*> ps;
  while (sched_problem* p = read_problem()) ps.push_back(p);
  CHECK(!ps.empty());
  g_fail_page_locked = 1 << 20;
  const Answers none = call_all(ps, 20, nullptr);
  CHECK(g_page_locked == 0 && g_slots == nullptr);
  g_fail_page_locked = 0;
  const Answers some = call_all(ps, 20, nullptr);
  CHECK(g_page_locked == 1 && g_slots_taken == 0);
  CHECK(some == none);
  {
    std::vector<std::unique_ptr<Slot>> all;
    for (int k = 0; k < kSlots; ++k) {
      all.push_back(std::make_unique<Slot>(nullptr));
      CHECK(all.back()->data() == g_slots + size_t(k) * kSlotBytes);
    }
    CHECK(Slot(nullptr).data() == nullptr);
    CHECK(call_all(ps, 20, nullptr) == none);
    all[3].reset();
    CHECK(Slot(nullptr).data() == g_slots + 3 * kSlotBytes);
    CHECK(call_all(ps, 20, nullptr) == none);
  }
  CHECK(g_page_locked == 1 && g_slots_taken == 0);
}

// Batches whose results fit a slot, fill it, and do not fit: each replica's
// answer is that of a search of its own.
static void check_replicas() {
  sched_problem* const p = read_problem();
  CHECK(p != nullptr);
  for (int R : {1, 2048, 2049, 3000}) {
    std::vector<int32_t> of(size_t(R), 0);
    std::vector<sched_lat> lat;
    for (int r = 0; r < R; ++r)
      for (const sched_tool& t : p->tools)
        lat.push_back({t.gpu_us + r % 37 * 1000, t.cpu_us + r % 5, t.load_us, t.xfer_us + r % 11});
    Workspace ws(bytes_for({p}, R));
    std::vector<sched_result> got(static_cast<size_t>(R));
    g_slots_held = 0;
    CHECK(sched_eval_batch(&p, 1, of.data(), lat.data(), R, ws.p, ws.bytes, nullptr, got.data()) ==
          SCHED_OK);
    CHECK(g_slots_held == (R <= 2048 ? 1u : 0u) && g_slots_taken == 0);
    for (int r = 0; r < R; r += R / 40 + 1) {
      sched_problem q = *p;
      CHECK(fill_latencies(q, &lat[size_t(r) * p->n], q.table_full.data(), true) == SCHED_OK);
      sched_result want{};
      CHECK(sched_bruteforce_argmin(&q, 0, q.n_mappings, ws.p, ws.bytes, nullptr, &want) == SCHED_OK);
      CHECK(want.best_index == got[r].best_index && want.makespan_us == got[r].makespan_us);
    }
  }
}

// Batches of the largest spaces: no launch has more blocks than the workspace
// has partials.
static void check_blocks() {
  g_plan_only = true;
  sched_problem* const p = read_problem();
  CHECK(p != nullptr);
  for (int R : {1, 2, 3, 7, 66000}) {
    const std::vector<int32_t> of(size_t(R), 0);
    std::vector<sched_lat> lat;
    for (int r = 0; r < R; ++r)
      for (const sched_tool& t : p->tools) lat.push_back({t.gpu_us, t.cpu_us, t.load_us, t.xfer_us});
    Workspace ws(bytes_for({p}, R));
    std::vector<sched_result> got(static_cast<size_t>(R));
    g_most_blocks = uint32_t(std::max(R, 65536));
    CHECK(sched_eval_batch(&p, 1, of.data(), lat.data(), R, ws.p, ws.bytes, nullptr, got.data()) ==
          SCHED_OK);
  }
}

// Workspaces from one table, the partials and a result upwards: every search
// takes them, a range in parts where they hold its tables.
static void check_room() {
  sched_problem* const p = read_problem();
  CHECK(p != nullptr);
  const size_t least = one_table_layout(*p).total, most = bytes_for({p}, 0);
  const uint64_t M = p->n_mappings;
  CHECK(range_in_parts(*p, 0, M) && most > least);
  Workspace ws(most);
  g_plan_only = true;
  for (size_t n : {least - 1, least, most - 1, most}) {
    const int want = n < least ? SCHED_E_WORKSPACE : SCHED_OK;
    sched_result r;
    std::vector<uint32_t> all(M);
    std::vector<sched_probe> pr(size_t(1 + 2 * p->n + p->n * (p->n - 1)));
    int32_t k = 0;
    CHECK(sched_bruteforce_argmin(p, 0, M, ws.p, n, nullptr, &r) == want);
    CHECK(sched_bruteforce_record(p, ws.p, n, nullptr, all.data(), M, &r) == want);
    CHECK(sched_eval_reprobes(p, 0, nullptr, ws.p, n, nullptr, pr.data(), int32_t(pr.size()), &k) ==
          want);
    g_max_tables = 0;
    CHECK(sched_bruteforce_argmin(p, 1, M, ws.p, n, nullptr, &r) == want);
    CHECK(n < least || (g_max_tables > 1) == (n == most));
  }
}

// A pruned search's launches over lists of children or prefixes: every mapping
// of a listed one is scored once, no other is; prints the answer and how many
// of either were listed.
static void check_children() {
  sched_problem* const p = read_problem();
  CHECK(p != nullptr && p->n_mappings >= kPruneMinSpace);
  const PrunePlan pl = plan_prune(*p);
  std::vector<uint8_t> times(p->n_mappings);
  g_times = &times;
  const size_t n = prune_layout(*p, pl).total;
  Workspace ws(n);
  sched_result r{};
  sched_prune_stats st{};
  CHECK(sched_pruned_argmin(p, ws.p, n, nullptr, &r, &st) == SCHED_OK);
  std::vector<uint32_t>& children = g_listed[pl.rest];
  std::vector<uint32_t>& prefixes = g_listed[pl.subspace];
  CHECK(g_listed.size() == 2 && pl.rest < pl.subspace && children.size() + prefixes.size() > 0);
  for (auto* list : {&children, &prefixes}) {
    std::sort(list->begin(), list->end());
    CHECK(std::adjacent_find(list->begin(), list->end()) == list->end());
  }
  std::vector<int32_t> upper(pl.prefix), modes(size_t(p->n));
  upper.insert(upper.end(), pl.ext.begin(), pl.ext.end());
  uint64_t scored = 0;
  for (uint64_t x = 0; x < p->n_mappings; ++x) {
    if (times[x] == 0) continue;
    CHECK(times[x] == 1);
    ++scored;
    CHECK(sched_mapping_modes(p, x, modes.data()) == SCHED_OK);
    uint64_t y = 0, w = 1;
    for (int32_t v : upper) {
      y += w * uint64_t(digit_of_mode(*p, v, modes[size_t(v)]));
      w *= p->radix[v];
    }
    CHECK(std::binary_search(children.begin(), children.end(), uint32_t(y)) !=
          std::binary_search(prefixes.begin(), prefixes.end(), uint32_t(y % pl.n_prefixes)));
  }
  CHECK(scored == children.size() * pl.rest + prefixes.size() * pl.subspace &&
        scored == st.mappings_searched);
  printf("%llu %lld %d %d %zu %zu\n", (unsigned long long)r.best_index, (long long)r.makespan_us,
         st.launches, st.shared_prefix_launches, children.size(), prefixes.size());
}

// The labels walked in closed form by a search of each problem (0: none), and
// by the launch each problem's replica has in a batch of one replica each.
static void check_closed() {
  std::vector<const sched_problem*> ps;
  while (const sched_problem* p = read_problem()) ps.push_back(p);
  std::vector<int32_t> of(ps.size()), order;
  std::iota(of.begin(), of.end(), 0);
  std::vector<Launch> launches;
  plan_batch(ps.data(), int32_t(ps.size()), of.data(), ps.size(), launches, order);
  std::vector<uint32_t> batch(ps.size());
  for (const Launch& l : launches)
    for (size_t i = l.first; i < l.last; ++i)
      batch[size_t(order[i])] = l.a.closed == kClosedNone ? 0 : l.a.inner_digits;
  for (size_t i = 0; i < ps.size(); ++i) {
    SearchArgs a{};
    plan_full(*ps[i], a);
    printf("%u %u\n", a.closed == kClosedNone ? 0 : a.inner_digits, batch[i]);
  }
}

// From how many mappings on a range of each problem goes in parts (0: never).
static void check_parts() {
  while (const sched_problem* p = read_problem()) {
    uint64_t lo = 0, hi = p->n_mappings;
    if (range_in_parts(*p, 0, hi))
      while (hi - lo > 1) (range_in_parts(*p, 0, lo + (hi - lo) / 2) ? hi : lo) = lo + (hi - lo) / 2;
    else
      hi = 0;
    printf("%llu\n", (unsigned long long)hi);
  }
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "stack") check_stack();
  else if (what == "stats") check_stats();
  else if (what == "slots") check_slots();
  else if (what == "replicas") check_replicas();
  else if (what == "blocks") check_blocks();
  else if (what == "room") check_room();
  else if (what == "closed") check_closed();
  else if (what == "allocations") check_failures(false);
  else if (what == "runtime") check_failures(true);
  else if (what == "parts") check_parts();
  else if (what == "children") check_children();
  else return 2;
  puts("ok");
  return 0;
}
