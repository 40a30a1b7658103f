// host_range.cpp -- test harness: a partial range searched in parts
// (split_range, stage_parts) with the kernels' per-lane code compiled for the
// host, one lane per wave, over every work item of every part.  Writes how
// often each mapping of [0, n_mappings) was scored (uint32) and its makespan
// (uint32, 0xFFFFFFFF infeasible) to argv[1], and prints the number of parts.
// The kernel is that for HOST_RANGE_N tools.  A problem with fewer tools (or
// hi = 0) is walked as a batch replica on it instead (lay_replica, with lo
// mappings in its launch).
//
// Input (text, stdin): n_tools lo hi share n_edges n_levels budget, then
// n_tools lines "gpu cpu load xfer mem allowed", n_edges lines "src dst", then
// the n_levels Q16 contention factors.
#include "../../paper_2607_22242_amd/csrc/api.cpp"
#include "../../paper_2607_22242_amd/csrc/kernels.h"

#include <cstdio>
#include <vector>

namespace devmap {
hipError_t launch_search(int, const SearchArgs&, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_eval(int, const uint32_t*, const uint64_t*, int64_t, uint64_t, int64_t*,
                       uint32_t, hipStream_t) {
  return hipErrorUnknown;
}
hipError_t launch_bound(int, const uint32_t*, uint32_t, uint64_t, int64_t, uint32_t, uint32_t*,
                        uint2*, hipStream_t) {
  return hipErrorUnknown;
}
hipError_t launch_valu_probe(uint32_t, uint32_t, uint32_t*, hipStream_t, double*) {
  return hipErrorUnknown;
}
hipError_t launch_wave_or_probe(const uint64_t*, const uint8_t*, uint32_t, uint64_t*, uint32_t*,
                                hipStream_t) {
  return hipErrorUnknown;
}
hipError_t scratch_buffer(void**, uint32_t**) { return hipErrorUnknown; }
}  // namespace devmap

using namespace devmap;

struct Count {
  uint32_t *times, *ms;
  bool on() const { return true; }
  void operator()(uint64_t x, uint32_t m) const {
    ++times[x];
    ms[x] = m;
  }
};

template <int N, bool SHARE>
static int run(const sched_problem& p, uint64_t lo, uint64_t hi, const char* path) {
  std::vector<uint32_t> stage(kStageWords), times(p.n_mappings, 0u), ms(p.n_mappings, 0u);
  const Count rec{times.data(), ms.data()};
  SearchArgs a{};
  size_t stride = p.table_words;
  if (p.n < N || hi == 0) {
    const Launch g{0, 1, N, lo, SearchArgs{}};
    a.n_tables = 1;
    stride = kStageWords;
    if (lay_replica(p, g, stage.data()) != SCHED_OK ||
        fill_latencies(p, nullptr, stage.data(), false) != SCHED_OK)
      return 1;
  } else if (stage_parts(p, lo, hi, a, stage.data()) > kStageWords) {
    return 1;
  }
  std::vector<uint32_t> snap(snap_words<N, SHARE>() * kBlock);
  uint64_t slot_word = 0;
  MaskT<N>* slot = reinterpret_cast<MaskT<N>*>(&slot_word);
  for (uint32_t t = 0; t < a.n_tables; ++t) {
    const uint32_t* tab = stage.data() + size_t(t) * stride;
    std::vector<uint32_t> lds(lds_words_for(N, tab[kHdrLevels]));
    stage_image<N>(tab, lds.data(), 0, 1);
    const TabWalk walk{Tab{tab}};
    const uint64_t items = (walk_n_outer(walk) + kBlock - 1) / kBlock;
    uint32_t bms = kInf;
    uint64_t bx = ~0ull;
    for (uint64_t item = 0; item < items; ++item)
      for (uint32_t lane = 0; lane < uint32_t(kBlock); ++lane) {
        if (tab[kHdrPrefix])
          lane_search_prefix<N, SHARE>(walk, tab, lds.data(), item, lane, slot, snap.data() + lane,
                                       bms, bx, rec);
        else
          lane_search<N, true, SHARE>(walk, tab, lds.data(), item, lane, slot, bms, bx, rec);
      }
  }
  FILE* f = fopen(path, "wb");
  if (!f || fwrite(times.data(), 4, times.size(), f) != times.size() ||
      fwrite(ms.data(), 4, ms.size(), f) != ms.size())
    return 1;
  fclose(f);
  printf("%u\n", a.n_tables);
  return 0;
}

int main(int argc, char** argv) {
  unsigned long long lo, hi;
  int n, share, ne, nl;
  long long budget;
  if (argc < 2 ||
      scanf("%d %llu %llu %d %d %d %lld", &n, &lo, &hi, &share, &ne, &nl, &budget) != 7)
    return 2;
  std::vector<sched_tool> tools(n);
  std::vector<uint8_t> allowed(n);
  for (int v = 0; v < n; ++v) {
    long long g, c, l, x, m;
    int al;
    if (scanf("%lld %lld %lld %lld %lld %d", &g, &c, &l, &x, &m, &al) != 6) return 2;
    tools[v] = sched_tool{g, c, l, x, m};
    allowed[v] = uint8_t(al);
  }
  std::vector<sched_edge> e(ne);
  for (auto& x : e)
    if (scanf("%d %d", &x.src, &x.dst) != 2) return 2;
  std::vector<uint32_t> f(nl);
  for (auto& x : f)
    if (scanf("%u", &x) != 1) return 2;
  sched_problem* p = nullptr;
  sched_problem_desc d{tools.data(), n, e.data(), ne, f.data(), nl, budget, allowed.data(), share};
  if (sched_problem_create_desc(&d, &p) != SCHED_OK) return 1;
  const int rc = share ? run<HOST_RANGE_N, true>(*p, lo, hi, argv[1])
                       : run<HOST_RANGE_N, false>(*p, lo, hi, argv[1]);
  sched_problem_destroy(p);
  return rc;
}
