// dispatch.hip -- run-time dispatch on the tool count, and the final
// per-table argmin reduction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <array>
#include <utility>

#include "devtab.h"
#include "launch.h"
#include "reduce.h"

namespace devmap {

template <int N>
hipError_t launch_search_n(const SearchArgs& a, hipStream_t s);
template <int N>
hipError_t launch_eval_n(const EvalArgs& e, uint32_t host_words, uint32_t flags, hipStream_t s);
template <int N>
hipError_t launch_bound_n(const uint32_t* tab, uint32_t K, uint64_t known, int64_t n,
                          uint32_t ub, uint32_t* count, uint2* out, hipStream_t s);

// Minimum over the partials of each result: per_result of them, or the blocks
// of one table each (first).  Bound by the latency of its loads (16 B per
// block of the search, at most 1 MB): four loads in flight per thread and
// 1,024 threads, as one block per result is all there is to launch.  65,536
// partials: 86 us with 256 threads and one load at a time, 16 us now.
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void reduce_kernel(const Partial* __restrict__ partials,
                                                                const uint32_t* __restrict__ first,
                                                                uint32_t per_result,
                                                                DevResult* __restrict__ out) {
  const uint32_t lo = first != nullptr ? first[blockIdx.x] : blockIdx.x * per_result;
  const uint32_t hi = first != nullptr ? first[blockIdx.x + 1] : lo + per_result;
  uint32_t ms = kInf;
  uint64_t x = ~0ull;
  for (uint32_t i = lo + threadIdx.x; i < hi; i += 4 * kReduceThreads) {
    Partial p[4];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t k = i + j * kReduceThreads;
      p[j] = partials[k < hi ? k : i];  // (past the end: this thread's first one again)
    }
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) lex_min(ms, x, p[j].makespan, p[j].index);
  }
  block_min<kReduceThreads>(ms, x);
  if (threadIdx.x == 0) {
    DevResult r;
    r.index = (ms == kInf) ? ~0ull : x;
    r.makespan = (ms == kInf) ? INT64_MAX : int64_t(ms);
    out[blockIdx.x] = r;
  }
}

using SearchFn = hipError_t (*)(const SearchArgs&, hipStream_t);
using EvalFn = hipError_t (*)(const EvalArgs&, uint32_t, uint32_t, hipStream_t);

template <size_t... I>
static constexpr auto make_search_table(std::index_sequence<I...>) {
  return std::array<SearchFn, sizeof...(I)>{&launch_search_n<int(I) + 1>...};
}
template <size_t... I>
static constexpr auto make_eval_table(std::index_sequence<I...>) {
  return std::array<EvalFn, sizeof...(I)>{&launch_eval_n<int(I) + 1>...};
}
using BoundFn = hipError_t (*)(const uint32_t*, uint32_t, uint64_t, int64_t, uint32_t, uint32_t*,
                               uint2*, hipStream_t);
template <size_t... I>
static constexpr auto make_bound_table(std::index_sequence<I...>) {
  return std::array<BoundFn, sizeof...(I)>{&launch_bound_n<int(I) + 1>...};
}

static const auto kSearchFns = make_search_table(std::make_index_sequence<kMaxTools>{});
static const auto kEvalFns = make_eval_table(std::make_index_sequence<kMaxTools>{});
static const auto kBoundFns = make_bound_table(std::make_index_sequence<kMaxTools>{});

hipError_t launch_search(int n_tools, const SearchArgs& a, hipStream_t s) {
  const hipError_t e =
      a.closed != kClosedNone ? launch_closed(a, s) : kSearchFns[n_tools - 1](a, s);
  if (e != hipSuccess || a.results == nullptr) return e;
  const uint32_t results = a.one_result ? 1u : a.n_tables;
  hipLaunchKernelGGL(reduce_kernel, dim3(results), dim3(kReduceThreads), 0, s, a.partials,
                     a.one_result ? nullptr : a.block_first, a.n_blocks / results, a.results);
  return hipGetLastError();
}

hipError_t launch_eval(int n_tools, const uint32_t* tab, const uint64_t* idx, int64_t n,
                       uint64_t n_mappings, int64_t* out, uint32_t flags, hipStream_t s) {
  const EvalArgs e{tab, idx, n, n_mappings, out};
  const uint32_t words =
      flags & kEvalHostTable ? bound_base(uint32_t(n_tools), tab[kHdrLevels]) : 0u;
  return kEvalFns[n_tools - 1](e, words, flags, s);
}

hipError_t launch_bound(int n_tools, const uint32_t* tab, uint32_t K, uint64_t known, int64_t n,
                        uint32_t ub, uint32_t* count, uint2* out, hipStream_t s) {
  return kBoundFns[n_tools - 1](tab, K, known, n, ub, count, out, s);
}

}  // namespace devmap
