// launch.h -- host-side entry points into the kernels (internal).
#pragma once
#include <hip/hip_runtime.h>

#include "devtab.h"

namespace devmap {

// The search over a.tables (or a.host_table) and the reduction of its partials
// into a.results, if given.
hipError_t launch_search(int n_tools, const SearchArgs& a, hipStream_t s);
// Searches in closed form (a.closed), without the reduction.
hipError_t launch_closed(const SearchArgs& a, hipStream_t s);
// flags: kEval*.  With kEvalHostTable, tab is the host's copy of a table of at
// most kArgWords words up to its bound table.
hipError_t launch_eval(int n_tools, const uint32_t* tab, const uint64_t* idx, int64_t n,
                       uint64_t n_mappings, int64_t* out, uint32_t flags, hipStream_t s);
hipError_t launch_bound(int n_tools, const uint32_t* tab, uint32_t K, uint64_t known, int64_t n,
                        uint32_t ub, uint32_t* count, uint2* out, hipStream_t s);
// Per-GPU memory of the entry point that allocates nothing: bytes of device
// memory (the tables of one search, 65,536 block partials and a result fit),
// and words of host memory in which a search's tables are put together.
constexpr size_t kScratchBytes = size_t(2) << 20;
constexpr size_t kStageWords = size_t(1) << 15;
hipError_t scratch_buffer(void** ptr, uint32_t** stage);
hipError_t launch_wave_or_probe(const uint64_t* in, const uint8_t* active, uint32_t blocks,
                                uint64_t* out64, uint32_t* out32, hipStream_t s);
hipError_t launch_valu_probe(uint32_t blocks, uint32_t iters, uint32_t* out, hipStream_t s,
                             double* lane_ops);

}  // namespace devmap
