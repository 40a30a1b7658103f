// inst.hip -- the kernels of one tool count, INST_N (set on the compiler command
// line): one unit per count, so that the 40 of them compile in parallel.
#include "kernels.h"

#ifndef INST_N
#error "INST_N must be defined"
#endif

namespace devmap {

template hipError_t launch_search_n<INST_N>(const SearchArgs&, hipStream_t);
template hipError_t launch_eval_n<INST_N>(const EvalArgs&, uint32_t, uint32_t, hipStream_t);
template hipError_t launch_bound_n<INST_N>(const uint32_t*, uint32_t, uint64_t, int64_t, uint32_t,
                                           uint32_t*, uint2*, hipStream_t);

}  // namespace devmap
