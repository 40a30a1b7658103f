// closed.hip -- full-order searches of the problems whose schedules follow in
// closed form: serial chains, and fan-outs that fit the budget together.
//
// Both kernels give a lane one combination of the outer tools (labels
// 0..n-J-1) and walk the combinations of the J last labels in it, so that what
// depends on the outer tools alone is computed once per lane, and a mapping
// costs its last step.  The walk visits every mapping and scores each.  They
// are not instantiated per tool count: their loops over tools run once per
// lane or once per inner pattern, outside the walk.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace devmap {

namespace {

// The block's table: its tools by label, options (radix 1 for a tool with one
// mode) and index weights of their digits.
struct ClosedTab {
  uint32_t opt[kMaxTools];
  uint64_t weight[kMaxTools];
};

__device__ __forceinline__ void stage_closed(Tab tab, uint32_t n, ClosedTab& t) {
  const uint64_t gn = uint64_t(tab[kHdrFixGnLo]) | (uint64_t(tab[kHdrFixGnHi]) << 32);
  const uint64_t gq = uint64_t(tab[kHdrFixGqLo]) | (uint64_t(tab[kHdrFixGqHi]) << 32);
  const uint32_t i = threadIdx.x;
  if (i < n) {
    const uint32_t m = ((gn >> i) & 1) ? 1u : (((gq >> i) & 1) ? 2u : 0u);
    t.opt[i] = 1u | (m << 2);
    t.weight[i] = 0;
  }
  __syncthreads();
  if (i < tab[kHdrPositions]) {
    const uint32_t lab = tab.p[enum_lab_base(n) + i];
    t.opt[lab] = tab.p[enum_opt_base(n) + i];
    t.weight[lab] = uint64_t(tab.p[enum_weight_base(n) + 2 * i]) |
                    (uint64_t(tab.p[enum_weight_base(n) + 2 * i + 1]) << 32);
  }
  __syncthreads();
}

// The block's table and its share of the table's work items.
struct Share {
  const uint32_t* tab;
  uint32_t bb, nb;
};

__device__ __forceinline__ Share my_share(const SearchArgs& a) {
  Share s;
  uint32_t table = 0;
  if (a.block_first != nullptr) {
    const Tab first{a.block_first};
    uint32_t hi = a.n_tables;
    while (hi - table > 1u) {
      const uint32_t mid = (table + hi) >> 1;
      if (first[mid] <= blockIdx.x) table = mid;
      else hi = mid;
    }
    s.bb = blockIdx.x - first[table];
    s.nb = first[table + 1u] - first[table];
  } else {
    table = blockIdx.x / a.blocks_per_table;
    s.nb = a.blocks_per_table;
    s.bb = blockIdx.x - table * s.nb;
  }
  s.tab = table_or_args(a.tables != nullptr ? a.tables + size_t(table) * a.table_stride : nullptr,
                        sizeof(SearchArgs));
  return s;
}

__device__ __forceinline__ void put_partial(const SearchArgs& a, uint32_t ms, uint64_t x) {
  block_min<kBlock>(ms, x);
  if (threadIdx.x == 0) {
    Partial p;
    p.index = x;
    p.makespan = ms;
    p.pad = 0;
    a.partials[blockIdx.x] = p;
  }
}

// Digit of y for a tool with options word o, which is taken off y.
__device__ __forceinline__ uint32_t take_digit(uint64_t& y, uint32_t o) {
  const uint32_t r = opt_radix(o);
  const uint64_t q = r == 3u ? y / 3u : (r == 2u ? y >> 1 : y);
  const uint32_t d = uint32_t(y - q * r);
  y = q;
  return r == 1u ? 0u : d;
}

constexpr uint32_t kClosedInf = 0xC0000000u;  // infeasible, with a time added to it or not

}  // namespace

// Serial chains (kClosedChain): one tool runs at a time, so nothing is slowed,
// queued behind another or kept waiting for VRAM, and the makespan is the sum
// of the durations and of the transfers between neighbours on different
// devices.  The inner tools' sum is the same for every lane but for the
// transfer into the first of them: the block forms it once per combination
// (in LDS, ascending index), and a mapping takes an add, a compare and two
// selects.  Bound by those: 1.22e9 mappings (256 replicas of 14 tools) in
// 0.41 ms, 25 ms through the event loop with shared prefixes.  A small search
// is bound by a step's LDS latency instead (about 0.1 us).
__global__ __launch_bounds__(kBlock) void chain_kernel(SearchArgs a, TableArg) {
  __shared__ ClosedTab t;
  __shared__ uint32_t s_dur[kMaxTools][3];  // per mode, kClosedInf if it never fits
  __shared__ uint32_t s_xfer[kMaxTools];
  __shared__ uint2 s_sum[kClosedInnerMost];     // sum, device of the first inner tool
  __shared__ uint64_t s_weight[kClosedInnerMost];
  const Share sh = my_share(a);
  const Tab tab{sh.tab};
  const uint32_t n = tab[kHdrN], levels = tab[kHdrLevels], J = a.inner_digits;
  stage_closed(tab, n, t);
  const uint32_t outer = n - J;
  if (threadIdx.x < n) {
    const uint32_t i = threadIdx.x;
    const uint32_t* rec = sh.tab + kHdrWords + kToolWords * i;
    const uint32_t* dur = sh.tab + tab[kHdrDurOff] + 2 * i * levels;
    const uint64_t big = uint64_t(tab[kHdrBigLo]) | (uint64_t(tab[kHdrBigHi]) << 32);
    s_dur[i][0] = rec[kToolCpu];
    s_dur[i][1] = (big >> i) & 1 ? kClosedInf : dur[0];
    s_dur[i][2] = (big >> i) & 1 ? kClosedInf : dur[levels];
    s_xfer[i] = rec[kToolXfer];
  }
  __syncthreads();
  uint32_t C = 1;
  for (uint32_t i = outer; i < n; ++i) C *= opt_radix(t.opt[i]);
  uint64_t n_outer = 1;
  for (uint32_t i = 0; i < outer; ++i) n_outer *= opt_radix(t.opt[i]);
  if (threadIdx.x < C) {
    // combination c: its digits in ascending index weight, so that index
    // grows with c and the first of equal sums is the lowest
    uint64_t c = threadIdx.x, weight = 0, done = 0;
    uint32_t mode[kClosedInner];
    for (uint32_t k = 0; k < J; ++k) {
      uint32_t next = 0;
      uint64_t least = ~0ull;
      for (uint32_t j = 0; j < J; ++j)
        if (!((done >> j) & 1) && t.weight[outer + j] < least) {
          least = t.weight[outer + j];
          next = j;
        }
      done |= 1ull << next;
      const uint32_t d = take_digit(c, t.opt[outer + next]);
#pragma unroll
      for (uint32_t j = 0; j < kClosedInner; ++j)
        if (j == next) mode[j] = opt_mode(t.opt[outer + next], d);
      weight += uint64_t(d) * t.weight[outer + next];
    }
    uint32_t sum = 0, last = 0, first = 0;
    bool never = false;
#pragma unroll
    for (uint32_t j = 0; j < kClosedInner; ++j)
      if (j < J) {
        const uint32_t dev = mode[j] != 0 ? 1u : 0u, d = s_dur[outer + j][mode[j]];
        never = never || d == kClosedInf;
        sum += d + (j > 0 && dev != last ? s_xfer[outer + j] : 0u);
        if (j == 0) first = dev;
        last = dev;
      }
    s_sum[threadIdx.x] = make_uint2(never ? kClosedInf : sum, first);
    s_weight[threadIdx.x] = weight;
  }
  __syncthreads();
  uint32_t best_ms = kInf;
  uint64_t best_x = ~0ull;
  for (uint64_t item = sh.bb; item * kBlock < n_outer; item += sh.nb) {
    uint64_t y = item * kBlock + threadIdx.x;
    if (y >= n_outer) break;
    uint64_t x = 0;
    uint32_t sum = 0, last = 0;
    bool never = false;
    for (uint32_t i = 0; i < outer; ++i) {
      const uint32_t o = t.opt[i], d = take_digit(y, o), m = opt_mode(o, d);
      const uint32_t dev = m != 0 ? 1u : 0u, b = s_dur[i][m];
      never = never || b == kClosedInf;
      sum += b + (i > 0 && dev != last ? s_xfer[i] : 0u);
      last = dev;
      x += uint64_t(d) * t.weight[i];
    }
    const uint32_t xf = outer > 0 ? s_xfer[outer] : 0u;
    const uint32_t to_cpu = never ? kClosedInf : sum + (last == 1 ? xf : 0u);
    const uint32_t to_gpu = never ? kClosedInf : sum + (last == 0 ? xf : 0u);
    uint32_t ms = kInf, at = 0;
    for (uint32_t c = 0; c < C; ++c) {
      const uint2 u = s_sum[c];
      const uint32_t from = __builtin_amdgcn_readfirstlane(u.y) ? to_gpu : to_cpu;
      // (both infeasible: the sum would wrap)
      const uint32_t m = umax32(from, u.x) >= kClosedInf ? kInf : from + u.x;
      if (a.record != nullptr) a.record[x + s_weight[c]] = m;
      at = m < ms ? c : at;
      ms = umin32(ms, m);
    }
    if (ms != kInf) lex_min(best_ms, best_x, ms, x + s_weight[at]);
  }
  put_partial(a, best_ms, best_x);
}

namespace {

// The three largest of the values inserted, largest first (0: none).
struct Top3 {
  uint32_t m1, m2, m3;
  __device__ __forceinline__ void insert(uint32_t f) {
    const uint32_t a = umin32(m1, f), b = umin32(m2, a);
    m1 = umax32(m1, f);
    m2 = umax32(m2, a);
    m3 = umax32(m3, b);
  }
};

// One lane's walk over the inner tools of a fan-out.
template <int J>
struct FanWalk {
  const uint32_t* s_dur;      // durations in LDS, level-major rows
  uint32_t row, inner;        // words per row; label of the first inner tool
  uint32_t cpu[J], opt[J];
  uint64_t w1[J], w2[J], w0[J];  // index contribution of modes gpu_now, gpu_queue, cpu
  uint32_t* record;
  uint64_t x;                 // index of the lane's outer digits
  Top3 top;                   // the latest finishes of the gpu_now tools
  uint32_t floor_ms;          // latest of them and of the outer CPU tools
  uint32_t alone;             // makespan without any queued tool, but for the inner CPU tools
  bool queued;                // an outer tool is queued
  uint32_t best_ms;
  uint64_t best_x;

  __device__ __forceinline__ uint32_t step(uint32_t s, uint32_t label) const {
    const uint32_t k = (s < top.m1 ? 1u : 0u) + (s < top.m2 ? 1u : 0u) + (s < top.m3 ? 1u : 0u);
    return s + s_dur[k * row + 2u * label + 1u];
  }
  // Inner tools D.. once the earlier ones are settled: those in g run on
  // gpu_now, those in Q (of the earlier ones) are queued, s is when the queue
  // frees and c the latest inner CPU tool.  A leaf costs a maximum, a compare
  // and a branch; its index is formed only if it may be the lane's best.
  template <int D, uint32_t Q>
  __device__ __forceinline__ void walk(uint32_t g, uint32_t s, uint32_t c) {
    if constexpr (D == J) {
      uint32_t ms = umax32(umax32(floor_ms, c), s);
      if constexpr (Q == 0) ms = queued ? ms : umax32(alone, c);
      if (record != nullptr || __any(ms <= best_ms)) {
        DEVMAP_KEEP_BRANCH();
        uint64_t at = x;
#pragma unroll
        for (int j = 0; j < J; ++j) at += (Q >> j) & 1 ? w2[j] : ((g >> j) & 1 ? w1[j] : w0[j]);
        if (record != nullptr) record[at] = ms;
        lex_min(best_ms, best_x, ms, at);
      }
    } else {
      const bool in = (g >> D) & 1;
      if (in || (opt[D] & 1u)) {
        DEVMAP_KEEP_BRANCH();
        walk<D + 1, Q>(g, s, in ? c : umax32(c, cpu[D]));
      }
      if (!in && (opt[D] & 4u)) {
        DEVMAP_KEEP_BRANCH();
        walk<D + 1, Q | (1u << D)>(g, step(s, inner + D), c);
      }
    }
  }
};

}  // namespace

// Fan-outs whose footprints all fit the budget together (kClosedFanout; the
// schedule is that of evaluate_fanout): with at most four contention levels, a
// queued tool that starts at s runs at 1 + (s < M1) + (s < M2) + (s < M3), M1
// to M3 the three latest finishes of the gpu_now tools, which is all that the
// queue's recursion needs of them.  Per lane and set of inner tools on gpu_now,
// the outer tools' queue is run once; the inner tools' queue is a walk over
// subsets in label order, one step of the recursion per mapping.  Bound by VALU
// issue and the LDS reads of those steps: 1.53e9 mappings (320 replicas of 14
// tools) in 1.87 ms; evaluated one by one, 17.5 ms.
template <int J>
__global__ __launch_bounds__(kBlock) void fanout_kernel(SearchArgs a, TableArg) {
  __shared__ ClosedTab t;
  __shared__ uint32_t s_dur[4 * 2 * 32];
  const Share sh = my_share(a);
  const Tab tab{sh.tab};
  const uint32_t n = tab[kHdrN], levels = tab[kHdrLevels];
  stage_closed(tab, n, t);
  const uint32_t row = 2u * n, outer = n - J;
  const uint32_t* dur = sh.tab + tab[kHdrDurOff];
  for (uint32_t w = threadIdx.x; w < row * 4u; w += kBlock) {
    const uint32_t lev = w / row, iq = w - lev * row;
    s_dur[w] = dur[iq * levels + umin32(lev, levels - 1u)];
  }
  __syncthreads();
  uint64_t n_outer = 1;
  for (uint32_t i = 0; i < outer; ++i) n_outer *= opt_radix(t.opt[i]);
  FanWalk<J> f;
  f.s_dur = s_dur;
  f.row = row;
  f.inner = outer;
  f.record = a.record;
  f.best_ms = kInf;
  f.best_x = ~0ull;
  uint32_t may = 0, must = 0;  // inner tools that may, and must, run on gpu_now
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const uint32_t o = __builtin_amdgcn_readfirstlane(t.opt[outer + j]);
    const uint64_t w = uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(t.weight[outer + j])))) |
                       (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(t.weight[outer + j] >> 32)))) << 32);
    f.cpu[j] = tab[kHdrWords + kToolWords * (outer + j) + kToolCpu];
    f.opt[j] = 0;
    f.w0[j] = f.w1[j] = f.w2[j] = 0;
    for (uint32_t d = 0; d < opt_radix(o); ++d) {
      const uint32_t m = opt_mode(o, d);
      f.opt[j] |= 1u << m;
      if (m == 0u) f.w0[j] = d * w;
      if (m == 1u) f.w1[j] = d * w;
      if (m == 2u) f.w2[j] = d * w;
    }
    if (f.opt[j] & 2u) may |= 1u << j;
    if (f.opt[j] == 2u) must |= 1u << j;
  }
  for (uint64_t item = sh.bb; item * kBlock < n_outer; item += sh.nb) {
    uint64_t y = item * kBlock + threadIdx.x;
    if (y >= n_outer) break;
    f.x = 0;
    uint32_t gn = 0, gq = 0, cpu = 0;
    for (uint32_t i = 0; i < outer; ++i) {
      const uint32_t o = t.opt[i], d = take_digit(y, o), m = opt_mode(o, d);
      gn |= m == 1u ? 1u << i : 0u;
      gq |= m == 2u ? 1u << i : 0u;
      cpu = m == 0u ? umax32(cpu, tab[kHdrWords + kToolWords * i + kToolCpu]) : cpu;
      f.x += uint64_t(d) * t.weight[i];
    }
    f.queued = gq != 0;
    const uint32_t now = uint32_t(__builtin_popcount(gn));
    // the outer gpu_now tools' latest finishes, were they to run at each level
    Top3 outer_top[4];
#pragma unroll
    for (int l = 0; l < 4; ++l) outer_top[l] = Top3{0, 0, 0};
    for (uint32_t i = 0; i < outer; ++i) {
      const bool on = (gn >> i) & 1;
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        const uint32_t d = s_dur[uint32_t(l) * row + 2u * i];
        outer_top[l].insert(on ? d : 0u);
      }
    }
    for (uint32_t g = 0; g < (1u << J); ++g) {
      if ((g & ~may) || (must & ~g)) continue;
      // rows of the concurrency at 0: the gpu_now tools, and the first queued
      const uint32_t k = now + uint32_t(__builtin_popcount(g));
      const uint32_t l0 = umin32(umax32(k, 1u), levels) - 1u, l1 = umin32(k + 1u, levels) - 1u;
      Top3 top = outer_top[0];
      uint32_t alone = outer_top[0].m1;
#pragma unroll
      for (int l = 1; l < 4; ++l) {
        top.m1 = l1 == uint32_t(l) ? outer_top[l].m1 : top.m1;
        top.m2 = l1 == uint32_t(l) ? outer_top[l].m2 : top.m2;
        top.m3 = l1 == uint32_t(l) ? outer_top[l].m3 : top.m3;
        alone = l0 == uint32_t(l) ? outer_top[l].m1 : alone;
      }
#pragma unroll
      for (int j = 0; j < J; ++j)
        if ((g >> j) & 1) {
          const uint32_t at = 2u * (outer + uint32_t(j));
          top.insert(s_dur[l1 * row + at]);
          alone = umax32(alone, s_dur[l0 * row + at]);
        }
      f.floor_ms = umax32(top.m1, cpu);
      f.alone = umax32(alone, cpu);
      // a tool runs at the last level stored at most
      if (levels < 4u) top.m3 = 0;
      if (levels < 3u) top.m2 = 0;
      if (levels < 2u) top.m1 = 0;
      f.top = top;
      uint32_t s = 0;
      for (uint32_t i = 0; i < outer; ++i)
        if ((gq >> i) & 1) s = f.step(s, i);
      f.template walk<0, 0>(g, s, 0u);
    }
  }
  put_partial(a, f.best_ms, f.best_x);
}

hipError_t launch_closed(const SearchArgs& a, hipStream_t s) {
  TableArg t;
  if (a.tables == nullptr) {
    if (a.host_words > kArgWords) return hipErrorInvalidValue;
    memcpy(t.w, a.host_table, size_t(a.host_words) * 4u);
  }
  const dim3 blocks(a.n_blocks), threads(kBlock);
  if (a.closed == kClosedChain) {
    if (a.inner_digits > kClosedInner || a.inner_digits == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(chain_kernel, blocks, threads, 0, s, a, t);
  } else {
    if (a.lds_levels > 4) return hipErrorInvalidValue;
    switch (a.inner_digits) {
      case 2: hipLaunchKernelGGL(fanout_kernel<2>, blocks, threads, 0, s, a, t); break;
      case 3: hipLaunchKernelGGL(fanout_kernel<3>, blocks, threads, 0, s, a, t); break;
      case 4: hipLaunchKernelGGL(fanout_kernel<4>, blocks, threads, 0, s, a, t); break;
      case 5: hipLaunchKernelGGL(fanout_kernel<5>, blocks, threads, 0, s, a, t); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

}  // namespace devmap
