// Kernels and host builder of work sets (see mss_work.h).
//
// Integrator: persistent waves take work items (64 / S consecutive
// intervals of one range, S lane-slices per interval) from an atomic
// counter until it passes the item count, so every wave exits once the
// queue is drained; no wave ever waits for another.
// Scan: level by level; a wave locates its sequence by binary search over
// the level's tile prefix and handles one tile of it.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "mss_scan.h"
#include "mss_work.h"

namespace mss {

int scan_top(int64_t K, int tile) {
  int top = 0;
  int64_t n = K;
  while (n > tile) {
    n = (n + tile - 1) / tile;
    ++top;
  }
  return top;
}

static size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t scan_scratch_bytes(int N, int64_t K, int tile) {
  size_t b = 0;
  int64_t n = K;
  while (n > tile) {
    n = (n + tile - 1) / tile;
    b += (size_t)n * (N * N + N) * 16;
  }
  return a256(b);
}

// ---------------------------------------------------------------------------
// device
// ---------------------------------------------------------------------------
// largest i in [0, n) with prefix[i] <= x (non-decreasing prefix, prefix[0] = 0)
__device__ __forceinline__ int find_segment(const int64_t* __restrict__ prefix, int n, int64_t x) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (as_constant(prefix)[mid] <= x) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

struct ScanWorkArgs {
  const SimDesc* sims;
  const int64_t* tiles;  // prefix over sequences at this level
  int64_t n_tiles;
  int32_t n_sims;
  int32_t level;
};

__global__ void work_reset_kernel(unsigned long long* counter) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *counter = 0ull;
}

// Field-program source of a descriptor: its slice of the term table.
struct TableSource {
  __device__ __forceinline__ TableTerms operator()(const IntegrateWorkArgs& A,
                                                   const SimDesc& s) const {
    return TableTerms{A.terms + s.term_off, s.n_terms, s.n_varying};
  }
};

__global__ void __launch_bounds__(256, 2) work_integrate_kernel(const IntegrateWorkArgs A) {
  work_integrate_loop(A, TableSource{});
}

__global__ void __launch_bounds__(256, 2) work_chained_kernel(const IntegrateWorkArgs A) {
  chained_integrate_loop(A, TableSource{});
}

// Before a chained run: unit counter and failure word to 0, every slot
// word to 0 (tag 0, which no unit writes).  Atomic stores, like every
// other access to these words; a kernel rather than a memset, so a captured
// graph replays it as such.
__global__ void chain_reset_kernel(ChainSync* s, unsigned long long* words, int64_t n_words) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    __hip_atomic_store(&s->counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&s->failed, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (i < n_words) __hip_atomic_store(words + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Element count of a sequence at a scan level and the start of that level's
// arrays in the sequence's scratch (levels >= 1).
template <int N, int E>
__device__ __forceinline__ int64_t level_geometry(const SimDesc& s, int level, size_t* mats_off) {
  int64_t n = s.K_total;
  size_t off = 0;
  for (int l = 1; l <= level; ++l) {
    if (l > 1) off += (size_t)n * (N * N + N) * 2;
    n = (n + 64 * E - 1) / (64 * E);
  }
  *mats_off = off;  // in doubles
  return n;
}

template <int N, int E, bool REV>
__device__ __forceinline__ void work_reduce_tile(const SimDesc& s, int level, int64_t local,
                                                 int lane) {
  size_t off = 0;
  const int64_t n = level_geometry<N, E>(s, level, &off);
  const double* M = level == 0 ? s.U : s.scan_ws + off;
  size_t up_off = 0;
  const int64_t n_up = level_geometry<N, E>(s, level + 1, &up_off);
  (void)n_up;
  double* out = s.scan_ws + up_off + (size_t)local * 2 * N * N;
  if (REV && level == 0) tile_reduce<N, E, REV>(M, n, local, lane, out);
  else tile_reduce<N, E>(M, n, local, lane, out);
}

template <int N, int E, bool REV>
__device__ __forceinline__ void work_apply_tile(const SimDesc& s, int level, int64_t local,
                                                int lane) {
  size_t off = 0;
  const int64_t n = level_geometry<N, E>(s, level, &off);
  const double* M = level == 0 ? s.U : s.scan_ws + off;
  double* before = level == 0 ? s.psi : s.scan_ws + off + (size_t)n * 2 * N * N;
  const double* start;
  if (level == s.top) {
    start = s.psi0;
  } else {
    size_t up_off = 0;
    const int64_t n_up = level_geometry<N, E>(s, level + 1, &up_off);
    start = s.scan_ws + up_off + (size_t)n_up * 2 * N * N + (size_t)local * 2 * N;
  }
  // the lane's operators stay in registers from the scan to the walk where
  // they fit, spin-1 at E = 4 included: that leaves one wave a SIMD, but the
  // second read of the operators (which at these sizes misses L2) is what the
  // pass waits for: scans of 9.3e5, 7.6e6 and 3.1e7 spin-1 operators 114, 839
  // and 3,279 us with it, 105, 738 and 2,743 without
  constexpr bool kKeep = E * 2 * N * N <= 72;
  double* last = level == 0 ? s.psi_final : nullptr;
  if (REV && level == 0)
    tile_apply<N, E, kKeep, REV>(M, n, local, lane, true, start, before, last);
  else
    tile_apply<N, E, kKeep>(M, n, local, lane, true, start, before, last);
}

template <int E, bool REV>
__global__ void __launch_bounds__(256) work_reduce_kernel(const ScanWorkArgs A) {
  const int lane = threadIdx.x & 63;
  const int64_t tile = (int64_t)blockIdx.x * (blockDim.x >> 6) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (tile >= A.n_tiles) return;  // the whole wave leaves together
  const int i = find_segment(A.tiles, A.n_sims, tile);
  const int64_t local = tile - as_constant(A.tiles)[i];
  const SimDesc s = load_constant(A.sims + i);
  if (s.spin_twice == 2) work_reduce_tile<3, E, REV>(s, A.level, local, lane);
  else work_reduce_tile<2, E, REV>(s, A.level, local, lane);
}

template <int E, bool REV>
__global__ void __launch_bounds__(256) work_apply_kernel(const ScanWorkArgs A) {
  const int lane = threadIdx.x & 63;
  const int64_t tile = (int64_t)blockIdx.x * (blockDim.x >> 6) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (tile >= A.n_tiles) return;  // the whole wave leaves together
  const int i = find_segment(A.tiles, A.n_sims, tile);
  const int64_t local = tile - as_constant(A.tiles)[i];
  const SimDesc s = load_constant(A.sims + i);
  if (s.spin_twice == 2) work_apply_tile<3, E, REV>(s, A.level, local, lane);
  else work_apply_tile<2, E, REV>(s, A.level, local, lane);
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
void WorkSet::add(const mss_problem& p, int slices_log2, int64_t k_first, int64_t k_count,
                  bool scan) {
  SimDesc d;
  memset(&d, 0, sizeof d);
  d.t_start = p.t_start;
  d.dt_out = p.dt_out;
  d.dt = p.dt_out / (double)p.n_fine;
  d.k_first = k_first;
  d.k_count = k_count;
  d.K_total = p.n_samples;
  d.spin_twice = p.spin_twice;
  d.n_terms = p.n_terms;
  d.n_fine = p.n_fine;
  d.tau = p.spin_twice == 2 ? p.n_squares : 0;
  d.frame = p.rotating_frame;
  d.method = p.method;
  d.full = api_full_basis(&p) ? 1 : 0;
  d.slices_log2 = slices_log2;
  d.top = scan ? scan_top(p.n_samples, 64 * scan_e) : -1;
  if (last_terms_ && last_n_terms_ == p.n_terms &&
      (p.n_terms == 0 || memcmp(last_terms_, p.terms, sizeof(mss_term) * p.n_terms) == 0)) {
    d.term_off = last_term_off_;
    d.n_varying = last_n_varying_;
  } else {
    d.term_off = (int32_t)terms.size();
    terms.resize(terms.size() + p.n_terms);
    d.n_varying = program_order(p.terms, p.n_terms, terms.data() + d.term_off);
    last_terms_ = p.terms;
    last_n_terms_ = p.n_terms;
    last_term_off_ = d.term_off;
    last_n_varying_ = d.n_varying;
  }
  sims.push_back(d);
}

void WorkSet::finalize() {
  const int n = (int)sims.size();
  int64_t item = 0;
  n_levels = 0;
  for (SimDesc& d : sims) {
    d.item_off = item;
    const int64_t per = 64 >> d.slices_log2;
    item += (d.k_count + per - 1) / per;
    n_levels = std::max(n_levels, d.top);
  }
  n_items = item;
  if (chained) {
    // unit counts per sequence (kChainPerLane 64 / S intervals each),
    // sequences by decreasing count; walking from the shortest up, each new
    // count starts a group of rounds in which exactly the sequences before
    // it (in `order`) and itself take part
    std::vector<int64_t> cnt(n);
    n_units = 0;
    for (int i = 0; i < n; ++i) {
      const int64_t per = (int64_t)kChainPerLane * (64 >> sims[i].slices_log2);
      cnt[i] = (sims[i].k_count + per - 1) / per;
      n_units += cnt[i];
    }
    order.resize(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return cnt[a] > cnt[b]; });
    group_item0.clear();
    group_round0.clear();
    group_count.clear();
    int64_t round = 0, at = 0;
    for (int j = n - 1; j >= 0; --j) {
      const int64_t m = cnt[order[j]];
      if (m <= round) continue;
      group_item0.push_back(at);
      group_round0.push_back(round);
      group_count.push_back(j + 1);
      at += (m - round) * (j + 1);
      round = m;
    }
  }
  reduce_tiles.assign(n_levels, std::vector<int64_t>(n + 1, 0));
  apply_tiles.assign(n_levels + 1, std::vector<int64_t>(n + 1, 0));
  const int tile = 64 * scan_e;
  for (int i = 0; i < n; ++i) {
    const SimDesc& d = sims[i];
    int64_t cnt = d.K_total;
    for (int l = 0; l <= n_levels; ++l) {
      const int64_t tiles = (cnt + tile - 1) / tile;
      const bool scans = d.top >= 0;
      if (l < n_levels) reduce_tiles[l][i + 1] = reduce_tiles[l][i] + (scans && l < d.top ? tiles : 0);
      apply_tiles[l][i + 1] = apply_tiles[l][i] + (scans && l <= d.top ? tiles : 0);
      cnt = tiles;
    }
  }
}

// chained tables: group_item0, group_round0, group_count, order
static size_t chain_table_bytes(size_t groups, size_t sims) {
  return 2 * a256(std::max<size_t>(1, groups) * sizeof(int64_t)) +
         a256(std::max<size_t>(1, groups) * sizeof(int32_t)) +
         a256(std::max<size_t>(1, sims) * sizeof(int32_t));
}

size_t WorkSet::packed_bytes() const {
  size_t b = a256(sims.size() * sizeof(SimDesc)) + a256(std::max<size_t>(1, terms.size()) * sizeof(mss_term));
  b += (reduce_tiles.size() + apply_tiles.size()) * a256((sims.size() + 1) * sizeof(int64_t));
  if (chained) b += chain_table_bytes(group_item0.size(), sims.size());
  return b;
}

void WorkSet::pack(char* dst, size_t* o_sims, size_t* o_terms, std::vector<size_t>* o_reduce,
                   std::vector<size_t>* o_apply, size_t* o_chain) const {
  size_t off = 0;
  *o_sims = off;
  memcpy(dst + off, sims.data(), sims.size() * sizeof(SimDesc));
  off += a256(sims.size() * sizeof(SimDesc));
  *o_terms = off;
  if (!terms.empty()) memcpy(dst + off, terms.data(), terms.size() * sizeof(mss_term));
  off += a256(std::max<size_t>(1, terms.size()) * sizeof(mss_term));
  const size_t tb = a256((sims.size() + 1) * sizeof(int64_t));
  o_reduce->clear();
  for (const auto& t : reduce_tiles) {
    o_reduce->push_back(off);
    memcpy(dst + off, t.data(), t.size() * sizeof(int64_t));
    off += tb;
  }
  o_apply->clear();
  for (const auto& t : apply_tiles) {
    o_apply->push_back(off);
    memcpy(dst + off, t.data(), t.size() * sizeof(int64_t));
    off += tb;
  }
  if (o_chain) *o_chain = off;
  if (chained) {
    const size_t g = group_item0.size();
    memcpy(dst + off, group_item0.data(), g * sizeof(int64_t));
    off += a256(std::max<size_t>(1, g) * sizeof(int64_t));
    memcpy(dst + off, group_round0.data(), g * sizeof(int64_t));
    off += a256(std::max<size_t>(1, g) * sizeof(int64_t));
    memcpy(dst + off, group_count.data(), g * sizeof(int32_t));
    off += a256(std::max<size_t>(1, g) * sizeof(int32_t));
    memcpy(dst + off, order.data(), order.size() * sizeof(int32_t));
  }
}

DevWork device_view(const WorkSet& w, const char* dev_base, size_t o_sims, size_t o_terms,
                    const std::vector<size_t>& o_reduce, const std::vector<size_t>& o_apply,
                    size_t o_chain) {
  DevWork d;
  if (w.chained) {
    const size_t g = w.group_item0.size();
    d.n_groups = (int32_t)g;
    size_t off = o_chain;
    d.group_item0 = (const int64_t*)(dev_base + off);
    off += a256(std::max<size_t>(1, g) * sizeof(int64_t));
    d.group_round0 = (const int64_t*)(dev_base + off);
    off += a256(std::max<size_t>(1, g) * sizeof(int64_t));
    d.group_count = (const int32_t*)(dev_base + off);
    off += a256(std::max<size_t>(1, g) * sizeof(int32_t));
    d.order = (const int32_t*)(dev_base + off);
  }
  d.sims = (const SimDesc*)(dev_base + o_sims);
  d.terms = (const mss_term*)(dev_base + o_terms);
  d.n_sims = (int32_t)w.sims.size();
  d.n_items = w.n_items;
  d.n_levels = w.n_levels;
  d.scan_e = w.scan_e;
  d.n_units = w.n_units;
  for (size_t l = 0; l < o_reduce.size(); ++l) {
    d.reduce_tiles.push_back((const int64_t*)(dev_base + o_reduce[l]));
    d.reduce_total.push_back(w.reduce_tiles[l].back());
  }
  for (size_t l = 0; l < o_apply.size(); ++l) {
    d.apply_tiles.push_back((const int64_t*)(dev_base + o_apply[l]));
    d.apply_total.push_back(w.apply_tiles[l].back());
  }
  return d;
}

// What one item of a descriptor costs its wave, in fine steps of a CF4 spin-1
// lane: the fine steps of a lane by the arithmetic of a step, and the set-up.
static double item_cost(const SimDesc& d) {
  const double step = (d.spin_twice == 1 ? 0.5 : d.full ? 1.5 : 1.0) * (d.method ? 0.6 : 1.0);
  const int s = 1 << d.slices_log2;
  return step * ((d.n_fine + s - 1) / s) + 1.0;
}

// A wave takes k items at a time, k = 4 or 2, while
//   * more than 2 k items for every wave are left, which leaves enough single
//     ones to even out the waves' rates (lines at half that: 200 mixed
//     simulations 584 us against 541; at twice that: a burst of 24 requests 10 %
//     longer), and
//   * k of the costliest items that the wave may be given take no longer than
//     a wave's even share of the work left (2 k: a burst of 24 requests 860 us
//     against 830).  A wave decides before it knows which items it gets: those
//     up to a grid's worth of chunks on.
// Items of one cost meet the second rule wherever they meet the first.
// Without it, simulations of 2,000 fine steps an interval among some of 2 ran
// four to a wave: 14.8 ms for 256 such items behind 6,144 of the cheap ones
// and before 18,432, which take 5.3 with it (alone 3.5).  What an item costs is
// told from the step counts and the arithmetic of a step; angles that take
// the squarings are not foreseen.
QueueLines queue_lines(const WorkSet& w, int grid_blocks) {
  const int64_t waves = 4 * (int64_t)grid_blocks, reach = 8 * waves;
  if (w.n_items <= 4 * waves) return {0, 0, 0};
  std::vector<int64_t> first;  // of every descriptor that has items
  std::vector<double> cost;
  for (const SimDesc& d : w.sims)
    if (d.k_count > 0) {
      first.push_back(d.item_off);
      cost.push_back(item_cost(d));
    }
  const size_t n = first.size();
  first.push_back(w.n_items);
  std::vector<double> work(n + 1, 0.0);  // from descriptor j to the end
  for (size_t j = n; j-- > 0;) work[j] = work[j + 1] + cost[j] * (double)(first[j + 1] - first[j]);
  // the longest run of items from `from` on at which k may be taken; with
  // here, only a run that holds `from`
  auto longest = [&](int k, int64_t from, bool here) {
    struct Run {
      int64_t begin, end;
    } best = {from, from}, run = {-1, -1};
    std::vector<size_t> top;  // descriptors in reach, by falling cost, from head on
    size_t head = 0, next = 0, j = 0;
    for (int64_t x = 0; x < w.n_items;) {
      while (first[j + 1] <= x) ++j;
      for (; next < n && first[next] <= x + reach; ++next) {
        while (top.size() > head && cost[top.back()] <= cost[next]) top.pop_back();
        top.push_back(next);
      }
      while (top[head] < j) ++head;
      // a piece with the same descriptors in reach; the rules hold at the
      // first of its items or at none
      int64_t end = first[j + 1];
      if (next < n) end = std::min(end, first[next] - reach);
      const double spare = (work[j] - k * cost[top[head]] * (double)waves) / cost[j];
      int64_t stop = std::min(end, w.n_items - 2 * k * waves);
      if (spare < (double)(stop - first[j])) stop = first[j] + (int64_t)std::max(0.0, ceil(spare));
      if (stop > x && stop > from) {
        if (run.end != x) run.begin = std::max(x, from);
        run.end = stop;
        if ((!here || run.begin == from) && run.end - run.begin > best.end - best.begin) best = run;
      }
      x = end;
    }
    return best;
  };
  const auto four = longest(4, 0, false);
  if (four.end > four.begin) return {four.begin, four.end, longest(2, four.end, true).end};
  const auto two = longest(2, 0, false);
  return {two.begin, two.begin, two.end};
}

hipError_t launch_work_integrate(const DevWork& w, unsigned long long* counter, int grid_blocks,
                                 hipStream_t st, hipFunction_t user_fn, bool counter_zeroed) {
  if (w.n_items == 0) return hipSuccess;
  if (!counter_zeroed) hipLaunchKernelGGL(work_reset_kernel, dim3(1), dim3(64), 0, st, counter);
  IntegrateWorkArgs a{w.sims, w.terms, counter, w.n_items, w.n_sims, w.lines};
  if (user_fn) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    void* args[] = {&a};
    return hipModuleLaunchKernel(user_fn, (unsigned)grid_blocks, 1, 1, 256, 1, 1, 0, st, args,
                                 nullptr);
  }
  hipLaunchKernelGGL(work_integrate_kernel, dim3(grid_blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}

size_t chain_workspace_bytes(int32_t n_sims) {
  return sizeof(ChainSync) + a256((size_t)std::max(1, n_sims) * sizeof(ChainSlot));
}

hipError_t launch_work_chained(const DevWork& w, void* ws, int grid_blocks, hipStream_t st,
                               hipFunction_t user_fn, unsigned long long wait_ticks) {
  if (w.n_units == 0) return hipSuccess;
  ChainSync* sync = (ChainSync*)ws;
  const int64_t n_words = (int64_t)w.n_sims * (sizeof(ChainSlot) / sizeof(unsigned long long));
  ChainSlot* slots = (ChainSlot*)((char*)ws + sizeof(ChainSync));
  hipLaunchKernelGGL(chain_reset_kernel, dim3((unsigned)((n_words + 255) / 256)), dim3(256), 0, st,
                     sync, (unsigned long long*)slots, n_words);
  IntegrateWorkArgs a{w.sims, w.terms, &sync->counter, w.n_units, w.n_sims};
  a.n_groups = w.n_groups;
  a.group_item0 = w.group_item0;
  a.group_round0 = w.group_round0;
  a.group_count = w.group_count;
  a.order = w.order;
  a.slots = slots;
  a.sync = sync;
  a.wait_ticks = wait_ticks;
  if (user_fn) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    void* args[] = {&a};
    return hipModuleLaunchKernel(user_fn, (unsigned)grid_blocks, 1, 1, 256, 1, 1, 0, st, args,
                                 nullptr);
  }
  hipLaunchKernelGGL(work_chained_kernel, dim3(grid_blocks), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int E, bool REV>
static void scan_levels(const DevWork& w, hipStream_t st) {
  for (int l = 0; l < w.n_levels; ++l) {
    const int64_t tiles = w.reduce_total[l];
    if (!tiles) continue;
    ScanWorkArgs a{w.sims, w.reduce_tiles[l], tiles, w.n_sims, l};
    hipLaunchKernelGGL((work_reduce_kernel<E, REV>), dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st,
                       a);
  }
  for (int l = w.n_levels; l >= 0; --l) {
    const int64_t tiles = w.apply_total[l];
    if (!tiles) continue;
    ScanWorkArgs a{w.sims, w.apply_tiles[l], tiles, w.n_sims, l};
    hipLaunchKernelGGL((work_apply_kernel<E, REV>), dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st,
                       a);
  }
}

hipError_t launch_work_scan(const DevWork& w, hipStream_t st) {
  if (w.reversed) scan_levels<kScanPerLane, true>(w, st);
  else if (w.scan_e == 2) scan_levels<2, false>(w, st);
  else if (w.scan_e == 8) scan_levels<8, false>(w, st);
  else scan_levels<4, false>(w, st);
  return hipGetLastError();
}

}  // namespace mss
