// Top-k under the memory cap: the k feasible candidates (flags == 0) with the
// smallest (makespan, index), ascending (paper Section 7.1: the tuner keeps the
// schedules whose bubble ratio is lowest; with fixed total work that is the
// least makespan).
//
// Each workgroup selects the k smallest of its part of the candidates, further launches the k smallest of what those left,
// the last one with one workgroup (a batch of one part needs one launch).  A workgroup collects candidates in LDS and sorts
// when the room is used up (block_sort.h); from then on only candidates in front of the k-th of the last sort
// are collected.  Before the first sort only those are that are not behind a bar which the first four batches give: each
// wavefront sorts its lanes' smallest, of which its share of k are in front of one, and the last of these is not in front of the
// k-th of all.  Of values in random order two to three times k get past it, so that a part is mostly sorted once, and all that
// it holds then: 4,096 candidates 15.6 -> 12.3 us at k = 1 and 18.3 -> 14.2 at k = 128, 65,536 at k = 16 18.0 -> 14.5, 262,144 at k = 64
// 34.5 -> 27.7 (all launches).  Not where a wavefront's share is more than a quarter of its lanes: the bar then drops too few
// (share of 64: 262,144 at k = 512 96.0 -> 100.6; of 16: at k = 128 49.1 -> 47.9).
//
// The time must not depend on the order of the values: a search that appends better and better candidates hands in falling
// ones, of which every element displaces the ones before it.  So a part is not walked from front to back but in strides of
// about 0.62 of its length (batch_step), which meets the best of a rising or falling sequence within a few
// batches, and a part has at most kTopkPartRooms times the elements that are sorted at a time, which bounds the sorts for
// any order.  Walked from the front, in at most 64 parts however large the batch, 1,048,576 values took 116 us (random
// order) and 702 us (falling) at k = 128, 1.2 ms (either) at k = 1024; now 68 and 72 us, 172 and 89 us.
//
// What bounds it: the latency of a few dependent steps on one compute unit (load, sort, launch): 12 us for 4,096
// candidates, 15 for 262,144 at k = 1, 48 at k = 128 (back to back; among other work a launch also waits for its code).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "block_sort.h"
#include "kernels.h"

namespace fpsched {

constexpr long long kInf = 0x7fffffffffffffffll;

namespace {

constexpr unsigned kNoPos = 0xffffffffu;

struct TopkSource {
  const long long* makespan;   // candidates: keys and flags
  const unsigned char* flags;
  const Key* keys;             // or survivors of the first launch
};

// Collects the k smallest of elements [first, first + n), ascending, in buf[0 .. *count), and more behind them (all
// threads get the same *count, at most k).  The elements are walked in `batches` >= n / threads batches of one per
// thread, `step` batches on at a time (step and batches have no common divisor).  P = NoPos: the key is
// value << 32 | position; returns false, in all threads, if some value does not fit.  P = unsigned: the value as an unsigned number in the order of the signed ones.
template <typename P>
__device__ bool select_smallest(const TopkSource& src, long long first, unsigned n, unsigned batches, unsigned step, int k,
                                const SortBuffer<P>& buf, int* taken, int* misfit, int* count) {
  constexpr bool kPacked = std::is_same<P, NoPos>::value;
  const int tid = threadIdx.x, threads = blockDim.x, lane = tid & 63, room = 2 * threads;
  constexpr int kBatch = 4;   // elements per thread on their way at a time
  SortElem<P> none{~0ull, P{}};
  if constexpr (!kPacked) none.pos = kNoPos;
  SortElem<P> bar = none;     // the k-th of the last sort: only elements in front of it are collected
  if (tid < 3) taken[tid] = 0;
  if (tid == 3) *misfit = 0;
  __syncthreads();
  int held = 0;               // elements in buf, the same number in all threads
  bool sorted = false;
  auto sort = [&]() {
    int size = 128;
    while (size < held) size <<= 1;
    const int ia = (tid >> 6) * 128 + lane, ib = ia + 64;
    SortElem<P> a = none, b = none;
    if (ia < held) a = buf.get(ia);
    if (ib < held) b = buf.get(ib);
    block_sort<P>(a, b, size, buf);
    if (ia < k) buf.put(ia, a);
    if (ib < k) buf.put(ib, b);
    __syncthreads();
    if (held >= k) bar = buf.get(k - 1);
    held = min(held, k);
    sorted = true;
  };
  const bool rough = n > 128u && 4 * k <= threads;
  int turn = 0;               // the counter of this try; those of the next two are 0 or about to be
  const unsigned stride = step * threads, wrap = batches * threads;
  unsigned at = 0;            // the batch's first element
  for (unsigned done = 0; done < batches; done += kBatch) {
    SortElem<P> e[kBatch];
    bool have[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const unsigned pos = at + tid;
      have[i] = pos < (done + i < batches ? n : 0u);
      at += stride;
      at = at >= wrap ? at - wrap : at;
      long long value = 0;
      if (have[i]) {
        const long long g = first + pos;
        if (src.keys) {
          const Key s = src.keys[g];
          value = s.makespan;
          have[i] = s.idx != kInf;
        } else {
          value = src.makespan[g];
          have[i] = src.flags[g] == 0;
        }
      }
      if constexpr (kPacked) {
        e[i].key = (unsigned long long)value << 32 | pos;
        if (have[i] && (unsigned long long)value >= 0xffffffffull) *misfit = 1;
      } else {
        e[i].key = (unsigned long long)value ^ (1ull << 63);
        e[i].pos = pos;
      }
    }
    if (done == 0 && rough) {
      // a first bar: the waves' share of k-th smallest lanes' smallest elements, the largest of them.  k elements are not
      // behind it.
      SortElem<P> least = none;
#pragma unroll
      for (int i = 0; i < kBatch; ++i)
        if (have[i] && elem_less(e[i], least)) least = e[i];
      sort_lanes(least);
      const int waves = threads >> 6, share = (k + waves - 1) / waves;   // (k <= threads: a lane's number)
      if (lane == share - 1) buf.put(tid >> 6, least);
      __syncthreads();
      bar = buf.get(0);
      for (int w = 1; w < waves; ++w) {
        const SortElem<P> o = buf.get(w);
        if (elem_less(bar, o)) bar = o;
      }
      // (the element itself is in front of the bar)
      if constexpr (kPacked) bar.key += bar.key != none.key ? 1ull : 0ull;
      else bar.pos += bar.pos != none.pos ? 1u : 0u;
      __syncthreads();
    }
    // the elements of a batch in front of the bar: a place for each in lane 0's `base`, and, a barrier later, their number
    int base = 0;
    bool take = false;
    unsigned long long takers = 0ull;
    auto count = [&](int i) {
      take = have[i] && elem_less(e[i], bar);
      takers = __ballot(take);
      base = 0;
      if (lane == 0 && takers != 0ull) base = held + atomicAdd(&taken[turn], __popcll(takers));
    };
    auto total = [&]() -> int {
      __syncthreads();
      const int more = taken[turn];
      // (read by all before the next barrier; in use again two barriers on)
      const int before = turn == 0 ? 2 : turn - 1;
      if (tid == 0) taken[before] = 0;
      turn = turn == 2 ? 0 : turn + 1;
      return more;
    };
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (done + i >= batches) break;
      // where there may not be room for what the batch adds: sort, which leaves k <= threads, if there is not
      if (__builtin_expect(held + threads > room, 0)) {
        count(i);
        if (held + total() > room) sort();
      }
      count(i);
      base = __shfl(base, 0);
      if (take) buf.put(base + __popcll(takers & ((1ull << lane) - 1ull)), e[i]);
      const int more = total();
      held += more;
      sorted = sorted && more == 0;
    }
  }
  if (kPacked && *misfit != 0) return false;
  if (!sorted && held > 0) sort();
  *count = held;
  return true;
}

}  // namespace

// One workgroup per part of n_part candidates; the last launch has one workgroup (final_* set) and writes the answer,
// any other the k survivors of each part, padded with keys behind all real ones.  batches, step: how a part is walked
// (select_smallest).  Dynamic LDS: 12 bytes per element of 2 * blockDim.x >= 2 * k.  wide_values: the caller knows that the values do not fit in 32 bits.
__global__ __launch_bounds__(kTopkThreads) void topk_kernel(
    const long long* __restrict__ in_makespan, const unsigned char* __restrict__ in_flags, const Key* __restrict__ in_keys,
    long long n, long long n_part, unsigned batches, unsigned step, int k, int wide_values, Key* __restrict__ out_keys, long long* __restrict__ final_idx,
    long long* __restrict__ final_makespan, int* __restrict__ final_count) {
  extern __shared__ unsigned long long topk_lds[];
  __shared__ int taken[3], misfit;
  const long long first = (long long)blockIdx.x * n_part;
  const unsigned here = (unsigned)min(n_part, n - first);
  const TopkSource src{in_makespan, in_flags, in_keys};
  const SortBuffer<unsigned> wide{topk_lds, reinterpret_cast<unsigned*>(topk_lds + 2 * blockDim.x)};
  int count;
  const bool packed = !wide_values && select_smallest<NoPos>(src, first, here, batches, step, k, SortBuffer<NoPos>{topk_lds, nullptr}, taken, &misfit, &count);
  if (!packed) {
    __syncthreads();
    select_smallest<unsigned>(src, first, here, batches, step, k, wide, taken, &misfit, &count);
  }
  for (int i = threadIdx.x; i < k; i += blockDim.x) {
    long long value = kInf, idx = kInf;
    if (i < count) {
      const unsigned long long key = topk_lds[i];
      const unsigned pos = packed ? (unsigned)key : wide.pos[i];
      value = packed ? (long long)(key >> 32) : (long long)(key ^ (1ull << 63));
      idx = in_keys ? in_keys[first + pos].idx : first + pos;
    }
    if (final_idx) {
      final_idx[i] = i < count ? idx : -1ll;
      final_makespan[i] = value;
    } else {
      out_keys[(long long)blockIdx.x * k + i] = Key{value, idx};
    }
  }
  if (final_idx && threadIdx.x == 0) *final_count = count;
}

// Ranking keys of evaluated candidates (one thread per candidate): the quantities the tuner can
// rank by besides the makespan -- the largest peak memory over the devices and the summed bubble
// time (Section 7.1: bubble ratio; Section 2: memory footprint as the second axis of a schedule).
// Two-part keys are packed primary << 32 | secondary (both below 2^31), so that the top-k kernel,
// which orders by (key, index), orders lexicographically.
__global__ void rank_keys_kernel(const long long* makespan, const long long* idle, const int* peak,
                                 const unsigned char* flags, long long n, int D, int mode, int include_over_cap,
                                 long long* key_out, unsigned char* excluded_out) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const unsigned fl = flags[c];
  const bool out = (fl & (kDeadlock | kIncomplete)) != 0 || (!include_over_cap && (fl & kOverCap) != 0);
  long long key = 0;
  if (!out) {
    int max_peak = 0;
    long long sum_idle = 0;
    for (int d = 0; d < D; ++d) {
      max_peak = max(max_peak, peak[c * D + d]);
      sum_idle += idle[c * D + d];
    }
    const long long ms = makespan[c];
    key = mode == 0 ? ms : (mode == 1 ? ((ms << 32) | (long long)max_peak)
                                      : (mode == 2 ? (((long long)max_peak << 32) | ms) : sum_idle));
  }
  key_out[c] = key;
  excluded_out[c] = out ? 1 : 0;
}

}  // namespace fpsched
