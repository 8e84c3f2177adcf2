// Pareto front of (makespan, largest peak[d]) over the candidates that completed, and the
// OVER_CAP flag recomputed for other caps.  A schedule has two properties in the paper, its bubble
// ratio (Section 7.1) and its memory footprint (Section 2); the front is every trade-off between
// the two that no other candidate beats, instead of one cut at a fixed cap.
//
// Two kernels.  pareto_tile_kernel: one workgroup per tile of kTile candidates sorts the tile by
// (makespan, peak, index), takes the running minimum of the peaks along the sorted order
// and keeps the entries whose peak is below every peak before them: the tile's own front, by
// ascending makespan and strictly descending peak, written compacted.  pareto_merge_kernel: one
// workgroup does the same with all tile fronts together if they fit in one tile (fronts are short: the peaks descend
// strictly), else it walks them, a cursor per tile.  The next point of the global front
// is the smallest (makespan, peak, index) among the entries whose peak is below the peak of the
// point found before; since peaks descend along a tile front, the entries a cursor skips can
// never qualify again, so every cursor only moves forward.  All steps are pure functions of the
// values, independent of workgroup scheduling.
//
// What bounds both: the latency of dependent steps on one compute unit, most of all the sort's (block_sort.h).  So a tile
// first drops what cannot be on its front, and sorts what is left, on evaluated schedules a few dozen of 2,048 candidates.  65,536
// candidates of 8 devices: tiles 16.8 us, merge 9.1 us (25 and 10 us where all of a tile was sorted and one thread fetched a
// tile's front).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "block_sort.h"
#include "kernels.h"

namespace fpsched {

namespace {

constexpr long long kInf = 0x7fffffffffffffffll;
constexpr int kNoPeak = 0x7fffffff;

// An element of the sort: makespan in the order of unsigned numbers, peak << 32 | index (a batch has fewer than 2^24
// candidates); kNoEntry behind all real ones.
using FrontElem = SortElem<unsigned long long>;
constexpr unsigned long long kNoEntry = ~0ull;
__device__ __forceinline__ FrontElem front_elem(long long makespan, int peak, unsigned idx) {
  return FrontElem{(unsigned long long)makespan ^ (1ull << 63), (unsigned long long)(unsigned)peak << 32 | idx};
}

// LDS of a workgroup of kTile / 2 threads
struct FrontBuffer {
  unsigned long long key[kTile], pos[kTile];
  int wave_min[kTile / 128], wave_kept[kTile / 128];
};

// Sorts the workgroup's elements (a, b as block_sort holds them; all within the first `size`) and hands the front's entries, in order, to
// emit(position, element); returns their number.  All threads call this.
template <typename Emit>
__device__ __forceinline__ int sorted_front(FrontElem a, FrontElem b, int size, FrontBuffer& buf, Emit emit) {
  block_sort<unsigned long long>(a, b, size, SortBuffer<unsigned long long>{buf.key, buf.pos});
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int peak_a = a.pos == kNoEntry ? kNoPeak : (int)(a.pos >> 32), peak_b = b.pos == kNoEntry ? kNoPeak : (int)(b.pos >> 32);
  // running minimum of the peaks within the wavefront, up to and with each element
  int min_a = peak_a, min_b = peak_b;
#pragma unroll
  for (int step = 1; step < 64; step <<= 1) {
    const int oa = __shfl_up(min_a, step), ob = __shfl_up(min_b, step);
    if (lane >= step) { min_a = min(min_a, oa); min_b = min(min_b, ob); }
  }
  min_b = min(min_b, __shfl(min_a, 63));
  if (lane == 63) buf.wave_min[wave] = min_b;
  __syncthreads();
  int ahead = kNoPeak;
  for (int w = 0; w < wave; ++w) ahead = min(ahead, buf.wave_min[w]);
  int before_a = __shfl_up(min_a, 1), before_b = __shfl_up(min_b, 1);
  const int all_a = __shfl(min_a, 63);
  before_a = lane == 0 ? ahead : min(ahead, before_a);
  before_b = min(ahead, lane == 0 ? all_a : before_b);
  // (the first entry of all is on the front whatever its peak)
  const bool keep_a = a.pos != kNoEntry && (peak_a < before_a || threadIdx.x == 0);
  const bool keep_b = b.pos != kNoEntry && peak_b < before_b;
  const unsigned long long kept_a = __ballot(keep_a), kept_b = __ballot(keep_b);
  if (lane == 0) buf.wave_kept[wave] = __popcll(kept_a) + __popcll(kept_b);
  __syncthreads();
  int at = 0, total = 0;
  for (int w = 0; w < kTile / 128; ++w) {
    if (w == wave) at = total;
    total += buf.wave_kept[w];
  }
  const unsigned long long lower = (1ull << lane) - 1ull;
  if (keep_a) emit(at + __popcll(kept_a & lower), a);
  if (keep_b) emit(at + __popcll(kept_a) + __popcll(kept_b & lower), b);
  return total;
}

// Classes of peaks for the candidates that a tile drops before it sorts: ascending in the peak, 32 per factor of two, so that
// peaks below 64 have one each.  (float rounds in order; 2^31 - 1 becomes 2^31 and class 993.)
constexpr int kPeakClasses = kTile / 2;
__device__ __forceinline__ int peak_class(unsigned peak) {
  return peak == 0u ? 0 : (int)(__float_as_uint((float)peak) >> 18) - 127 * 32 + 1;
}
static_assert((158 - 127) * 32 + 1 < kPeakClasses, "");

// Drops entries that are not on the front of the workgroup's and puts the others next to each other, in any order, into
// buf.key and buf.pos; returns their number.  Of a class stays what is faster than all of the classes in front of it, and of that the
// best (makespan, peak, index) and whatever has a smaller peak than it.  All threads call this.
__device__ __forceinline__ int drop_dominated(const FrontElem& a, const FrontElem& b, FrontBuffer& buf, unsigned long long (&wave_fastest)[kTile / 128], int& held) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned long long* const fastest = buf.key;                    // of a class: its smallest makespan,
  unsigned long long* const ahead = buf.key + kPeakClasses;       // that of the classes in front of it,
  unsigned long long* const best = buf.pos;                       // the first (peak, index) of the former
  fastest[tid] = ~0ull;
  best[tid] = ~0ull;
  if (tid == 0) held = 0;
  __syncthreads();
  const bool have_a = a.pos != kNoEntry, have_b = b.pos != kNoEntry;
  const int class_a = have_a ? peak_class((unsigned)(a.pos >> 32)) : 0, class_b = have_b ? peak_class((unsigned)(b.pos >> 32)) : 0;
  // (a look first: lanes at one address take turns)
  auto fastest_yet = [&](int c) { return __hip_atomic_load(&fastest[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  if (have_a && a.key < fastest_yet(class_a)) atomicMin(&fastest[class_a], a.key);
  if (have_b && b.key < fastest_yet(class_b)) atomicMin(&fastest[class_b], b.key);
  __syncthreads();
  if (have_a && a.key == fastest[class_a]) atomicMin(&best[class_a], a.pos);
  if (have_b && b.key == fastest[class_b]) atomicMin(&best[class_b], b.pos);
  unsigned long long least = fastest[tid];
#pragma unroll
  for (int step = 1; step < 64; step <<= 1) {
    const unsigned long long o = __shfl_up(least, step);
    if (lane >= step) least = min(least, o);
  }
  if (lane == 63) wave_fastest[wave] = least;
  __syncthreads();
  unsigned long long before = __shfl_up(least, 1);
  if (lane == 0) before = ~0ull;
  for (int w = 0; w < wave; ++w) before = min(before, wave_fastest[w]);
  ahead[tid] = before;
  __syncthreads();
  auto stays = [&](const FrontElem& e, int c) {
    const unsigned long long first = best[c];
    return (e.key < ahead[c] || e.key == ~0ull) && (e.pos == first || e.pos >> 32 < first >> 32);
  };
  const bool keep_a = have_a && stays(a, class_a), keep_b = have_b && stays(b, class_b);
  const unsigned long long kept_a = __ballot(keep_a), kept_b = __ballot(keep_b);
  int at = 0;
  if (lane == 0 && (kept_a | kept_b) != 0ull) at = atomicAdd(&held, __popcll(kept_a) + __popcll(kept_b));
  at = __shfl(at, 0);
  __syncthreads();   // (everyone has looked at the classes, whose place the entries take)
  const unsigned long long lower = (1ull << lane) - 1ull;
  if (keep_a) {
    const int to = at + __popcll(kept_a & lower);
    buf.key[to] = a.key;
    buf.pos[to] = a.pos;
  }
  if (keep_b) {
    const int to = at + __popcll(kept_a) + __popcll(kept_b & lower);
    buf.key[to] = b.key;
    buf.pos[to] = b.pos;
  }
  __syncthreads();
  return held;
}

// The front of the first `held` entries of buf, as sorted_front hands it out.
template <typename Emit>
__device__ __forceinline__ int front_of_held(int held, FrontBuffer& buf, Emit emit) {
  auto load = [&](int i) { return i < held ? FrontElem{buf.key[i], buf.pos[i]} : FrontElem{kNoEntry, kNoEntry}; };
  const int ia = (threadIdx.x >> 6) * 128 + (threadIdx.x & 63);
  const FrontElem a = load(ia), b = load(ia + 64);
  int size = 128;
  while (size < held) size <<= 1;
  __syncthreads();
  return sorted_front(a, b, size, buf, emit);
}

}  // namespace

__global__ __launch_bounds__(kTile / 2) void pareto_tile_kernel(
    const long long* __restrict__ makespan, const int* __restrict__ peak, const unsigned char* __restrict__ flags,
    long long n, int D, Key* __restrict__ front_keys, int* __restrict__ front_peak, int* __restrict__ tile_count) {
  __shared__ FrontBuffer buf;
  __shared__ unsigned long long wave_fastest[kTile / 128];
  __shared__ int held;
  const long long base = (long long)blockIdx.x * kTile;
  auto load = [&](int i) {
    const long long g = base + i;
    FrontElem e{kNoEntry, kNoEntry};
    if (g < n && (flags[g] & (kDeadlock | kIncomplete)) == 0) {
      int mp = 0;
      for (int d = 0; d < D; ++d) mp = max(mp, peak[g * D + d]);
      e = front_elem(makespan[g], mp, (unsigned)g);
    }
    return e;
  };
  const FrontElem a = load(threadIdx.x), b = load(threadIdx.x + kTile / 2);
  const int left = drop_dominated(a, b, buf, wave_fastest, held);
  const int total = front_of_held(left, buf, [&](int at, const FrontElem& e) {
    front_keys[base + at] = Key{(long long)(e.key ^ (1ull << 63)), (long long)(unsigned)e.pos};
    front_peak[base + at] = (int)(e.pos >> 32);
  });
  if (threadIdx.x == 0) tile_count[blockIdx.x] = total;
}

__global__ __launch_bounds__(kParetoMergeThreads) void pareto_merge_kernel(
    const Key* __restrict__ front_keys, const int* __restrict__ front_peak, const int* __restrict__ tile_count,
    int tiles, int kmax, long long* __restrict__ out_idx, long long* __restrict__ out_makespan,
    int* __restrict__ out_peak, int* __restrict__ out_count) {
  // the fronts together, if they fit in one tile
  __shared__ union {
    FrontBuffer front;
    int cursor[kParetoMaxTiles];
  } lds;
  __shared__ int held;
  if (threadIdx.x == 0) held = 0;
  __syncthreads();
  // (as many lanes of a wavefront to a tile as there are, so that its entries come side by side)
  int per_tile = 64;
  while (per_tile > 1 && tiles * per_tile > kParetoMergeThreads) per_tile >>= 1;
  const int of_tile = threadIdx.x & (per_tile - 1), first_tile = threadIdx.x / per_tile, tile_step = kParetoMergeThreads / per_tile;
  int mine = 0;
  for (int t = first_tile; t < tiles; t += tile_step) mine += tile_count[t];
  int my_first = of_tile == 0 && mine > 0 ? atomicAdd(&held, mine) : 0;
  my_first = __shfl(my_first, (threadIdx.x & 63) - of_tile);
  __syncthreads();
  if (held <= kTile) {
    int at = my_first;
    for (int t = first_tile; t < tiles; t += tile_step) {
      const long long base = (long long)t * kTile;
      const int cnt = tile_count[t];
      for (int i = of_tile; i < cnt; i += per_tile) {
        const Key k = front_keys[base + i];
        const FrontElem e = front_elem(k.makespan, front_peak[base + i], (unsigned)k.idx);
        lds.front.key[at + i] = e.key;
        lds.front.pos[at + i] = e.pos;
      }
      at += cnt;
    }
    __syncthreads();
    const int total = front_of_held(held, lds.front, [&](int to, const FrontElem& e) {
      if (to >= kmax) return;
      out_idx[to] = (long long)(unsigned)e.pos;
      out_makespan[to] = (long long)(e.key ^ (1ull << 63));
      out_peak[to] = (int)(e.pos >> 32);
    });
    for (int i = total + threadIdx.x; i < kmax; i += kParetoMergeThreads) {
      out_idx[i] = -1;
      out_makespan[i] = kInf;
      out_peak[i] = -1;
    }
    if (threadIdx.x == 0) *out_count = min(total, kmax);
    return;
  }
  int* const cursor = lds.cursor;
  constexpr int kWaves = kParetoMergeThreads / 64;
  __shared__ long long wave_ms[2][kWaves];
  __shared__ long long wave_idx[2][kWaves];
  __shared__ int wave_peak[2][kWaves];
  for (int t = threadIdx.x; t < tiles; t += kParetoMergeThreads) cursor[t] = 0;   // read back by the same thread only
  long long below = kInf;   // the next point needs a peak smaller than this
  int written = 0;
  while (written < kmax) {
    long long b_ms = kInf, b_idx = kInf;
    int b_peak = kNoPeak;
    for (int t = threadIdx.x; t < tiles; t += kParetoMergeThreads) {   // each tile has one owner thread
      const long long base = (long long)t * kTile;
      int cur = cursor[t];
      const int cnt = tile_count[t];
      while (cur < cnt && front_peak[base + cur] >= below) ++cur;
      cursor[t] = cur;
      if (cur < cnt) {
        const Key k = front_keys[base + cur];
        const int pk = front_peak[base + cur];
        if (k.makespan < b_ms || (k.makespan == b_ms && (pk < b_peak || (pk == b_peak && k.idx < b_idx)))) {
          b_ms = k.makespan; b_peak = pk; b_idx = k.idx;
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      const long long o_ms = __shfl_xor(b_ms, off), o_idx = __shfl_xor(b_idx, off);
      const int o_peak = __shfl_xor(b_peak, off);
      if (o_ms < b_ms || (o_ms == b_ms && (o_peak < b_peak || (o_peak == b_peak && o_idx < b_idx)))) {
        b_ms = o_ms; b_peak = o_peak; b_idx = o_idx;
      }
    }
    const int buf = written & 1;
    if ((threadIdx.x & 63) == 0) {
      wave_ms[buf][threadIdx.x >> 6] = b_ms;
      wave_idx[buf][threadIdx.x >> 6] = b_idx;
      wave_peak[buf][threadIdx.x >> 6] = b_peak;
    }
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) {
      const long long o_ms = wave_ms[buf][w], o_idx = wave_idx[buf][w];
      const int o_peak = wave_peak[buf][w];
      if (o_ms < b_ms || (o_ms == b_ms && (o_peak < b_peak || (o_peak == b_peak && o_idx < b_idx)))) {
        b_ms = o_ms; b_peak = o_peak; b_idx = o_idx;
      }
    }
    if (b_idx == kInf) break;   // the same value in every thread: no entry is left
    if (threadIdx.x == 0) {
      out_idx[written] = b_idx;
      out_makespan[written] = b_ms;
      out_peak[written] = b_peak;
    }
    below = b_peak;
    ++written;
  }
  for (int i = written + threadIdx.x; i < kmax; i += kParetoMergeThreads) {
    out_idx[i] = -1;
    out_makespan[i] = kInf;
    out_peak[i] = -1;
  }
  if (threadIdx.x == 0) *out_count = written;
}

__global__ void apply_caps_kernel(const int* __restrict__ peak, const int* __restrict__ caps, int per_candidate,
                                  long long n, int D, unsigned char* __restrict__ flags) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const unsigned fl = flags[c];
  bool over = false;
  for (int d = 0; d < D; ++d) over |= peak[c * D + d] > caps[per_candidate ? c * D + d : d];
  over &= (fl & (kDeadlock | kIncomplete)) == 0;
  flags[c] = (unsigned char)((fl & ~(unsigned)kOverCap) | (over ? kOverCap : 0));
}

}  // namespace fpsched
