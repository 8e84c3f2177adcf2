// Sorting within a workgroup: two elements per thread, bitonic network.
//
// Of the 66 stages for 2048 elements only the ten whose partners sit in another wavefront go through LDS with a
// barrier; the others exchange inside a wavefront by DPP moves (strides 1, 2, 4, 8), lane permutation (16, 32) or
// between the thread's two registers.  An element is a 64-bit key and, unless PACKED, a 32-bit position that breaks
// ties; PACKED elements carry both in 64 bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace fpsched {

struct NoPos {};   // the key alone orders
template <typename P>
struct SortElem {
  unsigned long long key;
  P pos;
};
template <typename P>
__device__ __forceinline__ bool elem_less(const SortElem<P>& a, const SortElem<P>& b) {
  if constexpr (std::is_same<P, NoPos>::value) return a.key < b.key;
  else return a.key < b.key || (a.key == b.key && a.pos < b.pos);
}

// the value of lane ^ S
template <int S>
__device__ __forceinline__ unsigned lane_xor(unsigned x) {
  if (S == 1) return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0xb1, 0xf, 0xf, true);   // quad_perm 1,0,3,2
  if (S == 2) return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x4e, 0xf, 0xf, true);   // quad_perm 2,3,0,1
  if (S == 4)   // mirrored half row, then mirrored quads
    return (unsigned)__builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
  if (S == 8) return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, true);  // row rotated by 8
  return __shfl_xor(x, S, 64);
}
template <int S>
__device__ __forceinline__ unsigned long long lane_xor(unsigned long long x) {
  return ((unsigned long long)lane_xor<S>((unsigned)(x >> 32)) << 32) | lane_xor<S>((unsigned)x);
}
template <int S>
__device__ __forceinline__ NoPos lane_xor(NoPos x) { return x; }
template <int S, typename P>
__device__ __forceinline__ void sort_stage(SortElem<P>& e, bool keep_small) {
  const SortElem<P> o{lane_xor<S>(e.key), lane_xor<S>(e.pos)};
  if (elem_less(o, e) == keep_small) e = o;
}
// strides FROM .. 1 within 64 lanes, ascending where `up`
template <int FROM, typename P>
__device__ __forceinline__ void merge_lanes(SortElem<P>& e, bool up) {
  const int lane = threadIdx.x & 63;
  if (FROM >= 32) sort_stage<32>(e, ((lane & 32) == 0) == up);
  if (FROM >= 16) sort_stage<16>(e, ((lane & 16) == 0) == up);
  if (FROM >= 8) sort_stage<8>(e, ((lane & 8) == 0) == up);
  if (FROM >= 4) sort_stage<4>(e, ((lane & 4) == 0) == up);
  if (FROM >= 2) sort_stage<2>(e, ((lane & 2) == 0) == up);
  sort_stage<1>(e, ((lane & 1) == 0) == up);
}
// one element per lane of a wavefront, ascending
template <typename P>
__device__ __forceinline__ void sort_lanes(SortElem<P>& e) {
  const int lane = threadIdx.x & 63;
  merge_lanes<1>(e, (lane & 2) == 0);
  merge_lanes<2>(e, (lane & 4) == 0);
  merge_lanes<4>(e, (lane & 8) == 0);
  merge_lanes<8>(e, (lane & 16) == 0);
  merge_lanes<16>(e, (lane & 32) == 0);
  merge_lanes<32>(e, true);
}
template <typename P>
__device__ __forceinline__ void merge_pair(SortElem<P>& a, SortElem<P>& b, bool up) {
  if (elem_less(b, a) == up) { const SortElem<P> t = a; a = b; b = t; }
  merge_lanes<32>(a, up);
  merge_lanes<32>(b, up);
}

// LDS: 2 x blockDim.x keys and as many positions
template <typename P>
struct SortBuffer {
  unsigned long long* key;
  P* pos;
  __device__ __forceinline__ void put(int i, const SortElem<P>& e) const {
    key[i] = e.key;
    if constexpr (!std::is_same<P, NoPos>::value) pos[i] = e.pos;
  }
  __device__ __forceinline__ SortElem<P> get(int i) const {
    if constexpr (std::is_same<P, NoPos>::value) return {key[i], NoPos{}};
    else return {key[i], pos[i]};
  }
};

// Sorts elements [0, n) ascending; thread t of wavefront w holds elements 128 w + lane (a) and 128 w + 64 + lane (b).
// n: a power of two from 128 to 2 * blockDim.x, the same in all threads, which all call this.
template <typename P>
__device__ __forceinline__ void block_sort(SortElem<P>& a, SortElem<P>& b, int n, const SortBuffer<P>& buf) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, threads = blockDim.x;
  const bool mine = wave * 128 < n;   // (the other wavefronts only take part in the barriers)
  if (mine) {
    merge_lanes<1>(a, (lane & 2) == 0); merge_lanes<1>(b, (lane & 2) == 0);
    merge_lanes<2>(a, (lane & 4) == 0); merge_lanes<2>(b, (lane & 4) == 0);
    merge_lanes<4>(a, (lane & 8) == 0); merge_lanes<4>(b, (lane & 8) == 0);
    merge_lanes<8>(a, (lane & 16) == 0); merge_lanes<8>(b, (lane & 16) == 0);
    merge_lanes<16>(a, (lane & 32) == 0); merge_lanes<16>(b, (lane & 32) == 0);
    merge_lanes<32>(a, true); merge_lanes<32>(b, false);
    merge_pair(a, b, n == 128 || (wave & 1) == 0);
  }
  for (int size = 256; size <= n; size <<= 1) {
    const bool up = size == n || (wave * 128 & size) == 0;
    for (int stride = size >> 1; stride >= 128; stride >>= 1) {
      __syncthreads();
      buf.put(tid, a);
      buf.put(threads + tid, b);
      __syncthreads();
      if (mine) {
        const int other = tid ^ (stride >> 1);
        const SortElem<P> oa = buf.get(other), ob = buf.get(threads + other);
        const bool keep_small = ((wave * 128 & stride) == 0) == up;
        if (elem_less(oa, a) == keep_small) a = oa;
        if (elem_less(ob, b) == keep_small) b = ob;
      }
    }
    if (mine) merge_pair(a, b, up);
  }
  __syncthreads();
}

}  // namespace fpsched
