// Order pass of the list evaluation: everything about a device's list that does not depend on time.
//
// Whether the ops of a list respect the activation state machine, the peak of the resident memory and the summed
// durations are functions of the order of the list alone: only a device's own ops change the states of its
// activations, and an op that is not legal where it stands can never issue.  So this pass walks every row on its
// own, one lane per (candidate, device) row and 64 rows per wavefront, no lane ever waiting for another, and
// leaves per row where the list stops, why, its peak and its busy time.  What is left for the timing pass
// (timing.hip), where most lanes wait for inputs most of the time, are the dependencies between devices.
//
// Per word: its table row (8 bytes in LDS, addressed by the top five bits of the word and the device) and its
// activation state, one byte per (chunk, micro-batch) in lane-private LDS.  A legal op's next state does not
// depend on the state found, so the eight words of a group read the old state and write the new one in list order
// without waiting for each other, and the comparisons follow when all have arrived.  A group in which some lane's
// list stops (its END word, or an op that is not legal) is gone over again for those lanes: the states behind the
// stop are put back, the sums taken up to it.
//
// What bounds it: per 64 words twelve vector instructions and twelve clocks of LDS, and the op words once from HBM; none
// of the three is at its limit (65,536 candidates of 32 devices, 128 micro-batches, two chunks, profiles/list_evaluation.md:
// vector units 55 % busy, LDS 58 %, 3.8 GB at 3.7 TB/s in 1.03 ms), what is left are waits with eight wavefronts per compute
// unit.  A row is read 64 bytes at a time.  (Fourteen vector instructions, the places of the states worked out word
// by word: 1.15 ms in the same run.  States without bank conflicts, a dword of all rows side by side: LDS 32 % busy, one
// instruction more, 1.14 ms.  128 bytes at a time: 5 % less on long batches of 16 devices, none on 32, 2 to 3 % more on
// short rows.)
//
// SHARED: a load in which every lane reads a row of its own asks for 64 lines, one after the other, and the three behind it
// for the same lines while they are on their way.  With twelve wavefronts per compute unit that is what the pass waits for
// (262,144 candidates of 16 devices, 64 micro-batches, two chunks: address units busy half the time, 0.97 ms).  Four lanes that read
// 64 bytes of each other's rows in turn ask for a quarter as many (0.77 ms); handing the words round takes 32 vector instructions
// per 64 bytes of 64 rows, which is more than is gained with eight wavefronts per compute unit or fewer (the batch of 32 devices
// above: 1.09 and 1.16 ms) and on rows of one or two requests (262,144 candidates of 4 devices, rows of 16 words, whole evaluation: 165 and
// 169 us; rows of 64 to 96 words the same either way, of 150 words 565 and 518 us).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "lds_access.h"

namespace fpsched {

namespace {

typedef unsigned short u16_pair __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned bits_of(u16_pair v) { return __builtin_bit_cast(unsigned, v); }
__device__ __forceinline__ u16_pair pair_of(unsigned v) { return __builtin_bit_cast(u16_pair, v); }

typedef unsigned uint4_of_row __attribute__((ext_vector_type(4)));
// Of two registers, lanes that differ in bit BIT (0 or 1) of their number trade: the one with 0 there gets the other's `a` as
// its second value, that one its `b` as its first.
template <int BIT>
__device__ __forceinline__ void exchange_lanes(const uint4& a, const uint4& b, uint4& first, uint4& second) {
  constexpr unsigned long long kLower = BIT == 0 ? 0x5555555555555555ull : 0x3333333333333333ull;
#define FPSCHED_TRADE(PERM)                                                              \
  asm volatile("s_nop 1\n\t"                                                             \
      "s_mov_b64 vcc, %16\n\t"                                                           \
      "v_cndmask_b32_dpp %0, %12, %8, vcc " PERM "\n\t"                                 \
      "v_cndmask_b32_dpp %1, %13, %9, vcc " PERM "\n\t"                                 \
      "v_cndmask_b32_dpp %2, %14, %10, vcc " PERM "\n\t"                                \
      "v_cndmask_b32_dpp %3, %15, %11, vcc " PERM "\n\t"                                \
      "s_not_b64 vcc, vcc\n\t"                                                           \
      "v_cndmask_b32_dpp %4, %8, %12, vcc " PERM "\n\t"                                 \
      "v_cndmask_b32_dpp %5, %9, %13, vcc " PERM "\n\t"                                 \
      "v_cndmask_b32_dpp %6, %10, %14, vcc " PERM "\n\t"                                \
      "v_cndmask_b32_dpp %7, %11, %15, vcc " PERM                                        \
      : "=&v"(first.x), "=&v"(first.y), "=&v"(first.z), "=&v"(first.w), "=&v"(second.x), "=&v"(second.y), "=&v"(second.z), \
        "=&v"(second.w)                                                                  \
      : "v"(a.x), "v"(a.y), "v"(a.z), "v"(a.w), "v"(b.x), "v"(b.y), "v"(b.z), "v"(b.w), "s"(kLower) \
      : "vcc", "scc")
  if constexpr (BIT == 0) FPSCHED_TRADE("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf");
  else FPSCHED_TRADE("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf");
#undef FPSCHED_TRADE
}

}  // namespace

// threads: of the workgroup.  counter: null where nothing is drawn.
// VBITS: bits of the chunk field that select a chunk's states (0, 1, 2: up to 1, 2, 4 stages per device)
template <int VBITS, bool NO_W, bool SHARED>
__device__ __forceinline__ void check_rows(
    const ListTables& T, const uint16_t* __restrict__ ops, long long n_rows, int stride, int rows_per_wave,
    long long* __restrict__ out_info, int* __restrict__ out_peak, unsigned long long* __restrict__ counter,
    unsigned long long counter_value, int draw_blocks, int dynamic, int threads) {
  extern __shared__ int32_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // where the timing pass draws its candidates from (dynamic: set, with the counter of this pass behind it, by a kernel
  // in front of this one)
  if (counter && !dynamic && blockIdx.x == 0 && tid == 0) *counter = counter_value;
  // The order rows, in columns or device by device (check_shape), and the dev rows.  The number of columns is a power of two:
  // the row of a word is where a shift and a mask leave the word's top five bits.
  constexpr int kRows = kNKinds * kMaxChunks;
  const int columns = T.check_columns, n_row_ints = 2 * kRows * (columns > 0 ? columns : T.D);
  const bool repeated = (T.D & (T.D - 1)) == 0;   // column c is of device c modulo D
  for (int i = tid; i < (kRows + 1) * T.D; i += threads) {
    const int2 from = reinterpret_cast<const int2*>(T.ints + T.off_check)[i];
    const int row = repeated ? i >> __builtin_ctz(T.D) : (int)((unsigned)i / (unsigned)T.D), of = i - row * T.D;
    int at = columns > 0 ? row * columns + of : of * kRows + (row ^ (of & (kRows - 1))), n = repeated && columns > 0 ? columns : 1;
    if (row == kRows) at = n_row_ints / 2 + of, n = 1;
    for (int c = 0; c < n; c += T.D, at += T.D) {
      lds[2 * at] = from.x;
      lds[2 * at + 1] = from.y;
    }
  }
  const unsigned lds0 = lds_address(lds);
  const int m = T.m;
  // the states of this wavefront's rows, then of this lane's: one byte per (chunk, micro-batch), m + 1 bytes per chunk
  const unsigned wave_states = lds0 + (unsigned)T.check_shared_bytes + (unsigned)wave * (unsigned)T.check_wave_bytes;
  const unsigned state = wave_states + (unsigned)(lane < rows_per_wave ? lane : 0) * (unsigned)T.state_bytes;
  __syncthreads();
  // The wavefronts of the resident workgroups take blocks of rows from a counter, none waiting for another: as one
  // workgroup per few blocks, a compute unit's LDS stays with the workgroup until its last row has ended, and with equal
  // shares the slowest wavefronts took a third longer than the average one.
  const long long n_blocks = (n_rows + rows_per_wave - 1) / rows_per_wave;
  const unsigned row_bytes = columns > 0 ? (unsigned)columns * 8u : 8u;
  const unsigned dev_table = lds0 + (unsigned)n_row_ints * 4u;
  // (from vector registers: an operand from a scalar one doubles what the instruction costs)
  unsigned shift_low = 11u - (unsigned)__builtin_ctz(row_bytes), shift_high = shift_low + 16u, row_mask = 31u * row_bytes;
  asm volatile("" : "+v"(shift_low), "+v"(shift_high), "+v"(row_mask));
  // The row that this lane walks, and the words of it or of the next one that are on their way or in registers: 64 bytes of
  // each row at a time, requested when the walk of those in front of them begins.  SHARED: by the row's four neighbouring
  // lanes, sixteen bytes each, row after row; what has arrived is then handed round among them.
  long long r = 0;
  int d = 0;
  bool active = false;
  constexpr int kGroups = 4;
  const unsigned quarter = lane & 3, row_bytes2 = (unsigned)stride * 2u;
  const unsigned lane_at = (unsigned)(lane & ~3) * row_bytes2 + quarter * 16u;
  const uint16_t* row = ops;
  int rows_here = 0;   // SHARED: of the block, less those in front of these four lanes'
  uint4 first[kGroups], second[kGroups], asked[SHARED ? kGroups : 1];
  auto request = [&](uint4 (&piece)[kGroups], int at) {
    if constexpr (SHARED) {
      typedef const __attribute__((address_space(1))) char global_bytes;
      typedef const __attribute__((address_space(1))) uint4_of_row global_piece;
      global_bytes* const block_at = (global_bytes*)of_first_lane((long long)row);   // (one address of the wavefront)
      const bool in_row = at + 8 * (int)quarter < stride;
      const unsigned from = lane_at + (unsigned)at * 2u;
#pragma unroll
      for (int i = 0; i < kGroups; ++i) {
        global_bytes* row_at = block_at + (size_t)i * row_bytes2;
        asm("" : "+s"(row_at));   // (and a lane's offset)
        if (in_row && i < rows_here) {
          const uint4_of_row v = *(global_piece*)(row_at + from);
          asked[i] = make_uint4(v.x, v.y, v.z, v.w);
        }
      }
    } else {
#pragma unroll
      for (int g = 0; g < kGroups; ++g)
        if (at + 8 * g < stride) piece[g] = *reinterpret_cast<const uint4*>(row + at + 8 * g);
    }
  };
  auto arrive = [&](uint4 (&piece)[kGroups]) {
    if constexpr (SHARED) {
      uint4 half[kGroups];
      exchange_lanes<0>(asked[0], asked[1], half[0], half[1]);
      exchange_lanes<0>(asked[2], asked[3], half[2], half[3]);
      exchange_lanes<1>(half[0], half[2], piece[0], piece[2]);
      exchange_lanes<1>(half[1], half[3], piece[1], piece[3]);
    }
  };
  auto take = [&](long long block) {
    r = block * rows_per_wave + lane;
    active = lane < rows_per_wave && r < n_rows;
    r = active ? r : 0;
    d = n_rows >> 31 ? (int)(r % T.D) : (int)((unsigned)r % (unsigned)T.D);
    row = ops + (size_t)(SHARED ? block * rows_per_wave : r) * (size_t)stride;
    rows_here = (int)min((long long)rows_per_wave, n_rows - block * rows_per_wave) - (lane & ~3);
    request(first, 0);
  };
  // (drawn several at a time: atomics on one address complete at some 8e7 per second)
  long long block = ((long long)blockIdx.x * (threads >> 6) + wave) * draw_blocks;
  int left = draw_blocks;
  if (block < n_blocks) take(block);
  while (block < n_blocks) {
  // the next block's number is on its way during the walk, its first words during the end of this block
  long long drawn = n_blocks;
  const bool draw = --left == 0;
  if (draw && dynamic && lane == 0) drawn = (long long)atomicAdd(counter + 1, (unsigned long long)draw_blocks);
  for (int i = lane * 16; i < T.check_wave_bytes; i += 1024) lds_write<lds_int4>(wave_states + i, lds_int4{0, 0, 0, 0});
  const lds_int2 dev = lds_read<lds_int2>(dev_table + (unsigned)d * 8u);
  const int n_chunks = dev.x, cap = dev.y;
  const unsigned meta = lds0 + (columns > 0 ? (unsigned)(d + (repeated ? lane & (columns - 1) & -T.D : 0)) * 8u : (unsigned)d * 256u + ((unsigned)d & 31u) * 8u);
  // (the items of a chunk's stage stand in its row of kind 0: m, or fewer where an item is a group of micro-batches)
  auto items_of = [&](unsigned c) -> int { return lds_read<int>((c * row_bytes ^ meta) + 4u); };
  auto pad = [&](unsigned value) {
    for (int c = 0; c < n_chunks; ++c)
      for (int i = items_of((unsigned)c); i <= m; ++i) lds_write<uint8_t>(state + c * (m + 1) + i, (uint8_t)value);
  };
  if (active) pad(kPadState);
  int mem = 0, pk = 0;
  unsigned busy = 0u;
  bool alive = active;
  int stop = stride;
  unsigned status = 0u;

  // A group is eight words, in three stages: fetch the table rows; read the old states and write the new ones, in list
  // order; compare and sum up.  The rows of a group are fetched before the comparisons of the group in front of it,
  // which cover their latency, as the fetching of the next rows covers that of the states.
  struct Group {
    uint4 q;
    unsigned x[8], y[8], old[8];
  };
  auto pair_word = [](const uint4& q, int k) -> unsigned { return k < 2 ? q.x : (k < 4 ? q.y : (k < 6 ? q.z : q.w)); };
  auto word_of = [&](const uint4& q, int k) -> unsigned { return (k & 1) ? pair_word(q, k) >> 16 : pair_word(q, k) & 0xffffu; };
  const u16_pair per_chunk = {(unsigned short)(m + 1), (unsigned short)(m + 1)};
  const u16_pair limit = {(unsigned short)m, (unsigned short)m};
  auto row_of = [&](const uint4& q, int k) -> unsigned {
    return __builtin_amdgcn_bitop3_b32(pair_word(q, k) >> ((k & 1) ? shift_high : shift_low), row_mask, meta, 0x6a);   // (a & b) ^ c
  };
  auto fetch = [&](Group& G, const uint4& q) {
    G.q = q;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const lds_int2 M = lds_read<lds_int2>(row_of(q, k));
      G.x[k] = (unsigned)M.x;
      G.y[k] = (unsigned)M.y;
    }
  };
  // where the state of a word's activation is: a micro-batch out of range looks at the byte behind its chunk, a chunk that
  // the device does not have at some chunk's bytes -- the op is found out either way and its write taken back
  auto states_of = [&](unsigned pair) -> unsigned {   // (of both words of a pair, 16 bits each, from this row's first on)
    unsigned at = bits_of(__builtin_elementwise_min(pair_of(pair & 0x07ff07ffu), limit));
    if (NO_W) {
      // a W item in range looks at the byte behind its chunk's items, whose state it asks for and leaves; one out of range
      // at item 0, which never has that state
      const u16_pair one = {1, 1}, zero = {0, 0};
      const unsigned other = bits_of(zero - __builtin_elementwise_min(pair_of((pair & 0xe000e000u) ^ 0x60006000u), one));
      const unsigned no_op = bits_of(__builtin_elementwise_min(limit - pair_of(at), one) * limit);
      at = (at & other) | (no_op & ~other);
    }
    if (VBITS > 0) {
      // (written out: the compiler makes comparisons and selects of it)
      unsigned chunk;
      asm("v_pk_lshrrev_b16 %0, 11, %1 op_sel_hi:[0,1]" : "=v"(chunk) : "v"(pair));
      chunk &= VBITS == 1 ? 0x00010001u : 0x00030003u;
      asm("v_pk_mad_u16 %0, %1, %2, %0" : "+v"(at) : "v"(chunk), "v"(bits_of(per_chunk)));
    }
    return at;
  };
  auto state_of = [&](unsigned two, int k) -> unsigned {
    unsigned at;
    if (k & 1) asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD src0_sel:DWORD src1_sel:WORD_1" : "=v"(at) : "v"(state), "v"(two));
    else asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD src0_sel:DWORD src1_sel:WORD_0" : "=v"(at) : "v"(state), "v"(two));
    return at;
  };
  auto exchange = [&](Group& G) {
    unsigned two = 0u;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if ((k & 1) == 0) two = states_of(pair_word(G.q, k));
      const unsigned at = state_of(two, k);
      G.old[k] = lds_read<uint8_t>(at);
      lds_write<uint8_t>(at, (uint8_t)G.x[k]);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) busy += G.y[k];
  };
  auto compare = [&](Group& G, int at) {
    const int mem0 = mem, pk0 = pk;
    unsigned long long bad[8], any = 0ull;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      asm volatile("v_cmp_ne_u32_sdwa %0, %1, %2 src0_sel:DWORD src1_sel:BYTE_1" : "=s"(bad[k]) : "v"(G.old[k]), "v"(G.x[k]));
      any |= bad[k];
      mem += (int)((G.x[k] >> 16) & 0xffu);
      pk = max(pk, mem);
      mem -= (int)(G.x[k] >> 24);
    }
    if (any != 0ull && __builtin_amdgcn_inverse_ballot_w64(any)) {
      // the list stops in this group: put back the states from the stop on, take the sums up to it
      int first_bad = 0;
#pragma unroll
      for (int k = 7; k >= 0; --k) first_bad = __builtin_amdgcn_inverse_ballot_w64(bad[k]) ? k : first_bad;
      mem = mem0; pk = pk0;
      unsigned stop_row = 0u, stop_word = 0u;
#pragma unroll
      for (int k = 7; k >= 0; --k)
        if (k >= first_bad) {
          lds_write<uint8_t>(state_of(states_of(pair_word(G.q, k)), k), (uint8_t)G.old[k]);
          busy -= lds_read<uint32_t>(row_of(G.q, k) + 4u);
        }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (k < first_bad) {
          mem += (int)((G.x[k] >> 16) & 0xffu);
          pk = max(pk, mem);
          mem -= (int)(G.x[k] >> 24);
        }
        if (k == first_bad) {
          stop_row = G.x[k];
          stop_word = word_of(G.q, k);
        }
      }
      // (an END word ends the list whatever its low bits are)
      if ((stop_word >> 13) != 0u)
        status = kRowStuck | ((((stop_row >> 8) & 0xffu) == kNoState || (int)(stop_word & 0x7ffu) >= items_of((stop_word >> 11) & 3u)) ? kRowMalformed : 0u);
      else if ((stop_word & 0x1000u) != 0u)
        status = kRowPlant;
      stop = at + first_bad;
      alive = false;
    }
  };

  Group A, B;
  auto walk = [&](uint4 (&piece)[kGroups], uint4 (&next)[kGroups], int at) {
    request(next, at + 8 * kGroups);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      Group& now = (g & 1) ? B : A;
      Group& then = (g & 1) ? A : B;
      if (g + 1 == kGroups) arrive(next);
      // (behind the end of the row this fetches rows of whatever words the registers hold, which nobody looks at)
      fetch(then, g + 1 < kGroups ? piece[g + 1] : next[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (alive) compare(now, at + 8 * g);
      alive = alive && at + 8 * g + 8 < stride;
      if (alive) exchange(then);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  arrive(first);
  fetch(A, first[0]);
  if (alive) exchange(A);
  for (int at = 0;; at += 16 * kGroups) {
    walk(first, second, at);
    if (__ballot(alive) == 0ull) break;
    walk(second, first, at + 8 * kGroups);
    if (__ballot(alive) == 0ull) break;
  }
  // (a list that fills its row stops at the row's end: stop is the stride)
  const long long r_done = r;
  const bool was_active = active;
  block = draw ? of_first_lane(drawn) : block + 1;
  if (draw) left = draw_blocks;
  if (block < n_blocks) take(block);
  if (was_active) {
  // every activation consumed?  (the bytes behind each chunk's items are set to the final state first)
  pad((unsigned)T.terminal);
  const unsigned want = (unsigned)T.terminal * 0x01010101u;
  const int n_bytes = n_chunks * (m + 1);
  unsigned differ = 0u;
  int i = 0;
  for (; i + 32 <= n_bytes; i += 32)
#pragma unroll
    for (int k = 0; k < 32; k += 4) differ |= lds_read<uint32_t>(state + i + k) ^ want;
  for (; i + 4 <= n_bytes; i += 4) differ |= lds_read<uint32_t>(state + i) ^ want;
  if (i < n_bytes) differ |= (lds_read<uint32_t>(state + i) ^ want) & ((1u << (8 * (n_bytes - i))) - 1u);
  if (differ != 0u) status |= kRowIncomplete;
  if (pk > cap) status |= kRowOverCap;
  out_info[r_done] = (long long)(((unsigned long long)((unsigned)stop | status) << 32) | busy);
  out_peak[r_done] = pk * T.unit_scale;
  }
  }
}

}  // namespace fpsched
