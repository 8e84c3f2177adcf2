// Weight-gradient sliding pass, second kernel (paper Section 5.2, "Bubble optimizations": the
// weight-gradient part of a backward pass is stashed and run in a later bubble of the same actor,
// so that what other actors wait for runs first).
//
// The rule: the W words of the input are dropped; every device walks its list under the
// evaluator's start rule; a B item that issues stashes its W item (first in, first out); in front
// of the next item of the list, which starts at t, the oldest stashed items run as long as they
// end by t; what is left when the list ends runs back to back.
//
// Because a stashed item only runs where it delays nothing, every item of the list starts exactly
// when it would start if there were no W items at all.  So the pass splits in two:
//   1. the lists are timed without their W items -- the only part with dependencies between devices -- by the order and
//      timing passes of the list evaluation in their forms for it (rows.h, timing.hip), or where those do not take the
//      problem or the model by the slot kernel in its TIMES form (eval_slots.hip); that leaves each op's start time and the
//      position at which each list stopped;
//   2. this kernel places the W items: one lane per (candidate, device) row, no interaction
//      between lanes until the final reduction.  A lane walks its row once.  One step per loop
//      iteration, the same code for all lanes: the oldest stashed item if it fits in front of the
//      item at the list cursor (or the list is over), else that item.  The new row is staged
//      in LDS and leaves in 32-byte pieces; memory is accounted along the new order.
// No global load sits on a step's critical path: op words and the low halves of their start times reach a
// lane through a 32-position LDS window that the whole wavefront tops up every eighth step, sixteen
// positions (32 bytes of each) at a time, the loads requested at one top-up landing at the next.  (With
// loads issued by each lane when it needs them the wavefront waited for memory in nearly every step:
// among 64 lanes at 64 different positions some lane always needs its next piece.)  The first kernel
// hands over sixteen bits per op: a start time is rebuilt from the device's free time in front of the op,
// start = free + ((low - free) mod 2^16), plus 2^16 times the entry of the row's escape list for the few
// ops that waited longer.  The stash is a ring of two bits per W item in LDS (the chunk; the micro-batch is
// counted); only a stash of more than kStash items, or one of a list whose B items are out of order, is
// read back from the device's own row, with the latency exposed.
//
// What bounds it: instruction issue and, with 11 wavefronts per compute unit, waits for LDS and loads.  32,768 candidates
// of 16 devices, 64 micro-batches, 2 chunks: 0.85 ms, some 75 vector instructions a step; 0.95 ms with 100, conditions as masks in vector
// registers and selects where now the lanes that an instruction is for execute it; 1.05 ms when the next entry of the escape list, loaded in a
// branch that is hardly ever taken, was waited for in every step, with all that was on its way for the windows; 1.2 ms with
// branches and scalar conditions in the step (150 vector and 110 scalar instructions); 2.6 ms with a stash
// ring of 16 words, which the lists of every loose in-flight limit overran, rows stored in 16-byte pieces (1.08 GB written
// instead of 0.50) and six wavefronts to a workgroup.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace fpsched {

namespace {

constexpr int kWin = 32;      // window: positions per lane (op words and the low halves of their start times)
constexpr int kPiece = 16;    // positions per load: 32 bytes of op words, 32 bytes of start times
constexpr int kRefillAt = 16; // a lane asks for its next piece when at most this many positions are unread
constexpr int kStash = 128;   // stash ring: entries of two bits per lane
constexpr int kOut = 32;      // staging ring of the new row: words per lane; stored sixteen (32 bytes) at a time
constexpr int kSteps = 8;     // between two top-ups
// conditions are sets of lanes in scalar registers, combined there
typedef unsigned long long Lanes;
__device__ __forceinline__ Lanes lanes(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool in(Lanes l) { return __builtin_amdgcn_inverse_ballot_w64(l); }
static_assert((2 * kWin + kStash / 8 + kOut) * 64 * 2 == kSlideWaveLdsBytes, "LDS of one wavefront");

}  // namespace

// FOUR: some device has more than two stages
template <bool FOUR>
__global__ __launch_bounds__(kSlideThreads) void wslide_place_kernel(
    SlotTables T, const uint16_t* __restrict__ ops, long long n_cand, int stride,
    const uint32_t* __restrict__ start_low, const uint32_t* __restrict__ escapes, int escape_cap,
    const int32_t* __restrict__ stop_pos,
    const unsigned char* __restrict__ timed_flags, uint16_t* __restrict__ ops_out, int stride_out,
    long long* __restrict__ out_makespan, long long* __restrict__ out_idle, int* __restrict__ out_peak,
    unsigned char* __restrict__ out_flags) {
  extern __shared__ int32_t lds[];
  const int lpc = T.lanes_per_cand;
  const int lpc_shift = __ffs(lpc) - 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // LDS: [of the metadata rows, per (kind * 4 + chunk, device): dur << 8, then units
  // allocated at the start (byte 0) | units freed at the end (byte 1)][per wavefront: window [position][lane],
  // op word | low half of its start time << 16; stash ring [entry][lane] and staging ring [dword][lane], 16 bits a word]
  const int n_meta_ints = kNKinds * kMaxChunks * lpc * 2;
  for (int i = threadIdx.x; i < n_meta_ints; i += blockDim.x) lds[i] = T.ints[i * 2 + (i & 1)];
  const int2* meta = reinterpret_cast<const int2*>(lds);
  uint32_t* window = reinterpret_cast<uint32_t*>(lds + n_meta_ints + wave * (kSlideWaveLdsBytes / 4)) + lane;   // position i at + i * 64
  uint32_t* ring = window + kWin * 64;                        // dword i (sixteen entries) at + i * 64
  uint32_t* staging = ring + kStash / 16 * 64;                // dword i at + i * 64
  __syncthreads();

  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long cand = t >> lpc_shift;
  const int d = (int)(t & (lpc - 1));
  const bool active = cand < n_cand && d < T.D;
  const size_t row_index = (size_t)(active ? cand : 0) * T.D + (active ? d : 0);
  const uint16_t* row = ops + row_index * (size_t)stride;
  // start times: [candidate][group of eight positions][lane of the candidate][8 x 16 bits], as dwords
  const uint32_t* start_row = start_low + (size_t)(active ? cand : 0) * ((size_t)stride >> 1) * (size_t)lpc + ((size_t)d << 2);
  const uint32_t* esc_row = escapes + row_index * (size_t)escape_cap;
  uint16_t* out_row = ops_out + row_index * (size_t)stride_out;
  int stop = active ? stop_pos[row_index] : 0;
  // a device that reached the end of its list runs what is still stashed back to back
  unsigned end_word = (active && stop < stride) ? row[stop] : 0u;
  // the first op that waited 2^16 time units or more (position << 8 | wait >> 16; all ones: none)
  unsigned esc = active ? esc_row[0] : 0xffffffffu;
  unsigned esc_pos = esc >> 8;
  int esc_at = 1;
  // have them in registers before the loop: a wait for them inside the loop would also wait for
  // the window loads in flight
  asm volatile("" : "+v"(stop), "+v"(end_word), "+v"(esc));
  const Lanes at_end = lanes(active && (end_word >> 13) == (unsigned)kEnd);

  // window: positions [loaded - kWin, loaded) of the row are in the rings; the whole wavefront tops
  // them up every eighth step, the loads requested at one top-up landing at the next
  int loaded = 0;
  uint4 pend_w0 = make_uint4(0u, 0u, 0u, 0u), pend_w1 = pend_w0, pend_s0 = pend_w0, pend_s1 = pend_w0;
  bool has_pend = false;
  auto land8 = [&](int q, uint4 wv, uint4 sv) {
    auto pair = [&](int i, unsigned w, unsigned s) {
      window[(q + i) * 64] = (w & 0xffffu) | (s << 16);
      window[(q + i + 1) * 64] = (w >> 16) | (s & 0xffff0000u);
    };
    pair(0, wv.x, sv.x); pair(2, wv.y, sv.y); pair(4, wv.z, sv.z); pair(6, wv.w, sv.w);
  };
  // a piece is sixteen positions, or eight at the end of a row whose stride is not a multiple of 16
  auto request = [&](int at) {
    pend_w0 = *reinterpret_cast<const uint4*>(row + at);
    pend_s0 = *reinterpret_cast<const uint4*>(start_row + ((size_t)(at >> 3) << (lpc_shift + 2)));
    if (at + 8 < stride) {
      pend_w1 = *reinterpret_cast<const uint4*>(row + at + 8);
      pend_s1 = *reinterpret_cast<const uint4*>(start_row + ((size_t)((at >> 3) + 1) << (lpc_shift + 2)));
    }
  };
  auto land = [&]() {
    const int q = loaded & (kWin - 1);
    land8(q, pend_w0, pend_s0);
    if (loaded + 8 < stride) land8(q + 8, pend_w1, pend_s1);
    loaded += (loaded + 8 < stride) ? kPiece : 8;
  };
  if (active)   // the head of the row is fetched before the first step
    for (int i = 0; i < 2 && loaded < stride; ++i) { request(loaded); land(); }

  int pos = 0, out_len = 0;
  unsigned t8 = 0u, busy8 = 0u;   // device free time and busy time, << 8
  unsigned u8 = 0u;               // the device's free time in the list without W items, << 8
  int mem = 0, pk = 0;
  Lanes done = lanes(!active);
  // Stash: a B item's W item is known by its chunk as long as the B items of each chunk come in ascending order of their
  // micro-batches (as in every list of the generator): entries [q_head, q_tail) of the ring are those chunks, two bits
  // each, and the micro-batch is a count.  `from_row`: B words from row position refill_pos on are not in the ring (it is
  // full, or a micro-batch is out of order); once it is empty they are read back from the row, one by one, until the list
  // cursor has been caught up with (an out-of-order chunk stays that way).
  unsigned q_head = 0u, q_tail = 0u, q_word_in = 0u;
  int refill_pos = 0;
  Lanes from_row = 0, out_of_order = 0;
  // next B word expected (without its kind), next W word, of chunks 0 and 1, 2 and 3, 16 bits each
  unsigned next_b[2] = {1u << 27, 2u << 11 | 3u << 27}, next_w[2] = {next_b[0] | 0x60006000u, next_b[1] | 0x60006000u};
  static_assert(kW << 13 == 0x6000, "");
  Lanes have_head = 0;         // q_word, q_dur8, q_free are those of the oldest stashed item
  unsigned q_word = 0u, q_dur8 = 0u;   // the oldest stashed item as a W word, its cost and what it frees
  int q_free = 0;
  // cost and freed units of the W item of each chunk of this device (rows kW * 4 + chunk of the metadata)
  // (as one vector value each: arrays would be indexed in memory)
  typedef int PerChunk __attribute__((ext_vector_type(kMaxChunks)));
  PerChunk w_dur8, w_free;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const int2 Mw = meta[(kW * kMaxChunks + c) * lpc + d];
    w_dur8[c] = Mw.x;
    w_free[c] = (int)(((unsigned)Mw.y >> 8) & 0xffu);
  }
  auto of_chunk = [&](const PerChunk& v, unsigned c) -> int {
    const int low = (c & 1u) != 0u ? v[1] : v[0];
    return FOUR && c > 1u ? ((c & 1u) != 0u ? v[3] : v[2]) : low;
  };
  // the next word of chunk c, and the one behind it
  auto next_of = [&](const unsigned (&n)[2], unsigned c) -> unsigned {
    const unsigned two = FOUR ? (c > 1u ? n[1] : n[0]) : n[0];
    return __builtin_amdgcn_ubfe(two, (c & 1u) << 4, 16u);
  };
  auto move_on = [&](unsigned (&n)[2], unsigned c) {
    const unsigned one = 1u << ((c & 1u) << 4);
    if (FOUR) {
      n[0] += c > 1u ? 0u : one;
      n[1] += c > 1u ? one : 0u;
    } else {
      n[0] += one;
    }
  };
  // the oldest stashed item becomes the next one of chunk c, or `word`
  auto set_head = [&](unsigned c, unsigned word) {
    q_word = word;
    move_on(next_w, c);
    q_dur8 = (unsigned)of_chunk(w_dur8, c);
    q_free = of_chunk(w_free, c);
  };
  // The new row is staged in LDS and stored sixteen words at a time when the window is topped up, behind the loads: lanes
  // fill up at different steps, so stores in the steps are issued in nearly every one, in pieces that the memory has to
  // merge, and a wait for the window's loads waits for them too.
  int stored = 0;
  const char* const meta_d = reinterpret_cast<const char*>(meta + d);
  const unsigned meta_row = (unsigned)lpc * 8u;
  auto meta_of = [&](unsigned top) -> int2 { return *reinterpret_cast<const int2*>(meta_d + __umul24(top, meta_row)); };
  typedef uint16_t half_of_dword __attribute__((may_alias));   // (stored in halves, read in dwords)
  auto put = [&](int at, unsigned word) { reinterpret_cast<half_of_dword*>(staging + ((at >> 1) & (kOut / 2 - 1)) * 64)[at & 1] = (uint16_t)word; };
  auto staged4 = [&](int at) {   // eight words from a multiple of eight on
    const uint32_t* w = staging + ((at >> 1) & (kOut / 2 - 1)) * 64;
    return make_uint4(w[0], w[64], w[128], w[192]);
  };

  // One step per iteration and lane, the same straight-line code for all: look at the word at the list
  // cursor (in the window unless the lane has outrun it: then it waits for the next top-up); the oldest
  // stashed item runs if it ends by the start of that item (or the list is over); else the item issues, or
  // a W word of the input is passed over.
  for (;;) {
    if (has_pend) {
      land();
      has_pend = false;
    }
    if (~done == 0ull) break;
    if (!in(done) && loaded - pos <= kRefillAt && loaded < stride) {
      request(loaded);
      has_pend = true;
    }
    if (out_len - stored >= 16) {
      // (the row keeps its first stride_out items; the candidate is reported as failed if there are more)
      if (stored + 8 <= stride_out) *reinterpret_cast<uint4*>(out_row + stored) = staged4(stored);
      if (stored + 16 <= stride_out) *reinterpret_cast<uint4*>(out_row + stored + 8) = staged4(stored + 8);
      stored += 16;
    }
    const int limit = min(stop, loaded);   // positions in front of it are in the window
#pragma unroll 2
    for (int step = 0; step < kSteps; ++step) {
      const unsigned e0 = window[(unsigned)(pos & (kWin - 1)) * 64u], e1 = window[(unsigned)((pos + 1) & (kWin - 1)) * 64u];
      const unsigned head_word = ring[__builtin_amdgcn_ubfe(q_head, 4u, 3u) * 64u];
      // a W word of the input at the cursor is passed over at once when the word behind it is there as well
      // (it is never in the escape list: in the first pass it starts the moment its device is free)
      const bool hop = in(lanes(__builtin_amdgcn_ubfe(e0, 13u, 3u) == (unsigned)kW) & lanes(pos + 1 < limit));
      pos += hop ? 1 : 0;
      const unsigned e = hop ? e1 : e0, kind = __builtin_amdgcn_ubfe(e, 13u, 3u);
      // (any 16-bit value indexes a row of the table: the top five bits of the word)
      const int2 M = meta_of(__builtin_amdgcn_ubfe(e, 11u, 5u));
      const Lanes have = lanes(pos < limit), over = lanes(pos >= stop);
      // the start time from its low half and the free time in front of the op, plus what the escape
      // list says for an op that waited 2^16 time units or more (of the word's bits below it none gets into the time)
      unsigned s8 = u8 + (((e >> 8) - u8) & 0x00ffff00u);
      const Lanes esc_here = lanes(esc_pos == (unsigned)pos);
      if (in(esc_here)) s8 += esc << 24;
      const Lanes item = have & lanes(kind != (unsigned)kW);   // where the input put its W items is not used
      const Lanes place = have_head & ((item & lanes(t8 + q_dur8 <= s8)) | (over & at_end & ~done));
      const Lanes issue = item & ~place;
      done |= over & ~place;
      put(out_len, in(place) ? q_word : e);   // (a word of a lane that does neither is overwritten by its next one)
      // an item of the list ends when it would without any W item; a W item takes its place in front of it
      asm volatile("s_mov_b64 exec, %[issue]\n\t"
                   "v_add_u32 %[t], %[start], %[cost]\n\t"
                   "v_add_u32_sdwa %[mem], %[mem], %[units] dst_sel:DWORD src0_sel:DWORD src1_sel:BYTE_0\n\t"
                   "v_add_u32 %[busy], %[busy], %[cost]\n\t"
                   "v_max_i32 %[pk], %[pk], %[mem]\n\t"
                   "v_mov_b32 %[u], %[t]\n\t"
                   "v_sub_u32_sdwa %[mem], %[mem], %[units] dst_sel:DWORD src0_sel:DWORD src1_sel:BYTE_1\n\t"
                   "s_mov_b64 exec, %[place]\n\t"
                   "v_add_u32 %[t], %[t], %[w_cost]\n\t"
                   "v_add_u32 %[busy], %[busy], %[w_cost]\n\t"
                   "v_sub_u32 %[mem], %[mem], %[w_units]\n\t"
                   "s_or_b64 exec, exec, %[issue]\n\t"
                   "v_add_u32 %[len], 1, %[len]\n\t"
                   "s_mov_b64 exec, -1"
                   : [t] "+&v"(t8), [u] "+&v"(u8), [mem] "+&v"(mem), [pk] "+&v"(pk), [busy] "+&v"(busy8), [len] "+&v"(out_len)
                   : [start] "v"(s8), [cost] "v"(M.x), [units] "v"(M.y), [w_cost] "v"(q_dur8), [w_units] "v"(q_free), [issue] "s"(issue),
                     [place] "s"(place)
                   : "scc");
      have_head &= ~place;
      // an issued B item stashes its W item
      const Lanes is_b = issue & lanes(kind == (unsigned)kB);
      const unsigned c = __builtin_amdgcn_ubfe(e, 11u, FOUR ? 2u : 1u);
      Lanes push = 0;
      const Lanes waiting = lanes(q_head != q_tail);   // (of those in front of this step's)
      if (is_b != 0ull) {
        out_of_order |= is_b & lanes(next_of(next_b, c) != (e & 0x1fffu));
        // (full: the next entry's word still holds older entries)
        const Lanes leave = is_b & (out_of_order | lanes(q_tail - (q_head & ~15u) == (unsigned)kStash));
        refill_pos = in(leave & ~from_row) ? pos : refill_pos;
        from_row |= leave;
        push = is_b & ~from_row;
        if (in(is_b)) move_on(next_b, c);
        if (in(push)) {
          const unsigned at = (q_tail & 15u) * 2u;
          q_word_in = (at == 0u ? 0u : q_word_in) | c << at;
          ring[__builtin_amdgcn_ubfe(q_tail, 4u, 3u) * 64u] = q_word_in;
          q_tail += 1u;
        }
      }
      const Lanes take = ~have_head & (waiting | push);
      if (in(take)) {
        const unsigned stashed = __builtin_amdgcn_ubfe(head_word, (q_head & 15u) * 2u, FOUR ? 2u : 1u), head = in(waiting) ? stashed : c;
        set_head(head, next_of(next_w, head));
        q_head += 1u;
      }
      have_head |= take;
      const Lanes refill = from_row & ~have_head;
      if (refill != 0ull) {
        // the ring is empty and B words wait in the row: the next one, up to the one just issued
        bool found = false, more = false;
        if (in(refill)) {
          const int end = pos + (in(issue) ? 1 : 0);
          while (refill_pos < end) {
            const unsigned b_word = row[refill_pos++];
            if ((b_word >> 13) == (unsigned)kB) {
              set_head((b_word >> 11) & 3u, (unsigned)kW << 13 | (b_word & 0x1fffu));
              found = true;
              break;
            }
          }
          more = refill_pos < end;
        }
        have_head |= lanes(found);
        from_row &= ~refill | out_of_order | lanes(more);
      }
      const Lanes advance = have & ~place;
      if (in(esc_here & advance)) {
        esc = esc_row[esc_at++];
        asm volatile("" : "+v"(esc));   // (waited for here, and not in every step together with all that is on its way for the window)
        esc_pos = esc >> 8;
      }
      pos += in(advance) ? 1 : 0;
    }
  }

  // ---- the rest of the new row: words still staged, then END words up to the stride
  if (active) {
    int at = min(out_len, stride_out);
    for (; at & 7; ++at) put(at, 0u);
    for (int i = stored; i < at; i += 8) *reinterpret_cast<uint4*>(out_row + i) = staged4(i);
    for (; at < stride_out; at += 8) *reinterpret_cast<uint4*>(out_row + at) = make_uint4(0u, 0u, 0u, 0u);
  }
  // ---- the evaluation of the new lists
  const int seg_base = (threadIdx.x & 63) & ~(lpc - 1);
  const unsigned long long seg_mask = (lpc == 64 ? ~0ull : ((1ull << lpc) - 1ull)) << seg_base;
  const int cap = active ? T.ints[T.off_dev + d * T.dev_ints + 1] : 0;
  const unsigned long long full = __ballot(active && out_len > stride_out) & seg_mask;
  const unsigned long long over = __ballot(active && pk > cap) & seg_mask;
  int ms = active ? (int)(t8 >> 8) : 0;
  for (int off = 1; off < lpc; off <<= 1) ms = max(ms, __shfl_xor(ms, off, 64));
  if (active) {
    unsigned fl = timed_flags[cand] & (kDeadlock | kIncomplete);
    if (full) fl |= kDeadlock | kIncomplete;
    const bool failed = fl != 0;
    if (!failed && over) fl = kOverCap;
    out_idle[cand * T.D + d] = failed ? -1ll : (long long)(ms - (int)(busy8 >> 8));
    out_peak[cand * T.D + d] = failed ? -1 : pk * T.unit_scale;
    if (d == 0) {
      out_makespan[cand] = failed ? 0x7fffffffffffffffll : (long long)ms;
      out_flags[cand] = (unsigned char)fl;
    }
  }
}

// The same for few candidates: one wavefront per row, a workgroup per candidate.  With a lane per row a step is some 200
// instructions and several LDS latencies long for the one item or W item it places, and few rows leave the GPU idle.  What a row
// needs is mostly local to its items: the gap in front of an item is its start less the end of the item in front of it, the W
// item of a B item stands at that item's number in the stash, and the memory in front of an item is a sum over the items and
// over the W items placed before it.  So 64 positions are read at a time, and only the gaps that a W item may fit are looked at
// one by one: how many fit follows from the summed costs of the stash's next 64 entries, compared by all lanes.
// 128 candidates of 32 devices, 128 micro-batches, 2 chunks: 0.42 ms with a lane per row, 0.19 here.
__global__ __launch_bounds__(kSlideThreads) void wslide_place_rows_kernel(
    SlotTables T, const uint16_t* __restrict__ ops, int stride, const uint32_t* __restrict__ start_low,
    const uint32_t* __restrict__ escapes, int escape_cap, const int32_t* __restrict__ stop_pos,
    const unsigned char* __restrict__ timed_flags, uint16_t* __restrict__ ops_out, int stride_out, int stash,
    long long* __restrict__ out_makespan, long long* __restrict__ out_idle, int* __restrict__ out_peak,
    unsigned char* __restrict__ out_flags) {
  extern __shared__ int32_t lds[];
  const int lpc = T.lanes_per_cand, D = T.D;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const long long cand = blockIdx.x;
  // LDS: [metadata rows as above][per device: end, busy time, peak, length of the new list][per wavefront: the new row; of the
  // first k W items of the stash, for each k, the summed costs and units (stash + 1 of each); their words]
  const int n_meta_ints = kNKinds * kMaxChunks * lpc * 2;
  for (int i = threadIdx.x; i < n_meta_ints; i += blockDim.x) lds[i] = T.ints[i * 2 + (i & 1)];
  const int2* meta = reinterpret_cast<const int2*>(lds);
  int32_t* ends = lds + n_meta_ints;
  int32_t *busies = ends + kMaxDevices, *peaks = busies + kMaxDevices, *lengths = peaks + kMaxDevices;
  char* own = reinterpret_cast<char*>(lengths + kMaxDevices) + (size_t)wave * (size_t)slide_rows_wave_bytes(stride_out, stash);
  uint16_t* out = reinterpret_cast<uint16_t*>(own);
  uint32_t* costs = reinterpret_cast<uint32_t*>(own + 2 * stride_out);
  uint32_t* units = costs + stash + 1;
  uint16_t* words = reinterpret_cast<uint16_t*>(units + stash + 1);
  __syncthreads();
  const unsigned long long up_to = lane == 63 ? ~0ull : (2ull << lane) - 1ull, below = up_to >> 1;
  for (int d = wave; d < D; d += waves) {
    const size_t r = (size_t)cand * D + d;
    const uint16_t* row = ops + r * (size_t)stride;
    const uint16_t* start16 = reinterpret_cast<const uint16_t*>(start_low) + (size_t)cand * (size_t)stride * (size_t)lpc + (size_t)d * 8;
    const uint32_t* esc_row = escapes + r * (size_t)escape_cap;
    const int stop = stop_pos[r];
    const bool at_end = stop >= stride || (row[stop] >> 13) == (unsigned)kEnd;
    unsigned esc = esc_row[0];
    int esc_at = 1;
    for (int i = lane * 8; i < stride_out; i += 512) *reinterpret_cast<uint4*>(out + i) = make_uint4(0u, 0u, 0u, 0u);
    if (lane == 0) { costs[0] = 0u; units[0] = 0u; }
    unsigned w_cost[kMaxChunks], w_units[kMaxChunks], least = ~0u;
    const int n_chunks = T.ints[T.off_dev + d * T.dev_ints];
#pragma unroll
    for (int c = 0; c < kMaxChunks; ++c) {
      const int2 M = meta[(kW * kMaxChunks + c) * lpc + d];
      w_cost[c] = c < n_chunks ? (unsigned)M.x >> 8 : 0u;
      w_units[c] = ((unsigned)M.y >> 8) & 0xffu;
      if (c < n_chunks) least = min(least, w_cost[c]);
    }
    // of the wavefront: items, W items stashed (and their cost and units) and placed (and their cost), memory of the items,
    // end of the last item; the 64 entries of the stash from `window` on are in registers, as they were with `known` entries
    int n_items = 0, n_stash = 0, placed = 0, window = 0, known = 0, mem = 0;
    unsigned stash_cost = 0u, stash_units = 0u, placed_cost = 0u, end16 = 0u, near_cost = 0u;
    uint16_t near_word = 0;
    // of the lane: shares of the sums over the items
    unsigned length = 0u, busy = 0u;
    int peak = 0;
    unsigned next_word = lane < stop ? row[lane] : 0u, next_start = lane < stop ? start16[(size_t)(lane >> 3) * lpc * 8 + (lane & 7)] : 0u;
    for (int base = 0; base < stop; base += 64) {
      const int p = base + lane;
      const unsigned w = next_word, start = next_start;
      if (p + 64 < stop) {
        next_word = row[p + 64];
        next_start = start16[(size_t)((p + 64) >> 3) * lpc * 8 + (p & 7)];
      }
      const int2 M = meta[(w >> 11) * lpc + d];
      const bool item = p < stop && (w >> 13) != (unsigned)kW, is_b = item && (w >> 13) == (unsigned)kB;
      const unsigned long long all = __ballot(item), all_b = __ballot(is_b);
      const int index = n_items + __popcll(all & below), stashed = n_stash + __popcll(all_b & below);
      const unsigned dur = (unsigned)M.x >> 8, my_end = (start + dur) & 0xffffu;
      // the gap in front of the item
      const unsigned long long earlier = all & below;
      const unsigned before = __shfl(my_end, 63 - __clzll((long long)(earlier | 1ull)));
      unsigned gap = (start - (earlier != 0ull ? before : end16)) & 0xffffu;
      while ((int)(esc >> 8) < base + 64) {
        if ((int)(esc >> 8) == p) gap += (esc & 0xffu) << 16;
        esc = esc_row[esc_at++];
      }
      if (item) { length += gap + dur; busy += dur; }
      // the B items' W items join the stash
      unsigned sum_cost = stash_cost, sum_units = stash_units;
#pragma unroll
      for (int c = 0; c < kMaxChunks; ++c) {
        const unsigned long long of_chunk = __ballot(is_b && ((w >> 11) & 3u) == (unsigned)c);
        const unsigned n = (unsigned)__popcll(of_chunk & up_to), n_all = (unsigned)__popcll(of_chunk);
        sum_cost += n * w_cost[c];
        sum_units += n * w_units[c];
        stash_cost += n_all * w_cost[c];
        stash_units += n_all * w_units[c];
      }
      if (is_b && stashed < stash) {
        costs[stashed + 1] = sum_cost;
        units[stashed + 1] = sum_units;
        words[stashed] = (uint16_t)((unsigned)kW << 13 | (w & 0x1fffu));
      }
      n_stash += __popcll(all_b);
      asm volatile("" : : : "memory");
      // the gaps that have room for some W item, in order
      int placed_before = placed;   // in front of this lane's item
      unsigned long long gaps = __ballot(item && gap >= least && stashed > placed);
      while (gaps != 0ull) {
        const int i = __ffsll((long long)gaps) - 1;
        gaps &= gaps - 1ull;
        const int there = __builtin_amdgcn_readlane(stashed, i), at_item = __builtin_amdgcn_readlane(index, i);
        const unsigned room = placed_cost + (unsigned)__builtin_amdgcn_readlane((int)gap, i);
        bool full = true;
        while (full && there > placed) {
          if (placed - window >= 32 || there > known) {
            window = placed;
            known = n_stash;
            const int entry = min(window + lane, stash - 1);
            near_cost = costs[entry + 1];
            near_word = words[entry];
          }
          const int entry = window + lane;
          const bool fits = entry >= placed && entry < there && near_cost <= room;
          const unsigned long long fit = __ballot(fits);
          if (fits && at_item + entry < stride_out) out[at_item + entry] = near_word;
          const int n = __popcll(fit);
          placed += n;
          if (n > 0) placed_cost = (unsigned)__builtin_amdgcn_readlane((int)near_cost, placed - 1 - window);
          full = fit >> 63 != 0ull;   // (more than the window holds)
        }
        placed_before = lane >= i ? placed : placed_before;
      }
      // the items in the new order, and the memory at their starts
      const unsigned allocated = item ? (unsigned)M.y & 0xffu : 0u, freed = item ? ((unsigned)M.y >> 8) & 0xffu : 0u;
      int sum = (int)allocated - (int)freed;
      for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(sum, off);
        if (lane >= off) sum += o;
      }
      if (item) {
        if (index + placed_before < stride_out) out[index + placed_before] = (uint16_t)w;
        peak = max(peak, mem + sum + (int)freed - (int)units[min(placed_before, stash)]);
      }
      mem += __builtin_amdgcn_readlane(sum, 63);
      if (all != 0ull) end16 = (unsigned)__builtin_amdgcn_readlane((int)my_end, 63 - __clzll((long long)all));
      n_items += __popcll(all);
    }
    // a device that reached the end of its list runs what is still stashed back to back
    asm volatile("" : : : "memory");
    const int last = at_end ? n_stash : placed;
    for (int k = placed + lane; k < last; k += 64)
      if (n_items + k < stride_out) out[n_items + k] = words[min(k, stash - 1)];
    for (int off = 32; off > 0; off >>= 1) {
      length += __shfl_xor(length, off);
      busy += __shfl_xor(busy, off);
      peak = max(peak, __shfl_xor(peak, off));
    }
    if (lane == 0) {
      const unsigned w_time = at_end ? stash_cost : placed_cost;
      ends[d] = (int)(length + (w_time - placed_cost));
      busies[d] = (int)(busy + w_time);
      peaks[d] = peak;
      lengths[d] = n_items + last;
    }
    asm volatile("" : : : "memory");
    uint16_t* out_row = ops_out + r * (size_t)stride_out;
    for (int i = lane * 8; i < stride_out; i += 512) *reinterpret_cast<uint4*>(out_row + i) = *reinterpret_cast<const uint4*>(out + i);
  }
  __syncthreads();
  // ---- the evaluation of the new lists
  if (wave != 0) return;
  const bool device = lane < D;
  int makespan = device ? ends[lane] : 0;
  for (int off = 32; off > 0; off >>= 1) makespan = max(makespan, __shfl_xor(makespan, off));
  const bool too_long = __ballot(device && lengths[lane] > stride_out) != 0ull;
  const bool over = __ballot(device && peaks[lane] > T.ints[T.off_dev + lane * T.dev_ints + 1]) != 0ull;
  unsigned flags = timed_flags[cand] & (kDeadlock | kIncomplete);
  if (too_long) flags |= kDeadlock | kIncomplete;
  const bool failed = flags != 0u;
  if (!failed && over) flags = kOverCap;
  if (device) {
    out_idle[cand * D + lane] = failed ? -1ll : (long long)(makespan - busies[lane]);
    out_peak[cand * D + lane] = failed ? -1 : peaks[lane] * T.unit_scale;
  }
  if (lane == 0) {
    out_makespan[cand] = failed ? 0x7fffffffffffffffll : (long long)makespan;
    out_flags[cand] = (unsigned char)flags;
  }
}

template __global__ void wslide_place_kernel<false>(SlotTables, const uint16_t*, long long, int, const uint32_t*, const uint32_t*, int, const int32_t*,
                                                    const unsigned char*, uint16_t*, int, long long*, long long*, int*, unsigned char*);
template __global__ void wslide_place_kernel<true>(SlotTables, const uint16_t*, long long, int, const uint32_t*, const uint32_t*, int, const int32_t*,
                                                   const unsigned char*, uint16_t*, int, long long*, long long*, int*, unsigned char*);

}  // namespace fpsched
