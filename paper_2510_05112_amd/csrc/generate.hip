// Schedule generator kernel: the actor-aware schedule of the paper's Section 5 for a batch of
// parameter sets, one schedule per set.
//
// The scheduling process is step-synchronous by definition (Section 5.2, Steps 2-5: in a step
// every actor runs the step function of Algorithm 1 on the state the previous step left, and
// what an actor schedules stays in its local buffer until the step is over), which is the shape
// of a wavefront: lane = actor, up to 64 / D parameter sets per wavefront, one step = one pass
// of straight-line code with a read phase and a write phase.
//
// State.  Items of one instruction type and stage are scheduled in ascending micro-batch order
// and become dependency-free in that order as well (a forward item needs the same micro-batch
// of the upstream stages, a backward item the same micro-batch of the own forward pass and of
// the downstream backward passes, a weight-gradient item its backward item), so the instruction
// pool and the reorder queues of Section 5.1 reduce to one counter per (type, stage): the number
// of micro-batches scheduled so far.  The next item of (type, stage) is in its reorder queue iff
// every counter it depends on is ahead of its own.  An actor keeps its own counters in registers, two
// stages side by side in one register; the forward and backward counters also stand in LDS, where the lanes of the
// neighbouring stages read them in the read phase and the owner stores a new value in the write phase.
//
// What bounds it: a set's steps are a serial chain, and the steps of a set differ by a factor of ten (a low in-flight
// limit makes a micro-batch's way through the stages the chain).  So the time is that of the longest sets where they
// are few, else the vector instructions of a step (a step's LDS latency is hidden by the other wavefronts of a SIMD).
// A step of the form with the sliding pass takes 57 vector instructions at two stages per actor, and the placing of W items
// behind it some 20 more; conditions are combined and state is changed by sets of lanes in scalar registers, and an item is
// timed in the step behind its own, before which nothing waits for LDS that the next step does not wait for as well.
// 16,384 sets of 32 devices, 2 stages each, 128 micro-batches (2,657 steps a set, 8,884 the longest): sliding form 4.84 ms
// with 73 instructions, conditions as masks in vector registers, and 12 wavefronts per compute unit in one workgroup, 4.22
// with 57 instructions, 3.97 with larger rings, 3.89 with fewer wavefronts (fpsched_api.hip, gen_shape), 3.82 since the placing of W items
// has its conditions as sets of lanes too (some 35 instead of 48 vector instructions a round); results only 5.49, 4.66, then 3.42,
// lists 5.04, 3.96, then 2.94; 4,096 sets of 16 devices, 64 micro-batches (the longest sets' chain): 0.77 and 0.75, 0.74 and
// 0.67, 0.66 and 0.54 ms; 65,536 of 8 devices, 32 micro-batches: 0.90 and 0.81, 0.77 and 0.72, 0.78 and 0.67 ms.
// Priorities (Section 5.2; Table of built-in values): computation type traversal priority
// bwdpass-first / fwdpass-first / interleaved(unit1, unit2); stage traversal priority
// breadth-first / depth-first with an optional interval, separately for forward and backward
// items; the check function is the per-stage limit of in-flight micro-batches (Section 4.2,
// config_inflight_micros).  How the corners are read (type fallback, when an interval position
// moves, weight-gradient items last) is stated with the host declaration of fpsched_generate.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "lds_access.h"

namespace fpsched {

namespace {

enum GenType : int { kGenF = 0, kGenB = 1, kGenW = 2 };

// lowest set bit of a non-zero mask
__device__ __forceinline__ int low_bit(unsigned x) { return __ffs(x) - 1; }
// two 16-bit counters side by side: those of an actor's two stages
typedef short pair16 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned bits_of(pair16 v) { return __builtin_bit_cast(unsigned, v); }
__device__ __forceinline__ pair16 pair_of(unsigned v) { return __builtin_bit_cast(pair16, v); }
constexpr unsigned kBothSigns = 0x80008000u;
// Four stages per actor: which pair of them, as a mask (all ones or 0) that is also combined with values.
__device__ __forceinline__ unsigned mask_of(bool b) { return b ? ~0u : 0u; }
__device__ __forceinline__ unsigned choose(unsigned mask, unsigned a, unsigned b) { return (a & mask) | (b & ~mask); }
// Conditions are sets of lanes in scalar registers, combined there, beside the vector instructions.
typedef unsigned long long Lanes;
__device__ __forceinline__ bool in(Lanes l) { return __builtin_amdgcn_inverse_ballot_w64(l); }
template <class A>
__device__ __forceinline__ A of(Lanes l, A a, A b) { return in(l) ? a : b; }
// An actor's traversal state of one direction (V > 1), in one register: the position (the chunk) from bit kPositionBit on
// (two chunks: bit 4, so that the register is the shift that brings the position's half of a pair to the front), the
// upper half the items until the position moves on by itself, less one (negative: it does).  No position
// sees more than kMaxChunks * m < kFarInterval items, so longer intervals are all the same.  Without an interval the
// position never moves: the first eligible stage from the first (breadth-first) or last one (depth-first) on is picked.
constexpr unsigned kPosition = 0x30u, kPositionBit = 4u, kOneItem = 0x10000u, kFarInterval = 0x3fffu;

// one value per chunk of an actor, as one vector value (an array would be indexed in memory)
template <int V>
struct GenPerChunk { typedef int type __attribute__((ext_vector_type(V))); };
template <int V>
__device__ __forceinline__ int gen_pick(typename GenPerChunk<V>::type a, unsigned c) {
  int r = a[0];
#pragma unroll
  for (int i = 1; i < V; ++i) r = (c == (unsigned)i) ? a[i] : r;
  return r;
}

// steps between two looks at whether a set is done
constexpr int kStepsPerLook = 8;
constexpr int kStagingWords = kGenStagingWords;   // 15 op words and those of a look
static_assert(2 * kStagingWords >= 15 + kStepsPerLook && (kStagingWords & (kStagingWords - 1)) == 0, "");
constexpr int kRoundsPerLook = 4;   // rounds of settle between two looks at whether there are enough of them
static_assert(kGenFewEvents > kStepsPerLook + 1, "a look's items fit");

}  // namespace

// Order in which the sets of a batch are worked on: those with many steps first, so that the batch does not end on a few
// wavefronts that have just begun a long one.  A set's steps are nearly those of the slower of two bounds: its actors'
// items, and for each stage micro-batches x (steps from a micro-batch's forward item to its backward item) / in-flight
// limit (measured correlation with the true steps: 0.99 for chains of 8 to 64 stages).  One wavefront per set writes
// the set's class, a power of two of the ratio of the two, into the set's status byte, which the generator overwrites
// when the set is done; the generator draws all sets once per class.
__global__ void generate_order_kernel(DevTables T, const int32_t* __restrict__ inflight, const long long* __restrict__ select,
                                      long long n_src, long long n_sets, int work_steps,
                                      unsigned char* __restrict__ out_status, unsigned long long* __restrict__ next_set) {
  const int lane = threadIdx.x & 63;
  const long long set = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (blockIdx.x == 0 && threadIdx.x == 0) *next_set = 0ull;
  if (set >= n_sets) return;
  const long long src = select ? select[set] : set;
  float longest = 0.f;
  if (src >= 0 && src < n_src)
    for (int s = lane; s < T.S; s += 64)
      longest = fmaxf(longest, (float)T.ints[T.off_turnaround + s] / (float)max(inflight[src * T.S + s], 1));
  for (int off = 32; off > 0; off >>= 1) longest = fmaxf(longest, __shfl_xor(longest, off, 64));
  if (lane == 0) {
    const float ratio = longest * (float)T.m / (float)work_steps;
    out_status[set] = (unsigned char)(kGenClassMark | (ratio >= 8.f ? 0 : (ratio >= 4.f ? 1 : (ratio >= 2.f ? 2 : 3))));
  }
}

// V = bound on the stages per device (1, 2, 4).  DEG = bound on the DAG in- and out-degree of a
// stage (1 or 2): the LDS addresses of the neighbours' counters are then kept in registers;
// DEG = 0 walks the edge lists in LDS instead (any degree).
// GRAPH: DEG, or kGenOneNeighbour (V = 2, DEG = 1): what an actor's two stages wait for in a direction is on one actor, as in a chain
// laid round the devices.  An actor's two counters of a direction are then one word, read with one instruction instead of two, its
// halves put in order for the reader (a stage that waits for nothing finds m): 32,768 sets of 16 x 64 x 2 through lists 3012 and 2996 us,
// 16,384 of 32 x 128 x 2, sliding, with the winners 4480 and 4441 us.
//
// The grid is persistent: a segment (the lanes of one parameter set) that finishes its schedule
// writes it out, draws the next set from a global counter and starts over while the other segments
// of the wavefront keep stepping, so that sets that need few and many steps balance out.  Segment g begins with set g and,
// with n_classes = 0 (no more sets than segments), has no other; with n_classes = 1 the counter hands out those behind the
// first ones, all that a wavefront asks for with one atomic.  With more classes the counter runs over all sets
// once per class of generate_order_kernel from the beginning on, and a segment takes those of the class (a status byte that
// still holds the class and one that has been overwritten since both say what is to be done: a set is taken in the pass of
// its class only).  These are drawn one by one: a segment that drew four at a time kept several long ones to itself (14.0 ms
// instead of 7.9), and so did a wavefront that claimed as many numbers as were likely to hold what it asked for (8.6 instead of
// 5.3 ms).  A wavefront's priority is that of its longest set.  (fpsched_api.hip, order_sets, says which of the two when.)
//
// TIMED: generator and evaluator in one (fpsched_generate_evaluate).  An item is scheduled only
// after everything it depends on was scheduled in an earlier step, so its start time is known the
// moment it is placed: start = max(the actor's free time, the inputs' finish + latency), exactly
// what fpsched_evaluate computes for the generated lists (Section 5.1 data dependency; the
// estimator's start / end / cost).  The inputs' finish times travel through the mail slots of the
// slot kernel, here plain int32 words without tags (the counters already say that the value is
// there); resident memory is counted as the items are placed.  No op word is formed, nothing but
// the results is written.  Workgroups hold several wavefronts that share the cost rows; each
// wavefront keeps its own counters and slots and never looks at another's, so no barrier is needed
// after the start.
//
// FORM kGenSlide: the timed form with the weight-gradient sliding pass of Section 5.2 (bubble optimizations) in
// it: the results fpsched_wslide_evaluate gives for the generated lists.  A W item that the scheduler places is
// passed over (it fills a step in which nothing else is eligible: a count of those not placed yet is all that is kept);
// a B item stashes its W item, and in front of every other item the actor runs the oldest
// stashed items that end before the item starts.  None of this moves an F or B item, it only decides what memory is
// resident at their starts; so the steps only note each item (its gap: how long the actor waits in front of it) in a ring
// of T.gen_events words per lane, and a second loop (settle) places W items into gaps, for all lanes at once and only when
// some lane's ring is nearly full: its rounds are then full of work, where in the step itself a few lanes' W items
// would be waited for by all.  The stash is a queue of log2(V) bits per entry
// (the chunk) in LDS: an actor stashes no more than V * m items, so entry i simply stands in word i * log2(V) / 32.
template <int V, int GRAPH, int FORM>
__global__ __launch_bounds__(kGenThreads) void generate_kernel(
    DevTables T, const int32_t* __restrict__ policy, const int32_t* __restrict__ inflight,
    const long long* __restrict__ select, long long n_src, long long n_sets, int n_classes, int stride,
    uint16_t* __restrict__ ops, int32_t* __restrict__ out_steps, unsigned char* out_status,
    unsigned long long* __restrict__ next_set, GenResults R) {
  constexpr bool ONE_NEIGHBOUR = GRAPH == kGenOneNeighbour;
  constexpr int DEG = ONE_NEIGHBOUR ? 1 : GRAPH;
  static_assert(!ONE_NEIGHBOUR || V == 2, "");
  constexpr bool TIMED = FORM != kGenPlain;
  constexpr bool SLIDE = FORM == kGenSlide;
  constexpr int NP = (V + 1) / 2;   // pairs of stages
  // SLIDE: bits per queue entry, entries per queue word
  constexpr unsigned kQueueBits = V > 2 ? 2u : 1u, kQueueEntries = 32u / kQueueBits;
  extern __shared__ int32_t lds[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6, waves_per_block = blockDim.x >> 6;
  const int S = T.S, m = T.m, D = T.D;
  const int cpw = T.gen_sets;
  const bool has_w = T.has_w != 0;
  // LDS: [SLIDE: rings of all wavefronts][edge lists, only if DEG == 0 | cost rows, only if TIMED: the first halves, then the second halves if they are
  // needed] then per wavefront
  // [sets of the wavefront: counters [2][S]][a word holding m][a word: may there be sets left to draw]
  // [row staging: 32 op words per lane, as 16 dwords laid out [dword][lane] | TIMED: the sets' slots, SLIDE: queues]
  const unsigned ring_bytes = SLIDE ? (unsigned)T.gen_events * 256u : 0u;   // of a wavefront
  int32_t* tab = lds + waves_per_block * (int)(ring_bytes / 4u);
  const int n_rows = 3 * V * D;
  constexpr bool kSecondHalves = DEG > 1 || FORM == kGenTimed;
  const int n_tab = TIMED ? n_rows * (kSecondHalves ? 8 : 4) : (DEG == 0 ? T.n_table_ints : 0);
  if (TIMED) {
    for (int i = threadIdx.x; i < n_tab; i += blockDim.x) tab[i] = T.ints[T.off_gen_rows + i];
  } else if (DEG == 0) {
    for (int i = threadIdx.x; i < n_tab; i += blockDim.x) lds[i] = T.ints[i];
  }
  const int n_count_ints = (cpw * 2 * S + 2 + 3) & ~3;
  const int slot_words = T.gen_slot_words;
  const int queue_words = SLIDE ? T.gen_queue_words : 0;   // per lane
  int32_t* counts = tab + n_tab + wave * (n_count_ints + (TIMED ? cpw * slot_words + (SLIDE ? 64 * queue_words : 0) : kStagingWords * 64));
  // a counter that is always "done" (value m) stands in for a missing neighbour
  const int at_m = cpw * 2 * S;
  if (lane == 0) { counts[at_m] = m; counts[at_m + 1] = 1; }
  // a lane collects 16 op words (32 bytes) of its row before it stores them: HBM is written in
  // 32-byte pieces, not a quarter of that.  They are stored between the steps: the lanes fill up at different steps, and in
  // most steps some lane would.
  uint32_t* staging = reinterpret_cast<uint32_t*>(counts + n_count_ints) + lane;   // dword i at + i * 64
  // (a lane's place in them: the dword from bit 8 on, its half in bit 1; what stands between is not looked at)
  const unsigned staging_at = lds_address(staging);
  constexpr unsigned kPlaceMask = (unsigned)(kStagingWords - 1) << 8 | 2u;
  // TIMED: slots never hold anything but finish times (an item without an input reads some word of
  // them and adds -2^30)
  if (TIMED)
    for (int i = lane; i < cpw * slot_words; i += 64) counts[n_count_ints + i] = 0;
  __syncthreads();

  const int seg = lane / D;       // (lanes from cpw * D on have no device)
  const int d = lane - seg * D;
  const bool has_dev = seg < cpw;
  const int base = has_dev ? seg * 2 * S : 0;   // this segment's counters: counts[base + type * S + stage]
  const unsigned slot = lds_address(counts + n_count_ints + (has_dev ? seg : 0) * slot_words);   // TIMED: this segment's slots

  // what depends on the actor only
  const int nch = has_dev ? T.ints[T.off_n_chunks + d] : 0;
  int stage[V];
  unsigned own_at[V];   // LDS address of this actor's forward counter of chunk c (backward: 4 S bytes on)
  int pred_at[V][DEG > 0 ? DEG : 1], succ_at[V][DEG > 0 ? DEG : 1];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    stage[c] = c < nch ? T.ints[T.off_local_stage + d * kMaxChunks + c] : 0;
    own_at[c] = lds_address(counts + (c < nch ? base + stage[c] : at_m));
    asm("" : "+v"(own_at[c]));   // (whole addresses stay in registers)
#pragma unroll
    for (int k = 0; k < (DEG > 0 ? DEG : 1); ++k) {
      pred_at[c][k] = at_m;
      succ_at[c][k] = at_m;
      if (DEG > 0 && c < nch) {
        const int s = stage[c];
        const int pe = T.ints[T.off_pred_off + s] + k, se = T.ints[T.off_succ_off + s] + k;
        if (pe < T.ints[T.off_pred_off + s + 1]) pred_at[c][k] = base + T.ints[T.off_pred_stage + pe];
        if (se < T.ints[T.off_succ_off + s + 1]) succ_at[c][k] = base + S + T.ints[T.off_succ_stage + se];
      }
    }
  }

  // ONE_NEIGHBOUR: counters [direction][device] instead, and where the neighbours' are; which bytes of such a word and of m the stages'
  // counters are (v_perm)
  unsigned ahead_at[2] = {lds_address(counts + at_m), lds_address(counts + at_m)}, ahead_bytes[2] = {0x01000100u, 0x01000100u};
  const unsigned both_m = (unsigned)m * 0x00010001u;
  if constexpr (ONE_NEIGHBOUR) {
    // (where each stage is, in the place of the counters until the first set.  A lane reads what others of the wavefront have written:
    // not before all of them have, whichever way the compiler lays out the conditions.  Both lines order, neither is an instruction)
#pragma unroll
    for (int c = 0; c < V; ++c)
      if (c < nch) counts[base + stage[c]] = d * kMaxChunks + c;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < V; ++c)
#pragma unroll
      for (int dir = 0; dir < 2; ++dir) {
        if (c >= nch) continue;
        const int first = dir == 0 ? T.off_pred_off : T.off_succ_off, s = stage[c];
        if (T.ints[first + s] >= T.ints[first + s + 1]) continue;
        const int other = T.ints[(dir == 0 ? T.off_pred_stage : T.off_succ_stage) + T.ints[first + s]];
        const int at = counts[base + other];
        ahead_at[dir] = lds_address(counts + base + dir * D + at / kMaxChunks);
        ahead_bytes[dir] = (ahead_bytes[dir] & ~(0xffffu << 16 * c)) | (at % kMaxChunks == 0 ? 0x0504u : 0x0706u) << 16 * c;
      }
    own_at[0] = lds_address(counts + (has_dev ? base + d : at_m));
  }

  // TIMED: what the actor's items cost together, and its memory cap
  long long busy_total = 0;
  int cap = 0x7fffffff;
  if (TIMED && has_dev) {
    cap = T.ints[T.off_mem_cap + d];
#pragma unroll
    for (int c = 0; c < V; ++c)
      if (c < nch)
        busy_total += (long long)m * ((long long)T.ints[T.off_dur + kF * S + stage[c]] + T.ints[T.off_dur + kB * S + stage[c]] +
                                      (has_w ? T.ints[T.off_dur + kW * S + stage[c]] : 0));
  }
  int free_at = 0, mem = 0, peak = 0;
  // SLIDE: units of an F item, cost and freed units of a W item of each chunk, what all W items cost
  typename GenPerChunk<V>::type f_units, w_dur, w_free;
  int w_total = 0;
#pragma unroll
  for (int c = 0; c < V; ++c) {
    f_units[c] = 0; w_dur[c] = 0; w_free[c] = 0;
    if (SLIDE && has_dev && c < nch) {
      const int32_t* first = T.ints + T.off_gen_rows;
      const int32_t* second = first + n_rows * 4;
      f_units[c] = second[(c * D + d) * 4];
      w_dur[c] = first[((2 * V + c) * D + d) * 4];
      w_free[c] = second[((2 * V + c) * D + d) * 4 + 1];
    }
    w_total += m * w_dur[c];
  }
  // SLIDE: the ring of items (LDS address of the next one in and out), the one whose gap is being filled and what is
  // left of its gap, the queue (entries in and out, the word being filled)
  const unsigned ring = lds_address(lds) + wave * ring_bytes + lane * 4;   // entry i at + i * 256; a multiple of its size + lane * 4
  const unsigned queue = lds_address(counts + n_count_ints + cpw * slot_words) + lane * 4;   // word i at + i * 256
  unsigned ring_in = ring, ring_out = ring, gap = 0u, q_in = 0u, q_out = 0u, q_tail = 0u;
  int w_placed = 0;
  unsigned event = 0u;
  Lanes has_event = 0;
  const unsigned ring_mask = ring_bytes - 256u;
  // one round: the oldest stashed W item runs if what is left of the gap has room for it; unless there is room for the one behind it
  // too, the gap's item starts, and the next one's gap opens
  auto settle = [&]() {
    const unsigned next = lds_read<unsigned>(ring_out);
    unsigned dur = (unsigned)w_dur[0], freed = (unsigned)w_free[0], units = (unsigned)f_units[0], dur_behind = dur;
    const unsigned q_behind = q_out + 1u;
    Lanes unseen = 0;   // the one behind it is in the queue's next word: looked at in the next round
    if constexpr (V > 1) {
      const unsigned word = lds_read<unsigned>(queue + q_out / kQueueEntries * 256u);
      if constexpr (V == 2) {
        const Lanes second = __ballot(__builtin_amdgcn_ubfe(word, q_out, 1u) != 0u), of_second = __ballot((event & 1u) != 0u);
        const Lanes second_behind = __ballot(__builtin_amdgcn_ubfe(word, q_behind, 1u) != 0u);
        dur_behind = of(second_behind, (unsigned)w_dur[V - 1], dur);
        dur = of(second, (unsigned)w_dur[V - 1], dur);
        freed = of(second, (unsigned)w_free[V - 1], freed);
        units = of(of_second, (unsigned)f_units[V - 1], units);
      } else {
        const unsigned c = word >> (q_out % kQueueEntries * kQueueBits) & 3u;
        dur_behind = (unsigned)gen_pick<V>(w_dur, word >> q_behind % kQueueEntries * kQueueBits & 3u);
        dur = (unsigned)gen_pick<V>(w_dur, c);
        freed = (unsigned)gen_pick<V>(w_free, c);
        units = (unsigned)gen_pick<V>(f_units, event & 3u);
      }
      unseen = __ballot(q_behind % kQueueEntries == 0u);
    }
    const Lanes run_w = __ballot(q_in != q_out) & __ballot(dur <= gap);
    const Lanes stay = run_w & (unseen | (__ballot(q_in != q_behind) & __ballot(dur + dur_behind <= gap)));
    const Lanes start = has_event & ~stay, is_b = __ballot((event & 4u) != 0u);
    const Lanes more = __ballot(ring_in != ring_out);
    [[maybe_unused]] unsigned scratch;
    // a B item's W item is stashed
    if constexpr (V > 1) {
      const unsigned shift = q_in * kQueueBits, at = queue + q_in / kQueueEntries * 256u, chunk = event & 3u;   // (of a shift five bits are looked at)
      asm volatile("s_mov_b64 exec, %[stashes]\n\t"
                   "v_lshl_or_b32 %[tail], %[chunk], %[shift], %[tail]\n\t"
                   "v_add_u32 %[in], 1, %[in]\n\t"
                   "ds_write_b32 %[at], %[tail]\n\t"
                   "v_and_b32 %[left], %[last], %[in]\n\t"
                   "v_cmp_ne_u32 vcc, 0, %[left]\n\t"
                   "s_andn2_b64 exec, exec, vcc\n\t"
                   "v_mov_b32 %[tail], 0\n\t"
                   "s_mov_b64 exec, -1"
                   : [tail] "+&v"(q_tail), [in] "+&v"(q_in), [left] "=&v"(scratch)
                   : [chunk] "v"(chunk), [shift] "v"(shift), [at] "v"(at), [last] "s"(kQueueEntries - 1u), [stashes] "s"(start & is_b)
                   : "memory", "vcc", "scc");
    } else {
      asm volatile("s_mov_b64 exec, %[stashes]\n\t"
                   "v_add_u32 %[in], 1, %[in]\n\t"
                   "s_mov_b64 exec, -1"
                   : [in] "+&v"(q_in) : [stashes] "s"(start & is_b));
    }
    asm volatile("s_mov_b64 exec, %[runs]\n\t"
                 "v_add_u32 %[placed], %[placed], %[dur]\n\t"
                 "v_add_u32 %[out], 1, %[out]\n\t"
                 "v_sub_u32 %[mem], %[mem], %[freed]\n\t"
                 "v_sub_u32 %[gap], %[gap], %[dur]\n\t"
                 "s_mov_b64 exec, %[starts]\n\t"
                 "v_add_u32 %[mem], %[mem], %[units]\n\t"
                 "v_max_i32 %[peak], %[peak], %[mem]\n\t"
                 "s_mov_b64 exec, %[opens]\n\t"
                 "v_mov_b32 %[gap], 0\n\t"
                 "s_and_b64 exec, exec, %[more]\n\t"
                 "v_lshrrev_b32 %[gap], 3, %[next]\n\t"
                 "v_mov_b32 %[event], %[next]\n\t"
                 "v_add_u32 %[at], 0x100, %[at]\n\t"
                 "v_and_or_b32 %[at], %[at], %[mask], %[ring]\n\t"
                 "s_mov_b64 exec, -1"
                 : [placed] "+&v"(w_placed), [out] "+&v"(q_out), [mem] "+&v"(mem), [peak] "+&v"(peak), [gap] "+&v"(gap), [event] "+&v"(event),
                   [at] "+&v"(ring_out)
                 : [dur] "v"(dur), [freed] "v"(freed), [units] "v"(units), [next] "v"(next), [ring] "v"(ring), [mask] "s"(ring_mask), [runs] "s"(run_w),
                   [starts] "s"(start & ~is_b), [opens] "s"(~stay), [more] "s"(more)
                 : "scc");
    has_event = (has_event & stay) | (more & ~stay);
  };

  // the actor's own counters, two stages per register
  // (n_bl: the backward counters + in-flight limits)
  unsigned n_f[NP], n_b[NP], n_w[NP], n_bl[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) { n_f[i] = 0u; n_b[i] = 0u; n_w[i] = 0u; n_bl[i] = 0u; }

  // TIMED: the items scheduled in the last step, not timed yet: the lanes that have one, its row and where its
  // micro-batch's slots are (of every other step in registers of their own: a lane without an item keeps an older one's)
  unsigned row_f = lds_address(tab) + d * 16, row_b = row_f + V * D * 16;
  asm("" : "+v"(row_f), "+v"(row_b));
  struct Item { int4 a, b; unsigned slot; };
  Item items_of[2] = {{make_int4(0, 0, 0, 0), make_int4(0, 0, 0, 0), slot}, {make_int4(0, 0, 0, 0), make_int4(0, 0, 0, 0), slot}};
  Lanes items = 0;
  // where the actor's counters are: of chunk 0, and how much further that of the last chunk is (V == 2)
  const unsigned own_f = own_at[0], own_b = own_at[0] + 4u * (unsigned)(ONE_NEIGHBOUR ? D : S);
  const int own_step = (int)(own_at[V - 1] - own_at[0]);

  // The neighbouring stages' counters (DEG > 0: two of each pair, as they stand in LDS), requested as soon as a step's own counters
  // have been stored: on their way while the step's items are timed.
  short ahead_f[NP][2 * (DEG > 0 ? DEG : 1)], ahead_b[NP][2 * (DEG > 0 ? DEG : 1)];
  unsigned ahead_words[2] = {0u, 0u};
  auto look_ahead = [&]() {
    if constexpr (ONE_NEIGHBOUR) {
      ahead_words[0] = lds_read<unsigned>(ahead_at[0]);
      ahead_words[1] = lds_read<unsigned>(ahead_at[1]);
    } else if constexpr (DEG > 0) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        constexpr int kLast = V - 1;
        const int c0 = 2 * i, c1 = min(2 * i + 1, kLast);
#pragma unroll
        for (int k = 0; k < DEG; ++k) {
          ahead_f[i][2 * k] = lds_read<short>(lds_address(counts + pred_at[c0][k]));
          ahead_f[i][2 * k + 1] = lds_read<short>(lds_address(counts + pred_at[c1][k]));
          ahead_b[i][2 * k] = lds_read<short>(lds_address(counts + succ_at[c0][k]));
          ahead_b[i][2 * k + 1] = lds_read<short>(lds_address(counts + succ_at[c1][k]));
        }
      }
    }
  };

  // per-set state
  long long set = ((long long)blockIdx.x * waves_per_block + wave) * cpw + seg;   // the first set of a segment is its global index
  bool first_draw = n_classes <= 1;
  int set_class = 3;
  bool has_set = false;   // the segment is working on a set (possibly finished and not yet written out)
  bool fresh = true;      // the segment wants its next set
  unsigned walk_f = 0u, walk_b = 0u, again_f = 0u, again_b = 0u;   // traversal states, and what they become on a move
  bool moves_f = false, moves_b = false, up_f = true, up_b = true;   // an interval is set; breadth-first
  Lanes moving_f = 0, moving_b = 0, upward_f = 0, upward_b = 0;      // (of all lanes)
  // The instruction type tried first in a step: F where it is not negative, else B; fixed, or the interleaved priority's
  // turn: an item of the type whose turn it is counts down from unit_f - 1 to -unit_b and then begins anew
  int turn_at = 0, turn_end = 0, turn_begin = 0;
  bool live = false;   // the set's process is still running
  int status = 0, stored = 0;
  unsigned place = 0u;   // of the next op word
  auto words_at = [](unsigned p) -> int { return (int)(p >> 8 << 1 | (p >> 1 & 1u)); };
  unsigned first_step = 0u;   // the loop's step counter when the set's process began
  // the step behind the one in which this actor scheduled its last item so far (first_step: none).  SLIDE: the step behind
  // the last W item if those up to here filled the steps from then on in which nothing else is eligible
  unsigned next_step = 0u;
  int steps = 0;
  uint16_t* row = ops;
  // "does any lane of my segment ...": the ballot against the lanes of the segment
  const unsigned long long seg_lanes = !has_dev ? 0ull : (D == 64 ? ~0ull : ((1ull << D) - 1ull) << (seg * D));
  const unsigned seg_lo = (unsigned)seg_lanes, seg_hi = (unsigned)(seg_lanes >> 32);
  auto any_in_segment = [&](unsigned long long ballot) -> bool {
    return (((unsigned)ballot & seg_lo) | ((unsigned)(ballot >> 32) & seg_hi)) != 0u;
  };
  // the largest value of the segment, in all of its lanes
  auto segment_max = [&](int v) -> int {
    for (int off = 1; off < D; off <<= 1) {
      const int o = __shfl_down(v, off, 64);
      if (d + off < D) v = max(v, o);
    }
    return __shfl(v, lane - d, 64);
  };

  // Every step but the last of a set schedules at least one of its 3 S m items, and a segment
  // cannot draw more than all sets: the bound below is never reached, it only makes sure that the
  // wavefront leaves the loop whatever happens.  A wavefront's counters are its own: its LDS instructions
  // execute in program order, so the reads of a step see the counters as the previous step left them
  // and no barrier is needed between the phases.
  const unsigned long long per_set = 3ull * (unsigned)S * (unsigned)m + 32ull;
  const unsigned long long bound = per_set * ((unsigned long long)n_sets + 1ull) / kStepsPerLook + 1ull;
  for (unsigned long long look = 0; look < bound; ++look) {
    const unsigned step_0 = (unsigned)look * kStepsPerLook;
    if (__ballot(fresh) != 0ull) {
      has_event &= ~__ballot(fresh);
      // ---- segments that finished write their schedule out and start on the next set
      if (fresh) {
        fresh = false;
        if (TIMED) {
          if (has_set) {
            // the segment's results, in the form fpsched_evaluate gives them for the generated lists; a
            // schedule that is not complete (stuck, bad policy) has items that never ran
            // (SLIDE: what is still stashed runs back to back behind the actor's last item)
            int makespan = SLIDE ? free_at + (w_total - w_placed) : free_at;
            bool over = peak > cap;
            makespan = segment_max(makespan);
            over = any_in_segment(__ballot(over));
            const bool complete = status == 0;
            if (has_dev) {
              R.idle[set * D + d] = complete ? (long long)makespan - busy_total : -1ll;
              R.peak[set * D + d] = complete ? peak : -1;
            }
            if (d == 0 && has_dev) {
              R.makespan[set] = complete ? (long long)makespan : 0x7fffffffffffffffll;
              R.flags[set] = (unsigned char)(complete ? (over ? kOverCap : 0) : kIncomplete);
              out_steps[set] = steps;
              out_status[set] = (unsigned char)status;
            }
          }
        } else if (has_set && has_dev) {
          // rows are END-padded to the stride; words still staged (less than 16) go out with the padding
          const int len = words_at(place);
          int at = len & ~15;
          if (len & 15) {
            typedef uint16_t half_of_dword __attribute__((may_alias));   // (stored in halves, read in dwords)
            for (int i = len & 15; i < 16; ++i) reinterpret_cast<half_of_dword*>(staging + (((at + i) >> 1) & (kStagingWords - 1)) * 64)[i & 1] = 0;
            const uint32_t* w = staging + ((at >> 1) & (kStagingWords - 1)) * 64;
            if (at < stride) *reinterpret_cast<uint4*>(row + at) = make_uint4(w[0], w[64], w[128], w[192]);
            if (at + 8 < stride) *reinterpret_cast<uint4*>(row + at + 8) = make_uint4(w[256], w[320], w[384], w[448]);
            at += 16;
          }
          for (; at < stride; at += 8) *reinterpret_cast<uint4*>(row + at) = make_uint4(0u, 0u, 0u, 0u);
          if (d == 0) {
            out_steps[set] = steps;
            out_status[set] = (unsigned char)status;
          }
        }
        if (!first_draw) {
          long long drawn = -1;
          const bool asks = d == 0 && has_dev;
          const unsigned long long asking = __ballot(asks);
          if (n_classes == 1) {
            // (one atomic for all of the wavefront's, which once it has come away empty does not ask again)
            const int leader = __ffsll((long long)asking) - 1;
            unsigned long long first = (unsigned long long)n_sets;
            if (lane == leader && counts[at_m + 1] != 0) {
              first = atomicAdd(next_set, (unsigned long long)__popcll(asking));
              if (first >= (unsigned long long)n_sets) counts[at_m + 1] = 0;
            }
            drawn = (long long)__shfl(first, leader) + __popcll(asking & ((1ull << lane) - 1ull));
          } else if (n_classes > 1 && asks) {
            for (;;) {
              long long q = (long long)atomicAdd(next_set, 1ull);
              int cls = 0;
              while (cls < n_classes && q >= n_sets) { q -= n_sets; ++cls; }
              if (cls == n_classes) break;
              if (out_status[q] == (unsigned char)(kGenClassMark | cls)) { drawn = q; set_class = cls; break; }
            }
          }
          set = __shfl(drawn, lane - d, 64);
        }
        first_draw = false;
        has_set = has_dev && set >= 0 && set < n_sets;
        const bool has_row = has_set && has_dev;
        if (has_dev)   // (also without a set: what the counters hold is compared with this actor's m items done)
          for (int i = d; i < 2 * S; i += D) counts[base + i] = 0;
        int cttp = 0, unit_f = 1, unit_b = 1, f_dir = 0, f_int = 0, b_dir = 0, b_int = 0;
        // (with a selection, output row `set` is the schedule of parameter set select[set]; an entry that
        // is negative or not below n_src selects nothing and counts as a bad set)
        const long long src = (has_set && select) ? select[set] : set;
        const bool has_src = has_row && src >= 0 && src < n_src;
        if (has_src) {
          const int32_t* pol = policy + (src * D + d) * 8;
          cttp = pol[0]; unit_f = pol[1]; unit_b = pol[2];
          f_dir = pol[3]; f_int = pol[4]; b_dir = pol[5]; b_int = pol[6];
        }
        int limit[V];
#pragma unroll
        for (int c = 0; c < V; ++c) limit[c] = (has_src && c < nch) ? inflight[src * S + stage[c]] : 1;
        // (no stage has more than m <= 2048 micro-batches in flight; a chunk the actor does not have is done)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const int c0 = 2 * i, c1 = 2 * i + 1 < V ? 2 * i + 1 : 2 * i;
          const unsigned none0 = c0 < nch ? 0u : (unsigned)m, none1 = (2 * i + 1 < V && c1 < nch) ? 0u : (unsigned)m << 16;
          n_f[i] = none0 | none1;
          n_b[i] = none0 | none1;
          n_bl[i] = (unsigned)min(limit[c0], 0x1fff) | (unsigned)min(limit[c1], 0x1fff) << 16;
          n_bl[i] += n_b[i];
          n_w[i] = has_w ? none0 | none1 : (unsigned)m * 0x00010001u;
        }
        // a parameter set with a value outside its domain generates nothing (status 4)
        bool bad = (has_row && !has_src) || cttp < 0 || cttp > 2 || unit_f < 1 || unit_b < 1 || f_dir < 0 || f_dir > 1 || f_int < 0 ||
                   b_dir < 0 || b_dir > 1 || b_int < 0 || (cttp != 2 && (unit_f != 1 || unit_b != 1));
#pragma unroll
        for (int c = 0; c < V; ++c) bad = bad || limit[c] < 1;
        const bool set_bad = any_in_segment(__ballot(bad && has_row));
        turn_begin = unit_f - 1;
        turn_end = cttp == 2 ? -unit_b : (int)0x80000000;
        turn_at = cttp == 2 ? turn_begin : (cttp != 0 ? 0x7fffffff : -1);
        const unsigned last_chunk = nch > 0 ? (unsigned)(nch - 1) << kPositionBit : 0u;
        moves_f = f_int > 0; moves_b = b_int > 0;
        up_f = f_dir == 0; up_b = b_dir == 0;
        again_f = f_int > 0 ? (min((unsigned)f_int, kFarInterval) - 2u) << 16 : 0u;
        again_b = b_int > 0 ? (min((unsigned)b_int, kFarInterval) - 2u) << 16 : 0u;
        walk_f = again_f + kOneItem + (up_f ? 0u : last_chunk);
        walk_b = again_b + kOneItem + (up_b ? 0u : last_chunk);
        const bool any_item = has_row && !set_bad && nch > 0 && m > 0;
        if (!any_item)   // (nothing is ever eligible)
          for (int i = 0; i < NP; ++i) { n_f[i] = n_b[i] = n_w[i] = (unsigned)m * 0x00010001u; }
        live = any_in_segment(__ballot(any_item));
        first_step = step_0; steps = 0; next_step = step_0;
        status = set_bad ? 4 : 0; place = 0u; stored = 0;
        free_at = 0; mem = 0; peak = 0;
        ring_in = ring; ring_out = ring; event = 0u; gap = 0u; q_in = 0u; q_out = 0u; q_tail = 0u; w_placed = 0;
        if (!TIMED) row = ops + (size_t)(has_row ? set * D + d : 0) * (size_t)stride;
        fresh = has_set && !live;   // nothing to schedule (a bad set, no stages): written out next time round
      }
      moving_f = __ballot(moves_f);
      moving_b = __ballot(moves_b);
      if (V > 2) { upward_f = __ballot(up_f); upward_b = __ballot(up_b); }
      if (__ballot(has_set) == 0ull) break;   // every segment of the wavefront is out of work
      if (n_classes > 1) {
        const int longest = __ballot(has_set && set_class == 0) ? 3 : (__ballot(has_set && set_class == 1) ? 2 : (__ballot(has_set && set_class == 2) ? 1 : 0));
        if (longest == 3) __builtin_amdgcn_s_setprio(3);
        else if (longest == 2) __builtin_amdgcn_s_setprio(2);
        else if (longest == 1) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
      look_ahead();
    }
    Lanes picked = 0;
    auto take_step = [&](const unsigned step, Item& now, const Item& last) {
      // ---- read phase: the neighbouring stages' counters, then for which stages the next item of each type is eligible
      // (dependencies resolved, and for forward items the in-flight rule): every comparison a packed subtraction whose
      // sign bits (bit 15: first stage, bit 31: second) say "eligible".  A missing stage never is.
      pair16 f_ahead[NP], b_ahead[NP];
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        constexpr int kLast = V - 1;
        const int c0 = 2 * i, c1 = min(2 * i + 1, kLast);
        if (ONE_NEIGHBOUR) {
          f_ahead[i] = pair_of(__builtin_amdgcn_perm(ahead_words[0], both_m, ahead_bytes[0]));
          b_ahead[i] = pair_of(__builtin_amdgcn_perm(ahead_words[1], both_m, ahead_bytes[1]));
        } else if (DEG > 0) {
          f_ahead[i] = pair16{ahead_f[i][0], ahead_f[i][1]};
          b_ahead[i] = pair16{ahead_b[i][0], ahead_b[i][1]};
#pragma unroll
          for (int k = 1; k < DEG; ++k) {
            f_ahead[i] = __builtin_elementwise_min(f_ahead[i], pair16{ahead_f[i][2 * k], ahead_f[i][2 * k + 1]});
            b_ahead[i] = __builtin_elementwise_min(b_ahead[i], pair16{ahead_b[i][2 * k], ahead_b[i][2 * k + 1]});
          }
        } else {
          int fa[2], ba[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int c = h == 0 ? c0 : c1;
            fa[h] = m; ba[h] = m;
            if (c >= nch) continue;
            const int32_t* pred_off = lds + T.off_pred_off;
            const int32_t* succ_off = lds + T.off_succ_off;
            const int s = stage[c];
            for (int e = pred_off[s]; e < pred_off[s + 1]; ++e) fa[h] = min(fa[h], counts[base + lds[T.off_pred_stage + e]]);
            for (int e = succ_off[s]; e < succ_off[s + 1]; ++e) ba[h] = min(ba[h], counts[base + S + lds[T.off_succ_stage + e]]);
          }
          f_ahead[i].x = (short)fa[0]; f_ahead[i].y = (short)fa[1];
          b_ahead[i].x = (short)ba[0]; b_ahead[i].y = (short)ba[1];
        }
      }
      // (TIMED: the inputs of the last step's items, all timed by now; a lane without one reads some slot)
      int ready = 0, ready2 = 0;
      if (TIMED) {
        ready = lds_read<int>(last.slot + (last.a.y & 0xffff));
        if (DEG > 1) ready2 = lds_read<int>(last.slot + (last.b.z & 0xffff));
      }
      unsigned el_f[NP], el_b[NP], el_w[NP];
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const pair16 nf = pair_of(n_f[i]), nb = pair_of(n_b[i]);
        el_f[i] = bits_of(nf - f_ahead[i]) & bits_of(nf - pair_of(n_bl[i])) & kBothSigns;
        el_b[i] = bits_of(nb - __builtin_elementwise_min(nf, b_ahead[i])) & kBothSigns;
        el_w[i] = SLIDE ? 0u : bits_of(pair_of(n_w[i]) - nb) & kBothSigns;
      }
      // ---- the step function: the first instruction type, in priority order, with an eligible item
      unsigned any_f = el_f[0], any_b = el_b[0], any_w = el_w[0];
      if (V > 2) { any_f |= el_f[NP - 1]; any_b |= el_b[NP - 1]; any_w |= el_w[NP - 1]; }
      const Lanes b_first = __ballot(turn_at < 0);
      const unsigned any_first = of(b_first, any_b, any_f), any_other = of(b_first, any_f, any_b);
      const Lanes hit = __ballot(any_first != 0u), is_f = hit ^ b_first;
      const unsigned any_fb = of(hit, any_first, any_other);
      const Lanes some_fb = __ballot(any_fb != 0u), is_w = SLIDE ? 0ull : ~some_fb;
      picked = SLIDE ? some_fb : __ballot((any_fb | any_w) != 0u);
      const Lanes picked_f = some_fb & is_f, picked_b = some_fb & ~is_f;
      auto by_type = [&](unsigned f, unsigned b, unsigned w) {
        const unsigned fb = of(is_f, f, b);
        return SLIDE ? fb : of(is_w, w, fb);
      };
      const Lanes timed = items;
      if (TIMED) items = picked;
      // ... then the stage.  (From here on all lanes do what those with an item need; where that changes the actor's state
      // it is done for those only.  A branch around it would make the items' timing wait for what stands behind it.)
      unsigned pick = 0u;   // chunk << kPositionBit
      [[maybe_unused]] unsigned walk = 0u;
      [[maybe_unused]] Lanes move = 0;
      if constexpr (V > 1) {
        walk = by_type(walk_f, walk_b, kOneItem);
        if constexpr (V == 2) {
          // the eligible ones with the position's half in the low half: it is taken unless it is not eligible or has had
          // its items and the other one is eligible
          const unsigned el = SLIDE ? any_fb : of(is_w, any_w, any_fb);
          const unsigned turned = __builtin_amdgcn_alignbit(el, el, walk);
          const unsigned other = turned & (walk | ~(turned << 16));   // (its sign)
          pick = (walk ^ (other >> 27)) & 16u;
          move = __ballot((int)(walk | other) < 0);
        } else {
          const unsigned el0 = by_type(el_f[0], el_b[0], el_w[0]), el1 = by_type(el_f[NP - 1], el_b[NP - 1], el_w[NP - 1]);
          const unsigned ok = (el0 >> 15 & 1u) | (el0 >> 30 & 2u) | (el1 >> 13 & 4u) | (el1 >> 28 & 8u);
          // the next stage after p0, in the traversal direction and cyclically, that has an eligible item:
          // lay the mask out twice, shift it so that the stage after p0 is at bit 0, take the lowest bit
          // (depth-first: the same on the mirrored mask)
          const Lanes up = (is_f & upward_f) | (~is_f & upward_b) | is_w;
          const int p0 = (int)((walk & kPosition) >> kPositionBit);
          move = __ballot((int)walk < 0) | __ballot(((ok >> p0) & 1u) == 0u);
          const unsigned mirrored = __brev(ok) >> (32 - nch);   // (without an item ok is 0 and the chunk some number)
          const unsigned line = of(up, ok, mirrored);
          const int q0 = of(up, p0, nch - 1 - p0);
          const unsigned twice = line | (line << nch);
          int q1 = q0 + 1 + low_bit(twice >> (q0 + 1));
          q1 = q1 >= nch ? q1 - nch : q1;
          const int moved_to = of(up, q1, nch - 1 - q1);
          pick = ((unsigned)of(move, moved_to, p0) & 3u) << kPositionBit;
        }
        asm("" : "+v"(pick));   // (not taken apart again)
      }
      // ---- write phase: the choice becomes visible for the next step; the counter's old value is the micro-batch of the
      // item.  Counts go up with the lanes of each type in turn, one instruction each.  (next_step: SLIDE, a step in which
      // nothing else is eligible takes a W item while there is one.)
      const unsigned half = V > 2 ? pick & 16u : pick, one = V > 1 ? 1u << (half & 31u) : 1u;
      unsigned old, own = of(is_f, own_f, own_b);
      unsigned hi = 0u;
      if constexpr (V <= 2) {
        old = by_type(n_f[0], n_b[0], n_w[0]);
        // (the second chunk's counter: the upper half of `one` is 1)
        if constexpr (V == 2 && !ONE_NEIGHBOUR) asm("v_mad_i32_i16 %0, %1, %2, %0 op_sel:[1,0,0,0]" : "+v"(own) : "v"(one), "v"(own_step));
      } else {
        hi = mask_of((pick & 32u) != 0u);
        old = choose(hi, by_type(n_f[NP - 1], n_b[NP - 1], n_w[NP - 1]), by_type(n_f[0], n_b[0], n_w[0]));
        unsigned first = own_at[0];
#pragma unroll
        for (int c = 1; c < V; ++c) first = pick == (unsigned)c << kPositionBit ? own_at[c] : first;
        own += first - own_at[0];
      }
      const unsigned j = V > 1 ? __builtin_amdgcn_ubfe(old, half, 16u) : old & 0xffffu, behind = ONE_NEIGHBOUR ? old + one : j + 1u;
#define FPSCHED_COUNT                                                                                                    \
  "s_mov_b64 exec, %[is_b]\n\t"                                                                                          \
  "v_add_u32 %[b], %[b], %[by]\n\t"                                                                                     \
  "v_add_u32 %[bl], %[bl], %[by]\n\t"                                                                                   \
  "s_mov_b64 exec, %[is_f]\n\t"                                                                                          \
  "v_add_u32 %[f], %[f], %[by]\n\t"                                                                                     \
  "s_mov_b64 exec, -1"
      if constexpr (V > 2) {
        const unsigned by = one & ~hi;
        asm volatile(FPSCHED_COUNT : [b] "+&v"(n_b[0]), [bl] "+&v"(n_bl[0]), [f] "+&v"(n_f[0]) : [by] "v"(by), [is_b] "s"(picked_b), [is_f] "s"(picked_f));
        if constexpr (!SLIDE) n_w[0] += of(picked & is_w, by, 0u);
      }
      const unsigned by = V > 2 ? one & hi : one;
      if constexpr (TIMED) {
        // The new item's row is on its way until the next step: cost, where its inputs' finish times are and where its own goes
        // (byte offsets), memory.  (What is read in front of the counters is there when it is asked for; behind them it would be
        // waited for with them.)
        const unsigned next_row = __umul24(pick, (unsigned)D) + by_type(row_f, row_b, row_b + V * D * 16);
        now.a = lds_read<int4>(next_row);
        if (kSecondHalves) now.b = lds_read<int4>(next_row + n_rows * 16);
        // (not before the row's place is known: the inputs' times are on their way until here)
        asm volatile("v_add_u32 %0, %0, %1" : "+v"(ready) : "v"(last.a.z), "v"(next_row), "v"(behind));
        if (DEG > 1) ready = max(ready, ready2 + last.b.w);
      }
      const Lanes counted = SLIDE ? picked : some_fb;
      if constexpr (SLIDE) {
        asm volatile("s_mov_b64 exec, %[all]\n\t"
                     "ds_write_b32 %[own], %[behind]\n\t"
                     "v_lshl_add_u32 %[slot], %[j], 2, %[slots]\n\t"
                     "v_max_u32 %[next], %[step], %[next]\n\t"
                     "v_addc_co_u32 %[next], vcc, 1, %[next], %[is_b]\n\t" FPSCHED_COUNT
                     : [b] "+&v"(n_b[NP - 1]), [bl] "+&v"(n_bl[NP - 1]), [f] "+&v"(n_f[NP - 1]), [next] "+&v"(next_step), [slot] "+&v"(now.slot)
                     : [by] "v"(by), [own] "v"(own), [behind] "v"(behind), [j] "v"(j), [slots] "v"(slot), [step] "s"(step), [all] "s"(counted),
                       [is_b] "s"(picked_b), [is_f] "s"(picked_f)
                     : "memory", "vcc");
      } else {
        asm volatile("s_mov_b64 exec, %[all]\n\t"
                     "ds_write_b32 %[own], %[behind]\n\t" FPSCHED_COUNT
                     : [b] "+&v"(n_b[NP - 1]), [bl] "+&v"(n_bl[NP - 1]), [f] "+&v"(n_f[NP - 1])
                     : [by] "v"(by), [own] "v"(own), [behind] "v"(behind), [all] "s"(counted), [is_b] "s"(picked_b), [is_f] "s"(picked_f)
                     : "memory");
        n_w[NP - 1] += of(picked & is_w, by, 0u);
        if (TIMED) {
          next_step = of(picked, step + 1u, next_step);
          now.slot = of(picked, slot + j * 4u, now.slot);
        }
      }
#undef FPSCHED_COUNT
      look_ahead();
      if constexpr (TIMED) {
        // the last step's items are timed
        const unsigned out_at = last.slot + ((unsigned)last.a.y >> 16), out_at2 = DEG > 1 ? last.slot + ((unsigned)last.b.z >> 16) : 0u;
        if constexpr (SLIDE) {
          [[maybe_unused]] unsigned wait;
          // (all W items of an actor together cost less than 2^29)
#define FPSCHED_TIME                                                                                                     \
  "s_mov_b64 exec, %[timed]\n\t"                                                                                         \
  "v_max_i32 %[start], %[free], %[start]\n\t"                                                                           \
  "v_sub_u32 %[wait], %[start], %[free]\n\t"                                                                            \
  "v_min_u32 %[wait], 0x1fffffff, %[wait]\n\t"                                                                          \
  "v_lshl_or_b32 %[wait], %[wait], 3, %[event]\n\t"                                                                     \
  "v_add_u32 %[free], %[start], %[cost]\n\t"                                                                            \
  "ds_write_b32 %[at], %[wait]\n\t"                                                                                     \
  "v_add_u32 %[at], 0x100, %[at]\n\t"                                                                                   \
  "ds_write_b32 %[out], %[free]\n\t"
          if constexpr (DEG > 1) {
            asm volatile(FPSCHED_TIME
                         "ds_write_b32 %[out2], %[free]\n\t"
                         "v_and_or_b32 %[at], %[at], %[mask], %[ring]\n\t"
                         "s_mov_b64 exec, -1"
                         : [start] "+&v"(ready), [free] "+&v"(free_at), [at] "+&v"(ring_in), [wait] "=&v"(wait)
                         : [event] "v"(last.a.w), [cost] "v"(last.a.x), [out] "v"(out_at), [out2] "v"(out_at2), [mask] "s"(ring_mask), [ring] "v"(ring), [timed] "s"(timed)
                         : "memory");
          } else {
            asm volatile(FPSCHED_TIME
                         "v_and_or_b32 %[at], %[at], %[mask], %[ring]\n\t"
                         "s_mov_b64 exec, -1"
                         : [start] "+&v"(ready), [free] "+&v"(free_at), [at] "+&v"(ring_in), [wait] "=&v"(wait)
                         : [event] "v"(last.a.w), [cost] "v"(last.a.x), [out] "v"(out_at), [mask] "s"(ring_mask), [ring] "v"(ring), [timed] "s"(timed)
                         : "memory");
          }
#undef FPSCHED_TIME
        } else if (in(timed)) {
          free_at = max(free_at, ready) + last.a.x;
          lds_write<int>(out_at, free_at);
          if (DEG > 1) lds_write<int>(out_at2, free_at);
          mem += last.b.x;
          peak = max(peak, mem);
          mem -= last.b.y;
        }
      } else {
        const unsigned word = (pick << (11u - kPositionBit) | by_type(1u << 13, 2u << 13, 3u << 13)) | j, at = (place & kPlaceMask) + staging_at;
        asm volatile("s_mov_b64 exec, %[all]\n\t"
                     "ds_write_b16 %[at], %[word]\n\t"
                     "v_or_b32 %[place], 0xfc, %[place]\n\t"
                     "v_add_u32 %[place], 2, %[place]\n\t"
                     "v_mov_b32 %[next], %[behind]\n\t"
                     "s_mov_b64 exec, -1"
                     : [place] "+&v"(place), [next] "+&v"(next_step) : [at] "v"(at), [word] "v"(word), [behind] "s"(step + 1u), [all] "s"(picked) : "memory");
      }
      // The traversal's and the interleaved priority's next state: while the counters are on their way (not before them).
      asm volatile("v_subb_co_u32 %0, vcc, %0, 0, %2" : "+v"(turn_at), "+v"(walk) : "s"(hit) : "vcc");   // (less 1 where it is)
      turn_at = turn_at < turn_end ? turn_begin : turn_at;
      if constexpr (V > 1) {
        const unsigned left = of(move, of(is_f, again_f, again_b), walk - kOneItem);
        const unsigned walked = (left & ~kPosition) | pick;
        walk_f = of(moving_f & picked_f, walked, walk_f);
        walk_b = of(moving_b & picked_b, walked, walk_b);
      }
      __builtin_amdgcn_wave_barrier();
    };
    for (unsigned turn = 0; turn < kStepsPerLook; turn += 2) {
      take_step(step_0 + turn, items_of[0], items_of[1]);
      take_step(step_0 + turn + 1u, items_of[1], items_of[0]);
    }
    // ---- has the set's process ended?  Looked at every kStepsPerLook steps only: it has if a step schedules nothing (no
    // later step can then; SLIDE: W items, on which nothing depends, aside), and stays ended, so the few steps a segment
    // runs on change nothing, and the number of steps the process took is one more than the step of its last item.
    const bool any_pick = any_in_segment(picked);
    if (!TIMED && words_at(place) - stored >= 16) {
      const uint32_t* w = staging + ((stored >> 1) & (kStagingWords - 1)) * 64;
      uint4* dst = reinterpret_cast<uint4*>(row + stored);
      dst[0] = make_uint4(w[0], w[64], w[128], w[192]);
      dst[1] = make_uint4(w[256], w[320], w[384], w[448]);
      stored += 16;
    }
    if (SLIDE) {
      // (a look adds at most kStepsPerLook items, and one place of the ring stays empty)
      const Lanes ended = __ballot(live && !any_pick);
      while ((__ballot(((ring_in - ring_out) & (ring_bytes - 1u)) > ring_bytes - (1 + kStepsPerLook) * 256u) |
              (ended & (has_event | __ballot(ring_in != ring_out)))) != 0ull)
#pragma unroll
        for (int i = 0; i < kRoundsPerLook; ++i) settle();
    }
    if (live && !any_pick) {
      bool done = true;   // else items remain and nothing can move
#pragma unroll
      for (int i = 0; i < NP; ++i) done = done && (SLIDE || !has_w ? n_b[i] : n_w[i]) == (unsigned)m * 0x00010001u;
      status = any_in_segment(__ballot(!done)) ? 1 : status;
      // (SLIDE: the W items that are left follow, one a step)
      steps = segment_max((int)(next_step - first_step));
      live = false;
      fresh = true;
    }
  }
}

#define FPSCHED_INSTANTIATE(V, G, FORM)                                                                     \
  template __global__ void generate_kernel<V, G, FORM>(DevTables, const int32_t*, const int32_t*,            \
                                                        const long long*, long long, long long, int, int, uint16_t*, int32_t*, \
                                                        unsigned char*, unsigned long long*, GenResults);
FPSCHED_INSTANTIATE(1, 1, false)
FPSCHED_INSTANTIATE(2, 1, false)
FPSCHED_INSTANTIATE(4, 1, false)
FPSCHED_INSTANTIATE(1, 2, false)
FPSCHED_INSTANTIATE(2, 2, false)
FPSCHED_INSTANTIATE(4, 2, false)
FPSCHED_INSTANTIATE(1, 0, false)
FPSCHED_INSTANTIATE(2, 0, false)
FPSCHED_INSTANTIATE(4, 0, false)
FPSCHED_INSTANTIATE(1, 1, true)
FPSCHED_INSTANTIATE(2, 1, true)
FPSCHED_INSTANTIATE(4, 1, true)
FPSCHED_INSTANTIATE(1, 2, true)
FPSCHED_INSTANTIATE(2, 2, true)
FPSCHED_INSTANTIATE(4, 2, true)
FPSCHED_INSTANTIATE(2, kGenOneNeighbour, kGenPlain)
FPSCHED_INSTANTIATE(2, kGenOneNeighbour, kGenTimed)
FPSCHED_INSTANTIATE(2, kGenOneNeighbour, kGenSlide)
FPSCHED_INSTANTIATE(1, 1, kGenSlide)
FPSCHED_INSTANTIATE(2, 1, kGenSlide)
FPSCHED_INSTANTIATE(4, 1, kGenSlide)
FPSCHED_INSTANTIATE(1, 2, kGenSlide)
FPSCHED_INSTANTIATE(2, 2, kGenSlide)
FPSCHED_INSTANTIATE(4, 2, kGenSlide)
#undef FPSCHED_INSTANTIATE

}  // namespace fpsched
