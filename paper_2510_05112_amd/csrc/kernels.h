// Kernel declarations shared by the translation units of libfpsched.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_tables.h"

namespace fpsched {

// a value that all lanes agree on, in scalar registers
__device__ __forceinline__ long long of_first_lane(long long v) {
  return (long long)((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)v));
}

struct Key {
  long long makespan;
  long long idx;
};
constexpr int kTile = 2048;
constexpr int kTopkThreads = 1024;
constexpr int kTopkPartRooms = 16;   // most elements of a part of the top-k, in what its workgroup sorts at a time

// dur_mb: nullptr, or costs per micro-batch [kinds][S][m] in device memory that replace the table's.
__global__ void eval_general_kernel(DevTables T, const uint16_t* ops, long long n_cand, int stride,
                                    long long* out_makespan, long long* out_idle, int* out_peak,
                                    unsigned char* out_flags, const int32_t* dur_mb);

// Synchronisation stages and dependency pairs (eval_sync.hip): the table form of the evaluator with one
// dependency list per (kind, stage) and items that stand for groups of micro-batches.
// COPY: offload and reload items run on a copy engine beside the computation (T.copy_depth transfers at
// most in the engine); needs 1536 more dwords of LDS per workgroup and one more table per candidate.
template <bool COPY>
__global__ void eval_sync_kernel(SyncTables T, const uint16_t* ops, long long n_cand, int stride,
                                 long long* out_makespan, long long* out_idle, int* out_peak,
                                 unsigned char* out_flags);

constexpr int kSlotMaxWaves = 16;
constexpr int kSlotMaxThreads = 64 * kSlotMaxWaves;

// V = compile-time bound on the stages (chunks) per device: 1, 2 or 4.  DEG2 = some stage
// has two inputs or two outputs in the stage DAG.  ONE_CLASS = the DAG is a single chain.
// next_candidate: a counter in device memory, preset to the number of segments in the grid, from
// which wavefronts draw their work, draw_block candidates per atomic (1 <= draw_block <= 64).
// MODE kSlotTimes: first pass of the weight-gradient sliding; writes out_start8 [n_cand][stride / 8][lanes per
// candidate][8 x 16 bits] (low half of the start time of the op at each position), out_escape [n_cand][D][escape_cap]
// (position << 8 | wait >> 16 of the ops that waited 2^16 time units or more, ended by an all-ones word), out_stop
// [n_cand][D] (words issued per device) and out_flags (DEADLOCK / INCOMPLETE only) instead of makespan, idle and peak;
// needs 16 bytes of LDS more.
// MODE kSlotPerMicrobatch: durations from mb_rows [32][lanes per candidate][m] (cost << 8 per metadata
// row, device and micro-batch) instead of the metadata rows.
// MODE kSlotTimesLinks: the timing pass of the sliding under the link model: every ordered pair of devices is a link that
// carries one value at a time; a producer holds its value back until its link is free (T.link_words, the longer dev rows).
// MODE kSlotCopy: offload and reload items run on a copy engine beside the computation (T.copy_depth transfers
// at most in the engine; T.link_words = 32 dwords per lane behind its state words: the finish times and keys of
// the last eight transfers, and a ring of eight pending memory events).
// MODE kSlotSync: synchronisation stages (one item per group of micro-batches) and dependency pairs of the
// forms the mail slots can carry (forward to forward, backward to backward); the dev rows then have V more ints:
// per chunk the micro-batches per item | items << 16.
// MODE kSlotSlide: the weight-gradient sliding pass without its lists: the results of the lists the two-pass form
// would write, in one kernel (tables as for kSlotTimes plus the W items' costs at T.off_w; 16 bytes of LDS more).
constexpr int kSlotTimes = 1, kSlotPerMicrobatch = 2, kSlotTimesLinks = 3, kSlotCopy = 4, kSlotSync = 5, kSlotSlide = 6,
              kSlotSlideLinks = 7;   // kSlotSlide under the link model
constexpr int kSlotCopyWords = 32;
template <int V, bool DEG2, bool ONE_CLASS, int MODE>
__global__ void eval_slot_kernel(SlotTables T, const uint16_t* ops, long long n_cand, int stride,
                                 long long* out_makespan, long long* out_idle, int* out_peak,
                                 unsigned char* out_flags, unsigned long long* next_candidate, int draw_block,
                                 uint32_t* out_start8, int32_t* out_stop, const int32_t* mb_rows,
                                 uint32_t* out_escape, int escape_cap);

// The list evaluation in two passes.  check_rows_kernel: one lane per (candidate, device) row, rows_per_wave of them per
// wavefront; per row out_info (kRow* | stop, then the busy time in the low half) and out_peak.  dynamic: more blocks of
// rows than resident wavefronts, taken draw_blocks at a time, the further ones from counter[1]; else it sets *counter for the timing pass.
// time_lists_kernel: reads out_info from out_idle, writes the results.  DEG2 = some stage has two inputs or outputs;
// WIDE = times beyond 24 bits; MB: bytes of a value of the cost table (0: none);
// COPY: copy engine, transfers that a lane keeps (3, 4, 7; T.copy_depth <= COPY; 0: another form).
constexpr int kCheckMaxThreads = 512;
constexpr int kCheckWavesPerSimd = 3;
constexpr int kTimeMaxThreads = 1024;
constexpr int kCopyShallow = 3;   // copy engine: transfers that a lane keeps in the form with few registers
constexpr int kTimeCopyMaxThreads = 512, kTimeCopyWavesPerSimd = 3;   // copy-engine form (up to 168 registers)
constexpr int kTimeMaxStride = (1 << 23) - 32;   // longest rows that the timing pass has positions for
constexpr int kTimeWindowBytes = 2 * 64 * 32;   // op windows of a wavefront of the timing pass
// VBITS 0, 1, 2: up to 1, 2, 4 stages per device.  NO_W: W items are no-ops that only have to be in range (tables: their
// rows ask for kPadState and leave it).  SHARED: four lanes read each other's rows.
template <int VBITS, bool NO_W, bool SHARED>
__global__ void check_rows_kernel(ListTables T, const uint16_t* ops, long long n_rows, int stride, int rows_per_wave,
                                  long long* out_info, int* out_peak, unsigned long long* counter,
                                  unsigned long long counter_value, int draw_blocks, int dynamic);
// TIMES: the first pass of the weight-gradient sliding (wslide.hip) on the plain model: what eval_slot_kernel<.., kSlotTimes>
// leaves, for lists the NO_W order pass has walked (out_flags and `starts`; makespan, idle and peak are not written).
struct StartTimes {
  uint32_t* low;        // [n_cand][stride / 8][lanes][8 x 16 bits]
  uint32_t* escapes;    // [n_cand][D][escape_cap]
  int32_t* stops;       // [n_cand][D]
  int32_t escape_cap, lanes;
};
// ALONE: 1 + VBITS: both passes in one launch, from a batch of kAloneLeast candidates to as many as the wavefronts hold, T.cands_per_wave each, whose
// rows are a lane's each (0: the timing pass only).
constexpr int kAloneMaxThreads = 512, kAloneLeast = 64;
template <bool DEG2, bool WIDE, bool LINKS, int MB, bool SYNC, bool TIMES, int ALONE, int COPY>
__global__ void time_lists_kernel(ListTables T, const uint16_t* ops, long long n_cand, int stride,
                                  long long* out_makespan, long long* out_idle, int* out_peak,
                                  unsigned char* out_flags, unsigned long long* next_candidate, int draw_block,
                                  unsigned draw_share, StartTimes starts);
// counter[0] = value, counter[1] = value2
__global__ void reset_counter_kernel(unsigned long long* counter, unsigned long long value, unsigned long long value2 = 0);

// V as above; DEG = bound on the in- and out-degree of a stage (1, 2, or 0 = any).  Wavefronts that work
// apart, T.gen_sets <= 64 / D parameter sets at a time each; next_set: a counter in device memory from
// which segments draw their sets.  n_classes = 0: not looked at, no more sets than segments; 1: preset to the number of
// segments in the grid; kGenClasses: set to 0 by generate_order_kernel, which has left each set's class in out_status.
// select: null, or which of the n_src parameter sets each output row takes (outside 0 .. n_src - 1: none).
// TIMED (DEG 1 or 2 only): the schedules are timed as they are generated and only the results R are
// written (ops and select unused).
struct GenResults {
  long long* makespan;
  long long* idle;
  int32_t* peak;
  unsigned char* flags;
};
constexpr int kGenThreads = 256;   // of a workgroup: a wavefront per SIMD
// FORM: kGenPlain writes the lists; kGenTimed times them instead (above); kGenSlide times them after the
// weight-gradient sliding pass (T.gen_events + T.gen_queue_words dwords of LDS more per lane)
constexpr int kGenPlain = 0, kGenTimed = 1, kGenSlide = 2;
constexpr int kGenFewEvents = 16, kGenMoreEvents = 32;   // kGenSlide: items noted per lane (T.gen_events)
constexpr int kGenStagingWords = 16;   // kGenPlain: dwords of op words staged per lane
constexpr int kGenOneNeighbour = 3;   // GRAPH of generate_kernel: two stages per actor, whose neighbours in a direction are on one actor
template <int V, int DEG, int FORM>
__global__ void generate_kernel(DevTables T, const int32_t* policy, const int32_t* inflight, const long long* select,
                                long long n_src, long long n_sets, int n_classes, int stride, uint16_t* ops,
                                int32_t* out_steps, unsigned char* out_status, unsigned long long* next_set,
                                GenResults R);
// classes of the sets by their expected steps, in the status bytes (kGenClassMark | class)
constexpr int kGenClasses = 4, kGenClassMark = 0x80;
__global__ void generate_order_kernel(DevTables T, const int32_t* inflight, const long long* select, long long n_src,
                                      long long n_sets, int work_steps, unsigned char* out_status,
                                      unsigned long long* next_set);

__global__ void topk_kernel(const long long* in_makespan, const unsigned char* in_flags, const Key* in_keys, long long n,
                            long long n_part, unsigned batches, unsigned step, int k, int wide_values, Key* out_keys, long long* final_idx,
                            long long* final_makespan, int* final_count);

__global__ void rank_keys_kernel(const long long* makespan, const long long* idle, const int* peak,
                                 const unsigned char* flags, long long n, int D, int mode, int include_over_cap,
                                 long long* key_out, unsigned char* excluded_out);

// Second kernel of the weight-gradient sliding: one lane per (candidate, device) row places the W
// items into the idle time in front of the ops timed by the pass in front of it.
constexpr int kSlideThreads = 1024;
// dynamic LDS of a workgroup: the metadata rows, then 14 KB per wavefront (windows, stash ring, staged rows)
constexpr int kSlideWaveLdsBytes = 14336;
template <bool FOUR>
__global__ void wslide_place_kernel(SlotTables T, const uint16_t* ops, long long n_cand, int stride,
                                    const uint32_t* start_low, const uint32_t* escapes, int escape_cap,
                                    const int32_t* stop_pos,
                                    const unsigned char* timed_flags, uint16_t* ops_out, int stride_out,
                                    long long* out_makespan, long long* out_idle, int* out_peak,
                                    unsigned char* out_flags);

// ... and for few candidates: one wavefront per row, a workgroup per candidate; dynamic LDS: the metadata rows, 4 ints per
// device, slide_rows_wave_bytes per wavefront.  stash: bound on the B items of a row that are issued.
__host__ __device__ constexpr int64_t slide_rows_wave_bytes(int64_t stride_out, int64_t stash) {
  return 2 * stride_out + ((10 * stash + 8 + 15) & ~15ll);
}
__global__ void wslide_place_rows_kernel(SlotTables T, const uint16_t* ops, int stride, const uint32_t* start_low,
                                         const uint32_t* escapes, int escape_cap, const int32_t* stop_pos,
                                         const unsigned char* timed_flags, uint16_t* ops_out, int stride_out, int stash,
                                         long long* out_makespan, long long* out_idle, int* out_peak,
                                         unsigned char* out_flags);

// Pareto front: at most kParetoMaxTiles tiles of kTile candidates (one cursor per tile in LDS).
constexpr int kParetoMergeThreads = kTile / 2;
constexpr int kParetoMaxTiles = 8192;

__global__ void pareto_tile_kernel(const long long* makespan, const int* peak, const unsigned char* flags,
                                   long long n, int D, Key* front_keys, int* front_peak, int* tile_count);

__global__ void pareto_merge_kernel(const Key* front_keys, const int* front_peak, const int* tile_count, int tiles,
                                    int kmax, long long* out_idx, long long* out_makespan, int* out_peak,
                                    int* out_count);

__global__ void apply_caps_kernel(const int* peak, const int* caps, int per_candidate, long long n, int D,
                                  unsigned char* flags);

}  // namespace fpsched
