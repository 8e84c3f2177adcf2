// Device-side view of one problem: small integer tables that every candidate of a
// batch shares.  Built on the host by fpsched_problem_create and passed to the
// kernels by value (the pointers are DEVICE pointers into one upload).
#pragma once
#include <stdint.h>

namespace fpsched {

constexpr int kMaxDevices = 64;
constexpr int kMaxChunks = 4;
constexpr int kNKinds = 8;

enum Kind : int { kEnd = 0, kF = 1, kB = 2, kW = 3, kR = 4, kO = 5, kL = 6, kFD = 7 };

// Activation state of one (stage, micro-batch); all transitions happen on the
// stage's own device.
enum ActState : int { kAbsent = 0, kRes = 1, kDisc = 2, kOff = 3, kBDone = 4, kDone = 5 };

enum Flag : int { kDeadlock = 1, kIncomplete = 2, kOverCap = 4 };

struct DevTables {
  int32_t D, S, m, has_w;
  int32_t lanes_per_cand;   // power of two >= D
  int32_t cands_per_wave;   // <= 64 / lanes_per_cand, limited by LDS
  int32_t n_table_ints;     // length of `ints`
  // offsets (in int32 units) into `ints`
  int32_t off_dur;          // [kNKinds][S]
  int32_t off_mem_units;    // [S]
  int32_t off_pred_off;     // [S+1]
  int32_t off_pred_stage;   // [E]
  int32_t off_pred_comm;    // [E]  latency, already 0 for same-device edges
  int32_t off_succ_off;     // [S+1]
  int32_t off_succ_stage;   // [E]
  int32_t off_succ_comm;    // [E]
  int32_t off_local_stage;  // [D][kMaxChunks], -1 = none
  int32_t off_n_chunks;     // [D]
  int32_t off_mem_cap;      // [D]
  // Timed form of the generator (generate.hip): one row per (instruction type F / B / W,
  // chunk < gen_row_chunks, device); -1 if the DAG has a stage with more than two inputs or
  // outputs.  A row has two halves of four ints, all first halves stand in front of all second halves:
  //   0 duration   1 byte offset of the first input slot | of the first output slot << 16
  //   2 latency of the first input, or -2^30 if there is none   3 chunk | 4 for B
  //   4 units allocated at the start   5 units freed at the end   6, 7 as 1, 2 for the second input and output
  // Slots of one parameter set: one word per (direction, class, micro-batch) as in the slot kernel
  // (backward class k at k m, forward class k at (classes + k) m) holding a plain finish time, then m
  // words that take what items without an out-edge write (and that items without an input read).
  int32_t off_gen_rows;
  int32_t gen_row_chunks;   // 1, 2 or 4
  int32_t gen_slot_words;   // (2 * classes + 1) * m
  int32_t gen_sets;         // parameter sets per wavefront, at most 64 / D: as many as LDS holds, set per launch
  int32_t gen_events;       // sliding form of the timed generator: items noted per lane, a power of two, set per launch
  int32_t gen_queue_words;  // sliding form of the timed generator: queue words per lane in LDS, set per launch
  int32_t off_turnaround;   // [S] generator steps from a micro-batch's forward item to its backward item, 2 * (longest path to a sink) + 1
  const int32_t* ints;      // DEVICE
};

// Slot kernel tables.  `ints` = [meta][meta2][pad to 512 ints][costs per micro-batch, if any][dev][expect]:
//   meta  [kNKinds * 4][lanes_per_cand] x 4 ints, one 16-byte row per (top five bits of the op
//     word = kind * 4 + chunk, device):
//     x = dur << 8
//     y = (latency of the first input edge << 8) - tag expected on the first input
//     z = required state (low nibble of byte 0) | state transition need ^ next (byte 1)
//         | byte offset of the first output slot, or of the dump region (16) << 16
//     w = units allocated at the op's start (byte 0) | units freed at its end (byte 1)
//         | own stage (byte 2) | 0xff if the op has a first input edge, else 0 (byte 3)
//     Rows of words that may not appear on the device (no such chunk, kind 0, W without split
//     backward) require state 15, which no activation is ever in.
//   meta2 [2 * 4 + 1][lanes_per_cand] x 2 ints, second input/output edge per (direction, chunk,
//     device); the last row is all zero (read by kinds without cross-stage edges):
//     x = (latency of the second input edge << 8) - its tag
//     y = byte offset of the second output slot (16) | kMetaHasProd | kMetaHasCons
//   dev   [lanes_per_cand] x (2 + 4V) ints: chunks on the device, memory cap / unit_scale, then per
//     chunk the slot offsets of the first forward / first backward / second forward / second
//     backward input
//   expect [lanes_per_cand][state_words]: the device's state words when every activation is done
// A slot is one dword, finish << 8 | producer stage; offsets count from the candidate's slot
// base: class * m slots for backward values, (classes + class) * m for forward values; the dump
// region (m slots written by ops without an output edge, never read) starts at 2 * classes * m.
// Memory units are divided by their greatest common divisor (unit_scale) and must then fit a byte.
constexpr unsigned kMetaHasProd = 1u << 30;
constexpr unsigned kMetaHasCons = 1u << 31;
constexpr unsigned kEmptySlot = 0x000000ffu;  // finish 0, tag 0xff = no stage

struct SlotTables {
  int32_t D, m;
  int32_t lanes_per_cand;   // power of two >= D
  int32_t cands_per_wave;
  int32_t n_classes;        // slot classes (1 for a chain)
  int32_t slots_per_cand;   // (2 * classes + 1) * m, rounded up to a multiple of 8
  int32_t unit_scale;       // common divisor of the memory units
  int32_t state_words;      // dwords of 4-bit activation states per lane
  int32_t wave_ints;        // LDS dwords owned by one wavefront (512 of them its op window)
  int32_t n_shared_ints;    // meta + meta2 + pad to a multiple of 512, copied to LDS once per workgroup
  int32_t off_meta2;        // in ints
  int32_t off_dev;          // in ints
  int32_t dev_ints;         // 2 + 4V
  int32_t off_expect;       // in ints
  int32_t link_words;       // link mode: dwords per lane behind its state words, one per device this device
                            // sends to, one for values that stay on the device and, last, one that takes
                            // what ops without an out-edge write (0 = plain model);
                            // the dev rows then have 4V more ints: per chunk the first forward / first backward /
                            // second forward / second backward out-edge as latency << 16 | byte offset of its
                            // link word (link index * 256)
  int32_t copy_depth;       // copy-engine form: transfers the engine holds at most (1..7), else 0; link_words is
                            // then the number of ring dwords per lane behind its state words
  int32_t off_w;            // in ints; sliding form: per device [lanes_per_cand][2 * kMaxChunks + 1]: cost << 8 of the
                            // W item of each chunk, the units it frees, then (cost << 8 of all W items of the device)
  const int32_t* ints;      // DEVICE
};

// Tables of the two-pass list evaluation (rows.h, timing.hip).  `ints` = [timing rows][link or group rows]
// [cost table][order rows][dev], those in the middle in their forms only:
//   timing rows [kNKinds * 4][D, the even devices first] x 4 ints, addressed by the top five bits of the op word and
//   the device:
//     0 (latency of the first input << 8) - tag expected on it (kEmptySlot's tag if the op starts a class, kOwnTag if
//       it has no cross-stage edge); 1: the op never issues
//     1 dur << 8 | tag it leaves: its stage, or kOwnTag
//     2 byte offset of its slot for micro-batch 0 | mask of the bits of (word << 2) that are added to it << 16
//     3 if the op has a second input or output (not in the plain form): byte offset of a second row | kRowTwoOut | sign bit: two inputs.  An op
//       with two inputs waits for its second one first: words 0 and 2 are then the second input's.
//     Narrow forms without second rows beside the row: 2 the mask | 16-byte rows in front of the row that follows << 18
//     (0: none), 3 the offset.  The plain form keeps second edges in rows that follow: [takes in the second input: no cost,
//     leaves an empty slot] [the op] [leaves the second output: expects an empty slot, no cost].  In the other forms:
//   second rows x 4 ints: 0 and 1 words 0 and 2 of the first edge, 2 the slot of the second output (as word 2), 3 the
//     second output's link row in the links form
//   Copy-engine form: rows that follow others as in the plain form; the upper half of word 3 has the units the op allocates |
//     those it frees << 8.
//   Wide form (times beyond 24 bits; a slot is two dwords, the time and the tag): word 0 is the latency, word 1 the
//   duration, word 3 the tag the op leaves | the tag it expects << 8 | number of 16-byte rows in front of its second row
//   << 16 | the two flags (problems without second edges: word 2 the mask, word 3 the two tags | the slot's offset << 16);
//   word 3 of a second row is the tag expected on the first edge << 8.
//   Slots of a candidate, in dwords: [0, D) the devices' own words, D + 1
//   for the makespan, then from list_slots_at(D) on class * m for backward values, (backward classes + class) * m for
//   forward values; finish << 8 | producer stage, kEmptySlot at first.
//   link rows: byte offset of the word of the link that the first output goes over | latency << 16; an op that sends nothing
//     to another device has the last word.
//   cost table: per kind (kinds with the same costs share) and stage a row of mb_bytes per micro-batch, an odd number of
//     dwords long; word 1 of a timing row then has the byte offset of that row instead of the duration, and the order
//     rows' durations are 0.
//   items of groups (synchronisation form): the timing row never issues, its word 1 is kGroupRow and it names, as a row that
//     follows, two group rows, of the first edge and of the second: 0 as in a timing row (without an input: 0), 1 (first)
//     dur << 8 | stage, 2 (first) micro-batches per item | kGroupIn if it has an input | kGroupOut if an output, 3 byte offset
//     of the slots
//   order rows [kNKinds * 4][D] x 2 ints:
//     0 next state | required state << 8 | units allocated << 16 | units freed << 24   1 dur
//     Rows of words that may not appear on the device require kNoState; word 1 of the rows of kind 0 has the items of the
//     chunk's stage.
//   dev [D] x 2: chunks on the device, memory cap / unit_scale
// Memory units are divided by their greatest common divisor (unit_scale) and must then fit a byte.
struct ListTables {
  int32_t D, m;
  int32_t cands_per_wave;   // candidates of one wavefront of the timing pass: ceil(D / 2) lanes each
  int32_t cand_slots;       // slots per candidate, a multiple of 4
  int32_t wave_bytes;       // LDS of one wavefront of the timing pass: op windows, link words, slots
  int32_t n_time_ints;      // timing rows, padded to a multiple of 8
  int32_t chunks;           // most stages of a device
  int32_t row_step;         // timing rows in LDS: bytes from one (kind, chunk) to the next,
  int32_t odd_at;           // ... from the even devices' rows to the odd ones',
  int32_t row_bytes;        // ... and in all
  int32_t off_links;        // links form: link rows, one int per timing row in the same order, in ints
  int32_t link_words;       // links form: words per lane and half (one behind the links for ops that send nothing)
  int32_t copy_depth;       // copy-engine form: transfers the engine holds at most, else 0
  int32_t mb_bytes;         // costs per micro-batch: bytes of a value, 1 or 2
  int32_t off_sync;         // synchronisation form: group rows, in ints (0: another form)
  int32_t off_check;        // order rows, in ints
  int32_t n_check_ints;
  int32_t check_columns;    // order rows in LDS: columns of each (kind, chunk), a power of two from D on; 0: device by device
  int32_t check_shared_bytes;   // order rows and dev rows in LDS, a multiple of 16
  int32_t off_dev;          // in ints
  int32_t state_bytes;      // states of one row in the order pass: an odd number of dwords
  int32_t check_wave_bytes; // LDS of one wavefront of the order pass, a multiple of 16
  int32_t terminal;         // state of a consumed activation
  int32_t unit_scale;
  const int32_t* ints;      // DEVICE
};
constexpr unsigned kRowTwoOut = 1u << 30;
// LDS of the timing pass's tables, and where what stands behind the rows is: an offset in `ints` counts from here on
constexpr int list_dense_row_bytes(const ListTables& T) { return kNKinds * kMaxChunks * 16 * T.D; }
constexpr int list_behind_rows(const ListTables& T) { return T.row_bytes - list_dense_row_bytes(T); }
constexpr int list_table_bytes(const ListTables& T) { return list_behind_rows(T) + 4 * T.n_time_ints; }
// LDS of the order pass in a workgroup that does both passes; the timing pass's is behind it, from a multiple of the bytes of a
// half's op windows on
constexpr int alone_check_bytes(const ListTables& T, int waves) { return (T.check_shared_bytes + waves * T.check_wave_bytes + 2047) & ~2047; }
constexpr int kCheckColumns = 32;   // of 8 bytes, all banks
constexpr int kRowColumns = 16;   // of 16 bytes, all banks (timing.hip); column c is of the pair of devices c modulo their number
constexpr int kGroupRow = -1;
constexpr unsigned kGroupIn = 1u << 16, kGroupOut = 1u << 17;
constexpr unsigned kWideNever = 0xffu << 8;   // wide form: the tag of an empty slot, expected on a device's own word
constexpr unsigned kOwnTag = 0xfeu;   // (no stage's op looks at a device's own word)
constexpr int list_slots_at(int D) { return (D + 2 + 3) & ~3; }
constexpr unsigned kNoState = 15u;
constexpr unsigned kPadState = 14u;   // order pass: state of the bytes behind a chunk's last item
// the upper half of what the order pass leaves per row: the position at which the list stops (its END word, the end
// of the row, or the first op that may not issue there), and
constexpr unsigned kRowStop = 0x07ffffffu;
constexpr unsigned kRowPlant = 1u << 27;       // the END word that the list stops at is of a third or fourth stage: its row may be another word's
constexpr unsigned kRowStuck = 1u << 28;       // the list stops at an op that can never issue
constexpr unsigned kRowMalformed = 1u << 29;   // ... whose word is malformed
constexpr unsigned kRowIncomplete = 1u << 30;  // not every activation is consumed at the stop
constexpr unsigned kRowOverCap = 1u << 31;     // the peak exceeds the device's cap

// Tables of the evaluation with synchronisation stages and dependency pairs (eval_sync.hip).  Every
// dependency of an item -- the edges of the stage DAG and the user's pairs alike -- is one entry of a list
// per (kind, stage): which finish-time table it looks into (0 forward, 1 backward, 2 weight gradient), the
// producing stage, and the latency (already 0 when both stages sit on one device).
struct SyncTables {
  int32_t D, S, m, has_w;
  int32_t lanes_per_cand;   // power of two >= D
  int32_t cands_per_wave;   // limited by LDS
  int32_t n_fin_tables;     // 2, or 3 if some pair waits for a weight-gradient item
  int32_t copy_depth;       // copy-engine form: transfers the engine holds at most (1..7), else 0
  int32_t n_table_ints;     // length of `ints`
  // offsets (in int32 units) into `ints`
  int32_t off_dur;          // [kNKinds][S]
  int32_t off_mem_units;    // [S]
  int32_t off_group;        // [S] micro-batches per item of the stage
  int32_t off_items;        // [S] items per kind: ceil(m / group)
  int32_t off_dep_off;      // [kNKinds * S + 1] first entry of (kind, stage) in the dependency list
  int32_t off_dep;          // [entries][3]: table, producing stage, latency
  int32_t off_local_stage;  // [D][kMaxChunks], -1 = none
  int32_t off_n_chunks;     // [D]
  int32_t off_mem_cap;      // [D]
  const int32_t* ints;      // DEVICE
};

}  // namespace fpsched
