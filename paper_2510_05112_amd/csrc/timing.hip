// Timing pass of the list evaluation: start and finish times across the devices, for lists the order pass (rows.h)
// has walked.  Any per-device op order, any stage DAG with at most two inputs and two outputs per stage.
//
// Mapping: lane = (candidate, pair of neighbouring devices), ceil(D / 2) lanes per candidate, as many candidates per
// wavefront as fit its 64 lanes; the wavefronts of a workgroup are independent and only share one LDS copy of the op
// table.  The grid is persistent: a segment (the lanes of one candidate) that finishes takes the next unevaluated
// candidate, from a global counter through a small pool per wavefront, while the other segments keep going.  A lane
// walks the lists of its two devices with cursors in registers, in turn: the even devices issue in one step (every
// device whose next op has its inputs), the odd ones in the next.  A pair of steps in which no lane of a segment moves
// ends that candidate (lists exhausted, or deadlock).
//
// Why in turn: a step costs the wavefront the same instructions however few of its lanes issue, and what a schedule's
// steps are spent on are chains of dependencies from device to neighbouring device, forward down the pipeline,
// backward up again.  With all devices in every step such a chain takes a step per device and most lanes wait; with
// even and odd devices in turn each link of the chain is the other half's turn, so twice as many candidates per
// wavefront move at the same speed along the chains, and only ops that follow each other on one device take two steps.
// Counted on the CPU over the candidates of the benchmark configurations: 1.25 to 1.9 times fewer wavefront steps.
//
// Finish times travel through per-micro-batch mail slots in LDS.  The edges of the stage DAG are split on the host
// into classes (chains of edges in which each edge starts at the stage the previous one ends in; a plain pipeline is
// one class).  For one micro-batch at most one edge of a class carries a live value at a time -- the value of F(a,j)
// on edge a->b is dead once F(b,j) has issued, and only then can the next edge of the class be produced -- so a
// class needs ONE slot per micro-batch and direction, tagged with the stage that produced it:
// slot[dir][class][j] = finish << 8 | producer stage.  A consumer finds its input iff the tag names its upstream
// stage.  No order of micro-batches is assumed and a producer never has to wait for room.
//
// Second inputs and outputs (DEG2), plain form: an op is up to three rows that follow each other, each of them a step like
// any other op's: the first takes in the second input (no cost; it leaves the slot it has read empty), the second is the op,
// the third leaves the second output (no cost).  So a step has one comparison more, and nothing that only few ops need: with
// a second row beside the first, read by every lane in every step, 131,072 candidates of 16 devices (two towers), 64
// micro-batches, offload took 0.88 ms instead of 0.77.  The other forms still have that.
//
// WIDE: finish times of up to 31 bits (durations in microseconds: 16 devices x 64 micro-batches pass 2^24 within a few
// dozen ops) take two words per slot, the time and the tag, and the tag is compared on its own; otherwise the same.  The
// host picks it where the bound on all times does not fit 24 bits or a latency not 16; the table kernel that such
// problems ran on before took 5.2 ms for 8,192 candidates of that size.
//
// LINKS, the link-occupancy variant of the cost model: a link between two devices carries one value at a time.  An op
// with an output to another device leaves in its slot not its finish time but the time its value leaves, max(finish, link
// busy until), and keeps the link busy for the edge's latency from then; the consumer adds the latency as before.  The
// lane keeps that time of each link its devices send over in a word of LDS, and the op's row has a word more: the link
// and the latency.  An op without such an output has a link of its own of latency 0, which only ever holds earlier
// finish times of the device.  The word is read together with the slot, since only the lane itself writes it.
//
// MB, costs per micro-batch: the row has, instead of the cost, where the costs of its (kind, stage) begin in a table in
// LDS; the cost is read together with the slot as well.  The busy time is then summed up here.  Both forms, 20,011
// candidates of 11 devices, 45 micro-batches, 3 chunks: 2.01 ms as forms of the slot kernel with all devices in every round and
// 16 lanes to a candidate; 0.64 + 0.06 ms here with the step as the compiler makes it, 0.55 + 0.06 without branches, and
// what the link and the cost take read ahead with the slot (FPSCHED_COST_STEP).  Such a batch has one candidate per segment:
// the time is its longest chain's, a step's instructions and waits one after the other.  So has one in microseconds: 8,192
// candidates of 16 devices, 64 micro-batches, 2 chunks 0.21 and 0.17 ms (FPSCHED_WIDE_STEP).
//
// SYNC, stages whose items stand for groups of micro-batches (a synchronisation every n micro-batches, Section 4.2 / 7.2
// of the paper) and dependency pairs between items of one direction.  An item of a stage with group n waits for the n
// values of its micro-batches and leaves its own in the n slots.  Its row never issues; every fourth round the devices at such
// an item take in up to four values each and run it with the last one (groups), so that the steps are those of the plain form.
// A pair is an edge of its own slot class in one direction only.  (The host only picks this form when the neighbours of
// such a stage have one item per micro-batch.)  65,536 candidates of 12 devices, 64 micro-batches, groups of four: 1.03 ms
// with one value a step in a step with branches, 0.76 now; groups looked after every second round 0.81, every eighth 0.84.
//
// COPY, the copy-engine model (the paper names CPU offloading without saying how an offload is timed): offload and reload
// items run on a copy timeline of the device.  The walk hands such an item over when it reaches it and goes on at once, unless
// copy_depth transfers are unfinished (then it waits for the oldest of them); a transfer starts at max(hand-over, finish of the
// transfer before it).  A backward item waits for the reload of its activation.  Memory is a sum over events in time order: a
// reload allocates at its start, an offload releases at its end, compute events come first at equal times; so the peak is
// found here and not in the order pass.  Transfers are no busy time; the makespan covers both timelines.  The last transfers
// and the events to come stand in registers, shifted along: in LDS every lane's loop over them was a wait for all lanes.
// 20,011 candidates of 16 devices (two towers), 45 micro-batches, depth 3: 0.72 ms as a form of the slot kernel, all devices
// in every round; 1.43 ms here with rings in LDS, 0.50 (and 0.05 for the order pass) with registers, 0.32 with conditions as sets
// of lanes and state changes on the lanes they are for (110 vector instructions a step as the compiler made them of selects).
// (COPY transfers are kept, and an event more: 65,536 of them, 64 micro-batches, 1.54, 1.68 and 1.90 ms with three, four and seven, 2.77
// ms as the slot kernel.)
//
// TIMES, the first pass of the weight-gradient sliding (wslide.hip) on problems of the plain form: the lists without their W
// items (a W word is an op of the device's own without a cost), of which it leaves the low sixteen bits of each op's start
// time, the ops that waited 2^16 time units or more, and where the lists stop.  A start time takes the place of the op's
// word in the ring and leaves eight at a time when the next piece lands there, so that a step has four vector instructions
// more and no store.  32,768 candidates of 16 devices, 64 micro-batches, 2 chunks: 0.15 ms (order pass) + 0.51 ms; 1.46 ms
// as a form of the slot kernel, with all devices in every round.
//
// Start rule (paper Section 5.1 "Data dependency"; estimator sketch after Section 6): start = max(device free, finish
// of each cross-stage input + latency if the input ran on another device); finish = start + dur[kind][stage].
//
// What bounds it: LDS and vector issue (busy 85 and 80 % of the time; one launch over 65,536 candidates of
// 32 devices, 128 micro-batches, two chunks, profiles/list_evaluation.md).  Everything that does not need the order
// between devices is the order pass's, which also says where each list stops, so that no word in front of that needs
// a check.  A step is four vector instructions to decide (the slot's address from the row; an addition that gives the
// ready time with a low byte that is zero iff the slot carries the expected tag; one byte compare) and nine to issue and
// to decode the next word; in LDS the slot read (random addresses: half of it bank conflicts), the row, the next word
// and the slot written.  The row is fetched when the device issues and first looked at in its next step, so the other
// half's step covers the wait.  That batch took 4.88 ms when one kernel with all devices in every round did the order
// pass's work as well; then 1.10 ms (rows.h) + 2.05 ms; the pass takes 1.67 ms since the step of the plain form is
// without branches (FPSCHED_STEP below: half of the gain), the rings are read without bank conflicts and requests are
// twice as large.
//
// Op words reach a device through a ring of sixteen words in LDS that is topped up every eighth round, eight words at a
// time, where at most seven are unread.  A device that issues one op per round so never runs dry (it reads the word two
// behind the one it issues; after every top-up eight or more are unread), and sixteen places hold the words unread, at
// most fifteen, and the END word that is planted behind a full row.  The ring of a lane is a column of dwords in a bank of
// its own: read in lanes' own 32 bytes, some eight lanes shared their banks (6.6 clocks a read instead of 2.2).  Words are
// requested 64 bytes (forms with the compiler's step: 32) at a time, as soon as the registers they arrive in are free: with the rows of a
// compute unit's candidates in flight the 128-byte lines mostly do not stay in the L2 cache from one request to the next
// (12.8 GB fetched for that batch of 3.76 GB with 32 bytes, 6.8 with 64).  (Rings of 32 words leave room for 11 instead
// of 16 wavefronts per compute unit: 3.3 ms.  Top-ups every fourth round: 2.19 ms.  Loads that bypass L2: 2.8 ms.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"
#include "lds_access.h"
#include "rows.h"

namespace fpsched {

namespace {

constexpr unsigned kRounds = 8;          // rounds (a step of either half) between two top-ups
constexpr unsigned kWindowBytes = 64u * 32u;   // the rings (sixteen words) of one half of a wavefront's devices, [dword][lane]
// Positions in a list and in its ring: the dword from bit 8 on (256 bytes are a dword of all lanes), the half of the dword
// in bit 1; what stands in the bits between is not looked at.
constexpr unsigned kPosMask = 0x702u;    // of a position: its place in the ring
constexpr unsigned kPosBetween = 0xfcu;
constexpr unsigned kPiece = 4u << 8;     // what is landed at a time: eight words, 16 bytes
constexpr unsigned kNoList = 0x40000000u;
// (a request reaches up to three pieces beyond the row, and no position may be kNoList)
static_assert(((unsigned)kTimeMaxStride >> 1 << 8) + 3u * kPiece < kNoList, "");
__device__ __forceinline__ unsigned position_of(unsigned word) { return word >> 1 << 8 | (word & 1u) << 1; }
__device__ __forceinline__ unsigned word_at(unsigned pos) { return pos >> 8 << 1 | (pos >> 1 & 1u); }
// COPY: a step's conditions are sets of lanes in scalar registers
typedef unsigned long long Lanes;
__device__ __forceinline__ Lanes lanes(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool in(Lanes l) { return __builtin_amdgcn_inverse_ballot_w64(l); }

}  // namespace

// The rounds between two looks at the lists, in one statement: what a step requests is waited for in the next one or the
// one behind it, by count, and nothing may come between that does not know it (a copy of such a register, say).  As written
// by the compiler a step has a branch around what the issuing lanes do, and waits in front of its decision for all that the
// step before it has requested; here
//   - the decision becomes the execution mask itself, and nothing branches;
//   - the slots that a half writes are the only thing the other half's read of its slots has to follow, so that read is
//     made before this half's issued ops give way to the next ones, and their rows and words are on their way while the
//     other half decides.
// In flight at the beginning of a step, oldest first: its half's slot, the other half's row and the word behind it; at the
// end of the statement nothing.
// S, O: this half and the other one, `even` or `odd`.  Registers of their rows' four words, and of the two of a wide slot:
#define FPSCHED_even_X "v40"
#define FPSCHED_even_Y "v41"
#define FPSCHED_even_Z "v42"
#define FPSCHED_even_W "v43"
#define FPSCHED_even_ROW "v[40:43]"
#define FPSCHED_even_IN "v48"
#define FPSCHED_even_TAG "v49"
#define FPSCHED_even_SLOT "v[48:49]"
#define FPSCHED_odd_X "v44"
#define FPSCHED_odd_Y "v45"
#define FPSCHED_odd_Z "v46"
#define FPSCHED_odd_W "v47"
#define FPSCHED_odd_ROW "v[44:47]"
#define FPSCHED_odd_IN "v50"
#define FPSCHED_odd_TAG "v51"
#define FPSCHED_odd_SLOT "v[50:51]"

// STEP(S, what is read ahead), AHEAD(O): of a form
#define FPSCHED_FIRST_LOOK(AHEAD) "s_waitcnt lgkmcnt(0)\n\t" AHEAD(even) "s_waitcnt lgkmcnt(0)\n\t"
#define FPSCHED_ROUND(STEP, AHEAD) STEP(even, AHEAD(odd)) STEP(odd, AHEAD(even))
#define FPSCHED_FOUR_ROUNDS(STEP, AHEAD)                                                                                 \
  FPSCHED_FIRST_LOOK(AHEAD) FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD)              \
  STEP(even, AHEAD(odd)) STEP(odd, "") "s_waitcnt lgkmcnt(0)"
#define FPSCHED_EIGHT_ROUNDS(STEP, AHEAD)                                                                                \
  FPSCHED_FIRST_LOOK(AHEAD) FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD)              \
  FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD) FPSCHED_ROUND(STEP, AHEAD)             \
  STEP(even, AHEAD(odd)) STEP(odd, "") "s_waitcnt lgkmcnt(0)"
// Operands of all forms.  (Every output is written while inputs are still to be read.)
#define FPSCHED_STATE(S)                                                                                                 \
  [S##_free] "+&v"(S.free_at), [S##_next] "+&v"(S.w_next), [S##_j] "+&v"(S.j_slot), [S##_pos] "+&v"(S.pos),               \
  [S##_row] "+&{" FPSCHED_##S##_ROW "}"(S.R), [S##_at] "=&v"(at_##S), [S##_moved] "=&s"(moved_##S)
#define FPSCHED_PLACES(S) [S##_rows] "v"(S.meta), [S##_ring] "v"(S.win)
#define FPSCHED_SHARED [stride] "s"(row_stride), [mask] "s"(kPosMask), [slots] "v"(slot_base), [form] "n"(kForm)
// Where the rounds begin in memory, set in front of the loop that they are in.  Instructions arrive 32 bytes at a time, and the few
// wavefronts of a small batch wait for those that lie across two such pieces.  Of the eight places that four bytes more in front of the
// loop give, best and worst: plain form 1005 us at a multiple of 32 bytes, 1017 sixteen behind one (462 candidates of 36 x 117 x 4, the
// whole evaluation); times of two words 189 and 191 (8,192 of 16 x 64 x 2), links with costs 588 and 591 (20,011 of 11 x 45 x 3), the best place
// the same; synchronisation, whose two statements lie apart, 820 sixteen bytes behind it, 838 eight behind it (65,536 of 12 devices).
// NAME: rounds, or alone in the kernel that does both passes.
#define FPSCHED_BEGIN(NAME) ".ifndef .L" NAME "_%c[form]\n\t.L" NAME "_%c[form]:\n\t.endif\n\t"
#define FPSCHED_PLACE_ROUNDS(NAME, AT)                                                                                         \
  asm volatile(".p2align 5\n\t"                                                                                         \
               ".fill ((%c[at] - (.L" NAME "_%c[form] - .Lplace_%c[form])) & 31) / 4, 4, 0xbf800000\n\t" /* (s_nop 0) */  \
               ".Lplace_%c[form]:" :: [form] "n"(kForm), [at] "n"(AT))

// ... the plain form.  (FOLLOW: for rows that another row follows in the place of the next word's, in the form with second
// edges)
#define FPSCHED_STEP(S, AHEAD, FOLLOW, NOT_FOLLOWED)                                                                     \
  "s_waitcnt lgkmcnt(2)\n\t"                                                                                             \
  "v_add_u32 %[" #S "_in], %[" #S "_in], " FPSCHED_##S##_X "\n\t"                                                        \
  "v_cmpx_eq_u32_sdwa %[" #S "_moved], %[" #S "_in], %[zero] src0_sel:BYTE_0 src1_sel:DWORD\n\t"                         \
  "v_max_u32 %[t], %[" #S "_free], %[" #S "_in]\n\t"                                                                     \
  "v_add_u32 %[t], %[t], " FPSCHED_##S##_Y "\n\t"                                                                        \
  "ds_write_b32 %[" #S "_at], %[t]\n\t"                                                                                  \
  "s_mov_b64 exec, -1\n\t" AHEAD                                                                                         \
  "s_mov_b64 exec, %[" #S "_moved]\n\t"                                                                                  \
  "v_and_b32 %[" #S "_free], 0xffffff00, %[t]\n\t"                                                                       \
  "v_lshrrev_b32 %[t], 11, %[" #S "_next]\n\t"                                                                           \
  "v_mad_u32_u24 %[t], %[t], %[stride], %[" #S "_rows]\n\t" FOLLOW                                                       \
  "ds_read_b128 " FPSCHED_##S##_ROW ", %[t]\n\t" NOT_FOLLOWED                                                            \
  FPSCHED_NEXT_WORD(S)
#define FPSCHED_NEXT_WORD(S)                                                                                             \
  "v_or_b32 %[" #S "_pos], 0xfc, %[" #S "_pos]\n\t"                                                                     \
  "v_add_u32 %[" #S "_pos], 2, %[" #S "_pos]\n\t"                                                                       \
  "v_bitop3_b32 %[t], %[" #S "_pos], %[mask], %[" #S "_ring] bitop3:0x6a\n\t"                                           \
  "v_lshlrev_b32 %[" #S "_j], 2, %[" #S "_next]\n\t"                                                                    \
  "ds_read_u16 %[" #S "_next], %[t]\n\t"                                                                                \
  "s_mov_b64 exec, -1\n\t"
// the other half's slot, whose row is there when as many requests as this half's have been made since are still out
#define FPSCHED_AHEAD_SLOT(O, OWN)                                                                                       \
  "s_waitcnt lgkmcnt(" OWN ")\n\t"                                                                                      \
  "v_and_b32 %[" #O "_at], %[" #O "_j], " FPSCHED_##O##_Z "\n\t"                                                        \
  "v_add3_u32 %[" #O "_at], %[" #O "_at], " FPSCHED_##O##_W ", %[slots]\n\t"                                            \
  "ds_read_b32 %[" #O "_in], %[" #O "_at]\n\t"
#define FPSCHED_PLAIN_STEP(S, AHEAD) FPSCHED_STEP(S, AHEAD, "", "")
#define FPSCHED_PLAIN_AHEAD(O) FPSCHED_AHEAD_SLOT(O, "2")
// lanes whose row (its mask) has another one behind it fetch that and stay at their word
#define FPSCHED_FOLLOW(S)                                                                                                \
  "v_cmp_lt_u32 vcc, 0x3ffff, " FPSCHED_##S##_Z "\n\t"                                                                  \
  "s_cbranch_vccz 1f\n\t"                                                                                               \
  "s_mov_b64 exec, vcc\n\t"                                                                                             \
  "v_lshrrev_b32 %[t], 14, " FPSCHED_##S##_Z "\n\t"                                                                     \
  "v_add_u32 %[t], %[tables], %[t]\n\t"                                                                                 \
  "s_mov_b64 exec, %[" #S "_moved]\n\t"                                                                                 \
  "1:\n\t"
#define FPSCHED_FOLLOW_STEP(S, AHEAD) FPSCHED_STEP(S, AHEAD, FPSCHED_FOLLOW(S), "s_andn2_b64 exec, exec, vcc\n\t")
#define FPSCHED_ROUNDS(NAME, TEXT)                                                                                       \
  asm volatile(FPSCHED_BEGIN(NAME) TEXT                                                                                        \
               : FPSCHED_STATE(even), FPSCHED_STATE(odd), [even_in] "=&v"(in_even), [odd_in] "=&v"(in_odd), [t] "=&v"(scratch) \
               : FPSCHED_PLACES(even), FPSCHED_PLACES(odd), FPSCHED_SHARED, [zero] "v"(0u), [tables] "s"(behind)        \
               : "memory", "vcc", "scc")

// ... the form that leaves start times: an op's start goes where its own word was in the ring (own: that place; at_next: the
// place of the word behind it, read already).  The few ops that waited 2^16 time units or more cannot be rebuilt from the low
// half of their start times and go to the row's escape list, while that has room: position << 8 | wait >> 16.
#define FPSCHED_TIMES_STEP(S, AHEAD)                                                                                     \
  "s_waitcnt lgkmcnt(3)\n\t"                                                                                             \
  "v_add_u32 %[" #S "_in], %[" #S "_in], " FPSCHED_##S##_X "\n\t"                                                        \
  "v_cmpx_eq_u32_sdwa %[" #S "_moved], %[" #S "_in], %[zero] src0_sel:BYTE_0 src1_sel:DWORD\n\t"                         \
  "v_max_u32 %[start], %[" #S "_free], %[" #S "_in]\n\t"                                                                 \
  "v_add_u32 %[t], %[start], " FPSCHED_##S##_Y "\n\t"                                                                    \
  "ds_write_b32 %[" #S "_at], %[t]\n\t"                                                                                  \
  "s_mov_b64 exec, -1\n\t" AHEAD                                                                                         \
  "s_mov_b64 exec, %[" #S "_moved]\n\t"                                                                                  \
  "v_sub_u32 %[wait], %[start], %[" #S "_free]\n\t"                                                                      \
  "v_lshrrev_b32 %[start], 8, %[start]\n\t"                                                                              \
  "ds_write_b16 %[" #S "_own], %[start]\n\t"                                                                             \
  "v_and_b32 %[" #S "_free], 0xffffff00, %[t]\n\t"                                                                       \
  "v_cmp_lt_u32 vcc, %[most], %[wait]\n\t"                                                                               \
  "s_cbranch_vccz 1f\n\t"                                                                                                \
  "v_cmp_lt_i32 %[far], 0, %[" #S "_room]\n\t"                                                                          \
  "s_and_b64 exec, vcc, %[far]\n\t"                                                                                     \
  "v_lshrrev_b32 %[t], 8, %[" #S "_pos]\n\t"                                                                             \
  "v_bfe_u32 %[start], %[" #S "_pos], 1, 1\n\t"                                                                          \
  "v_lshl_or_b32 %[t], %[t], 1, %[start]\n\t"                                                                            \
  "v_add_u32 %[t], -1, %[t]\n\t"                                                                                         \
  "v_lshrrev_b32 %[wait], 24, %[wait]\n\t"                                                                               \
  "v_lshl_or_b32 %[t], %[t], 8, %[wait]\n\t"                                                                             \
  "global_store_dword %[" #S "_escape], %[t], off\n\t"                                                                   \
  "v_lshl_add_u64 %[" #S "_escape], %[" #S "_escape], 0, 4\n\t"                                                          \
  "v_add_u32 %[" #S "_room], -1, %[" #S "_room]\n\t"                                                                     \
  "s_mov_b64 exec, %[" #S "_moved]\n\t"                                                                                  \
  "1:\n\t"                                                                                                               \
  "v_lshrrev_b32 %[t], 11, %[" #S "_next]\n\t"                                                                           \
  "v_mad_u32_u24 %[t], %[t], %[stride], %[" #S "_rows]\n\t"                                                              \
  "v_mov_b32 %[" #S "_own], %[" #S "_at_next]\n\t"                                                                       \
  "v_or_b32 %[" #S "_pos], 0xfc, %[" #S "_pos]\n\t"                                                                      \
  "ds_read_b128 " FPSCHED_##S##_ROW ", %[t]\n\t"                                                                         \
  "v_add_u32 %[" #S "_pos], 2, %[" #S "_pos]\n\t"                                                                        \
  "v_bitop3_b32 %[" #S "_at_next], %[" #S "_pos], %[mask], %[" #S "_ring] bitop3:0x6a\n\t"                               \
  "v_lshlrev_b32 %[" #S "_j], 2, %[" #S "_next]\n\t"                                                                     \
  "ds_read_u16 %[" #S "_next], %[" #S "_at_next]\n\t"                                                                    \
  "s_mov_b64 exec, -1\n\t"
#define FPSCHED_TIMES_AHEAD(O) FPSCHED_AHEAD_SLOT(O, "2")
#define FPSCHED_LEFT(S)                                                                                                  \
  [S##_own] "+&v"(S.own_place), [S##_at_next] "+&v"(S.next_place), [S##_escape] "+&v"(S.escape), [S##_room] "+&v"(S.escape_room)
#define FPSCHED_TIMES_ROUNDS(TEXT)                                                                                       \
  asm volatile(FPSCHED_BEGIN("rounds") TEXT                                                                                        \
               : FPSCHED_STATE(even), FPSCHED_STATE(odd), [even_in] "=&v"(in_even), [odd_in] "=&v"(in_odd),             \
                 FPSCHED_LEFT(even), FPSCHED_LEFT(odd), [t] "=&v"(scratch), [start] "=&v"(start_time), [wait] "=&v"(waited), [far] "=&s"(long_waits) \
               : FPSCHED_PLACES(even), FPSCHED_PLACES(odd), FPSCHED_SHARED, [zero] "v"(0u), [most] "s"(0xffffffu)       \
               : "memory", "vcc", "scc")

// ... the forms with link occupancy and costs per micro-batch.  COST: how the op's cost and tag are added to its start; LEAVE: when
// the value leaves, over the link, and until when that keeps the link busy, in front of the other half's requests, whose row is on its
// way meanwhile; OWN: what else only the own device needs; SEND: the link's word, behind the request for the next row, which the
// device waits for; LINK_ROW: the next op's link row is fetched in front of its row.  With the slot, the other half's link word and cost
// are read ahead.  (All of the link's word in front of the slot / behind the other half's requests and in front of the own / as it is, the
// pass: 4,096 candidates of 4 x 32 x 2 73.2, 75.4 and 73.3 us, of 7 x 20 x 3 112.0, 115.6 and 112.2; 20,000 of 16 x 64 x 2 301, 290 and 286,
// 20,011 of 11 x 45 x 3 479, 462 and 455, with costs 541, 527 and 517.)
#define FPSCHED_COST_STEP(S, AHEAD, COST, LEAVE, OWN, SEND, REQUESTED, LINK_ROW)                                         \
  "s_waitcnt lgkmcnt(" REQUESTED ")\n\t"                                                                                 \
  "v_add_u32 %[" #S "_in], %[" #S "_in], " FPSCHED_##S##_X "\n\t"                                                        \
  "v_cmpx_eq_u32_sdwa %[" #S "_moved], %[" #S "_in], %[zero] src0_sel:BYTE_0 src1_sel:DWORD\n\t"                         \
  "v_max_u32 %[t], %[" #S "_free], %[" #S "_in]\n\t" COST LEAVE                                                          \
  "s_mov_b64 exec, -1\n\t" AHEAD                                                                                         \
  "s_mov_b64 exec, %[" #S "_moved]\n\t" OWN                                                                              \
  "v_lshrrev_b32 %[t], 11, %[" #S "_next]\n\t" LINK_ROW                                                                  \
  "v_mad_u32_u24 %[t], %[t], %[stride], %[" #S "_rows]\n\t"                                                              \
  "ds_read_b128 " FPSCHED_##S##_ROW ", %[t]\n\t" SEND                                                                    \
  FPSCHED_NEXT_WORD(S)
#define FPSCHED_COST_PLAIN(S) "v_add_u32 %[t], %[t], " FPSCHED_##S##_Y "\n\t"
#define FPSCHED_COST_TABLE(S)                                                                                            \
  "v_lshl_add_u32 %[t], %[" #S "_cost], 8, %[t]\n\t"                                                                     \
  "v_add_u32_sdwa %[t], %[t], " FPSCHED_##S##_Y " dst_sel:DWORD src0_sel:DWORD src1_sel:BYTE_0\n\t"
#define FPSCHED_COST_BUSY(S) "v_add_u32 %[" #S "_busy], %[" #S "_busy], %[" #S "_cost]\n\t"
#define FPSCHED_COST_FREE(S) "v_and_b32 %[" #S "_free], 0xffffff00, %[t]\n\t"
#define FPSCHED_LEAVE(S) "ds_write_b32 %[" #S "_at], %[t]\n\t"
#define FPSCHED_LEAVE_LINK(S)                                                                                            \
  "v_and_or_b32 %[u], " FPSCHED_##S##_Y ", %[byte], %[" #S "_sent]\n\t"                                                  \
  "v_max_u32 %[" #S "_in], %[t], %[u]\n\t"                                                                               \
  "ds_write_b32 %[" #S "_at], %[" #S "_in]\n\t" FPSCHED_COST_FREE(S)                                                     \
  "v_lshrrev_b32 %[" #S "_sent], 16, %[" #S "_link]\n\t"                                                                 \
  "v_and_b32 %[u], 0xffffff00, %[" #S "_in]\n\t"                                                                         \
  "v_lshl_add_u32 %[" #S "_sent], %[" #S "_sent], 8, %[u]\n\t"
#define FPSCHED_SEND_LINK(S) "ds_write_b32 %[" #S "_link_at], %[" #S "_sent]\n\t"
#define FPSCHED_LINK_ROW(S)                                                                                              \
  "v_mad_u32_u24 %[u], %[t], %[link_stride], %[" #S "_link_rows]\n\t"                                                   \
  "ds_read_b32 %[" #S "_link], %[u]\n\t"
#define FPSCHED_AHEAD_LINK(O)                                                                                            \
  "v_add_u32_sdwa %[" #O "_link_at], %[" #O "_links], %[" #O "_link] dst_sel:DWORD src0_sel:DWORD src1_sel:WORD_0\n\t"  \
  "ds_read_b32 %[" #O "_sent], %[" #O "_link_at]\n\t"
#define FPSCHED_AHEAD_COST(O, SHIFT, READ)                                                                               \
  "v_lshrrev_b32 %[" #O "_cost], 8, " FPSCHED_##O##_Y "\n\t"                                                            \
  "v_bfe_u32 %[u], %[" #O "_j], 2, 11\n\t"                                                                              \
  "v_lshl_add_u32 %[" #O "_cost], %[u], " SHIFT ", %[" #O "_cost]\n\t" READ " %[" #O "_cost], %[" #O "_cost]\n\t"
#define FPSCHED_LINKS_STEP(S, AHEAD) FPSCHED_COST_STEP(S, AHEAD, FPSCHED_COST_PLAIN(S), FPSCHED_LEAVE_LINK(S), "", FPSCHED_SEND_LINK(S), "4", FPSCHED_LINK_ROW(S))
#define FPSCHED_LINKS_AHEAD(O) FPSCHED_AHEAD_SLOT(O, "3") FPSCHED_AHEAD_LINK(O)
#define FPSCHED_MB_STEP(S, AHEAD) FPSCHED_COST_STEP(S, AHEAD, FPSCHED_COST_TABLE(S), FPSCHED_LEAVE(S), FPSCHED_COST_BUSY(S) FPSCHED_COST_FREE(S), "", "2", "")
#define FPSCHED_MB1_AHEAD(O) FPSCHED_AHEAD_SLOT(O, "2") FPSCHED_AHEAD_COST(O, "0", "ds_read_u8")
#define FPSCHED_MB2_AHEAD(O) FPSCHED_AHEAD_SLOT(O, "2") FPSCHED_AHEAD_COST(O, "1", "ds_read_u16")
#define FPSCHED_LINKS_MB_STEP(S, AHEAD) FPSCHED_COST_STEP(S, AHEAD, FPSCHED_COST_TABLE(S), FPSCHED_LEAVE_LINK(S), FPSCHED_COST_BUSY(S), FPSCHED_SEND_LINK(S), "4", FPSCHED_LINK_ROW(S))
#define FPSCHED_LINKS_MB1_AHEAD(O) FPSCHED_LINKS_AHEAD(O) FPSCHED_AHEAD_COST(O, "0", "ds_read_u8")
#define FPSCHED_LINKS_MB2_AHEAD(O) FPSCHED_LINKS_AHEAD(O) FPSCHED_AHEAD_COST(O, "1", "ds_read_u16")
#define FPSCHED_COST_STATE(S)                                                                                            \
  [S##_link] "+&v"(S.link), [S##_busy] "+&v"(S.busy), [S##_link_at] "=&v"(link_at_##S), [S##_sent] "=&v"(sent_##S),       \
  [S##_cost] "=&v"(cost_##S)
#define FPSCHED_COST_ROUNDS(TEXT)                                                                                        \
  asm volatile(FPSCHED_BEGIN("rounds") TEXT                                                                                        \
               : FPSCHED_STATE(even), FPSCHED_STATE(odd), [even_in] "=&v"(in_even), [odd_in] "=&v"(in_odd),             \
                 FPSCHED_COST_STATE(even), FPSCHED_COST_STATE(odd), [t] "=&v"(scratch), [u] "=&v"(scratch2)             \
               : FPSCHED_PLACES(even), FPSCHED_PLACES(odd), FPSCHED_SHARED, [zero] "v"(0u), [byte] "s"(0xffu),          \
                 [link_stride] "s"(4u * (unsigned)D), [even_link_rows] "v"(even.link_rows), [odd_link_rows] "v"(odd.link_rows), \
                 [even_links] "v"(even.links), [odd_links] "v"(odd.links)                                               \
               : "memory", "scc")

// ... and the form with times of two words (rows: latency; cost; mask; own tag, expected tag, slot's offset).
#define FPSCHED_WIDE_STEP(S, AHEAD)                                                                                      \
  "s_waitcnt lgkmcnt(2)\n\t"                                                                                            \
  "v_cmpx_eq_u32_sdwa %[" #S "_moved], " FPSCHED_##S##_TAG ", " FPSCHED_##S##_W " src0_sel:BYTE_0 src1_sel:BYTE_1\n\t"   \
  "v_add_u32 " FPSCHED_##S##_IN ", " FPSCHED_##S##_IN ", " FPSCHED_##S##_X "\n\t"                                       \
  "v_max_u32 %[" #S "_free], %[" #S "_free], " FPSCHED_##S##_IN "\n\t"                                                  \
  "v_add_u32 %[" #S "_free], %[" #S "_free], " FPSCHED_##S##_Y "\n\t"                                                   \
  "ds_write2_b32 %[" #S "_at], %[" #S "_free], " FPSCHED_##S##_W " offset1:1\n\t"                                       \
  "s_mov_b64 exec, -1\n\t" AHEAD                                                                                        \
  "s_mov_b64 exec, %[" #S "_moved]\n\t"                                                                                 \
  "v_lshrrev_b32 %[t], 11, %[" #S "_next]\n\t"                                                                          \
  "v_mad_u32_u24 %[t], %[t], %[stride], %[" #S "_rows]\n\t"                                                             \
  "v_or_b32 %[" #S "_pos], 0xfc, %[" #S "_pos]\n\t"                                                                     \
  "ds_read_b128 " FPSCHED_##S##_ROW ", %[t]\n\t"                                                                        \
  "v_add_u32 %[" #S "_pos], 2, %[" #S "_pos]\n\t"                                                                       \
  "v_bitop3_b32 %[t], %[" #S "_pos], %[mask], %[" #S "_ring] bitop3:0x6a\n\t"                                           \
  "v_lshlrev_b32 %[" #S "_j], 3, %[" #S "_next]\n\t"                                                                    \
  "ds_read_u16 %[" #S "_next], %[t]\n\t"                                                                                \
  "s_mov_b64 exec, -1\n\t"
#define FPSCHED_WIDE_AHEAD(O)                                                                                            \
  "s_waitcnt lgkmcnt(2)\n\t"                                                                                             \
  "v_and_b32 %[" #O "_at], %[" #O "_j], " FPSCHED_##O##_Z "\n\t"                                                        \
  "v_add_u32_sdwa %[" #O "_at], %[" #O "_at], " FPSCHED_##O##_W " dst_sel:DWORD src0_sel:DWORD src1_sel:WORD_1\n\t"     \
  "v_add_u32 %[" #O "_at], %[" #O "_at], %[slots]\n\t"                                                                  \
  "ds_read_b64 " FPSCHED_##O##_SLOT ", %[" #O "_at]\n\t"
#define FPSCHED_WIDE_ROUNDS(NAME, TEXT)                                                                                  \
  asm volatile(FPSCHED_BEGIN(NAME) TEXT                                                                                        \
               : FPSCHED_STATE(even), FPSCHED_STATE(odd), [t] "=&v"(scratch)                                            \
               : FPSCHED_PLACES(even), FPSCHED_PLACES(odd), FPSCHED_SHARED                                              \
               : "memory", "scc", "v48", "v49", "v50", "v51")

// ALONE: both passes in one launch, behind the order pass of the same candidates, no more of them than segments (1 + VBITS of that pass, or
// 0); for batches that leave the GPU one or two wavefronts per SIMD.  Such a batch takes as long as a candidate does: the start of a
// kernel, its tables and the first words of the rows, in both of two kernels, are a part of it that is not small, and a step waits less
// for LDS with fewer lanes in it, so the candidates are spread over all SIMDs (with four stages on a few devices over the compute units,
// run_list_evaluation).  Each wavefront walks the rows of its own candidates and
// then times them.  Two launches / this one: 1,024 candidates of 4 x 8 x 1 19.0 and 15.5 us, 4,096 18.2 and 16.8, 1,024 of 8 x 32 x 2 108.9
// and 101.3, of 16 x 64 x 2 162.4 and 155.2, 4,096 172.5 and 163.5, 2,048 of 24 x 30 x 2 100.0 and 90.2.
template <bool DEG2, bool WIDE, bool LINKS, int MB, bool SYNC, bool TIMES, int ALONE, int COPY>
__global__ __launch_bounds__(COPY ? kTimeCopyMaxThreads : (ALONE ? kAloneMaxThreads : kTimeMaxThreads)) __attribute__((amdgpu_waves_per_eu(COPY ? kTimeCopyWavesPerSimd : (ALONE ? 2 : 4)))) void time_lists_kernel(
    ListTables T, const uint16_t* __restrict__ ops, long long n_cand, int stride, long long* __restrict__ out_makespan,
    long long* __restrict__ out_idle, int* __restrict__ out_peak, unsigned char* __restrict__ out_flags,
    unsigned long long* __restrict__ next_candidate, int draw_block, unsigned draw_share, StartTimes starts) {
  static_assert(!WIDE || !(LINKS || MB || SYNC || COPY != 0), "these forms have times of 24 bits");
  static_assert(!COPY || (DEG2 && !LINKS && !MB && !SYNC && !TIMES), "rows that follow others");
  static_assert(!SYNC || (DEG2 && !LINKS && !MB), "rows that follow others");
  static_assert(!TIMES || !(DEG2 || WIDE || LINKS || MB || SYNC), "");
  constexpr unsigned kRowBytes = 16u;
  constexpr bool PLAIN = !WIDE && !LINKS && !MB && !COPY;   // (TIMES and SYNC too)
  constexpr bool STRAIGHT = PLAIN || !DEG2;   // the step without branches
  constexpr bool SPLIT = !WIDE && (!DEG2 || PLAIN || COPY);   // rows with the slot's mask and offset in a word each
  // pieces of a request.  (The 128-byte lines mostly do not stay in the L2 cache from one request to the next.)
  constexpr int kPieces = STRAIGHT ? 4 : 2;
  constexpr unsigned kSlotBytes = WIDE ? 8u : 4u;
  [[maybe_unused]] constexpr int kForm = (DEG2 ? 1 : 0) + (WIDE ? 2 : 0) + (LINKS ? 4 : 0) + 8 * MB + (SYNC ? 32 : 0) + (TIMES ? 64 : 0) + 128 * ALONE;
  extern __shared__ int32_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int D = T.D, cpw = T.cands_per_wave, P = (D + 1) >> 1;
  // LDS: [op windows of all wavefronts][rows][the tables behind them][per wavefront: link words, slots]
  const unsigned lds_from = ALONE ? (unsigned)alone_check_bytes(T, (int)(blockDim.x >> 6)) : 0u;
  const unsigned lds0 = lds_address(lds) + lds_from, tables = lds0 + (blockDim.x >> 6) * (unsigned)kTimeWindowBytes;
  const unsigned behind = tables + (unsigned)list_behind_rows(T);   // (of an offset in the image)
  // Rows with columns (fpsched_api.hip, timing_shape): a row read of sixteen bytes is served for sixteen lanes at a time, without bank
  // conflicts if these read sixteen different columns of 256 bytes, whatever kind and chunk each of them reads.  As dense as in the
  // image the rows of two candidates met in a bank at 16 devices, those of four at 8: 8 and 10 clocks a read instead of 4.7, in a pass
  // that LDS is busy in for 90 % of its time (whole evaluation: 262,144 candidates of 16 devices, 64 micro-batches, two chunks 2478 and
  // 2313 us; 65,536 of 8, 32 micro-batches 311 and 299 us).  On 32 devices the rows are the same columns; of two stages they take half as
  // much, which is a wavefront more for each compute unit where tables are large (the pass, 65,536 of 128 micro-batches: links 2.78 and 2.57
  // ms, costs 2.44 and 2.31, both 3.50 and 3.20; plain the same).
  const bool columns = T.odd_at != 16 * P;
  const int n_rows = T.row_bytes / 16, image_rows = kNKinds * kMaxChunks * D;
  for (int i = tid; i < n_rows; i += blockDim.x) {
    int from = i;
    if (columns) {
      const int row = (i >> 4) & 31, k = T.chunks <= 2 ? row >> 1 & 1 : i >> 9;
      from = (T.chunks <= 2 ? row & ~2 : row) * D + min(k * P + ((i & 15) & (P - 1)), D - 1);
    }
    lds_int4 R = reinterpret_cast<const lds_int4*>(T.ints)[from];
    if (MB != 0) R.y += (int)(behind << 8);   // (where the costs begin becomes an LDS address)
    lds_write<lds_int4>(tables + (unsigned)i * 16u, R);
  }
  for (int i = 4 * image_rows + tid; i < T.n_time_ints; i += blockDim.x) lds_write<int>(behind + (unsigned)i * 4u, T.ints[i]);
  if constexpr (ALONE != 0) {
    check_rows<ALONE - 1, false, false>(T, ops, n_cand * D, stride, cpw * D, out_idle, out_peak, nullptr, 0ull, 1, 0, (int)blockDim.x);
    __syncthreads();   // (what the rows' lanes have left in memory is read by the candidates')
  }
  const int seg = lane / P, pair = lane - seg * P;
  const bool lane_ok = seg < cpw;
  const int d0 = 2 * pair;
  const bool has_odd = d0 + 1 < D;
  const unsigned wave_at = behind + (unsigned)T.n_time_ints * 4u + (unsigned)wave * (unsigned)(T.wave_bytes - kTimeWindowBytes);
  const unsigned links_bytes = LINKS ? (unsigned)T.link_words * 512u : 0u;   // of the wavefront: [half][link][lane]
  unsigned slot_base = wave_at + links_bytes + (unsigned)(lane_ok ? seg : 0) * (unsigned)T.cand_slots * kSlotBytes;
  asm volatile("" : "+v"(slot_base));   // one register, not a sum to be re-associated every round
  const unsigned own_word = slot_base + (unsigned)(lane_ok ? d0 : 0) * kSlotBytes;
  const int own_at = (lane_ok ? d0 : 0) * (int)kSlotBytes;   // that word as a row's slot field
  const unsigned at_max = slot_base + ((unsigned)D + 1u) * kSlotBytes;
  auto clear_own = [&](unsigned at) {
    if (WIDE) lds_write<lds_int2>(at, lds_int2{0, (int)kOwnTag});
    else lds_write<uint32_t>(at, kOwnTag);
  };
  clear_own(own_word);   // what a lane without an op looks at
  __syncthreads();

  // segment bookkeeping on the scalar unit: bit seg * P stands for segment seg
  unsigned long long base_bits = 0ull;
  for (int s = 0; s < cpw; ++s) base_bits |= 1ull << (s * P);
  const unsigned long long high_bits = base_bits << (P - 1);
  const unsigned long long seg_lanes = ((1ull << P) - 1ull) << (seg * P & 63);   // (P <= 32)
  const unsigned seg_lo = (unsigned)seg_lanes, seg_hi = (unsigned)(seg_lanes >> 32);
  auto any_in_segment = [&](unsigned long long ballot) -> bool {
    return (((unsigned)ballot & seg_lo) | ((unsigned)(ballot >> 32) & seg_hi)) != 0u;
  };

  const unsigned row_stride = (unsigned)T.row_step;
  const unsigned stride2 = (unsigned)stride * 2u, stride_pos = position_of((unsigned)stride);

  // (a transfer more may have its memory event to come than may be unfinished: of equal times the compute event is first)
  constexpr int kTransfers = COPY ? COPY : 1, kEvents = COPY ? COPY + 1 : 1;
  // one device of the lane: its op window, and the op under its cursor, decoded.  A device without an op looks at its
  // own word with an L that keeps it waiting.
  struct Device {
    unsigned win, meta;
    unsigned free_at;       // narrow: << 8
    unsigned j_slot, w_next;   // the word under the cursor times the bytes of a slot, and the word behind it
    lds_int4 R;             // the op's table row: L, dur | tag, slot, second edge
    unsigned loaded;    // position up to which the row has been in the ring (kNoList: no list, or all of it)
    unsigned asked;     // ... up to which it has been requested
    unsigned pos;       // position of w_next; the device has issued one op less than words in front of it
    unsigned info;      // what the order pass left for this row: kRow* | stop
    unsigned busy;
    unsigned link_rows, links;   // LINKS: where its devices' link rows are, the lane's link words
    // COPY: the copy timeline, the last COPY transfers: finish << 8 and key (a reload's word without its kind, else all ones),
    // newest first (0: none); the memory events that the walk has not passed, oldest first, time << 8 | units (all ones: none),
    // with a bit each for those that allocate
    unsigned copy_end[kTransfers], copy_key[kTransfers], event[kEvents], event_adds, n_events;
    int mem, pk, cap;
    unsigned taken;              // SYNC: values of its group's item taken in
    unsigned link;               // the op's link row: byte offset of the link word, latency << 16
    unsigned own_place, next_place;   // TIMES: places in the ring of the words under and behind the cursor
    uint32_t* escape;                 // TIMES: next entry of the row's escape list
    int escape_room;                  // TIMES: ... and how many it has room for, one for its end aside
    uint4 pend[kPieces];   // what has been requested and is not in the ring, in order
  };
  Device even, odd;
  auto idle_device = [&](Device& x) {
    x.R = WIDE ? (STRAIGHT ? lds_int4{0, 0, 0, own_at << 16 | (int)kWideNever} : lds_int4{0, 0, own_at, (int)kWideNever}) : (SPLIT ? lds_int4{1, 0, 0, own_at} : lds_int4{1, 0, own_at, 0});
    x.link = 0u;
    x.taken = 0u;
    x.loaded = kNoList;
    x.asked = 0u;
    x.pos = position_of(1u);
    x.info = 0u;
  };
  auto no_transfers = [&](Device& x) {
#pragma unroll
    for (int i = 0; i < kTransfers; ++i) { x.copy_end[i] = 0u; x.copy_key[i] = ~0u; }
#pragma unroll
    for (int i = 0; i < kEvents; ++i) x.event[i] = ~0u;
    x.event_adds = 0u; x.n_events = 0u; x.mem = 0; x.pk = 0;
  };
  auto set_up = [&](Device& x, int k) {
    x.win = lds0 + (unsigned)wave * (unsigned)kTimeWindowBytes + (unsigned)k * kWindowBytes + (unsigned)lane * 4u;
    x.meta = tables + (unsigned)(k * T.odd_at) + (unsigned)(columns ? lane & 15 : pair) * kRowBytes;
    x.link_rows = LINKS ? behind + (unsigned)T.off_links * 4u + (unsigned)(k * P + pair) * 4u : 0u;
    x.links = LINKS ? wave_at + (unsigned)k * (links_bytes / 2u) + (unsigned)lane * 4u : 0u;
    x.free_at = 0u; x.j_slot = 0u; x.w_next = 0u; x.busy = 0u;
    x.cap = COPY && (k == 0 || has_odd) && lane_ok ? T.ints[T.off_dev + 2 * (d0 + k) + 1] : 0x7fffffff;
    no_transfers(x);
    x.own_place = x.win; x.next_place = x.win; x.escape = starts.escapes; x.escape_room = 0;
    for (int i = 0; i < kPieces; ++i) x.pend[i] = make_uint4(0u, 0u, 0u, 0u);
    idle_device(x);
  };
  set_up(even, 0);
  set_up(odd, 1);

  long long cand = 0;
  uint32_t* start_row = starts.low;   // TIMES: of the even device
  const char* row = reinterpret_cast<const char*>(ops);   // of the even device; the odd one's follows it
  bool running = false, fresh = true, priming = false;
  bool any_special = true;          // wave-uniform: some segment starts, or has just started, a candidate
  bool any_stuck = false;           // wave-uniform: some device's list stops at a word that is not to be looked at
  unsigned long long idle_lanes = ~0ull;
  bool first_draw = true;
  // Drawn from the counter and not handed to a segment: [pool_next, pool_end); behind a draw that reached past the last candidate
  // pool_end is there too, and nothing is drawn any more.  (Where there are no more candidates than segments nothing is ever drawn,
  // and a segment that ends changes nothing for the others: a draw that comes back empty costs the wavefront some 4,500 clocks, which
  // were 8 to 13 % of the pass on such batches.)
  // Drawn at a time: draw_share / 2^32 of the candidates that were left at this wavefront's last draw, up to one a segment, and
  // draw_block at least.  All of it is worked out on the scalar unit: the SYNC form has no vector register left (with what every
  // lane agrees on in vector registers it kept four in memory; 65,536 candidates of 12 devices, the whole evaluation: 850 and 837 us).
  unsigned long long pool_next = (unsigned long long)gridDim.x * (blockDim.x >> 6) * (unsigned)cpw, pool_end = pool_next;

  // fetch the row of the word that comes under the cursor; what follows from the row is worked out when the device's
  // next step begins, so that the other half's step covers the wait for it
  auto decode = [&](Device& x, unsigned word) {
    const unsigned at = __umul24(word >> 11, row_stride) + x.meta;
    x.j_slot = word * kSlotBytes;
    x.R = lds_read<lds_int4>(at);
    if (LINKS) x.link = lds_read<unsigned>(__umul24(word >> 11, 4u * (unsigned)D) + x.link_rows);
  };
  // address of a position in the device's ring (the windows of a wavefront begin at a multiple of their size)
  auto in_ring = [&](const Device& x, unsigned pos) -> unsigned {
    return __builtin_amdgcn_bitop3_b32(pos, kPosMask, x.win, 0x6a);   // (pos & mask) ^ win
  };
  auto store_piece = [&](Device& x) {
    const unsigned at = in_ring(x, x.loaded);
    lds_write<uint32_t>(at, x.pend[0].x);
    lds_write<uint32_t>(at + 256u, x.pend[0].y);
    lds_write<uint32_t>(at + 512u, x.pend[0].z);
    lds_write<uint32_t>(at + 768u, x.pend[0].w);
#pragma unroll
    for (int i = 1; i < kPieces; ++i) x.pend[i - 1] = x.pend[i];
  };
  auto request = [&](Device& x, const char* from, unsigned pos) {
    const unsigned at2 = pos >> 6;   // (a piece begins with a dword)
    const uint4* piece = reinterpret_cast<const uint4*>(from + at2);
    x.asked = pos + (unsigned)kPieces * kPiece;
    if ((stride2 & (16u * kPieces - 1u)) == 0u) {
#pragma unroll
      for (int i = 0; i < kPieces; ++i) x.pend[i] = piece[i];
    } else {
#pragma unroll
      for (int i = 0; i < kPieces; ++i)
        if (at2 + 16u * (unsigned)i < stride2) x.pend[i] = piece[i];
    }
  };
  // TIMES: the start times of the eight ops from a position on, whose words' places in the ring they have taken
  auto leave_starts = [&](const Device& x, unsigned pos, int odd_device) {
    const unsigned at = in_ring(x, pos);
    const uint4 eight = make_uint4(lds_read<uint32_t>(at), lds_read<uint32_t>(at + 256u), lds_read<uint32_t>(at + 512u), lds_read<uint32_t>(at + 768u));
    *reinterpret_cast<uint4*>(start_row + (size_t)(pos >> 10) * (unsigned)starts.lanes * 4u + odd_device * 4) = eight;
  };
  // land what has been asked for, where at most seven words are unread
  // (TIMES: where all ops whose places are taken have issued, which is at most six unread: the word behind the cursor may
  // have been read too early and is read again.  Behind a full row comes a piece of nothing but the END word.)
  auto land = [&](Device& x, int odd_device) {
    if constexpr (TIMES) {
      if ((int)(x.loaded - (x.pos & ~kPosBetween)) <= (int)kPiece - 2 && (x.loaded != x.asked || x.loaded == stride_pos)) {
        if (x.loaded >= 2u * kPiece) leave_starts(x, x.loaded - 2u * kPiece, odd_device);
        if (x.loaded < stride_pos) {
          store_piece(x);
          if (any_stuck) {
            const unsigned stop = position_of(x.info & kRowStop);
            if (stop - x.loaded < kPiece) lds_write<uint16_t>(in_ring(x, stop), (uint16_t)0);
          }
          x.loaded += kPiece;
        } else {
          lds_write<uint16_t>(in_ring(x, stride_pos), (uint16_t)0);
          x.loaded = kNoList;
        }
        x.w_next = lds_read<uint16_t>(in_ring(x, x.pos));
      }
    } else if ((int)(x.loaded - x.pos) <= (int)kPiece && x.loaded != x.asked) {
      store_piece(x);
      // the device goes no further than where the order pass says its list stops (an END word does that by itself)
      if (any_stuck) {
        const unsigned stop = position_of(x.info & kRowStop);
        if (stop - x.loaded < kPiece) lds_write<uint16_t>(in_ring(x, stop), (uint16_t)0);
      }
      x.loaded += kPiece;
      // a row that fills its stride has no END word: plant one behind it
      if (x.loaded >= stride_pos) {
        lds_write<uint16_t>(in_ring(x, stride_pos), (uint16_t)0);
        x.loaded = kNoList;
      }
    }
  };
  auto ask = [&](Device& x, const char* from) {
    if (x.loaded == x.asked && (!TIMES || x.loaded < stride_pos)) request(x, from, x.loaded);
  };
  // the head of the row has arrived: the device joins in
  auto join = [&](Device& x, int odd_device) {
    x.loaded = 0u;
    store_piece(x);
    x.loaded = kPiece;
    if (stride_pos > kPiece) {
      store_piece(x);
      x.loaded = 2u * kPiece;
    }
    const unsigned stop = x.info & kRowStop, stop_pos = position_of(stop);
    const unsigned w = stop == 0u ? 0u : lds_read<uint16_t>(in_ring(x, 0u));
    x.w_next = stop <= 1u ? 0u : lds_read<uint16_t>(in_ring(x, position_of(1u)));
    if (TIMES ? stop_pos < x.loaded : stop_pos <= x.loaded) lds_write<uint16_t>(in_ring(x, stop_pos), (uint16_t)0);   // (behind a full row of one or two pieces too)
    if (!TIMES && x.loaded >= stride_pos) x.loaded = kNoList;
    if (TIMES) {
      x.own_place = in_ring(x, 0u);
      x.next_place = in_ring(x, position_of(1u));
      x.escape = starts.escapes + ((size_t)cand * D + d0 + odd_device) * (size_t)starts.escape_cap;
      x.escape_room = starts.escape_cap - 1;
    }
    decode(x, w);
    x.pos = position_of(1u);
  };
  // where the second row of an op with a second input or output is
  auto second_row = [&](int w) -> unsigned {
    return behind + (WIDE ? ((unsigned)w >> 12) & 0xfff0u : (unsigned)w & 0xffffu);
  };
  // one step of one half of the devices with second edges in the wide form and under link occupancy or costs per
  // micro-batch; returns the lanes that issued
  auto step = [&](Device& x) -> unsigned long long {
    asm volatile("" : "+v"(x.R), "+v"(x.j_slot));   // (the row stays one value until here: no earlier wait for it)
    const unsigned j_slot = x.j_slot;
    const unsigned at_slot = (j_slot & ((unsigned)x.R.z >> 16)) + (slot_base + ((unsigned)x.R.z & 0xffffu));
    unsigned ready, cost_tag = (unsigned)x.R.y, link_free = 0u;
    unsigned long long moved;
    unsigned cost = 0u;
    if (MB) {
      // (a row without a cost table reads some word of LDS and does not issue)
      const unsigned at = (cost_tag >> 8) + (((x.j_slot >> 2) & 0x7ffu) << (MB - 1));
      cost = MB == 1 ? lds_read<uint8_t>(at) : lds_read<uint16_t>(at);
      cost_tag = cost << 8 | (cost_tag & 0xffu);
    }
    // (the second row comes with the slot: read where it is needed, some lane of a wavefront waits for it in most steps)
    const lds_int4 second_r = lds_read<lds_int4>(second_row(x.R.w));
    if (LINKS) link_free = lds_read<unsigned>(x.links + (x.link & 0xffffu));
    if (WIDE) {
      // the slot's second word is the tag, the row's last one the expected tag (byte 1) and the op's own (byte 0)
      const lds_int2 in = lds_read<lds_int2>(at_slot);
      ready = (unsigned)in.x + (unsigned)x.R.x;
      asm volatile("v_cmp_eq_u32_sdwa %0, %1, %2 src0_sel:DWORD src1_sel:BYTE_1" : "=s"(moved) : "v"(in.y), "v"(x.R.w));
    } else {
      ready = lds_read<uint32_t>(at_slot) + (unsigned)x.R.x;
      const unsigned zero = 0u;
      asm volatile("v_cmp_eq_u32_sdwa %0, %1, %2 src0_sel:BYTE_0 src1_sel:DWORD" : "=s"(moved) : "v"(ready), "v"(zero));
    }
    // an op with two inputs waits for its second one first: once that is there the device's free time takes it in
    // (nothing but the start of this op looks at that time) and the op waits for its first
    unsigned long long issue = moved;
    const unsigned long long absorb = issue & __ballot(x.R.w < 0);
    if (absorb != 0ull) {
      if (__builtin_amdgcn_inverse_ballot_w64(absorb)) {
        x.free_at = max(x.free_at, ready);
        x.R.x = second_r.x;
        x.R.z = second_r.y;
        x.R.w = WIDE ? (x.R.w & 0x7fff00ff) | second_r.w : x.R.w & 0x7fffffff;
      }
      issue &= ~absorb;
    }
    if (__builtin_amdgcn_inverse_ballot_w64(issue)) {
      unsigned val = max(x.free_at, ready) + cost_tag;
      x.free_at = WIDE ? val : val & 0xffffff00u;
      if (MB) x.busy += cost;
      if (LINKS) {
        // (the tag stays in the low byte, which the link words do not have)
        const unsigned leaves = max(val, link_free | (cost_tag & 0xffu));
        lds_write<unsigned>(x.links + (x.link & 0xffffu), (leaves & 0xffffff00u) + (x.link >> 16 << 8));
        val = leaves;
      }
      auto leave = [&](unsigned at) {
        if (WIDE) lds_write<lds_int2>(at, lds_int2{(int)val, x.R.w & 0xff});
        else lds_write<uint32_t>(at, val);
      };
      leave(at_slot);
      if (((unsigned)x.R.w & kRowTwoOut) != 0u) {
        const unsigned second = (unsigned)second_r.z;
        if (LINKS) {
          const unsigned link = (unsigned)second_r.w;
          val = max(x.free_at, lds_read<unsigned>(x.links + (link & 0xffffu))) | (cost_tag & 0xffu);
          lds_write<unsigned>(x.links + (link & 0xffffu), (val & 0xffffff00u) + (link >> 16 << 8));
        }
        leave((j_slot & (second >> 16)) + slot_base + (second & 0xffffu));
      }
      decode(x, x.w_next);
      x.pos = (x.pos | kPosBetween) + 2u;
      x.w_next = lds_read<uint16_t>(in_ring(x, x.pos));
    }
    return moved;
  };
  // COPY: the memory events in front of a time are summed up, and `units` that come in at an earlier time among them
  auto pass_events = [&](Device& x, unsigned until, unsigned from, int units) {
    while (x.event[0] < until) {
      const int now = x.event[0] >= from ? units : 0, change = (int)(x.event[0] & 0xffu);
      units -= now;
      x.mem += now;
      x.pk = max(x.pk, x.mem);
      x.mem += (x.event_adds & 1u) != 0u ? change : -change;
      x.pk = max(x.pk, x.mem);
#pragma unroll
      for (int i = 0; i + 1 < kEvents; ++i) x.event[i] = x.event[i + 1];
      x.event[kEvents - 1] = ~0u;
      x.event_adds >>= 1;
      --x.n_events;
    }
    x.mem += units;
    x.pk = max(x.pk, x.mem);
  };
  auto copy_step = [&](Device& x) -> unsigned long long {
    const unsigned offset = (unsigned)x.R.w;
    const unsigned at_slot = (x.j_slot & (unsigned)x.R.z) + ((offset & 0xffffu) + slot_base);
    const unsigned ready = lds_read<uint32_t>(at_slot) + (unsigned)x.R.x;
    Lanes moved;
    const unsigned zero = 0u;
    asm volatile("v_cmp_eq_u32_sdwa %0, %1, %2 src0_sel:BYTE_0 src1_sel:DWORD" : "=s"(moved) : "v"(ready), "v"(zero));
    const unsigned kind = x.j_slot >> 15, key = __builtin_amdgcn_ubfe(x.j_slot, 2u, 13u);
    const Lanes transfers = moved & lanes(kind - (unsigned)kO < 2u), computes = moved & ~transfers;
    unsigned start = max(x.free_at, ready);
    // a B item waits for the reload of its activation, which may still run if it is among the last transfers (one copy_depth or
    // more back has finished before the device got here, so a match there changes nothing)
    const Lanes reloaded = computes & lanes(kind == (unsigned)kB) & lanes(x.copy_end[0] > start);
    if (reloaded != 0ull) {
#pragma unroll
      for (int i = 0; i < kTransfers; ++i)
        start = in(reloaded & lanes(x.copy_key[i] == key)) ? max(start, x.copy_end[i]) : start;
    }
    // a transfer is handed over when the engine is done with the one copy_depth transfers back
    if (transfers != 0ull) {
      unsigned gate = x.copy_end[0];
#pragma unroll
      for (int i = 1; i < kTransfers; ++i) gate = T.copy_depth > i ? x.copy_end[i] : gate;
      start = in(transfers) ? max(start, gate) : start;
    }
    unsigned val;
    asm volatile("s_mov_b64 exec, %[computes]\n\t"
                 "v_add_u32 %[val], %[start], %[cost]\n\t"
                 "ds_write_b32 %[at], %[val]\n\t"
                 "v_and_b32 %[free], 0xffffff00, %[val]\n\t"
                 "s_mov_b64 exec, %[transfers]\n\t"
                 "v_mov_b32 %[free], %[start]\n\t"
                 "s_mov_b64 exec, -1"
                 : [val] "=&v"(val), [free] "+&v"(x.free_at)
                 : [start] "v"(start), [cost] "v"(x.R.y), [at] "v"(at_slot), [computes] "s"(computes), [transfers] "s"(transfers)
                 : "memory");
    // the memory in front of the op's start and up to its end, with the op's own
    const Lanes passes = moved & lanes(x.event[0] < x.free_at);
    if (in(passes)) pass_events(x, x.free_at, start, in(computes) ? (int)__builtin_amdgcn_ubfe(offset, 16u, 8u) : 0);
    asm volatile("s_mov_b64 exec, %[alone]\n\t"
                 "v_add_u32_sdwa %[mem], %[mem], %[units] dst_sel:DWORD src0_sel:DWORD src1_sel:BYTE_2\n\t"
                 "v_max_i32 %[pk], %[pk], %[mem]\n\t"
                 "s_mov_b64 exec, %[computes]\n\t"
                 "v_sub_u32_sdwa %[mem], %[mem], %[units] dst_sel:DWORD src0_sel:DWORD src1_sel:BYTE_3\n\t"
                 "s_mov_b64 exec, -1"
                 : [mem] "+&v"(x.mem), [pk] "+&v"(x.pk)
                 : [units] "v"(offset), [alone] "s"(computes & ~passes), [computes] "s"(computes));
    if (in(transfers)) {
      // a reload allocates when it starts, an offload releases when it ends
      const bool reload = kind == (unsigned)kL;
      const unsigned begin = max(start, x.copy_end[0]), end = begin + ((unsigned)x.R.y & 0xffffff00u);
      const unsigned event = reload ? begin | __builtin_amdgcn_ubfe(offset, 16u, 8u) : end | offset >> 24;
#pragma unroll
      for (int i = kTransfers - 1; i > 0; --i) { x.copy_end[i] = x.copy_end[i - 1]; x.copy_key[i] = x.copy_key[i - 1]; }
      x.copy_end[0] = end;
      x.copy_key[0] = reload ? key : ~0u;
#pragma unroll
      for (int i = 0; i < kEvents; ++i) x.event[i] = x.n_events == (unsigned)i ? event : x.event[i];
      x.event_adds |= (reload ? 1u : 0u) << x.n_events;
      ++x.n_events;
    }
    const Lanes followed = moved & lanes((unsigned)x.R.z > 0x3ffffu);
    if (in(moved & ~followed)) {
      decode(x, x.w_next);
      x.pos = (x.pos | kPosBetween) + 2u;
      x.w_next = lds_read<uint16_t>(in_ring(x, x.pos));
    }
    if (in(followed)) x.R = lds_read<lds_int4>(behind + ((unsigned)x.R.z >> 14 & ~15u));
    return moved;
  };
  // SYNC, every fourth round: the devices at an item of a group of micro-batches (their rows never issue and name another
  // one, then one of the second edge) take in what has arrived of the values it waits for, up to four at a time; with the last one the
  // item runs, and leaves its value in the slots of its micro-batches.  Returns the lanes that took in a value or issued.
  // (stepped: the lanes that have issued in this round, which do not again: the ring has words for one op a round)
  auto groups = [&](Device& x, unsigned long long stepped) -> unsigned long long {
    const unsigned long long at_group = __ballot(x.R.y == kGroupRow) & ~stepped;
    if (at_group == 0ull) return 0ull;
    unsigned long long moved = 0ull;
    if (__builtin_amdgcn_inverse_ballot_w64(at_group)) {
      const unsigned at = behind + ((unsigned)x.R.z >> 14);
      const lds_int4 first = lds_read<lds_int4>(at), second = lds_read<lds_int4>(at + 16u);
      const unsigned n = (unsigned)first.z & 0xffffu;
      const unsigned first_j = __umul24((x.j_slot >> 2) & 0x7ffu, n), n_slots = min(n, (unsigned)T.m - first_j);
      const unsigned first_at = slot_base + (unsigned)first.w + (first_j << 2), second_at = slot_base + (unsigned)second.w + (first_j << 2);
      const unsigned of_first = ((unsigned)first.z & kGroupIn) != 0u ? n_slots : 0u, of_second = ((unsigned)second.z & kGroupIn) != 0u ? n_slots : 0u;
      // (up to four values of one edge at a time)
      const bool at_first = x.taken < of_first;
      const unsigned done = at_first ? x.taken : x.taken - of_first, left = (at_first ? of_first : of_second) - done;
      const unsigned from = (at_first ? first_at : second_at) + (done << 2), wait = (unsigned)(at_first ? first.x : second.x);
      unsigned value[4];
#pragma unroll
      for (unsigned k = 0; k < 4; ++k) value[k] = lds_read<unsigned>(from + (k < left ? k << 2 : 0u));
      bool there = true;
      unsigned got = 0u;
#pragma unroll
      for (unsigned k = 0; k < 4; ++k) {
        const unsigned ready = value[k] + wait;
        there = there && k < left && (ready & 0xffu) == 0u;
        x.free_at = there ? max(x.free_at, ready) : x.free_at;
        got += there ? 1u : 0u;
      }
      x.taken += got;
      const bool issue = x.taken == of_first + of_second;
      moved = __ballot(issue || got != 0u);
      if (issue) {
        const unsigned val = x.free_at + (unsigned)first.y;
        x.free_at = val & 0xffffff00u;
        for (unsigned k = 0; k < n_slots; ++k) {
          lds_write<unsigned>(first_at + (k << 2), val);
          if (((unsigned)second.z & kGroupOut) != 0u) lds_write<unsigned>(second_at + (k << 2), val);
        }
        x.taken = 0u;
        decode(x, x.w_next);
        x.pos = (x.pos | kPosBetween) + 2u;
        x.w_next = lds_read<uint16_t>(in_ring(x, x.pos));
      }
    }
    return __shfl(moved, __ffsll((long long)at_group) - 1);
  };

  // Every candidate ends after at most 3 D * stride + 2 rounds (each round but its last issues at least one of its at
  // most D * stride ops, takes in the second input of one or leaves the second output), so the bound below is never reached;
  // it only makes sure the wavefront leaves the loop whatever happens.
  // (SYNC: an op takes in at most 2 m values, in every fourth round)
  const unsigned long long bound = (3ull * (unsigned)D * (unsigned)stride * (SYNC ? 4ull * (unsigned)T.m : 1ull) + 16ull) * ((unsigned long long)n_cand + 1ull);
  const unsigned max_rounds = bound > 0xfffffff0ull ? 0xfffffff0u : (unsigned)bound;
  if constexpr (ALONE != 0) FPSCHED_PLACE_ROUNDS("alone", 0);
  else if constexpr (STRAIGHT) FPSCHED_PLACE_ROUNDS("rounds", SYNC ? 16 : 0);
  for (unsigned round = 0; round < max_rounds; round += kRounds) {
    // (vmcnt(0): the requests of the last top-up.  Waited for behind the first start times that leave, they would take these
    // stores with them, which have only just been issued.)
    if constexpr (TIMES) __builtin_amdgcn_s_waitcnt(0x0f70);
    land(even, 0);
    land(odd, 1);
    // ---- the rare part, only when some segment starts or has just started a candidate
    if (any_special) {
      // segments restarted at the previous top-up: the heads of their rows have arrived, they join in and ask for
      // their second pieces like any other, below
      if (priming) {
        join(even, 0);
        if (has_odd) join(odd, 1);
      }
      any_stuck = __ballot(running && ((even.info | odd.info) & (kRowStuck | kRowPlant)) != 0u) != 0ull;
      priming = false;
      // hand the segments that ask for one (lane 0 of each speaks for it) their next candidate
      const unsigned long long want = __ballot(fresh && !first_draw && pair == 0 && lane_ok);
      unsigned long long from_pool = 0ull;
      if (want != 0ull) {
        const int n_want = __popcll(want), have = (int)(pool_end - pool_next), lacking = n_want - have;
        const int rank = __popcll(want & ((1ull << lane) - 1ull));   // among the asking segments
        if (lacking > 0 && pool_end < (unsigned long long)n_cand) {
          const unsigned left = (unsigned)min((unsigned long long)n_cand - pool_end, 0xffffffffull);
          const int amount = max(max(draw_block, lacking), min((int)__umulhi(left, draw_share), cpw));
          unsigned long long base = 0ull;
          if (lane == 0) base = atomicAdd(next_candidate, (unsigned long long)amount);
          base = (unsigned long long)of_first_lane((long long)base);
          from_pool = (rank < have ? pool_next : base - (unsigned)have) + (unsigned)rank;
          pool_next = base + (unsigned)lacking;
          pool_end = base + (unsigned)amount;
        } else {
          from_pool = rank < have ? pool_next + (unsigned)rank : (unsigned long long)n_cand;
          pool_next += (unsigned)min(n_want, have);
        }
      }
      if (fresh) {
        fresh = false;
        unsigned long long drawn = ((unsigned long long)blockIdx.x * (blockDim.x >> 6) + wave) * cpw + seg;
        if (!first_draw) drawn = __shfl(from_pool, lane_ok ? seg * P : 0, 64);
        first_draw = false;
        cand = (long long)drawn;
        running = lane_ok && cand < n_cand;
        priming = running;
        even.free_at = 0u;
        odd.free_at = 0u;
        if (running) {
          const int n4 = T.cand_slots * (int)kSlotBytes / 16, unused = WIDE ? 0 : (int)kEmptySlot;
          for (int i = pair; i < n4; i += P)
            lds_write<lds_int4>(slot_base + (unsigned)i * 16u, lds_int4{unused, (int)kEmptySlot, unused, (int)kEmptySlot});
          clear_own(own_word);
          if (has_odd) clear_own(own_word + kSlotBytes);
          if (pair == 0) lds_write<uint32_t>(at_max, 0u);
          if (COPY) { no_transfers(even); no_transfers(odd); }
          if (LINKS)
            for (unsigned i = 0; i < links_bytes / 2u; i += 256u) { lds_write<unsigned>(even.links + i, 0u); lds_write<unsigned>(odd.links + i, 0u); }
          const long long r = cand * D + d0;
          row = reinterpret_cast<const char*>(ops + (size_t)r * (size_t)stride);
          if (TIMES) start_row = starts.low + (size_t)cand * ((size_t)stride >> 1) * (unsigned)starts.lanes + (unsigned)d0 * 4u;
          request(even, row, 0u);
          const unsigned long long left = (unsigned long long)out_idle[r];
          even.info = (unsigned)(left >> 32);
          even.busy = (unsigned)left;
          if (has_odd) {
            request(odd, row + stride2, 0u);
            const unsigned long long left_odd = (unsigned long long)out_idle[r + 1];
            odd.info = (unsigned)(left_odd >> 32);
            odd.busy = (unsigned)left_odd;
          }
        }
      }
      // segments that are priming do not count as running yet (nothing can move in them)
      const unsigned long long all_running = __ballot(running);
      const unsigned long long primers = __ballot(priming);
      idle_lanes = ~(all_running & ~primers);
      any_special = primers != 0ull;
      if (all_running == 0ull) break;   // every segment of the wave is out of work
    }
    ask(even, row);
    ask(odd, row + stride2);
    if (ALONE != 0 && idle_lanes == ~0ull) continue;   // (the first words of all its candidates are on their way)
    unsigned long long moved_even = 0ull, moved_odd = 0ull;
    if constexpr (STRAIGHT) {
      [[maybe_unused]] unsigned in_even, in_odd, at_even, at_odd, scratch, scratch2, start_time, waited;
      [[maybe_unused]] unsigned long long long_waits;
      [[maybe_unused]] unsigned link_at_even, link_at_odd, sent_even, sent_odd, cost_even, cost_odd;
      if constexpr (SYNC) {
#pragma unroll
        for (unsigned sub = 0; sub < kRounds; sub += 4u) {
          FPSCHED_ROUNDS("rounds", FPSCHED_FOUR_ROUNDS(FPSCHED_FOLLOW_STEP, FPSCHED_PLAIN_AHEAD));
          moved_even |= groups(even, moved_even);
          moved_odd |= groups(odd, moved_odd);
        }
      } else if constexpr (TIMES) {
        FPSCHED_TIMES_ROUNDS(FPSCHED_EIGHT_ROUNDS(FPSCHED_TIMES_STEP, FPSCHED_TIMES_AHEAD));
      } else if constexpr (WIDE) {
        if constexpr (ALONE != 0) FPSCHED_WIDE_ROUNDS("alone", FPSCHED_EIGHT_ROUNDS(FPSCHED_WIDE_STEP, FPSCHED_WIDE_AHEAD));
        else FPSCHED_WIDE_ROUNDS("rounds", FPSCHED_EIGHT_ROUNDS(FPSCHED_WIDE_STEP, FPSCHED_WIDE_AHEAD));
      } else if constexpr (LINKS && MB == 0) {
        FPSCHED_COST_ROUNDS(FPSCHED_EIGHT_ROUNDS(FPSCHED_LINKS_STEP, FPSCHED_LINKS_AHEAD));
      } else if constexpr (LINKS && MB == 1) {
        FPSCHED_COST_ROUNDS(FPSCHED_EIGHT_ROUNDS(FPSCHED_LINKS_MB_STEP, FPSCHED_LINKS_MB1_AHEAD));
      } else if constexpr (LINKS) {
        FPSCHED_COST_ROUNDS(FPSCHED_EIGHT_ROUNDS(FPSCHED_LINKS_MB_STEP, FPSCHED_LINKS_MB2_AHEAD));
      } else if constexpr (MB == 1) {
        FPSCHED_COST_ROUNDS(FPSCHED_EIGHT_ROUNDS(FPSCHED_MB_STEP, FPSCHED_MB1_AHEAD));
      } else if constexpr (MB == 2) {
        FPSCHED_COST_ROUNDS(FPSCHED_EIGHT_ROUNDS(FPSCHED_MB_STEP, FPSCHED_MB2_AHEAD));
      } else if constexpr (DEG2) {
        if constexpr (ALONE != 0) FPSCHED_ROUNDS("alone", FPSCHED_EIGHT_ROUNDS(FPSCHED_FOLLOW_STEP, FPSCHED_PLAIN_AHEAD));
        else FPSCHED_ROUNDS("rounds", FPSCHED_EIGHT_ROUNDS(FPSCHED_FOLLOW_STEP, FPSCHED_PLAIN_AHEAD));
      } else {
        if constexpr (ALONE != 0) FPSCHED_ROUNDS("alone", FPSCHED_EIGHT_ROUNDS(FPSCHED_PLAIN_STEP, FPSCHED_PLAIN_AHEAD));
        else FPSCHED_ROUNDS("rounds", FPSCHED_EIGHT_ROUNDS(FPSCHED_PLAIN_STEP, FPSCHED_PLAIN_AHEAD));
      }
    } else {
#pragma unroll
      for (unsigned sub = 0; sub < kRounds; ++sub) {
        moved_even = COPY ? copy_step(even) : step(even);
        moved_odd = COPY ? copy_step(odd) : step(odd);
      }
    }
    // A segment none of whose lanes issued is finished, and stays so: nothing it reads changes any more.  It could
    // only be restarted at the next top-up anyway, so only the last round in front of it looks.  Cheap scalar
    // pre-test: does the issue mask, with the lanes of idle segments set, contain an all-zero field of P bits?
    // (x - lows) & ~x & highs is non-zero iff some field of x is zero.
    const unsigned long long x = moved_even | moved_odd | idle_lanes;
    if (((x - base_bits) & ~x & high_bits) != 0ull) {
      const bool ended = running && !priming && !any_in_segment(x);
      const bool more = pool_next < (unsigned long long)n_cand;   // (of the pool or the counter)
      // (a device that a lane does not have counts as one whose list is exhausted)
      const unsigned even_issued = word_at(even.pos) - 1u, odd_issued = has_odd ? word_at(odd.pos) - 1u : 0u;
      const unsigned both = even.info | odd.info;
      const bool even_stops = even_issued == (even.info & kRowStop), odd_stops = odd_issued == (odd.info & kRowStop);
      const bool stuck = any_in_segment(__ballot(!even_stops || !odd_stops || (both & kRowStuck) != 0u));
      const bool malformed = any_in_segment(__ballot((even_stops && (even.info & kRowMalformed) != 0u) || (odd_stops && (odd.info & kRowMalformed) != 0u)));
      const bool unfinished = any_in_segment(__ballot((both & kRowIncomplete) != 0u));
      if (COPY && ended) {
        // what the engine still had to do; the makespan covers both timelines
        pass_events(even, ~0u, ~0u, 0);
        pass_events(odd, ~0u, ~0u, 0);
        even.free_at = max(even.free_at, even.copy_end[0]);
        odd.free_at = max(odd.free_at, odd.copy_end[0]);
      }
      const bool over = any_in_segment(__ballot(COPY ? even.pk > even.cap || odd.pk > odd.cap : (both & kRowOverCap) != 0u));
      if (ended) {
        const unsigned flags = stuck ? kDeadlock | (malformed ? kIncomplete : 0u)
                                     : (unfinished ? (unsigned)kIncomplete : (over ? (unsigned)kOverCap : 0u));
        if constexpr (TIMES) {
          // the start times still in the rings, the ends of the escape lists, and where the lists stopped
          auto leave = [&](const Device& x, int odd_device, unsigned issued) {
            const unsigned landed = x.loaded == kNoList ? stride_pos + kPiece : x.loaded;
            for (unsigned back = 2u * kPiece; back > 0u; back -= kPiece)
              if (landed >= back && (landed - back) >> 7 < issued) leave_starts(x, landed - back, odd_device);
            const size_t r = (size_t)cand * D + d0 + odd_device;
            *x.escape = 0xffffffffu;
            starts.stops[r] = (int)issued;
          };
          leave(even, 0, even_issued);
          if (has_odd) leave(odd, 1, odd_issued);
          if (pair == 0) out_flags[cand] = (unsigned char)(flags & (kDeadlock | kIncomplete));
        } else {
          // the latest finish, in a word that was cleared when the segment started
          atomicMax(reinterpret_cast<unsigned*>(reinterpret_cast<char*>(lds) + (at_max - lds0 + lds_from)), max(even.free_at, odd.free_at));
          const unsigned ms = lds_read<uint32_t>(at_max) >> (WIDE ? 0 : 8);
          const bool failed = (flags & (kDeadlock | kIncomplete)) != 0u;
          const long long r = cand * D + d0;
          out_idle[r] = failed ? -1ll : (long long)((int)ms - (int)even.busy);
          if (COPY || failed) out_peak[r] = failed ? -1 : even.pk * T.unit_scale;
          if (has_odd) {
            out_idle[r + 1] = failed ? -1ll : (long long)((int)ms - (int)odd.busy);
            if (COPY || failed) out_peak[r + 1] = failed ? -1 : odd.pk * T.unit_scale;
          }
          if (pair == 0) {
            out_makespan[cand] = failed ? 0x7fffffffffffffffll : (long long)ms;
            out_flags[cand] = (unsigned char)flags;
          }
        }
        running = false;
        fresh = more;
        idle_device(even);
        idle_device(odd);
      }
      // the finished segments stop counting as running at once
      const unsigned long long all_running = __ballot(running);
      idle_lanes = ~(all_running & ~__ballot(priming));
      any_special = any_special || more;
      if (all_running == 0ull && !more) break;
    }
  }
}

#define FPSCHED_INSTANTIATE_FORM(DEG2, WIDE, LINKS, MB, SYNC, TIMES, ALONE, COPY)                                                   \
  template __global__ void time_lists_kernel<DEG2, WIDE, LINKS, MB, SYNC, TIMES, ALONE, COPY>(ListTables, const uint16_t*, long long, int, long long*, \
                                                                    long long*, int*, unsigned char*, unsigned long long*, int, unsigned, StartTimes);
#define FPSCHED_INSTANTIATE(DEG2, WIDE, LINKS, MB, SYNC, TIMES, COPY) FPSCHED_INSTANTIATE_FORM(DEG2, WIDE, LINKS, MB, SYNC, TIMES, 0, COPY)
#define FPSCHED_INSTANTIATE_ALONE(DEG2, WIDE)                              \
  FPSCHED_INSTANTIATE_FORM(DEG2, WIDE, false, 0, false, false, 1, 0)       \
  FPSCHED_INSTANTIATE_FORM(DEG2, WIDE, false, 0, false, false, 2, 0)       \
  FPSCHED_INSTANTIATE_FORM(DEG2, WIDE, false, 0, false, false, 3, 0)
#define FPSCHED_INSTANTIATE_MODELS(DEG2)                            \
  FPSCHED_INSTANTIATE(DEG2, false, false, 0, false, false, 0)   \
  FPSCHED_INSTANTIATE(DEG2, true, false, 0, false, false, 0)    \
  FPSCHED_INSTANTIATE(DEG2, false, true, 0, false, false, 0)    \
  FPSCHED_INSTANTIATE(DEG2, false, false, 1, false, false, 0)   \
  FPSCHED_INSTANTIATE(DEG2, false, false, 2, false, false, 0)   \
  FPSCHED_INSTANTIATE(DEG2, false, true, 1, false, false, 0)    \
  FPSCHED_INSTANTIATE(DEG2, false, true, 2, false, false, 0)
FPSCHED_INSTANTIATE_MODELS(false)
FPSCHED_INSTANTIATE_MODELS(true)
FPSCHED_INSTANTIATE(true, false, false, 0, true, false, 0)
FPSCHED_INSTANTIATE(false, false, false, 0, false, true, 0)
FPSCHED_INSTANTIATE(true, false, false, 0, false, false, kCopyShallow)
FPSCHED_INSTANTIATE(true, false, false, 0, false, false, 4)
FPSCHED_INSTANTIATE(true, false, false, 0, false, false, 7)
FPSCHED_INSTANTIATE_ALONE(false, false)
FPSCHED_INSTANTIATE_ALONE(true, false)
FPSCHED_INSTANTIATE_ALONE(false, true)
#undef FPSCHED_INSTANTIATE_ALONE
#undef FPSCHED_INSTANTIATE_FORM
#undef FPSCHED_INSTANTIATE_MODELS
#undef FPSCHED_INSTANTIATE

}  // namespace fpsched
