// C ABI of libfpsched: problem handles, host-side helpers and kernel launches.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <numeric>
#include <vector>

#include "../../include/fpsched.h"
#include "kernels.h"

using namespace fpsched;

// The list evaluation's tables and launch shape under link occupancy, costs per micro-batch, or both
struct ListVariant {
  bool ok = false, deg2 = false;
  ListTables tab{};
  int32_t* d_image = nullptr;
  size_t capacity = 0;             // ints
  int32_t waves = 0, grid = 0;     // of the timing pass: wavefronts per workgroup, resident workgroups
};

struct fpsched_problem {
  int32_t D = 0, S = 0, m = 0, has_w = 0;
  int device_id = -1;
  int32_t max_stride = 0;
  std::vector<int32_t> stage_device, stage_chunk, local_stage, n_chunks;
  std::vector<int32_t> host_ints;  // the table image uploaded to the GPU
  DevTables tables{};
  int32_t* d_ints = nullptr;
  int32_t lds_bytes = 0;           // dynamic LDS of the general kernel (one wave per group)
  int32_t max_lds = 0;
  int32_t max_degree = 0;          // largest in- or out-degree of a stage in the DAG
  int32_t n_cu = 0;                // compute units of the device
  void* d_static_scratch = nullptr; // this device's copy of the library's static scratch array
  bool general_ok = false, slots_ok = false;  // which kernels fit this problem in LDS (slots_ok: the forms of eval_slots.hip)
  bool use_slots = false;          // selected kernels: those with mail slots (default when they fit) or the general one
  int32_t slot_v = 0;              // template bound on chunks per device
  bool slot_deg2 = false;          // some stage has two inputs or two outputs
  int32_t slot_lds_bytes = 0;      // dynamic LDS of one slot-kernel workgroup
  int32_t slot_waves = 0;          // wavefronts per slot-kernel workgroup
  int32_t slot_grid = 0;           // resident workgroups: the persistent grid
  bool slide_ok = false;           // the sliding pass is available (split backward, slot tables)
  SlotTables stab_times{};         // the slot tables of the lists without their W items
  int32_t* d_times_ints = nullptr;
  bool slide_eval_ok = false;      // the one-kernel form of the sliding pass (results only) is available
  SlotTables stab_slide{};         // stab_times plus the costs of the W items
  int32_t* d_slide_ints = nullptr;
  std::vector<int32_t> slide_w_table;   // host copy of those costs (layout: SlotTables::off_w)
  bool links_slide_eval_ok = false;     // ... and its form under the link model
  SlotTables stab_slide_links{};
  int32_t* d_slide_links_image = nullptr;
  SlotTables stab{};
  std::vector<int32_t> slot_ints;
  int32_t* d_slot_ints = nullptr;
  // the two-pass list evaluation: order pass, timing pass
  bool lists_ok = false;
  bool lists_deg2 = false, lists_wide = false;
  ListTables ltab{};
  int32_t* d_list_ints = nullptr;
  int32_t check_rows_per_wave = 0, check_waves = 0, check_grid = 0, check_vbits = 0;
  int32_t time_waves = 0, time_grid = 0;   // wavefronts per workgroup, resident workgroups
  std::vector<int32_t> list_image;         // host copy of d_list_ints
  // what the variants' tables are made from: as ltab and its image, second edges as the variants read them
  ListTables variants_tab{};
  std::vector<int32_t> variants_image;
  ListVariant lists_links, lists_mb, lists_both, lists_sync, lists_copy, lists_copy_deep;
  // (an engine of more than kCopyShallow transfers is a form of its own)
  ListVariant& copy_lists(int depth) { return depth > kCopyShallow ? lists_copy_deep : lists_copy; }
  const ListVariant& copy_lists(int depth) const { return depth > kCopyShallow ? lists_copy_deep : lists_copy; }
  ListVariant lists_times;                 // the lists without their W items, first pass of the sliding pass
  // costs per micro-batch (fpsched_problem_set_microbatch_costs)
  int64_t max_comm = 0;
  bool mb_set = false;
  bool mb_slots_ok = false;        // the table's values fit the slot kernel's 24-bit times
  int32_t* d_mb_raw = nullptr;     // [kinds][S][m]
  int32_t* d_mb_rows = nullptr;    // [32 metadata rows][lanes per candidate][m], << 8
  // link occupancy (fpsched_problem_set_link_occupancy): a table image with longer dev rows
  int64_t max_dur = 0;
  bool links_on = false;
  SlotTables stab_links{};         // of the sliding pass's forms
  std::vector<int32_t> mb_raw;          // host copy of the cost table that is set, [kinds][S][m]
  int64_t mb_max_dur = 0;               // largest value of the cost table that is set
  std::vector<int32_t> times_ints;      // host copy of the timing pass's table image
  bool links_slide_ok = false;          // the sliding pass has a link form (its LDS fits)
  SlotTables stab_times_links{};
  int32_t* d_times_links_image = nullptr;
  int32_t links_waves = 0, links_grid = 0, links_lds_bytes = 0;
  // synchronisation stages and dependency pairs (fpsched_problem_set_sync)
  bool sync_on = false;
  int32_t copy_depth = 0;               // copy-engine form (fpsched_problem_set_copy_engine), 0 = off
  bool sync_slots_ok = false;           // the synchronisation model has a slot-kernel form for this setting
  SlotTables stab_sync{};
  bool sync_deg2 = false;
  int32_t* d_sync_slot_image = nullptr;
  size_t sync_slot_image_ints = 0;
  int32_t sync_slot_waves = 0, sync_slot_grid = 0, sync_slot_lds_bytes = 0;
  bool copy_slots_ok = false;           // ... which the slot kernel can run (its rings fit LDS)
  SlotTables stab_copy{};
  int32_t copy_waves = 0, copy_grid = 0, copy_lds_bytes = 0;
  std::vector<int32_t> sync_items;      // [S] items per kind of each stage (m while the model is off)
  SyncTables sync_tab{};
  int32_t* d_sync_ints = nullptr;
  size_t sync_ints_capacity = 0;
  int32_t sync_lds_bytes = 0;
};

namespace {

int check_hip(hipError_t e) { return e == hipSuccess ? FPSCHED_OK : FPSCHED_EHIP; }

// Device memory of fpsched_evaluate_topk_static, the entry point for callers that cannot allocate: the
// work counter and the top-k key buffers that the other entry points take from the caller's workspace.
// Every GPU the library runs on holds its own copy of the array until the process ends.  In host code the
// array's name is only a stand-in: the address on a device comes from hipGetSymbolAddress, asked once per
// device with that device current, and only that pointer is ever handed to a kernel.
constexpr size_t kStaticScratchBytes = FPSCHED_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxGpus = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxGpus] = {nullptr};

// The device must be current.  FPSCHED_EHIP if the runtime does not give the address.
int static_scratch_of(int device_id, void** out) {
  *out = nullptr;
  if (device_id < 0 || device_id >= kMaxGpus) return FPSCHED_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device_id]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return FPSCHED_EHIP;
    }
    g_scratch_ptr[device_id] = ptr;
  }
  *out = g_scratch_ptr[device_id];
  return FPSCHED_OK;
}

struct DeviceGuard {
  int prev = -1;
  bool ok = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) return;
    ok = (prev == dev) || hipSetDevice(dev) == hipSuccess;
    if (prev == dev) prev = -1;
  }
  ~DeviceGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

using SlotKernel = void (*)(SlotTables, const uint16_t*, long long, int, long long*, long long*, int*,
                            unsigned char*, unsigned long long*, int, uint32_t*, int32_t*, const int32_t*, uint32_t*, int);
template <int MODE>   // kSlotPlain, kSlotTimes, ...
SlotKernel slot_kernel_of(int v, bool deg2, bool one_class) {
  if (deg2)
    return v == 1 ? &eval_slot_kernel<1, true, false, MODE>
                  : (v == 2 ? &eval_slot_kernel<2, true, false, MODE> : &eval_slot_kernel<4, true, false, MODE>);
  if (one_class)
    return v == 1 ? &eval_slot_kernel<1, false, true, MODE>
                  : (v == 2 ? &eval_slot_kernel<2, false, true, MODE> : &eval_slot_kernel<4, false, true, MODE>);
  return v == 1 ? &eval_slot_kernel<1, false, false, MODE>
                : (v == 2 ? &eval_slot_kernel<2, false, false, MODE> : &eval_slot_kernel<4, false, false, MODE>);
}

// Launch shape of the slot kernel for a batch: `waves` wavefronts per workgroup and `grid` workgroups fill the
// chip; a batch too small for that is spread over as many compute units as it has wavefronts' worth of
// candidates (a wavefront that has a SIMD to itself runs its rounds faster than three that share one), with
// fewer wavefronts per workgroup and the LDS that goes with them.
struct SlotLaunch { int waves; int64_t blocks; size_t lds_bytes; };
static SlotLaunch slot_launch(const SlotTables& tab, int waves, int grid, size_t lds_bytes, int64_t n_cand) {
  const int64_t cpw = tab.cands_per_wave;
  const int64_t spread = (n_cand + cpw * grid - 1) / (cpw * grid);   // wavefronts per workgroup that cover the batch
  const int w = (int)std::clamp<int64_t>(spread, 1, waves);
  SlotLaunch L;
  L.waves = w;
  L.blocks = std::min<int64_t>((n_cand + cpw * w - 1) / (cpw * w), grid);
  L.lds_bytes = lds_bytes - (size_t)(waves - w) * (size_t)tab.wave_ints * 4u;
  return L;
}

// Workgroup shape of the slot kernel for a shared LDS part of n_shared_ints dwords: candidates per
// wavefront, then the split of a compute unit's LDS into workgroups that keeps the most wavefronts
// resident (LDS is the only limiter: ~50 VGPRs).  Returns wavefronts per workgroup (0 = does not fit).
struct SlotGeometry { int cands_per_wave, wave_ints, waves, groups; };
SlotGeometry slot_geometry(int64_t n_shared_ints, int lanes_per_cand, int state_words, int slots_per_cand, int max_lds,
                           int max_cands_per_wave = 64) {
  int scpw = std::min(64 / lanes_per_cand, max_cands_per_wave);
  const int64_t fixed = 64ll * (8 + state_words);  // 16 op words + state words per lane
  const int64_t lds_ints = max_lds / 4;
  while (scpw > 1 && n_shared_ints + fixed + (int64_t)scpw * slots_per_cand > lds_ints) scpw >>= 1;
  const int64_t wave_ints = fixed + (int64_t)scpw * slots_per_cand;
  int best_waves = 0, best_groups = 0, best_total = 0;
  for (int groups = 1; groups <= 8; ++groups) {
    const int64_t per_group = lds_ints / groups - n_shared_ints - 64;  // allocation slack
    int wv = per_group > 0 ? (int)std::min<int64_t>(per_group / wave_ints, kSlotMaxWaves) : 0;
    wv = std::min(wv, 32 / groups);  // 8 wavefronts per SIMD, 4 SIMDs per compute unit
    if (wv * groups > best_total) { best_total = wv * groups; best_waves = wv; best_groups = groups; }
  }
  // tuning knob: FPSCHED_SLOT_WAVES=n caps the wavefronts per workgroup (one workgroup per CU)
  if (const char* env = getenv("FPSCHED_SLOT_WAVES")) {
    const int cap_waves = atoi(env);
    if (cap_waves >= 1 && cap_waves < best_waves * best_groups) { best_waves = std::min(cap_waves, best_waves); best_groups = 1; }
  }
  return SlotGeometry{scpw, (int)wave_ints, best_waves, std::max(best_groups, 1)};
}

// Wavefronts per workgroup and workgroups per compute unit that keep the most wavefronts resident, for a shared part
// of `shared` bytes of LDS per workgroup and `per_wave` bytes per wavefront (0 = does not fit).  At equal numbers the
// fewer workgroups win: each has a copy of the shared part to fetch.
struct WorkgroupShape { int waves, groups; };
// max_waves: of a workgroup; per_simd: resident wavefronts per SIMD that the registers allow; even: keep the four SIMDs
// of a compute unit equally loaded (for kernels whose wavefronts are given equal shares of the work).
WorkgroupShape workgroup_shape(int64_t shared, int64_t per_wave, int64_t max_lds, int max_waves = 16, int per_simd = 8,
                               bool even = false) {
  WorkgroupShape best{0, 1};
  for (int groups = 1; groups <= 8; ++groups) {
    const int64_t room = max_lds / groups - shared - 512;   // allocation slack
    int waves = room > 0 ? (int)std::min<int64_t>(room / per_wave, max_waves) : 0;
    waves = std::min(waves, 4 * per_simd / groups);   // 4 SIMDs per compute unit
    if (even && waves > 4) waves &= ~3;
    if (waves * groups > best.waves * best.groups) best = WorkgroupShape{waves, groups};
  }
  // tuning knob: FPSCHED_SLOT_WAVES=n caps the wavefronts per workgroup (one workgroup per CU)
  if (const char* env = getenv("FPSCHED_SLOT_WAVES")) {
    const int cap = atoi(env);
    if (cap >= 1 && cap < best.waves * best.groups) best = WorkgroupShape{std::min(cap, best.waves), 1};
  }
  return best;
}

int next_pow2(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

using CheckKernel = void (*)(ListTables, const uint16_t*, long long, int, int, long long*, int*, unsigned long long*, unsigned long long, int, int);
template <bool NO_W, bool SHARED>
CheckKernel check_kernel_of(int vbits) {
  return vbits == 0 ? &check_rows_kernel<0, NO_W, SHARED> : (vbits == 1 ? &check_rows_kernel<1, NO_W, SHARED> : &check_rows_kernel<2, NO_W, SHARED>);
}
CheckKernel check_kernel_of(int vbits, bool no_w, bool shared) {
  return no_w ? (shared ? check_kernel_of<true, true>(vbits) : check_kernel_of<true, false>(vbits))
              : (shared ? check_kernel_of<false, true>(vbits) : check_kernel_of<false, false>(vbits));
}

using TimeKernel = void (*)(ListTables, const uint16_t*, long long, int, long long*, long long*, int*, unsigned char*, unsigned long long*, int, unsigned, StartTimes);
template <bool DEG2>
TimeKernel time_kernel_of(const ListTables& T, bool wide) {
  const bool links = T.link_words > 0;
  if (wide) return &time_lists_kernel<DEG2, true, false, 0, false, false, 0, 0>;
  if (T.mb_bytes == 1) return links ? &time_lists_kernel<DEG2, false, true, 1, false, false, 0, 0> : &time_lists_kernel<DEG2, false, false, 1, false, false, 0, 0>;
  if (T.mb_bytes == 2) return links ? &time_lists_kernel<DEG2, false, true, 2, false, false, 0, 0> : &time_lists_kernel<DEG2, false, false, 2, false, false, 0, 0>;
  return links ? &time_lists_kernel<DEG2, false, true, 0, false, false, 0, 0> : &time_lists_kernel<DEG2, false, false, 0, false, false, 0, 0>;
}
// the form that reads these tables
TimeKernel time_kernel_of(const ListTables& T, bool deg2, bool wide) {
  if (T.off_sync > 0) return &time_lists_kernel<true, false, false, 0, true, false, 0, 0>;
  if (T.copy_depth > 4) return &time_lists_kernel<true, false, false, 0, false, false, 0, FPSCHED_MAX_COPY_DEPTH>;
  if (T.copy_depth > kCopyShallow) return &time_lists_kernel<true, false, false, 0, false, false, 0, 4>;
  if (T.copy_depth > 0) return &time_lists_kernel<true, false, false, 0, false, false, 0, kCopyShallow>;
  return deg2 ? time_kernel_of<true>(T, wide) : time_kernel_of<false>(T, wide);
}
// both passes in one launch (null: second edges and times of two words, whose step has branches)
template <bool DEG2, bool WIDE>
TimeKernel alone_kernel_of(int vbits) {
  return vbits == 0 ? &time_lists_kernel<DEG2, WIDE, false, 0, false, false, 1, 0>
                    : (vbits == 1 ? &time_lists_kernel<DEG2, WIDE, false, 0, false, false, 2, 0> : &time_lists_kernel<DEG2, WIDE, false, 0, false, false, 3, 0>);
}
TimeKernel alone_kernel_of(int vbits, bool deg2, bool wide) {
  return wide ? (deg2 ? nullptr : alone_kernel_of<false, true>(vbits)) : (deg2 ? alone_kernel_of<true, false>(vbits) : alone_kernel_of<false, false>(vbits));
}
TimeKernel times_kernel() { return &time_lists_kernel<false, false, false, 0, false, true, 0, 0>; }

// What the list evaluation needs to know about one stage: per direction (0 forward, 1 backward) its inputs and outputs.
struct StageEdge { int32_t cls, tag, latency; };
struct StageEdges { std::vector<StageEdge> in[2], out[2]; };

// timing pass: as many candidates per wavefront as its lanes and LDS hold (waves 0: it does not fit)
WorkgroupShape timing_shape(ListTables* T, int slot_bytes, int64_t max_lds) {
  const int pairs = (T->D + 1) / 2;
  for (int cpw = 64 / pairs; cpw >= 1; --cpw) {
    T->cands_per_wave = cpw;   // (rings are 32-byte aligned)
    T->wave_bytes = (int32_t)((kTimeWindowBytes + 512ll * T->link_words + (int64_t)cpw * slot_bytes * T->cand_slots + 31) & ~31ll);
    auto place = [&](bool columns) {
      // (where no device has more than two stages, the odd devices' rows take the place of the third and fourth stage's)
      T->row_step = columns ? 16 * kRowColumns : 16 * T->D;
      T->odd_at = !columns ? 16 * pairs : (T->chunks <= 2 ? 2 : kNKinds * kMaxChunks) * T->row_step;
      T->row_bytes = kNKinds * kMaxChunks * T->row_step * (columns && T->chunks > 2 ? 2 : 1);
      const int64_t tables = list_table_bytes(*T);
      return T->copy_depth > 0 ? workgroup_shape(tables, T->wave_bytes, max_lds, kTimeCopyMaxThreads / 64, kTimeCopyWavesPerSimd, T->copy_depth > kCopyShallow)
                               : workgroup_shape(tables, T->wave_bytes, max_lds);
    };
    const WorkgroupShape dense = place(false);
    // Columns where the lanes of a candidate divide them, so that a lane's column is its number's, and where they cost no wavefront
    // (a wavefront in fourteen is worth about what half of a row read is).  On one or two devices the rows of the image are eight to a
    // turn of the banks, about as many as a list has kinds of words, and in columns they only take longer to set up (the pass, in columns
    // and as in the image: 3,465 candidates of 2 x 8 x 2, links 21.4 and 20.3 us, costs 19.4 and 18.4; 74,761 of 2 x 60 x 2 180 either way);
    // with times of two words columns are worth it there too (whole evaluation, 40,000 of 2 x 32 x 2, 84 and 87 us).
    if ((pairs > 1 || slot_bytes == 8) && kRowColumns % pairs == 0) {
      const WorkgroupShape shape = place(true);
      if (shape.waves >= 1 && shape.waves * shape.groups >= dense.waves * dense.groups) return shape;
      (void)place(false);
    }
    if (dense.waves >= 1) return dense;
  }
  return WorkgroupShape{0, 1};
}

// The launch shape of the order pass, with as many rows per wavefront as the states leave room for, and where its table stands.
// Columns of eight bytes, a power of two of them for each (kind, chunk): as many as are all banks, with the devices over and
// over in them where they are a power of two themselves, so that no two lanes of half a wavefront that are at different rows
// read the same bank.  Fewer columns where those would cost a wavefront, and the rows of a device side by side, which take no
// more than the rows themselves, where these would too: on devices that are no power of two, 9 % of 2 to 40 devices, 6 to 160
// micro-batches and one to four stages.  (Columns against rows [kind][chunk][device], the row found by a multiplication: 262,144
// candidates of 16 devices, 64 micro-batches, two chunks, whole evaluation 2,298 and 2,276 us, the first the multiplication; 32 devices the
// same.  Device by device against that, the pass, both twice: 24 x 119 x 2 130 and 127 us, 33 x 74 x 2 96.8 and 95.0, 9 x 55 x 3 99.3 and 97.7,
// 11 x 47 x 4 113.0 and 111.9, 17 x 75 x 3 101.8 and 100.5, 3 x 118 x 2 114.0 and 112.1; 5 x 98 x 2, 12 x 105 x 4, 23 x 86 x 2, 36 x 148 x 2 and
// 40 x 70 x 2 within 1 %.)
WorkgroupShape check_shape(ListTables* T, int64_t max_lds, int* rows) {
  WorkgroupShape best{0, 1};
  for (*rows = 64; *rows >= 4; *rows >>= 1) {
    T->check_wave_bytes = (*rows * T->state_bytes + 15) & ~15;
    for (int columns : {0, next_pow2(T->D), std::max(next_pow2(T->D), kCheckColumns)}) {
      const int shared = (4 * (2 * kNKinds * kMaxChunks * (columns > 0 ? columns : T->D) + 2 * T->D) + 15) & ~15;
      const WorkgroupShape shape = workgroup_shape(shared, T->check_wave_bytes, max_lds, kCheckMaxThreads / 64, kCheckWavesPerSimd, true);
      if (shape.waves < 1 || shape.waves * shape.groups < best.waves * best.groups) continue;
      best = shape;
      T->check_columns = columns;
      T->check_shared_bytes = shared;
    }
    if (best.waves >= 1) break;
  }
  return best;
}

void take_check_place(const ListTables& from, ListTables* to) {
  to->check_columns = from.check_columns;
  to->check_shared_bytes = from.check_shared_bytes;
  to->check_wave_bytes = from.check_wave_bytes;
}

// Edge slots of an op: an input and the output that continues its class share one, an output (or input) of a class of its
// own has one.
struct EdgeSlot { int32_t cls; const StageEdge* in; bool out; };
std::vector<EdgeSlot> edge_slots(const StageEdges& e, int dir) {
  std::vector<EdgeSlot> slots;
  for (const StageEdge& in : e.in[dir]) slots.push_back(EdgeSlot{in.cls, &in, false});
  for (const StageEdge& out : e.out[dir]) {
    size_t i = 0;
    while (i < slots.size() && slots[i].cls != out.cls) ++i;
    if (i == slots.size()) slots.push_back(EdgeSlot{out.cls, nullptr, true});
    else slots[i].out = true;
  }
  // (the output of the first slot goes with the op's first row)
  if (slots.size() > 1 && !slots[0].out && slots[1].out) std::swap(slots[0], slots[1]);
  return slots;
}

// Table image of the two-pass list evaluation (layout: device_tables.h): rows and sizes, not yet the launch shapes.
// n_forward, n_backward: slot classes of either direction.  items: per stage (m, or fewer where an item is a group of micro-batches).  Returns false if the problem does not fit:
// more than two edge slots of a stage in one direction, or times, latencies,
// stages or slots beyond the widths of their fields.
// follow: second edges are rows of their own that follow the op's (the plain narrow form; device_tables.h).
bool fill_list_image(const fpsched_problem* p, const std::vector<StageEdges>& edges, int n_forward, int n_backward, bool wide,
                     bool follow, const std::vector<int32_t>& items, ListTables* tables, bool* deg2, std::vector<int32_t>* image) {
  const int D = p->D, S = p->S, m = p->m;
  const int32_t* dur = &p->host_ints[p->tables.off_dur];
  const int32_t* mem_units = &p->host_ints[p->tables.off_mem_units];
  const int32_t* mem_cap = &p->host_ints[p->tables.off_mem_cap];
  int64_t unit_scale = 0;
  for (int s = 0; s < S; ++s) unit_scale = std::gcd<int64_t, int64_t>(unit_scale, mem_units[s]);
  unit_scale = std::max<int64_t>(unit_scale, 1);
  const int64_t cand_slots = (list_slots_at(D) + (int64_t)(n_forward + n_backward) * m + 3) & ~3ll;
  const int slot_bytes = wide ? 8 : 4;
  if (slot_bytes * cand_slots > 0xffff || S > 255) return false;
  *deg2 = false;
  int n_second = 0;   // (F, FD and B rows of a stage may each have a second row)
  for (int s = 0; s < S; ++s) {
    if (mem_units[s] / unit_scale > 0xff) return false;
    for (int dir = 0; dir < 2; ++dir) {
      const size_t n = edge_slots(edges[s], dir).size();
      if (n > 2) return false;
      if (n > 1) { *deg2 = true; n_second += (dir == 0 ? 2 : 1) * (follow ? 2 : 1); }
    }
  }
  const int row_ints = 4;
  ListTables& T = *tables;
  T = ListTables{};
  T.D = D; T.m = m;
  for (int d = 0; d < D; ++d) T.chunks = std::max(T.chunks, p->n_chunks[d]);
  T.n_time_ints = (kNKinds * kMaxChunks * D * row_ints + n_second * 4 + 7) & ~7;
  if (4ll * T.n_time_ints > 0xffff) return false;
  int second_at = kNKinds * kMaxChunks * D * row_ints;
  T.off_check = T.n_time_ints;
  T.n_check_ints = kNKinds * kMaxChunks * D * 2;
  T.off_dev = T.off_check + T.n_check_ints;
  T.cand_slots = (int32_t)cand_slots;
  T.terminal = p->has_w ? kDone : kBDone;
  T.unit_scale = (int32_t)unit_scale;
  T.state_bytes = ((((m + 1) * (1 << p->check_vbits) + 3) / 4) | 1) * 4;
  std::vector<int32_t>& J = *image;
  J.assign((size_t)T.off_dev + 2 * D, 0);
  static const int need_of[kNKinds] = {(int)kNoState, kAbsent, kRes, kBDone, kDisc, kRes, kOff, kAbsent};
  static const int next_of[kNKinds] = {0, kRes, kBDone, kDone, kRes, kOff, kRes, kDisc};
  for (int kind = 0; kind < kNKinds; ++kind)
    for (int c = 0; c < kMaxChunks; ++c)
      for (int d = 0; d < D; ++d) {
        const size_t row = ((size_t)kind * kMaxChunks + c) * D;
        int32_t* t = &J[(row + (d & 1) * ((D + 1) / 2) + d / 2) * row_ints];   // even devices first
        int32_t* o = &J[(size_t)T.off_check + (row + d) * 2];
        t[0] = wide ? 0 : 1;
        t[2] = slot_bytes * d;
        if (wide) t[3] = (int32_t)kWideNever;
        o[0] = (int32_t)(kNoState << 8);
        if (kind == kEnd && c < p->n_chunks[d]) o[1] = items[p->local_stage[(size_t)d * kMaxChunks + c]];
        if (c >= p->n_chunks[d] || kind == kEnd || (kind == kW && !p->has_w)) continue;
        const int s = p->local_stage[(size_t)d * kMaxChunks + c];
        const unsigned units = (unsigned)(mem_units[s] / unit_scale);
        const bool allocs = kind == kF || kind == kFD || kind == kR || kind == kL;
        const bool frees = kind == kFD || kind == kO || kind == (p->has_w ? kW : kB);
        o[0] = (int32_t)((unsigned)next_of[kind] | ((unsigned)need_of[kind] << 8) | ((allocs ? units : 0u) << 16) | ((frees ? units : 0u) << 24));
        o[1] = dur[kind * S + s];
        const int dir = kind == kF || kind == kFD ? 0 : (kind == kB ? 1 : -1);
        const std::vector<EdgeSlot> slots = dir < 0 ? std::vector<EdgeSlot>() : edge_slots(edges[s], dir);
        const bool crosses = !slots.empty();
        const unsigned own_tag = crosses ? (unsigned)s : kOwnTag;
        t[1] = wide ? dur[kind * S + s] : (int32_t)(((unsigned)dur[kind * S + s] << 8) | own_tag);
        if (wide) t[3] = (int32_t)own_tag;
        if (!crosses) {
          if (wide) t[3] |= (int32_t)(kOwnTag << 8);
          else t[0] = -(int32_t)kOwnTag;
          continue;
        }
        const int base = list_slots_at(D) + (dir == 0 ? n_backward * m : 0);
        for (size_t e = 0; e < slots.size(); ++e) {
          const StageEdge* in = slots[e].in;
          const int32_t slot = (int32_t)((unsigned)(slot_bytes * (base + slots[e].cls * m)) | ((unsigned)(0x7ff * slot_bytes) << 16));
          const unsigned expected = in ? (unsigned)in->tag : kEmptySlot & 0xffu;
          const unsigned latency = in ? (unsigned)in->latency : 0u;
          const int32_t wait = (int32_t)(wide ? latency : (latency << 8) - expected);
          if (e == 0) {
            t[0] = wait;
            t[2] = slot;
            if (wide) t[3] |= (int32_t)(expected << 8);
            continue;
          }
          int32_t* second = &J[second_at];
          if (follow) {
            // (SPLIT below: the row's number stands above the mask of 16 bits and two of the word that it is applied to)
            auto in_front_of = [&](int32_t* row, int32_t at) { row[3] = at / 4; };
            int32_t* main = t;
            if (in) {
              for (int i = 0; i < 4; ++i) second[i] = t[i];
              main = second;
              t[0] = wait; t[1] = (int32_t)(kEmptySlot & 0xffu); t[2] = slot;
              in_front_of(t, second_at);
              second_at += 4;
            }
            if (slots[e].out) {
              int32_t* last = &J[second_at];
              last[0] = -(int32_t)(kEmptySlot & 0xffu); last[1] = (int32_t)own_tag; last[2] = slot;
              in_front_of(main, second_at);
              second_at += 4;
            }
            continue;
          }
          second[0] = t[0]; second[1] = t[2]; second[2] = slot;
          if (wide) second[3] = t[3] & 0xff00;
          const unsigned flags = (slots[e].out ? kRowTwoOut : 0u) | (in ? 1u << 31 : 0u);
          const unsigned at_second = wide ? (unsigned)(second_at / 4) << 16 : (unsigned)(4 * second_at);
          t[3] = (int32_t)(((unsigned)t[3] & 0xffffu) | at_second | flags);
          if (in) {
            t[0] = wait; t[2] = slot;
            if (wide) t[3] = (int32_t)(((unsigned)t[3] & ~0xff00u) | (expected << 8));
          }
          second_at += 4;
        }
      }
  // (without second rows beside them: the slot's mask and offset in a word each, above the mask the row that follows)
  if ((!*deg2 || follow) && !wide)
    for (int i = 0; i < second_at / row_ints; ++i) {
      int32_t* t = &J[(size_t)i * row_ints];
      const uint32_t behind = (uint32_t)t[3];
      t[3] = t[2] & 0xffff;
      t[2] = (int32_t)((uint32_t)t[2] >> 16 | behind << 18);
    }
  // (wide: the mask, and the offset above the two tags)
  if (!*deg2 && wide)
    for (int i = 0; i < kNKinds * kMaxChunks * D; ++i) {
      int32_t* t = &J[(size_t)i * row_ints];
      t[3] = (int32_t)(((uint32_t)t[3] & 0xffffu) | (uint32_t)t[2] << 16);
      t[2] = (int32_t)((uint32_t)t[2] >> 16);
    }
  for (int d = 0; d < D; ++d) {
    J[(size_t)T.off_dev + 2 * d] = p->n_chunks[d];
    J[(size_t)T.off_dev + 2 * d + 1] = (int32_t)(mem_cap[d] / unit_scale);   // peak > cap  <=>  peak / scale > floor(cap / scale)
  }
  return true;
}

// The plain model's image and the launch shapes; leaves lists_ok false if the problem does not fit.
void build_list_tables(fpsched_problem* p, const std::vector<StageEdges>& edges, int n_classes, int64_t bound,
                       std::vector<int32_t>* image) {
  const bool wide = p->max_comm >= (1ll << 16) || bound >= (1ll << 24);
  const int slot_bytes = wide ? 8 : 4;
  int max_chunks = 1;
  for (int d = 0; d < p->D; ++d) max_chunks = std::max(max_chunks, p->n_chunks[d]);
  p->check_vbits = max_chunks <= 1 ? 0 : (max_chunks <= 2 ? 1 : 2);
  ListTables& T = p->ltab;
  bool deg2 = false;
  const std::vector<int32_t> items(p->S, p->m);
  if (!fill_list_image(p, edges, n_classes, n_classes, wide, false, items, &T, &deg2, image)) return;
  p->variants_tab = T;
  p->variants_image = *image;
  if (deg2 && !wide && !fill_list_image(p, edges, n_classes, n_classes, wide, true, items, &T, &deg2, image)) return;
  int rows = 64;
  const WorkgroupShape check = check_shape(&T, p->max_lds, &rows);
  const WorkgroupShape time = timing_shape(&T, slot_bytes, p->max_lds);
  if (check.waves < 1 || time.waves < 1) return;
  take_check_place(T, &p->variants_tab);
  p->check_rows_per_wave = rows;
  p->check_waves = check.waves;
  p->check_grid = p->n_cu * check.groups;
  p->time_waves = time.waves;
  p->time_grid = p->n_cu * time.groups;
  p->lists_deg2 = deg2;
  p->lists_wide = wide;
  p->lists_ok = true;
}

// The launch shape of a variant's tables and its image on the device.  FPSCHED_EUNSUPPORTED if fewer than min_waves
// wavefronts fit a compute unit.
int install_list_variant(fpsched_problem* p, ListTables T, const std::vector<int32_t>& J, bool deg2, int min_waves, ListVariant* v) {
  const WorkgroupShape shape = timing_shape(&T, 4, p->max_lds);
  if (shape.waves < 1 || shape.waves * shape.groups < min_waves) return FPSCHED_EUNSUPPORTED;
  DeviceGuard g(p->device_id);
  if (!g.ok || hipDeviceSynchronize() != hipSuccess) return FPSCHED_EHIP;   // an earlier image may be in use
  if (J.size() > v->capacity) {
    if (v->d_image) (void)hipFree(v->d_image);
    v->d_image = nullptr;
    v->capacity = 0;
    if (hipMalloc(&v->d_image, J.size() * sizeof(int32_t)) != hipSuccess) { v->d_image = nullptr; return FPSCHED_ENOMEM; }
    v->capacity = J.size();
  }
  const TimeKernel kernel = time_kernel_of(T, deg2, false);
  if (hipMemcpy(v->d_image, J.data(), J.size() * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) != hipSuccess)
    return FPSCHED_EHIP;
  T.ints = v->d_image;
  v->tab = T;
  v->deg2 = deg2;
  v->waves = shape.waves;
  v->grid = p->n_cu * shape.groups;
  v->ok = true;
  if (getenv("FPSCHED_VERBOSE"))
    fprintf(stderr, "[fpsched] list evaluation%s%s%s: %d x %d wavefronts per compute unit (plain: %d x %d), %d candidates each\n",
            T.copy_depth > kCopyShallow ? ", deep copy engine" : T.copy_depth > 0 ? ", copy engine" : T.link_words > 0 ? ", links" : "", T.mb_bytes > 0 ? ", costs per micro-batch" : "", T.off_sync > 0 ? ", synchronisation" : "",
            shape.groups, shape.waves, p->time_grid / std::max(p->n_cu, 1), p->time_waves, T.cands_per_wave);
  return FPSCHED_OK;
}

// The tables with link rows (links) and a table of costs per micro-batch (mb: [kinds][S][m]) between the timing rows and
// the order rows.  FPSCHED_EUNSUPPORTED if they do not fit.
int build_list_variant(fpsched_problem* p, bool links, const int32_t* mb, ListVariant* v) {
  v->ok = false;
  if (!p->lists_ok || p->lists_wide) return FPSCHED_EUNSUPPORTED;
  const ListTables& B = p->variants_tab;
  const int D = p->D, S = p->S, m = p->m, n_rows = kNKinds * kMaxChunks * D;
  const std::vector<int32_t>& I = p->host_ints;
  const DevTables& G = p->tables;
  ListTables T = B;
  std::vector<int32_t> J(p->variants_image.begin(), p->variants_image.begin() + B.n_time_ints);
  auto row_at = [&](int kind, int c, int d) { return (kind * kMaxChunks + c) * D + (d & 1) * ((D + 1) / 2) + d / 2; };
  if (links) {
    // links of a device: the devices its stages send to (activations to successor stages, gradients to predecessor
    // stages), numbered in the order they are met; one more for what sends nothing or stays on the device
    std::vector<std::vector<int>> sends_to(D);
    struct Sent { int d, link; int32_t latency; };
    auto out_edge = [&](int s, int dir, int k, Sent* e) {
      const int off = dir == 0 ? G.off_succ_off : G.off_pred_off, at = I[off + s] + k;
      if (at >= I[off + s + 1]) return false;
      const int from = p->stage_device[s], to = p->stage_device[I[(dir == 0 ? G.off_succ_stage : G.off_pred_stage) + at]];
      if (from == to) return false;
      std::vector<int>& known = sends_to[from];
      size_t link = 0;
      while (link < known.size() && known[link] != to) ++link;
      if (link == known.size()) known.push_back(to);
      *e = Sent{from, (int)link, I[(dir == 0 ? G.off_succ_comm : G.off_pred_comm) + at]};
      return true;
    };
    Sent e;
    for (int s = 0; s < S; ++s)
      for (int dir = 0; dir < 2; ++dir)
        for (int k = 0; k < 2; ++k) (void)out_edge(s, dir, k, &e);
    size_t most = 0;
    for (const std::vector<int>& known : sends_to) most = std::max(most, known.size());
    T.link_words = (int32_t)most + 1;
    if (256 * T.link_words > 0xffff) return FPSCHED_EUNSUPPORTED;
    const int32_t nowhere = 256 * (T.link_words - 1);
    T.off_links = (int32_t)J.size();
    J.resize(J.size() + n_rows, nowhere);
    for (int kind : {(int)kF, (int)kFD, (int)kB})
      for (int d = 0; d < D; ++d)
        for (int c = 0; c < p->n_chunks[d]; ++c) {
          const int s = p->local_stage[(size_t)d * kMaxChunks + c], dir = kind == kB ? 1 : 0, row = row_at(kind, c, d);
          auto packed = [&](int k) {
            return out_edge(s, dir, k, &e) ? (int32_t)((uint32_t)e.latency << 16 | (uint32_t)(256 * e.link)) : nowhere;
          };
          J[T.off_links + row] = packed(0);
          const uint32_t second = (uint32_t)J[4 * row + 3];
          if (second & kRowTwoOut) J[(second & 0xffffu) / 4 + 3] = packed(1);
        }
  }
  if (mb) {
    // kinds whose costs are the same (a forward item whether its activation is kept or dropped, a recomputation, ...)
    // share a block; values of two bytes, or one if all fit
    int32_t most = 0;
    for (size_t i = (size_t)S * m; i < (size_t)kNKinds * S * m; ++i) most = std::max(most, mb[i]);
    if (most >= 65536) return FPSCHED_EUNSUPPORTED;
    T.mb_bytes = most < 256 ? 1 : 2;
    std::vector<int> blocks;
    std::vector<unsigned char> costs;
    // (a stage's row is an odd number of dwords long: the lanes of a candidate mostly ask for the same micro-batch)
    const size_t row_bytes = ((((size_t)m * T.mb_bytes + 3) / 4) | 1) * 4, block_bytes = S * row_bytes, first = 4 * J.size();
    for (int kind = 1; kind < kNKinds; ++kind) {
      const int32_t* of_kind = mb + (size_t)kind * S * m;
      size_t b = 0;
      while (b < blocks.size() && !std::equal(of_kind, of_kind + (size_t)S * m, mb + (size_t)blocks[b] * S * m)) ++b;
      if (b == blocks.size()) {
        blocks.push_back(kind);
        costs.resize(blocks.size() * block_bytes, 0);
        for (int s = 0; s < S; ++s)
          for (int j = 0; j < m; ++j)
            for (int k = 0; k < T.mb_bytes; ++k)
              costs[b * block_bytes + s * row_bytes + (size_t)j * T.mb_bytes + k] = (unsigned char)((uint32_t)of_kind[s * m + j] >> (8 * k));
      }
      for (int d = 0; d < D; ++d)
        for (int c = 0; c < p->n_chunks[d]; ++c) {
          const int s = p->local_stage[(size_t)d * kMaxChunks + c];
          int32_t& word = J[4 * row_at(kind, c, d) + 1];
          const size_t at = first + b * block_bytes + s * row_bytes;
          if (at >= 1u << 24) return FPSCHED_EUNSUPPORTED;
          if (J[4 * row_at(kind, c, d)] != 1) word = (int32_t)((uint32_t)at << 8 | ((uint32_t)word & 0xffu));
        }
    }
    J.resize(J.size() + costs.size() / 4);
    memcpy(reinterpret_cast<char*>(J.data()) + first, costs.data(), costs.size());
  }
  J.resize((J.size() + 7) & ~(size_t)7, 0);
  T.n_time_ints = (int32_t)J.size();
  J.insert(J.end(), p->variants_image.begin() + B.off_check, p->variants_image.end());
  T.off_check = T.n_time_ints;
  T.off_dev = T.off_check + (B.off_dev - B.off_check);
  if (mb)   // (the busy time is the timing pass's)
    for (int i = kMaxChunks * D; i < T.n_check_ints / 2; ++i) J[(size_t)T.off_check + 2 * i + 1] = 0;
  // (costs from device memory, kSlotPerMicrobatch, are better than so few wavefronts)
  return install_list_variant(p, T, J, p->lists_deg2, mb && !links ? 6 : 1, v);
}

// The tables of the copy-engine form: the plain ones, with the units in the rows of the ops themselves; transfers are no
// busy time.
int build_copy_variant(fpsched_problem* p, int depth) {
  ListVariant& v = p->copy_lists(depth);
  v.ok = false;
  if (!p->lists_ok || p->lists_wide) return FPSCHED_EUNSUPPORTED;
  ListTables T = p->ltab;
  std::vector<int32_t> J = p->list_image;
  const int D = p->D;
  T.copy_depth = depth;
  for (int kind = 1; kind < kNKinds; ++kind)
    for (int c = 0; c < kMaxChunks; ++c)
      for (int d = 0; d < D; ++d) {
        const size_t row = ((size_t)kind * kMaxChunks + c) * D;
        int32_t* o = &J[(size_t)T.off_check + (row + d) * 2];
        int32_t* t = &J[(row + (d & 1) * ((D + 1) / 2) + d / 2) * 4];
        if (t[1] == (int32_t)(kEmptySlot & 0xffu)) t = &J[(size_t)((uint32_t)t[2] >> 18) * 4];   // (takes in the second input; the op follows)
        t[3] |= (int32_t)((uint32_t)o[0] & 0xffff0000u);
        if (kind == kO || kind == kL) o[1] = 0;
      }
  return install_list_variant(p, T, J, true, 1, &v);
}

// The tables of the lists without their W items: a W word is a no-op, an activation is consumed by its B item.
int build_times_variant(fpsched_problem* p) {
  ListVariant* v = &p->lists_times;
  ListTables T = p->ltab;
  std::vector<int32_t> J = p->variants_image;   // (no second edges: the plain model's too)
  const int D = p->D;
  for (int c = 0; c < kMaxChunks; ++c)
    for (int d = 0; d < D; ++d) {
      if (c >= p->n_chunks[d]) continue;
      const size_t row = ((size_t)kW * kMaxChunks + c) * D;
      J[(row + (d & 1) * ((D + 1) / 2) + d / 2) * 4 + 1] = (int32_t)kOwnTag;   // no cost
      int32_t* o = &J[(size_t)T.off_check + (row + d) * 2];
      o[0] = (int32_t)(kPadState | kPadState << 8);
      o[1] = 0;
    }
  T.terminal = kBDone;
  if (hipMalloc(&v->d_image, J.size() * sizeof(int32_t)) != hipSuccess) { v->d_image = nullptr; return FPSCHED_ENOMEM; }
  v->capacity = J.size();
  if (hipMemcpy(v->d_image, J.data(), J.size() * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess) return FPSCHED_EHIP;
  for (const void* kernel : {reinterpret_cast<const void*>(check_kernel_of(p->check_vbits, true, false)),
                             reinterpret_cast<const void*>(check_kernel_of(p->check_vbits, true, true)), reinterpret_cast<const void*>(times_kernel())})
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) != hipSuccess) return FPSCHED_EHIP;
  T.ints = v->d_image;
  v->tab = T;
  v->waves = p->time_waves;
  v->grid = p->time_grid;
  v->ok = true;
  return FPSCHED_OK;
}

}  // namespace

extern "C" {

int fpsched_version(void) { return FPSCHED_VERSION; }

const char* fpsched_strerror(int code) {
  switch (code) {
    case FPSCHED_OK: return "ok";
    case FPSCHED_EINVAL: return "invalid argument";
    case FPSCHED_ENOMEM: return "out of memory or workspace too small";
    case FPSCHED_EHIP: return "HIP runtime call failed";
    case FPSCHED_EOVERFLOW: return "time bound does not fit int32";
    case FPSCHED_ENODEV: return "host-only problem handle";
    case FPSCHED_EUNSUPPORTED: return "problem too large for the on-chip tables";
    case FPSCHED_ESCRATCH: return "batch too large for the library's static scratch memory";
    default: return "unknown error";
  }
}

int fpsched_problem_create(const fpsched_problem_desc* desc, int device_id, int32_t max_stride_words,
                           fpsched_problem** out) {
  if (!desc || !out) return FPSCHED_EINVAL;
  *out = nullptr;
  const int D = desc->n_devices, S = desc->n_stages, m = desc->n_microbatches, E = desc->n_edges;
  if (D < 1 || D > FPSCHED_MAX_DEVICES || S < 1 || S > D * FPSCHED_MAX_CHUNKS || m < 1 ||
      m > FPSCHED_MAX_MICROBATCHES || E < 0 || max_stride_words < 8 || (max_stride_words & 7))
    return FPSCHED_EINVAL;
  if (!desc->stage_device || !desc->dur || !desc->mem_units || !desc->mem_cap) return FPSCHED_EINVAL;
  if (E > 0 && (!desc->edge_src || !desc->edge_dst || !desc->edge_comm)) return FPSCHED_EINVAL;

  fpsched_problem* p = new (std::nothrow) fpsched_problem;
  if (!p) return FPSCHED_ENOMEM;
  p->D = D; p->S = S; p->m = m; p->has_w = desc->has_w ? 1 : 0;
  p->device_id = device_id < 0 ? -1 : device_id;
  p->max_stride = max_stride_words;
  p->stage_device.assign(desc->stage_device, desc->stage_device + S);
  p->stage_chunk.assign(S, 0);
  p->local_stage.assign((size_t)D * kMaxChunks, -1);
  p->n_chunks.assign(D, 0);
  p->sync_items.assign(S, m);
  int rc = FPSCHED_OK;
  for (int s = 0; s < S && rc == FPSCHED_OK; ++s) {
    const int d = p->stage_device[s];
    if (d < 0 || d >= D || p->n_chunks[d] >= kMaxChunks) { rc = FPSCHED_EINVAL; break; }
    p->stage_chunk[s] = p->n_chunks[d];
    p->local_stage[(size_t)d * kMaxChunks + p->n_chunks[d]++] = s;
  }
  // edges: range, non-negative latency, acyclic (Kahn over stages)
  int64_t max_dur = 0, max_comm = 0, units_total = 0;
  if (rc == FPSCHED_OK) {
    std::vector<int> indeg(S, 0);
    for (int e = 0; e < E; ++e) {
      const int a = desc->edge_src[e], b = desc->edge_dst[e];
      if (a < 0 || a >= S || b < 0 || b >= S || a == b || desc->edge_comm[e] < 0) { rc = FPSCHED_EINVAL; break; }
      indeg[b]++;
      max_comm = std::max<int64_t>(max_comm, desc->edge_comm[e]);
    }
    if (rc == FPSCHED_OK) {
      std::vector<int> order;
      for (int s = 0; s < S; ++s) if (!indeg[s]) order.push_back(s);
      for (size_t i = 0; i < order.size(); ++i)
        for (int e = 0; e < E; ++e)
          if (desc->edge_src[e] == order[i] && --indeg[desc->edge_dst[e]] == 0) order.push_back(desc->edge_dst[e]);
      if ((int)order.size() != S) rc = FPSCHED_EINVAL;
    }
  }
  if (rc == FPSCHED_OK) {
    for (int i = 0; i < kNKinds * S; ++i) {
      if (desc->dur[i] < 0) { rc = FPSCHED_EINVAL; break; }
      max_dur = std::max<int64_t>(max_dur, desc->dur[i]);
    }
    for (int s = 0; s < S && rc == FPSCHED_OK; ++s) {
      if (desc->mem_units[s] < 0) rc = FPSCHED_EINVAL;
      units_total += (int64_t)desc->mem_units[s] * m;
    }
    // (a negative cap would round towards zero when divided by the units' common divisor)
    for (int d = 0; d < D && rc == FPSCHED_OK; ++d)
      if (desc->mem_cap[d] < 0) rc = FPSCHED_EINVAL;
  }
  // every finish time is at most (number of listed ops) * (largest duration + largest
  // latency); resident memory is at most the sum of all activations
  if (rc == FPSCHED_OK) {
    const int64_t bound = (int64_t)D * max_stride_words * (max_dur + max_comm);
    if (bound >= (int64_t)1 << 31 || units_total >= (int64_t)1 << 31) rc = FPSCHED_EOVERFLOW;
  }
  if (rc != FPSCHED_OK) { delete p; return rc; }
  p->max_comm = max_comm;
  p->max_dur = max_dur;

  // table image
  std::vector<int32_t>& I = p->host_ints;
  DevTables& T = p->tables;
  T.D = D; T.S = S; T.m = m; T.has_w = p->has_w;
  auto append = [&](const int32_t* src, size_t n) { int32_t off = (int32_t)I.size(); I.insert(I.end(), src, src + n); return off; };
  T.off_dur = append(desc->dur, (size_t)kNKinds * S);
  T.off_mem_units = append(desc->mem_units, S);
  std::vector<int32_t> poff(S + 1, 0), soff(S + 1, 0), pst(E), pcm(E), sst(E), scm(E);
  for (int e = 0; e < E; ++e) { poff[desc->edge_dst[e] + 1]++; soff[desc->edge_src[e] + 1]++; }
  for (int s = 0; s < S; ++s) { poff[s + 1] += poff[s]; soff[s + 1] += soff[s]; }
  {
    std::vector<int32_t> pf(S, 0), sf(S, 0);
    for (int e = 0; e < E; ++e) {
      const int a = desc->edge_src[e], b = desc->edge_dst[e];
      const int32_t lat = p->stage_device[a] != p->stage_device[b] ? desc->edge_comm[e] : 0;
      pst[poff[b] + pf[b]] = a; pcm[poff[b] + pf[b]++] = lat;
      sst[soff[a] + sf[a]] = b; scm[soff[a] + sf[a]++] = lat;
    }
  }
  T.off_pred_off = append(poff.data(), S + 1);
  T.off_pred_stage = append(pst.data(), E);
  T.off_pred_comm = append(pcm.data(), E);
  T.off_succ_off = append(soff.data(), S + 1);
  T.off_succ_stage = append(sst.data(), E);
  T.off_succ_comm = append(scm.data(), E);
  for (int s = 0; s < S; ++s)
    p->max_degree = std::max({p->max_degree, poff[s + 1] - poff[s], soff[s + 1] - soff[s]});
  T.off_local_stage = append(p->local_stage.data(), (size_t)D * kMaxChunks);
  T.off_n_chunks = append(p->n_chunks.data(), D);
  T.off_mem_cap = append(desc->mem_cap, D);
  // Slot classes: chains of edges such that each edge starts at the stage the previous
  // one ends in.  Stages are visited in topological order; an out-edge continues the
  // class of a not yet continued in-edge of its stage, else it opens a new class.
  std::vector<int32_t> edge_cls(E, -1);
  int n_classes = 0;
  std::vector<int32_t> turnaround(S, 1);
  {
    std::vector<int> indeg(S, 0), order;
    for (int e = 0; e < E; ++e) indeg[desc->edge_dst[e]]++;
    for (int s = 0; s < S; ++s) if (!indeg[s]) order.push_back(s);
    for (size_t i = 0; i < order.size(); ++i) {
      const int s = order[i];
      std::vector<int32_t> arriving;
      for (int e = 0; e < E; ++e) if (desc->edge_dst[e] == s) arriving.push_back(edge_cls[e]);
      size_t used = 0;
      for (int e = 0; e < E; ++e) {
        if (desc->edge_src[e] != s) continue;
        edge_cls[e] = used < arriving.size() ? arriving[used++] : n_classes++;
        if (--indeg[desc->edge_dst[e]] == 0) order.push_back(desc->edge_dst[e]);
      }
    }
    if (n_classes == 0) n_classes = 1;
    for (size_t i = order.size(); i-- > 0;)
      for (int e = soff[order[i]]; e < soff[order[i] + 1]; ++e)
        turnaround[order[i]] = std::max(turnaround[order[i]], turnaround[sst[e]] + 2);
  }
  T.n_table_ints = (int32_t)I.size();   // what the table-walking kernels copy to LDS ends here
  T.off_turnaround = append(turnaround.data(), S);
  // Rows of the timed generator: what an item of (type, chunk) on a device costs, where its inputs'
  // finish times lie and where its own goes (layout: device_tables.h).
  T.off_gen_rows = -1;
  T.gen_row_chunks = 1;
  T.gen_slot_words = (2 * n_classes + 1) * m;
  if (p->max_degree <= 2 && 4ll * (2 * n_classes + 1) * m <= 0xffff) {
    int max_chunks = 1;
    for (int d = 0; d < D; ++d) max_chunks = std::max(max_chunks, p->n_chunks[d]);
    const int V = max_chunks <= 1 ? 1 : (max_chunks <= 2 ? 2 : 4);
    T.gen_row_chunks = V;
    std::vector<int32_t> pcl(E), scl(E), pf(S, 0), sf(S, 0);
    for (int e = 0; e < E; ++e) {
      const int a = desc->edge_src[e], b = desc->edge_dst[e];
      pcl[poff[b] + pf[b]++] = edge_cls[e];
      scl[soff[a] + sf[a]++] = edge_cls[e];
    }
    const int32_t dump = 4 * 2 * n_classes * m, none = -(1 << 30);   // slot offsets in bytes
    const size_t n_rows = (size_t)3 * V * D;
    std::vector<int32_t> rows(n_rows * 8, 0);
    for (size_t i = 0; i < n_rows; ++i) {
      int32_t* a = &rows[i * 4];
      int32_t* b = a + n_rows * 4;
      a[1] = b[2] = dump | (dump << 16);
      a[2] = b[3] = none;
    }
    for (int t = 0; t < 3; ++t)
      for (int c = 0; c < V; ++c)
        for (int d = 0; d < D; ++d) {
          int32_t* a = &rows[(((size_t)t * V + c) * D + d) * 4];
          int32_t* b = a + n_rows * 4;
          a[3] = c | (t == 1 ? 4 : 0);
          if (c >= p->n_chunks[d]) continue;
          const int s = p->local_stage[(size_t)d * kMaxChunks + c];
          const int kind = t == 0 ? kF : (t == 1 ? kB : kW);
          a[0] = desc->dur[kind * S + s];
          b[0] = t == 0 ? desc->mem_units[s] : 0;
          b[1] = (t == 2 || (t == 1 && !p->has_w)) ? desc->mem_units[s] : 0;
          if (t == 2) continue;
          // forward items read the values of their in-edges and write those of their out-edges; backward
          // items the other way round
          const std::vector<int32_t>& ioff = t == 0 ? poff : soff;
          const std::vector<int32_t>& icl = t == 0 ? pcl : scl;
          const std::vector<int32_t>& ilat = t == 0 ? pcm : scm;
          const std::vector<int32_t>& ooff = t == 0 ? soff : poff;
          const std::vector<int32_t>& ocl = t == 0 ? scl : pcl;
          const int32_t dir_base = t == 0 ? n_classes : 0;
          int32_t in[2] = {dump, dump}, lat[2] = {none, none}, out[2] = {dump, dump};
          for (int k = 0; k < ioff[s + 1] - ioff[s]; ++k) {
            in[k] = 4 * (dir_base + icl[ioff[s] + k]) * m;
            lat[k] = ilat[ioff[s] + k];
          }
          for (int k = 0; k < ooff[s + 1] - ooff[s]; ++k) out[k] = 4 * (dir_base + ocl[ooff[s] + k]) * m;
          a[1] = in[0] | (out[0] << 16); a[2] = lat[0];
          b[2] = in[1] | (out[1] << 16); b[3] = lat[1];
        }
    T.off_gen_rows = append(rows.data(), rows.size());
  }
  T.lanes_per_cand = next_pow2(D);
  T.cands_per_wave = 64 / T.lanes_per_cand;

  if (p->device_id >= 0) {
    DeviceGuard g(p->device_id);
    if (!g.ok) { delete p; return FPSCHED_EHIP; }
    int max_lds = 0;
    if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, p->device_id) != hipSuccess) {
      delete p; return FPSCHED_EHIP;
    }
    p->max_lds = max_lds;
    if (static_scratch_of(p->device_id, &p->d_static_scratch) != FPSCHED_OK) { delete p; return FPSCHED_EHIP; }
    // (The dynamic-LDS limit of a kernel is one value per process, not per handle: it is always raised
    // to the device's maximum, so that handles with different needs never undo each other's setting.)
    // general kernel geometry: finish-time tables and state bytes of whole candidates in LDS
    const int64_t SM = (int64_t)S * m;
    const int64_t per_cand = 4 * (2 * SM + ((SM + 3) >> 2));
    const int64_t table_bytes = 4ll * T.n_table_ints;
    int cpw = T.cands_per_wave;
    while (cpw > 1 && table_bytes + cpw * per_cand > max_lds) cpw >>= 1;
    p->general_ok = table_bytes + cpw * per_cand <= max_lds;
    T.cands_per_wave = cpw;
    p->lds_bytes = (int32_t)(table_bytes + cpw * per_cand);
    // ---- slot kernel: metadata per (kind, chunk, device), geometry, fit ----
    {
      SlotTables& ST = p->stab;
      int max_chunks = 1;
      for (int d = 0; d < D; ++d) max_chunks = std::max(max_chunks, p->n_chunks[d]);
      const int V = p->slot_v = max_chunks <= 1 ? 1 : (max_chunks <= 2 ? 2 : 4);
      const int lpc = T.lanes_per_cand;
      // memory units are carried in bytes: divide them (and the caps) by their common divisor
      int64_t unit_scale = 0;
      for (int s = 0; s < S; ++s) unit_scale = std::gcd<int64_t, int64_t>(unit_scale, desc->mem_units[s]);
      if (unit_scale < 1) unit_scale = 1;
      const int slot_stride = ((2 * n_classes + 1) * m + 7) & ~7;   // slots of one candidate
      // slot byte offsets are 16-bit, tags 8-bit (0xff = empty), finish times 24-bit
      bool fits = 4ll * slot_stride <= 0xffff && S <= 255 && max_comm < (1ll << 16) &&
                  (int64_t)D * max_stride_words * (max_dur + max_comm) < (1ll << 24);
      bool deg2 = false;
      for (int s = 0; s < S; ++s) {
        const int nin = poff[s + 1] - poff[s], nout = soff[s + 1] - soff[s];
        if (nin > 2 || nout > 2) fits = false;
        if (nin > 1 || nout > 1) deg2 = true;
        if (desc->mem_units[s] / unit_scale > 0xff) fits = false;
      }
      p->slot_deg2 = deg2;
      // classes of the edges in pred-CSR and succ-CSR order
      std::vector<int32_t> pcl(E), scl(E);
      {
        std::vector<int32_t> pf(S, 0), sf(S, 0);
        for (int e = 0; e < E; ++e) {
          const int a = desc->edge_src[e], b = desc->edge_dst[e];
          pcl[poff[b] + pf[b]++] = edge_cls[e];
          scl[soff[a] + sf[a]++] = edge_cls[e];
        }
      }
      const int n_meta = kNKinds * kMaxChunks * lpc * 4;
      const int n_meta2 = deg2 ? (2 * kMaxChunks + 1) * lpc * 2 : 0;   // + one all-zero row
      const int n_shared = (n_meta + n_meta2 + 511) & ~511;   // the op windows behind it are 2 KB-aligned
      const unsigned dump_bytes = (unsigned)(2 * n_classes * m) * 4u;
      const int dev_ints = 2 + 4 * V;
      const int words_per_chunk = (m + 7) / 8;
      const int state_words = V * words_per_chunk;
      std::vector<int32_t>& J = p->slot_ints;
      J.assign((size_t)n_shared + (size_t)lpc * dev_ints + (size_t)lpc * state_words, 0);
      static const int need_of[kNKinds] = {15, kAbsent, kRes, kBDone, kDisc, kRes, kOff, kAbsent};
      static const int next_of[kNKinds] = {0, kRes, kBDone, kDone, kRes, kOff, kRes, kDisc};
      for (int kind = 0; kind < kNKinds; ++kind)
        for (int c = 0; c < kMaxChunks; ++c)
          for (int d = 0; d < lpc; ++d) {
            int32_t* e = &J[(((size_t)kind * kMaxChunks + c) * lpc + d) * 4];
            e[2] = (int32_t)(15u | (dump_bytes << 16));
            if (d >= D || c >= p->n_chunks[d] || kind == kEnd || (kind == kW && !p->has_w)) continue;
            const int s = p->local_stage[(size_t)d * kMaxChunks + c];
            const unsigned units = (unsigned)(desc->mem_units[s] / unit_scale);
            const bool allocs = kind == kF || kind == kFD || kind == kR || kind == kL;
            const bool frees = kind == kFD || kind == kO || kind == (p->has_w ? kW : kB);
            unsigned has_in = 0, tag = 0, prod = dump_bytes;
            unsigned comm = 0;
            if (kind == kF || kind == kFD) {
              if (poff[s + 1] > poff[s]) { has_in = 0xffu; tag = (unsigned)pst[poff[s]]; comm = (unsigned)pcm[poff[s]]; }
              if (soff[s + 1] > soff[s]) prod = (unsigned)((n_classes + scl[soff[s]]) * m) * 4u;
            } else if (kind == kB) {
              if (soff[s + 1] > soff[s]) { has_in = 0xffu; tag = (unsigned)sst[soff[s]]; comm = (unsigned)scm[soff[s]]; }
              if (poff[s + 1] > poff[s]) prod = (unsigned)(pcl[poff[s]] * m) * 4u;
            }
            e[0] = (int32_t)((unsigned)desc->dur[kind * S + s] << 8);
            e[1] = (int32_t)((comm << 8) - tag);
            e[2] = (int32_t)((unsigned)need_of[kind] | ((unsigned)(need_of[kind] ^ next_of[kind]) << 8) | (prod << 16));
            e[3] = (int32_t)((allocs ? units : 0u) | ((frees ? units : 0u) << 8) | ((unsigned)s << 16) | (has_in << 24));
          }
      for (int dir = 0; dir < 2 && deg2; ++dir)
        for (int c = 0; c < kMaxChunks; ++c)
          for (int d = 0; d < D; ++d) {
            if (c >= p->n_chunks[d]) continue;
            const int s = p->local_stage[(size_t)d * kMaxChunks + c];
            int32_t* e = &J[(size_t)n_meta + (((size_t)dir * kMaxChunks + c) * lpc + d) * 2];
            unsigned y = 0;
            if (dir == 0) {
              if (poff[s + 1] - poff[s] > 1) { y |= kMetaHasCons; e[0] = (int32_t)(((unsigned)pcm[poff[s] + 1] << 8) - (unsigned)pst[poff[s] + 1]); }
              if (soff[s + 1] - soff[s] > 1) y |= kMetaHasProd | ((unsigned)((n_classes + scl[soff[s] + 1]) * m) * 4u);
            } else {
              if (soff[s + 1] - soff[s] > 1) { y |= kMetaHasCons; e[0] = (int32_t)(((unsigned)scm[soff[s] + 1] << 8) - (unsigned)sst[soff[s] + 1]); }
              if (poff[s + 1] - poff[s] > 1) y |= kMetaHasProd | ((unsigned)(pcl[poff[s] + 1] * m) * 4u);
            }
            e[1] = (int32_t)y;
          }
      for (int d = 0; d < D; ++d) {
        // state words of device d once every activation placed on it is consumed
        int32_t* x = &J[(size_t)n_shared + (size_t)lpc * dev_ints + (size_t)d * state_words];
        const unsigned terminal = p->has_w ? kDone : kBDone;
        for (int c = 0; c < p->n_chunks[d]; ++c)
          for (int j = 0; j < m; ++j)
            x[c * words_per_chunk + (j >> 3)] |= (int32_t)(terminal << ((j & 7) * 4));
      }
      for (int d = 0; d < D; ++d) {
        int32_t* e = &J[(size_t)n_shared + (size_t)d * dev_ints];
        e[0] = p->n_chunks[d];
        e[1] = (int32_t)(desc->mem_cap[d] / unit_scale);   // peak > cap  <=>  peak / scale > floor(cap / scale)
        for (int c = 0; c < p->n_chunks[d]; ++c) {
          const int s = p->local_stage[(size_t)d * kMaxChunks + c];
          const int nin = poff[s + 1] - poff[s], nout = soff[s + 1] - soff[s];
          e[2 + c] = nin > 0 ? (n_classes + pcl[poff[s]]) * m : 0;
          e[2 + V + c] = nout > 0 ? scl[soff[s]] * m : 0;
          e[2 + 2 * V + c] = nin > 1 ? (n_classes + pcl[poff[s] + 1]) * m : 0;
          e[2 + 3 * V + c] = nout > 1 ? scl[soff[s] + 1] * m : 0;
        }
      }
      ST.D = D; ST.m = m; ST.lanes_per_cand = lpc; ST.n_classes = n_classes;
      ST.slots_per_cand = slot_stride;
      ST.unit_scale = (int32_t)unit_scale;
      ST.state_words = state_words;
      ST.off_expect = n_shared + lpc * dev_ints;
      ST.n_shared_ints = n_shared;
      ST.off_meta2 = n_meta;
      ST.off_dev = n_shared;
      ST.dev_ints = dev_ints;
      ST.link_words = 0;
      const SlotGeometry geo = slot_geometry(ST.n_shared_ints, lpc, ST.state_words, ST.slots_per_cand, max_lds);
      const int scpw = geo.cands_per_wave, best_waves = geo.waves, best_groups = geo.groups;
      const int64_t wave_ints = geo.wave_ints;
      p->slots_ok = fits && best_waves >= 1;
      ST.cands_per_wave = scpw;
      ST.wave_ints = (int32_t)wave_ints;
      p->slot_waves = best_waves;
      p->slot_lds_bytes = (int32_t)(4ll * (ST.n_shared_ints + (int64_t)best_waves * wave_ints));
      int n_cu = 0;
      if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, p->device_id) != hipSuccess || n_cu < 1) {
        delete p; return FPSCHED_EHIP;
      }
      p->slot_grid = n_cu * std::max(best_groups, 1);
      p->n_cu = n_cu;
    }
    std::vector<int32_t> list_image;
    {
      std::vector<StageEdges> se(S);
      for (int e = 0; e < E; ++e) {
        const int a = desc->edge_src[e], b = desc->edge_dst[e];
        const int32_t lat = p->stage_device[a] != p->stage_device[b] ? desc->edge_comm[e] : 0;
        se[a].out[0].push_back({edge_cls[e], b, lat});
        se[b].in[0].push_back({edge_cls[e], a, lat});
        se[a].in[1].push_back({edge_cls[e], b, lat});
        se[b].out[1].push_back({edge_cls[e], a, lat});
      }
      build_list_tables(p, se, n_classes, (int64_t)D * max_stride_words * (max_dur + max_comm), &list_image);
    }
    if (!p->general_ok && !p->lists_ok) { delete p; return FPSCHED_EUNSUPPORTED; }
    p->use_slots = p->lists_ok;
    if (hipMalloc(&p->d_ints, I.size() * sizeof(int32_t)) != hipSuccess) { delete p; return FPSCHED_ENOMEM; }
    bool ok = hipMemcpy(p->d_ints, I.data(), I.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess;
    if (ok && p->general_ok)
      ok = hipFuncSetAttribute(reinterpret_cast<const void*>(&eval_general_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess;
    if (ok && p->lists_ok) {
      ok = hipMalloc(&p->d_list_ints, list_image.size() * sizeof(int32_t)) == hipSuccess &&
           hipMemcpy(p->d_list_ints, list_image.data(), list_image.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess;
      for (const void* kernel : {reinterpret_cast<const void*>(check_kernel_of(p->check_vbits, false, false)),
                                 reinterpret_cast<const void*>(check_kernel_of(p->check_vbits, false, true)),
                                 reinterpret_cast<const void*>(alone_kernel_of(p->check_vbits, p->lists_deg2, p->lists_wide)),
                                 reinterpret_cast<const void*>(time_kernel_of(p->ltab, p->lists_deg2, p->lists_wide))})
        ok = ok && (!kernel || hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess);
      p->ltab.ints = p->d_list_ints;
      p->list_image = list_image;
    }
    if (ok && p->slots_ok) {
      ok = hipMalloc(&p->d_slot_ints, p->slot_ints.size() * sizeof(int32_t)) == hipSuccess &&
           hipMemcpy(p->d_slot_ints, p->slot_ints.data(), p->slot_ints.size() * sizeof(int32_t),
                     hipMemcpyHostToDevice) == hipSuccess;
      p->stab.ints = p->d_slot_ints;
      // The sliding pass times the lists without their W items with the evaluation kernel's TIMES
      // form: the same tables, except that a W word is a no-op (any state, no cost, no memory) and a
      // (stage, micro-batch) is finished once its B item ran.
      if (ok && p->has_w) {
        std::vector<int32_t> J = p->slot_ints;
        const int lpc = p->stab.lanes_per_cand;
        for (int c = 0; c < kMaxChunks; ++c)
          for (int d = 0; d < D; ++d) {
            if (c >= p->n_chunks[d]) continue;
            int32_t* e = &J[(((size_t)kW * kMaxChunks + c) * lpc + d) * 4];
            e[0] = 0;
            e[1] = 0;
            e[2] = (int32_t)((unsigned)e[2] & 0xffff0000u);   // required state 0, no transition, same output slot
            e[3] = (int32_t)((unsigned)e[3] & 0x00ff0000u);   // own stage only
          }
        const int words_per_chunk = (m + 7) / 8;
        for (int d = 0; d < D; ++d) {
          int32_t* x = &J[(size_t)p->stab.off_expect + (size_t)d * p->stab.state_words];
          for (int i = 0; i < p->stab.state_words; ++i) x[i] = 0;
          for (int c = 0; c < p->n_chunks[d]; ++c)
            for (int j = 0; j < m; ++j) x[c * words_per_chunk + (j >> 3)] |= (int32_t)((unsigned)kBDone << ((j & 7) * 4));
        }
        p->stab_times = p->stab;
        p->times_ints = J;
        const bool up = hipMalloc(&p->d_times_ints, J.size() * sizeof(int32_t)) == hipSuccess &&
                        hipMemcpy(p->d_times_ints, J.data(), J.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess &&
                        hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotTimes>(p->slot_v, p->slot_deg2, p->stab.n_classes == 1)),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess &&
                        hipFuncSetAttribute(reinterpret_cast<const void*>(&wslide_place_rows_kernel),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess &&
                        hipFuncSetAttribute(reinterpret_cast<const void*>(p->slot_v > 2 ? &wslide_place_kernel<true> : &wslide_place_kernel<false>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess;
        if (up) {
          p->stab_times.ints = p->d_times_ints;
          p->slide_ok = true;
          // ... or, on the plain model, the two passes of the list evaluation do, with the same change to their tables
          // (without them the slot kernel stays in use)
          if (p->lists_ok && !p->lists_deg2 && !p->lists_wide && build_times_variant(p) != FPSCHED_OK) (void)hipGetLastError();
          // the one-kernel form: the same image, and behind it per device the cost << 8 of the W item of each
          // chunk, the units it frees, and the cost << 8 of all W items of the device
          std::vector<int32_t> JS = J;
          const int32_t off_w = (int32_t)JS.size();
          JS.resize(JS.size() + (size_t)lpc * (2 * kMaxChunks + 1), 0);
          for (int d = 0; d < D; ++d) {
            int32_t* w = &JS[(size_t)off_w + (size_t)d * (2 * kMaxChunks + 1)];
            int64_t total = 0;
            for (int c = 0; c < p->n_chunks[d]; ++c) {
              const int s = p->local_stage[(size_t)d * kMaxChunks + c];
              w[c] = (int32_t)((unsigned)desc->dur[kW * S + s] << 8);
              w[kMaxChunks + c] = (int32_t)(desc->mem_units[s] / p->stab.unit_scale);
              total += (int64_t)m * desc->dur[kW * S + s];
            }
            w[2 * kMaxChunks] = (int32_t)((uint32_t)total << 8);   // (below 2^24: the slot form's bound on all times)
          }
          p->slide_w_table.assign(JS.begin() + off_w, JS.end());
          if (hipMalloc(&p->d_slide_ints, JS.size() * sizeof(int32_t)) == hipSuccess &&
              hipMemcpy(p->d_slide_ints, JS.data(), JS.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess &&
              hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotSlide>(p->slot_v, p->slot_deg2, p->stab.n_classes == 1)),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess) {
            p->stab_slide = p->stab_times;
            p->stab_slide.ints = p->d_slide_ints;
            p->stab_slide.off_w = off_w;
            p->slide_eval_ok = true;
          } else {
            (void)hipGetLastError();
            if (p->d_slide_ints) { (void)hipFree(p->d_slide_ints); p->d_slide_ints = nullptr; }
          }
        } else {
          (void)hipGetLastError();
          if (p->d_times_ints) { (void)hipFree(p->d_times_ints); p->d_times_ints = nullptr; }
        }
      }
    }
    if (!ok) {
      (void)hipFree(p->d_ints);
      if (p->d_list_ints) (void)hipFree(p->d_list_ints);
      if (p->d_slot_ints) (void)hipFree(p->d_slot_ints);
      if (p->d_times_ints) (void)hipFree(p->d_times_ints);
      if (p->d_slide_ints) (void)hipFree(p->d_slide_ints);
      delete p;
      return FPSCHED_EHIP;
    }
    T.ints = p->d_ints;
  }
  *out = p;
  return FPSCHED_OK;
}

void fpsched_problem_destroy(fpsched_problem* p) {
  if (!p) return;
  if (p->d_ints || p->d_slot_ints || p->d_sync_ints) {
    DeviceGuard g(p->device_id);
    if (p->d_ints) (void)hipFree(p->d_ints);
    if (p->d_list_ints) (void)hipFree(p->d_list_ints);
    if (p->d_slot_ints) (void)hipFree(p->d_slot_ints);
    if (p->d_slide_ints) (void)hipFree(p->d_slide_ints);
    if (p->d_sync_slot_image) (void)hipFree(p->d_sync_slot_image);
    if (p->d_times_ints) (void)hipFree(p->d_times_ints);
    if (p->d_mb_raw) (void)hipFree(p->d_mb_raw);
    if (p->d_mb_rows) (void)hipFree(p->d_mb_rows);
    for (ListVariant* v : {&p->lists_links, &p->lists_mb, &p->lists_both, &p->lists_sync, &p->lists_copy, &p->lists_copy_deep, &p->lists_times})
      if (v->d_image) (void)hipFree(v->d_image);
    if (p->d_times_links_image) (void)hipFree(p->d_times_links_image);
    if (p->d_slide_links_image) (void)hipFree(p->d_slide_links_image);
    if (p->d_sync_ints) (void)hipFree(p->d_sync_ints);
  }
  delete p;
}

int fpsched_problem_info(const fpsched_problem* p, int32_t* lanes_per_candidate,
                         int32_t* candidates_per_wave, int32_t* lds_bytes_per_wave) {
  if (!p) return FPSCHED_EINVAL;
  const bool slots = p->use_slots;
  if (lanes_per_candidate) *lanes_per_candidate = slots ? (p->D + 1) / 2 : p->tables.lanes_per_cand;
  if (candidates_per_wave) *candidates_per_wave = slots ? p->ltab.cands_per_wave : p->tables.cands_per_wave;
  if (lds_bytes_per_wave) *lds_bytes_per_wave = slots ? 4 * p->ltab.n_time_ints / std::max(p->time_waves, 1) + p->ltab.wave_bytes : p->lds_bytes;
  return FPSCHED_OK;
}

int fpsched_problem_select_kernel(fpsched_problem* p, int which) {
  if (!p) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (which == FPSCHED_KERNEL_AUTO) p->use_slots = p->lists_ok;
  else if (which == FPSCHED_KERNEL_GENERAL) { if (!p->general_ok) return FPSCHED_EUNSUPPORTED; p->use_slots = false; }
  else if (which == FPSCHED_KERNEL_SLOTS) { if (!p->lists_ok) return FPSCHED_EUNSUPPORTED; p->use_slots = true; }
  else return FPSCHED_EINVAL;
  return FPSCHED_OK;
}

int fpsched_problem_active_kernel(const fpsched_problem* p) {
  if (!p) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (p->sync_on) return p->use_slots && p->sync_slots_ok ? FPSCHED_KERNEL_SLOTS : FPSCHED_KERNEL_GENERAL;
  if (p->copy_depth > 0) return p->use_slots && p->copy_slots_ok ? FPSCHED_KERNEL_SLOTS : FPSCHED_KERNEL_GENERAL;
  return p->use_slots && (!p->mb_set || p->mb_slots_ok) ? FPSCHED_KERNEL_SLOTS : FPSCHED_KERNEL_GENERAL;
}

size_t fpsched_workspace_bytes(const fpsched_problem* p, int64_t n_cand, int32_t k) {
  if (!p || n_cand < 0) return 0;
  // survivors of the top-k's first launch (at most k per tile of candidates), and a second buffer in proportion
  int64_t keys = 0;
  if (k > 0) {
    const int64_t per_part = std::min(k, 1024);
    const int64_t first = std::max<int64_t>(1, (n_cand + kTile - 1) / kTile) * per_part;
    keys = first + std::max<int64_t>(1, (first + kTile - 1) / kTile) * per_part;
  }
  return (size_t)(256 + keys * (int64_t)sizeof(Key));
}

// Candidates per atomic draw from a launch's work counter.  Atomics on one address complete at some 8e7 per second; a
// batch of long candidates stays far below that and is drawn one by one (best balance at the end of the batch), short
// rows are drawn several at a time: about one draw per 12 K op words.
static int draws_at_a_time(const fpsched_problem* p, int32_t stride_words, int cands_per_wave) {
  const int64_t row_words = (int64_t)p->D * stride_words;
  return (int)std::clamp<int64_t>((12288 + row_words - 1) / row_words, 1, cands_per_wave);
}

// ... and the timing pass, while many are left: a draw is a wait of some 4,500 clocks for a wavefront, whose segments need
// one every sixth of their top-ups or so; so a part of the wavefront's share of what is left is drawn at a time, up to one a segment:
// half of it, or a quarter on rows of 192 words and more where a step also asks for link words and has no branches (such a step waits
// for more than the draw gives back, and a wavefront that has drawn more than its equals ends later, the more so the longer its
// candidates).  Candidates of more than 16 K words are worth the wait and better drawn one by one.  Whole evaluation against one draw
// per 12 K words, a quarter / half / three quarters of the share, mean over batches of 1.3 to 9 candidates a segment, 14 problems of 2
// to 32 devices, 20 to 64 micro-batches:
//   plain model 0.96 to 1.00 / 0.93 to 1.005 / 0.91 to 1.003 (16 x 64 x 2 0.980 / 0.958 / 0.952; 262,144 of it 2605, 2408, 2395,
//   2412 us); at worst, 1.3 a segment of 2 x 64 x 1, 1.03 / 1.06 / 1.05;
//   links, with and without costs, no second edges, rows of 192 words and more 0.993 to 1.003 / 0.991 to 1.026 / 0.993 to 1.035
//   (configuration 3 3004, 2969, 2996, 3028 us, with costs 3353, 3328, 3381, 3415; at worst 1.02 / 1.08 / 1.09), of 120 words 0.994 to 1.003 /
//   0.987 to 1.001 / 0.98 to 1.002; with second edges 0.98 to 0.99 / 0.98 to 0.99 / 0.97 to 0.99;
//   costs per micro-batch 0.975 to 1.001 / 0.955 to 1.013 (12 x 40 x 4; 11 x 45 x 3 1.006) / 0.94 to 1.02;
//   synchronisation 1.00 / 0.995 to 1.0 / 1.0, copy engine 0.99 to 1.00 / 0.99 to 1.00 / 0.98 to 1.00.
// 65,536 of 32 x 128 x 2: 2597, 2586, 2663, 2661 us, under links 3657, 3674, 3771, 3839.
static uint32_t drawn_share(const fpsched_problem* p, const ListTables& T, bool deg2, int32_t stride_words, int64_t waves) {   // (times 2^32)
  const int64_t part = (int64_t)p->D * stride_words > 16384 ? 0 : 1ll << (T.link_words > 0 && !deg2 && stride_words >= 192 ? 30 : 31);
  return (uint32_t)((part + waves - 1) / waves);
}

// the two-pass list evaluation: the order pass over all rows, then the timing pass on a persistent grid
// (variant: its tables and launch shape under link occupancy or costs per micro-batch; null: the plain model; starts: what
// the first pass of the sliding pass leaves, with its variant)
static int run_list_evaluation(const fpsched_problem* p, const ListVariant* variant, const uint16_t* d_ops, int64_t n_cand, int32_t stride_words,
                               const fpsched_results& out, unsigned long long* counter, hipStream_t st,
                               const StartTimes* starts = nullptr) {
  ListTables T = variant ? variant->tab : p->ltab;
  const int64_t n_rows = n_cand * p->D, rpw = p->check_rows_per_wave;
  const int64_t n_cu = std::max(p->n_cu, 1), each = (n_cand + 4 * n_cu - 1) / (4 * n_cu);   // candidates for each SIMD
  // Both passes in one launch where every wavefront has room for the rows and the lanes of its share, with one wavefront per SIMD, or two.  Two
  // launches / one, 1,024 to 16,384 candidates, one wavefront per SIMD: 1.00 to 1.14 on 2 to 12 devices (at worst 0.99, 4 x 32 x 2; four stages: below), 1.01 to
  // 1.06 on 16, 1.04 to 1.11 on 24 to 40.  Two: 1.04 to 1.15 where the timing rows have no columns (12, 24, 40 devices), 1.1 on
  // 4 x 8 x 1; with columns and rows of 192 words and more 0.98 (8 x 32 x 2), 0.99 and 1.00 (16 x 64 x 2), 0.99 and 1.00 (32 x 128 x 2), 1.06 (32 x 64 x
  // 1).  (A handful of candidates, which is no batch, stays with the two.)
  const TimeKernel alone = variant ? nullptr : alone_kernel_of(p->check_vbits, p->lists_deg2, p->lists_wide);
  // Candidates of a wavefront: a SIMD's share; a compute unit's with four stages on up to six devices and no more than sixteen for each
  // (a step of one candidate costs LDS as much as one of four, and the chain of so many ops waits for it.  Two launches / one with a SIMD's
  // share / with a compute unit's, 1,024 of 4 x 80 x 4 282, 287 and 277 us, of 2 x 60 x 4 176, 177 and 171, 4,096 288, 294 and 285, 180, 182
  // and 176; 1,024 of 6 x 60 x 4 under links 362, 370 and 360; but of 3 x 40 x 3 121, 118 and 117, of 6 x 40 x 3 168, 159 and 163, of 4 x 60 x 2
  // 139, 129 and 130, of 8 x 40 x 3 204, 192 and 198, and 6,000 of 3 x 60 x 4 231, 217 and 223.)
  const int64_t share = T.chunks > 3 && T.D <= 6 && n_cand <= 16 * n_cu ? (n_cand + n_cu - 1) / n_cu : each;
  const int64_t room = std::min<int64_t>(64 / p->D, T.cands_per_wave), together = std::min(share, room);
  // (One or two devices are with those with columns: their rows are not in each other's way either)
  const bool columns = T.D <= 2 || T.odd_at != 16 * ((T.D + 1) / 2);
  if (alone && n_cand >= kAloneLeast && n_cand <= std::min(each, room) * n_cu * (columns && stride_words > 128 ? 4 : 8)) {
    ListTables A = T;
    const int64_t wavefronts = (n_cand + together - 1) / together;
    const int waves = (int)((wavefronts + n_cu - 1) / n_cu);
    A.cands_per_wave = (int)together;
    A.check_columns = std::min(T.check_columns, next_pow2(T.D));
    A.check_wave_bytes = ((int)together * T.D * T.state_bytes + 15) & ~15;
    A.wave_bytes = (kTimeWindowBytes + (int)together * (p->lists_wide ? 8 : 4) * T.cand_slots + 31) & ~31;
    const int64_t lds = alone_check_bytes(A, waves) + list_table_bytes(T) + (int64_t)waves * A.wave_bytes;
    if (lds <= p->max_lds) {
      hipLaunchKernelGGL(alone, dim3((unsigned)((wavefronts + waves - 1) / waves)), dim3(64 * waves), (size_t)lds, st, A, d_ops, (long long)n_cand,
                         (int)stride_words, reinterpret_cast<long long*>(out.makespan), reinterpret_cast<long long*>(out.idle), out.peak, out.flags, (unsigned long long*)nullptr,
                         1, 0u, StartTimes{});
      return check_hip(hipGetLastError());
    }
  }
  // (A wavefront's share, one candidate mostly, where there are no more than SIMDs: 800 of 11 x 45 x 2, links 163 and 152 us, costs 146 and 134, in
  // microseconds 128 and 119; with two for each SIMD no such gain, 2,048 of 4 x 32 x 2 67.6 and 68.9.  One workgroup to a compute unit,
  // whose wavefronts have a SIMD each, which those of two workgroups of two have not: 1,024 with costs, full wavefronts, two workgroups
  // and one, 7 x 20 x 3 122, 127 and 116 us, 5 x 20 x 3 98.7, 104.6 and 95.8, 9 x 24 x 3 168, 176 and 159; 600 of two towers, copy engine,
  // 245, 219 and 210.  It has no more wavefronts than a compute unit had room for in several workgroups.)
  int64_t grid = variant ? variant->grid : p->time_grid, max_waves = variant ? variant->waves : p->time_waves;
  if (each == 1 && n_cand <= grid * max_waves) {
    T.cands_per_wave = (int)std::min<int64_t>(share, T.cands_per_wave);
    grid = n_cu;
    max_waves = std::max(max_waves, (n_cand + n_cu - 1) / n_cu);
  }
  // (a small batch is spread over the compute units: fewer wavefronts per workgroup)
  const int64_t row_waves = (n_rows + rpw - 1) / rpw;
  const int cw = (int)std::clamp<int64_t>((row_waves + p->check_grid - 1) / p->check_grid, 1, p->check_waves);
  const int64_t check_blocks = std::min<int64_t>((row_waves + cw - 1) / cw, p->check_grid);
  const int64_t cpw = T.cands_per_wave;
  const int tw = (int)std::clamp<int64_t>((n_cand + cpw * grid - 1) / (cpw * grid), 1, max_waves);
  const int64_t time_blocks = std::min<int64_t>((n_cand + cpw * tw - 1) / (cpw * tw), grid);
  long long* idle = reinterpret_cast<long long*>(out.idle);
  // segment g starts on candidate g, wavefront w of the order pass on block w of rows; the counters hand out those behind
  const unsigned long long first_drawn = (unsigned long long)(time_blocks * cpw * tw);
  // (About four draws per wavefront even out the last blocks; with as many as there are blocks the counter's address is
  // what the pass waits for.  Up to eight blocks per wavefront are shared out equally.  Equal shares against draws of one
  // block, whole evaluation, 32 shapes of 2 to 40 devices with 2 to 31 blocks per wavefront: rows of up to 100 words 59
  // and 107 us (65,536 candidates of 4 x 8 x 1), 216 and 343 us (262,144 of 3 x 20 x 1); rows of 192 to 1,000 words 322
  // and 388 us (65,536 of 8 x 32 x 2) at best and 3 % worse at worst; 12 % worse on 24 x 100 x 4, whose rows of 1,200 words
  // leave room for four wavefronts.  Two, four, eight or sixteen draws beyond eight blocks: within 3 % of each other on
  // rows of 192 words and more.)
  const int64_t check_waves = check_blocks * cw, per_wave = (row_waves + check_waves - 1) / check_waves;
  const int draw_blocks = (int)(per_wave <= 8 ? per_wave : per_wave / 4);
  const bool dynamic = row_waves > check_waves * draw_blocks;
  // (Copies of the columns cost a workgroup more than they save in one block of rows: the pass, with and without them, 1,024 candidates of
  // 4 x 8 x 1 under links 5.5 and 5.1 us, 20,000 of 2 x 32 x 2 17.2 and 16.0, 8,192 of 4 x 32 x 2 14.6 and 14.2, on 16 and 32 devices the same)
  ListTables check = T;
  if (row_waves <= check_waves) check.check_columns = std::min(T.check_columns, next_pow2(T.D));
  // (How the rows are read, see there)
  const bool shared = (row_waves + draw_blocks - 1) / draw_blocks > 8 * (int64_t)p->n_cu && check_waves > 8 * (int64_t)p->n_cu && stride_words >= 64;
  if (dynamic) {
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, st, counter, first_drawn, (unsigned long long)(check_waves * draw_blocks));
    if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  }
  hipLaunchKernelGGL(check_kernel_of(p->check_vbits, starts != nullptr, shared), dim3((unsigned)check_blocks), dim3(64 * cw),
                     (size_t)(T.check_shared_bytes + (int64_t)cw * T.check_wave_bytes), st, check, d_ops, (long long)n_rows,
                     (int)stride_words, (int)rpw, idle, out.peak, counter, first_drawn, draw_blocks, (int)dynamic);
  if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  const bool deg2 = variant ? variant->deg2 : p->lists_deg2;
  hipLaunchKernelGGL(starts ? times_kernel() : time_kernel_of(T, deg2, p->lists_wide && !variant), dim3((unsigned)time_blocks),
                     dim3(64 * tw), (size_t)(list_table_bytes(T) + (int64_t)tw * T.wave_bytes), st, T, d_ops,
                     (long long)n_cand, (int)stride_words, reinterpret_cast<long long*>(out.makespan), idle, out.peak,
                     out.flags, counter, draws_at_a_time(p, stride_words, T.cands_per_wave), drawn_share(p, T, deg2, stride_words, time_blocks * tw), starts ? *starts : StartTimes{});
  return check_hip(hipGetLastError());
}

static int max_chunks_of(const fpsched_problem* p) {
  int max_chunks = 0;
  for (int d = 0; d < p->D; ++d) max_chunks = std::max(max_chunks, p->n_chunks[d]);
  return max_chunks;
}

// Copy engine: the two passes or the one kernel.  The two passes have the cheaper steps, the more so the fewer transfers a lane keeps,
// on half the lanes, and an order pass and a launch more; the one kernel has its candidates side by side in wavefronts until the chip
// is full (`resident`), and takes another turn for the rest.  Measured over 2 to 40 devices, 6 to 64 micro-batches, 1 to 4 stages per
// device, 256 to 65,536 candidates, one kernel / two passes, depths up to 3, 4, and 5 to 7:
//   more than one turn: 1.1 (65,536 of 32 x 8 x 1) to 2.6, 1.07 to 2.4, 0.99 (32 x 8 x 1) to 2.1;
//   one turn, rows of 96 items and more: 1.04 to 1.36, 0.97 (8,192 of 16 x 48 x 1: 1.00) to 1.31, and at two or more stages per device 1.0 to
//   1.18, at one 0.83 to 1.02; two devices, which are a lane per candidate in the one and two in the other: 1.0 to 1.03, 0.96 to 1.01, 0.83 to 0.87;
//   one turn, shorter rows: 0.99 (3 x 6 x 2) to 1.13, 0.95 to 1.09, 0.82 to 0.96; but where some stage has a second input or output, at depths
//   up to 3, 0.92 to 1.0 below 64 items and 1.03 to 1.07 from there on (towers with 8 to 18, and 24 and 30 micro-batches), and 0.88 to
//   0.98 on two devices.
static bool copy_takes_two_passes(const fpsched_problem* p, int64_t n_cand) {
  const int64_t resident = (int64_t)p->copy_grid * p->copy_waves * p->stab_copy.cands_per_wave;
  const int64_t items = (int64_t)max_chunks_of(p) * p->m * (p->has_w ? 3 : 2);
  if (n_cand > resident) return true;
  if (p->D <= 2) return false;
  return p->copy_depth <= kCopyShallow ? items >= 64 || !p->lists_deg2 : items >= 96 && (p->copy_depth == 4 || max_chunks_of(p) > 1);
}

int fpsched_evaluate(const fpsched_problem* p, const uint16_t* d_ops, int64_t n_cand,
                     int32_t stride_words, fpsched_results out, void* d_workspace,
                     size_t workspace_bytes, void* hip_stream) {
  if (!p || n_cand < 0) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (n_cand == 0) return FPSCHED_OK;
  if (!d_ops || !out.makespan || !out.idle || !out.peak || !out.flags) return FPSCHED_EINVAL;
  if (stride_words < 8 || (stride_words & 7) || stride_words > p->max_stride) return FPSCHED_EINVAL;
  if (reinterpret_cast<uintptr_t>(d_ops) & 15) return FPSCHED_EINVAL;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  // Rows too long for the timing pass's positions: the other kernels.  (Link occupancy needs D * stride * (the largest cost + two
  // latencies) below 2^24: such rows have a single device, or no costs and latencies at all, and the plain model's results.)
  const bool two_passes = stride_words <= kTimeMaxStride;
  const bool copy_on_slots = p->copy_depth > 0 && p->use_slots && p->copy_slots_ok;
  const bool sync_on_slots = p->sync_on && p->use_slots && p->sync_slots_ok && (two_passes || !p->lists_sync.ok);
  if ((p->sync_on || p->copy_depth > 0) && !copy_on_slots && !sync_on_slots) {
    const int cpw = p->sync_tab.cands_per_wave;
    const int64_t blocks = (n_cand + cpw - 1) / cpw;
    if (blocks > 0x7fffffffll) return FPSCHED_EINVAL;
    hipLaunchKernelGGL(p->copy_depth > 0 ? eval_sync_kernel<true> : eval_sync_kernel<false>, dim3((unsigned)blocks), dim3(64), (size_t)p->sync_lds_bytes,
                       static_cast<hipStream_t>(hip_stream), p->sync_tab, d_ops, (long long)n_cand,
                       (int)stride_words, reinterpret_cast<long long*>(out.makespan),
                       reinterpret_cast<long long*>(out.idle), out.peak, out.flags);
    return check_hip(hipGetLastError());
  }
  if (p->links_on && !p->use_slots) return FPSCHED_EUNSUPPORTED;   // the general kernel has no link form
  // (times or latencies beyond the 24-bit forms: the general kernel, which needs no workspace, takes calls without one)
  const bool usable_workspace = d_workspace && (reinterpret_cast<uintptr_t>(d_workspace) & 15) == 0 && workspace_bytes >= 256;
  const bool without_workspace = !usable_workspace && !p->slots_ok && p->general_ok;
  const bool rows_fit = two_passes || copy_on_slots || sync_on_slots || (p->mb_set && !p->links_on && !p->lists_mb.ok);
  if (!rows_fit && !p->general_ok) return FPSCHED_EUNSUPPORTED;
  if (copy_on_slots || sync_on_slots || (p->use_slots && (!p->mb_set || p->mb_slots_ok) && !without_workspace && rows_fit)) {
    // the first 8 bytes of the workspace hold the counter the segments draw candidates from
    if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
    if (workspace_bytes < 256) return FPSCHED_ENOMEM;
    unsigned long long* counter = static_cast<unsigned long long*>(d_workspace);
    const ListVariant& copy_lists = p->copy_lists(p->copy_depth);
    if (copy_on_slots && two_passes && copy_lists.ok && copy_takes_two_passes(p, n_cand))
      return run_list_evaluation(p, &copy_lists, d_ops, n_cand, stride_words, out, counter, static_cast<hipStream_t>(hip_stream));
    if (sync_on_slots && p->lists_sync.ok)
      return run_list_evaluation(p, &p->lists_sync, d_ops, n_cand, stride_words, out, counter, static_cast<hipStream_t>(hip_stream));
    if (!copy_on_slots && !sync_on_slots) {
      const ListVariant* variant = p->links_on ? (p->mb_set ? &p->lists_both : &p->lists_links) : (p->mb_set ? &p->lists_mb : nullptr);
      if (!variant || variant->ok)
        return run_list_evaluation(p, variant, d_ops, n_cand, stride_words, out, counter, static_cast<hipStream_t>(hip_stream));
      if (p->links_on) return FPSCHED_EUNSUPPORTED;   // (the setters made sure that it is there)
    }
    // copy engine, synchronisation stages; costs per micro-batch whose table does not fit LDS
    const SlotTables& tab = sync_on_slots ? p->stab_sync : copy_on_slots ? p->stab_copy : p->stab;
    const int waves = sync_on_slots ? p->sync_slot_waves : copy_on_slots ? p->copy_waves : p->slot_waves;
    const int grid = sync_on_slots ? p->sync_slot_grid : copy_on_slots ? p->copy_grid : p->slot_grid;
    const size_t lds_bytes = (size_t)(sync_on_slots ? p->sync_slot_lds_bytes : copy_on_slots ? p->copy_lds_bytes : p->slot_lds_bytes);
    const SlotLaunch L = slot_launch(tab, waves, grid, lds_bytes, n_cand);
    const int per_block = tab.cands_per_wave * L.waves;
    const int64_t blocks = L.blocks;
    // Candidates per atomic draw.  Atomics on one address complete at some 8e7 per second; a batch of
    // long candidates stays far below that and is drawn one by one (best balance at the end of the
    // batch), short rows are drawn several at a time: about one draw per 12 K op words.
    const int64_t row_words = (int64_t)p->D * stride_words;
    const int draw_block = (int)std::clamp<int64_t>((12288 + row_words - 1) / row_words, 1, tab.cands_per_wave);
    // segment g starts on candidate g; the counter hands out the candidates after those
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(hip_stream), counter,
                       (unsigned long long)(blocks * per_block), 0ull);
    const bool one_class = tab.n_classes == 1;
    const SlotKernel kernel = sync_on_slots ? slot_kernel_of<kSlotSync>(p->slot_v, p->sync_deg2, one_class)
                              : copy_on_slots ? slot_kernel_of<kSlotCopy>(p->slot_v, p->slot_deg2, one_class)
                              : slot_kernel_of<kSlotPerMicrobatch>(p->slot_v, p->slot_deg2, one_class);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(64 * L.waves), L.lds_bytes,
                       static_cast<hipStream_t>(hip_stream), tab, d_ops,
                       (long long)n_cand, (int)stride_words, reinterpret_cast<long long*>(out.makespan),
                       reinterpret_cast<long long*>(out.idle), out.peak, out.flags, counter, draw_block,
                       (uint32_t*)nullptr, (int32_t*)nullptr,
                       (const int32_t*)(p->mb_set ? p->d_mb_rows : nullptr), (uint32_t*)nullptr, 0);
    return check_hip(hipGetLastError());
  }
  const int cpw = p->tables.cands_per_wave;
  const int64_t blocks = (n_cand + cpw - 1) / cpw;
  if (blocks > 0x7fffffffll) return FPSCHED_EINVAL;
  hipLaunchKernelGGL(eval_general_kernel, dim3((unsigned)blocks), dim3(64), (size_t)p->lds_bytes,
                     static_cast<hipStream_t>(hip_stream), p->tables, d_ops, (long long)n_cand,
                     (int)stride_words, reinterpret_cast<long long*>(out.makespan),
                     reinterpret_cast<long long*>(out.idle), out.peak, out.flags,
                     (const int32_t*)(p->mb_set ? p->d_mb_raw : nullptr));
  return check_hip(hipGetLastError());
}

int fpsched_problem_set_microbatch_costs(fpsched_problem* p, const int32_t* dur_mb) {
  if (!p) return FPSCHED_EINVAL;
  if (!dur_mb) {
    p->mb_set = false;   // the tables stay allocated for the next call
    return FPSCHED_OK;
  }
  if (p->sync_on || p->copy_depth > 0) return FPSCHED_EUNSUPPORTED;   // those models know one cost per (type, stage)
  const int D = p->D, S = p->S, m = p->m;
  const size_t n_raw = (size_t)kNKinds * S * m;
  int64_t max_dur = 0;
  for (size_t i = 0; i < n_raw; ++i) {
    if (dur_mb[i] < 0) return FPSCHED_EINVAL;
    max_dur = std::max<int64_t>(max_dur, dur_mb[i]);
  }
  // (with links every item may add two transfers to the longest chain)
  const int64_t bound = (int64_t)D * p->max_stride * (max_dur + (p->links_on ? 2 : 1) * p->max_comm);
  if (bound >= (int64_t)1 << 31) return FPSCHED_EOVERFLOW;
  const bool fits_slots = bound < (1ll << 24);
  if (p->device_id < 0) {
    p->mb_set = true;
    p->mb_slots_ok = fits_slots;
    p->mb_max_dur = max_dur;
    return FPSCHED_OK;
  }
  if (p->links_on && !(p->slots_ok && fits_slots)) return FPSCHED_EUNSUPPORTED;   // the link form is the slot kernel's
  if (!(p->slots_ok && fits_slots) && !p->general_ok) return FPSCHED_EUNSUPPORTED;
  const int lpc = p->tables.lanes_per_cand;
  const size_t n_rows = (size_t)kNKinds * kMaxChunks * lpc * m;
  std::vector<int32_t> rows(n_rows, 0);
  for (int kind = 1; kind < kNKinds; ++kind)
    for (int c = 0; c < kMaxChunks; ++c)
      for (int d = 0; d < D; ++d) {
        if (c >= p->n_chunks[d]) continue;
        const int s = p->local_stage[(size_t)d * kMaxChunks + c];
        for (int j = 0; j < m; ++j)
          rows[(((size_t)kind * kMaxChunks + c) * lpc + d) * m + j] =
              fits_slots ? (int32_t)((unsigned)dur_mb[((size_t)kind * S + s) * m + j] << 8) : 0;
      }
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  // work that reads the previous table must be over before it is overwritten
  if (hipDeviceSynchronize() != hipSuccess) return FPSCHED_EHIP;
  p->mb_set = false;   // a failure from here on leaves the handle on the costs of its description
  if (!p->d_mb_raw && hipMalloc(&p->d_mb_raw, n_raw * sizeof(int32_t)) != hipSuccess) { p->d_mb_raw = nullptr; return FPSCHED_ENOMEM; }
  if (!p->d_mb_rows && hipMalloc(&p->d_mb_rows, n_rows * sizeof(int32_t)) != hipSuccess) { p->d_mb_rows = nullptr; return FPSCHED_ENOMEM; }
  if (hipMemcpy(p->d_mb_raw, dur_mb, n_raw * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(p->d_mb_rows, rows.data(), n_rows * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess)
    return FPSCHED_EHIP;
  if (p->slots_ok && fits_slots &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotPerMicrobatch>(p->slot_v, p->slot_deg2, p->stab.n_classes == 1)),
                          hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) != hipSuccess)
    return FPSCHED_EHIP;
  p->mb_raw.assign(dur_mb, dur_mb + n_raw);
  p->lists_mb.ok = p->lists_both.ok = false;
  if (p->slots_ok && fits_slots) {
    if (!getenv("FPSCHED_MB_GLOBAL")) {
      const int rc = build_list_variant(p, false, dur_mb, &p->lists_mb);
      if (rc != FPSCHED_OK && rc != FPSCHED_EUNSUPPORTED) return rc;
    }
    if (p->links_on) {   // both variants: only with the table in LDS; else the handle stays on the links alone
      const int rc = build_list_variant(p, true, dur_mb, &p->lists_both);
      if (rc != FPSCHED_OK) return rc;
    }
  }
  p->mb_set = true;
  p->mb_slots_ok = p->slots_ok && fits_slots;
  p->mb_max_dur = max_dur;
  return FPSCHED_OK;
}

int fpsched_problem_set_link_occupancy(fpsched_problem* p, int32_t on) {
  if (!p) return FPSCHED_EINVAL;
  if (!on) {
    p->links_on = false;   // the table image stays allocated for the next call
    return FPSCHED_OK;
  }
  if (p->sync_on || p->copy_depth > 0) return FPSCHED_EUNSUPPORTED;   // those models read transfers as latencies
  const int D = p->D, S = p->S;
  // every finish time is at most the sum of all costs and of all transfers (at most two per op here)
  const int64_t bound = (int64_t)D * p->max_stride * ((p->mb_set ? p->mb_max_dur : p->max_dur) + 2 * p->max_comm);
  if (bound >= (int64_t)1 << 31) return FPSCHED_EOVERFLOW;
  if (p->device_id < 0) {
    p->links_on = true;
    return FPSCHED_OK;
  }
  if (!p->slots_ok || bound >= (1ll << 24)) return FPSCHED_EUNSUPPORTED;
  if (p->mb_set) {   // both variants
    const int rc = build_list_variant(p, true, p->mb_raw.data(), &p->lists_both);
    if (rc != FPSCHED_OK) return rc;
  }
  if (p->lists_links.ok) {   // built by an earlier call
    p->links_on = true;
    return FPSCHED_OK;
  }
  const int rc = build_list_variant(p, true, nullptr, &p->lists_links);
  if (rc != FPSCHED_OK) return rc;
  p->links_on = true;
  // ---- the sliding pass under the link model, if it fits
  // links of a device: the devices its stages send to (activations to successor stages, gradients to
  // predecessor stages), numbered in the order they are met
  const std::vector<int32_t>& I = p->host_ints;
  const DevTables& T = p->tables;
  const SlotTables& ST = p->stab;
  const int V = p->slot_v, lpc = ST.lanes_per_cand;
  std::vector<std::vector<int>> sends_to(D);
  auto link_of = [&](int d, int to) {
    for (size_t i = 0; i < sends_to[d].size(); ++i) if (sends_to[d][i] == to) return (int)i;
    sends_to[d].push_back(to);
    return (int)sends_to[d].size() - 1;
  };
  struct OutEdge { int to, comm; };
  auto out_edge = [&](int s, bool forward, int k, OutEdge* e) {
    const int off = forward ? T.off_succ_off : T.off_pred_off;
    const int at = I[off + s] + k;
    if (at >= I[off + s + 1]) return false;
    e->to = p->stage_device[I[(forward ? T.off_succ_stage : T.off_pred_stage) + at]];
    e->comm = I[(forward ? T.off_succ_comm : T.off_pred_comm) + at];
    return true;
  };
  for (int s = 0; s < S; ++s)
    for (int fwd = 0; fwd < 2; ++fwd)
      for (int k = 0; k < 2; ++k) {
        OutEdge e;
        if (out_edge(s, fwd != 0, k, &e) && e.to != p->stage_device[s]) (void)link_of(p->stage_device[s], e.to);
      }
  // two more words per lane: one for values that stay on the device (latency 0; it only ever holds
  // earlier finish times of the device, so nothing waits for it) and one that takes what ops without an
  // out-edge write
  int link_words = 2;
  for (int d = 0; d < D; ++d) link_words = std::max(link_words, (int)sends_to[d].size() + 2);
  if (link_words * 256 > 0xffff) return FPSCHED_OK;
  const uint32_t spare = (uint32_t)(link_words - 2) * 256u;
  // (this form of the kernel needs no dump region behind the slots: ops without an out-edge write the
  // lane's last link word)
  const int slots_per_cand = (2 * ST.n_classes * p->m + 7) & ~7;
  // (as many candidates per wavefront as the plain tables: the per-lane constants are shared)
  SlotGeometry geo = slot_geometry(ST.n_shared_ints, lpc, ST.state_words + link_words, slots_per_cand, p->max_lds,
                                   ST.cands_per_wave);
  if (geo.waves < 1 || geo.cands_per_wave != ST.cands_per_wave) return FPSCHED_OK;
  // never more wavefronts than the plain kernel runs with: where this form would fit more (batches of
  // short candidates), more segments only lengthen the ragged end of a batch
  const int plain_groups = std::max(p->slot_grid / std::max(p->n_cu, 1), 1);
  if (geo.waves * geo.groups > p->slot_waves * plain_groups &&
      4ll * (ST.n_shared_ints + (int64_t)p->slot_waves * geo.wave_ints) + 256 <= p->max_lds / plain_groups) {
    geo.waves = p->slot_waves;
    geo.groups = plain_groups;
  }
  // the timing pass's table image with longer dev rows: [.. 2 + 4V ints as before ..][4V out-edges]
  const int dev_ints = ST.dev_ints + 4 * V;
  auto with_links = [&](const std::vector<int32_t>& base) {
  std::vector<int32_t> J((size_t)ST.n_shared_ints + (size_t)lpc * dev_ints + (size_t)lpc * ST.state_words, 0);
  std::copy(base.begin(), base.begin() + ST.n_shared_ints, J.begin());
  for (int d = 0; d < lpc; ++d) {
    int32_t* row = &J[(size_t)ST.n_shared_ints + (size_t)d * dev_ints];
    std::copy(base.begin() + ST.off_dev + (size_t)d * ST.dev_ints,
              base.begin() + ST.off_dev + (size_t)(d + 1) * ST.dev_ints, row);
    for (int i = 0; i < 4 * V; ++i) row[ST.dev_ints + i] = (int32_t)spare;
    if (d >= D) continue;
    for (int c = 0; c < p->n_chunks[d]; ++c) {
      const int s = p->local_stage[(size_t)d * kMaxChunks + c];
      for (int fwd = 0; fwd < 2; ++fwd)
        for (int k = 0; k < 2; ++k) {
          OutEdge e;
          if (!out_edge(s, fwd != 0, k, &e) || e.to == d) continue;
          // first forward / first backward / second forward / second backward
          row[ST.dev_ints + (2 * k + (fwd ? 0 : 1)) * V + c] =
              (int32_t)(((uint32_t)e.comm << 16) | (uint32_t)link_of(d, e.to) * 256u);
        }
    }
  }
  std::copy(base.begin() + ST.off_expect, base.end(), J.begin() + ST.n_shared_ints + (size_t)lpc * dev_ints);
  return J;
  };
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  const int32_t lds_bytes = (int32_t)(4ll * (ST.n_shared_ints + (int64_t)geo.waves * geo.wave_ints));
  p->stab_links = ST;
  p->stab_links.link_words = link_words;
  p->stab_links.slots_per_cand = slots_per_cand;
  p->stab_links.dev_ints = dev_ints;
  p->stab_links.off_expect = ST.n_shared_ints + lpc * dev_ints;
  p->stab_links.cands_per_wave = geo.cands_per_wave;
  p->stab_links.wave_ints = geo.wave_ints;
  p->links_waves = geo.waves;
  p->links_grid = p->n_cu * geo.groups;
  p->links_lds_bytes = lds_bytes;
  // the sliding pass's timing kernel under the link model: the timing image, widened the same way; it
  // needs 16 bytes of LDS more
  if (p->slide_ok && !p->times_ints.empty() && (int64_t)lds_bytes + 16 <= p->max_lds / geo.groups) {
    const std::vector<int32_t> JT = with_links(p->times_ints);
    int32_t* timg = nullptr;
    if (hipMalloc(&timg, JT.size() * sizeof(int32_t)) == hipSuccess &&
        hipMemcpy(timg, JT.data(), JT.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotTimesLinks>(p->slot_v, p->slot_deg2, ST.n_classes == 1)),
                            hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess) {
      p->d_times_links_image = timg;
      p->stab_times_links = p->stab_links;
      p->stab_times_links.ints = timg;
      p->links_slide_ok = true;
      // the one-kernel form of the pass under the link model: the same image with the W items' costs behind it
      if (p->slide_eval_ok && !p->slide_w_table.empty()) {
        std::vector<int32_t> JS = JT;
        JS.insert(JS.end(), p->slide_w_table.begin(), p->slide_w_table.end());
        int32_t* simg = nullptr;
        if (hipMalloc(&simg, JS.size() * sizeof(int32_t)) == hipSuccess &&
            hipMemcpy(simg, JS.data(), JS.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess &&
            hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotSlideLinks>(p->slot_v, p->slot_deg2, ST.n_classes == 1)),
                                hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess) {
          p->d_slide_links_image = simg;
          p->stab_slide_links = p->stab_links;
          p->stab_slide_links.ints = simg;
          p->stab_slide_links.off_w = (int32_t)JT.size();
          p->links_slide_eval_ok = true;
        } else {
          (void)hipGetLastError();
          if (simg) (void)hipFree(simg);
        }
      }
    } else {
      (void)hipGetLastError();
      if (timg) (void)hipFree(timg);
    }
  }
  return FPSCHED_OK;
}

// The table image and workgroup shape of eval_sync_kernel for one setting of the handle: groups and pairs
// (fpsched_problem_set_sync) or the copy-engine form (fpsched_problem_set_copy_engine, copy_depth > 0).
// On success the handle's table is replaced; on failure the handle is back on the plain model.
static int install_table_model(fpsched_problem* p, const std::vector<int32_t>& grp, const std::vector<int32_t>& items,
                               int32_t n_pairs, const fpsched_dependency* pairs, bool wants_w, int copy_depth) {
  const int D = p->D, S = p->S, m = p->m;
  const std::vector<int32_t>& I = p->host_ints;
  const DevTables& T = p->tables;
  std::vector<int32_t> J;
  SyncTables ST{};
  ST.D = D; ST.S = S; ST.m = m; ST.has_w = p->has_w;
  ST.lanes_per_cand = T.lanes_per_cand;
  ST.n_fin_tables = wants_w ? 3 : 2;
  ST.copy_depth = copy_depth;
  auto append = [&](const int32_t* src, size_t n) { const int32_t off = (int32_t)J.size(); J.insert(J.end(), src, src + n); return off; };
  ST.off_dur = append(&I[T.off_dur], (size_t)kNKinds * S);
  ST.off_mem_units = append(&I[T.off_mem_units], S);
  ST.off_group = append(grp.data(), S);
  ST.off_items = append(items.data(), S);
  // one dependency list per (kind, stage): the edges of the stage DAG, then the pairs
  std::vector<int32_t> dep_off((size_t)kNKinds * S + 1, 0), dep;
  for (int kind = 0; kind < kNKinds; ++kind)
    for (int s = 0; s < S; ++s) {
      dep_off[(size_t)kind * S + s] = (int32_t)(dep.size() / 3);
      if (kind == kF || kind == kFD)
        for (int e = I[T.off_pred_off + s]; e < I[T.off_pred_off + s + 1]; ++e) {
          dep.push_back(0); dep.push_back(I[T.off_pred_stage + e]); dep.push_back(I[T.off_pred_comm + e]);
        }
      if (kind == kB)
        for (int e = I[T.off_succ_off + s]; e < I[T.off_succ_off + s + 1]; ++e) {
          dep.push_back(1); dep.push_back(I[T.off_succ_stage + e]); dep.push_back(I[T.off_succ_comm + e]);
        }
      for (int i = 0; i < n_pairs; ++i) {
        const fpsched_dependency& q = pairs[i];
        if (q.stage_to != s || !(q.kind_to == kind || (q.kind_to == FPSCHED_F && kind == kFD))) continue;
        dep.push_back(q.kind_from == FPSCHED_F ? 0 : (q.kind_from == FPSCHED_B ? 1 : 2));
        dep.push_back(q.stage_from);
        dep.push_back(p->stage_device[q.stage_from] != p->stage_device[s] ? q.latency : 0);
      }
    }
  dep_off[(size_t)kNKinds * S] = (int32_t)(dep.size() / 3);
  ST.off_dep_off = append(dep_off.data(), dep_off.size());
  ST.off_dep = append(dep.data(), dep.size());
  ST.off_local_stage = append(p->local_stage.data(), (size_t)D * kMaxChunks);
  ST.off_n_chunks = append(p->n_chunks.data(), D);
  ST.off_mem_cap = append(&I[T.off_mem_cap], D);
  ST.n_table_ints = (int32_t)J.size();
  // candidates per wavefront: whole finish-time tables (and reload times) and state bytes of each in LDS;
  // the copy-engine form adds three rings of eight dwords per lane
  const int64_t SM = (int64_t)S * m;
  const int64_t per_cand = 4 * ((ST.n_fin_tables + (copy_depth > 0 ? 1 : 0)) * SM + ((SM + 3) >> 2));
  const int64_t fixed_bytes = 4ll * ST.n_table_ints + (copy_depth > 0 ? 3 * 8 * 64 * 4 : 0);
  int cpw = 64 / ST.lanes_per_cand;
  while (cpw > 1 && fixed_bytes + cpw * per_cand > p->max_lds) cpw >>= 1;
  if (fixed_bytes + cpw * per_cand > p->max_lds) return FPSCHED_EUNSUPPORTED;
  ST.cands_per_wave = cpw;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  if (hipDeviceSynchronize() != hipSuccess) return FPSCHED_EHIP;   // an earlier table may be in use
  auto back_to_plain = [&]() {
    p->sync_on = false;
    p->copy_depth = 0;
    p->sync_items.assign(S, m);
  };
  if (J.size() > p->sync_ints_capacity) {
    int32_t* fresh = nullptr;
    if (hipMalloc(&fresh, J.size() * sizeof(int32_t)) != hipSuccess) { (void)hipGetLastError(); return FPSCHED_ENOMEM; }
    if (p->d_sync_ints) (void)hipFree(p->d_sync_ints);
    p->d_sync_ints = fresh;
    p->sync_ints_capacity = J.size();
    back_to_plain();   // the table the handle ran on is gone
  }
  if (hipMemcpy(p->d_sync_ints, J.data(), J.size() * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&eval_sync_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          p->max_lds) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(&eval_sync_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          p->max_lds) != hipSuccess) {
    back_to_plain();
    return FPSCHED_EHIP;
  }
  ST.ints = p->d_sync_ints;
  p->sync_tab = ST;
  p->sync_lds_bytes = (int32_t)(fixed_bytes + cpw * per_cand);
  return FPSCHED_OK;
}

// The slot kernel's form of the synchronisation model (mode kSlotSync): possible when every dependency pair runs
// forward-to-forward or backward-to-backward, no stage has more than two inputs or outputs in either direction
// (pairs included), and the neighbours of a stage with more than one micro-batch per item all have one.  The
// table image has the plain layout; a pair is an edge of a slot class of its own that exists in one direction.  The
// two-pass evaluation takes those settings in which an op's edges need no more than two slots (p->lists_sync).
// Leaves p->sync_slots_ok false when the setting does not fit.
static void build_sync_slot_tables(fpsched_problem* p, const std::vector<int32_t>& grp, const std::vector<int32_t>& items,
                                   int32_t n_pairs, const fpsched_dependency* pairs, int64_t max_lat) {
  p->sync_slots_ok = false;
  p->lists_sync.ok = false;
  if (!p->slots_ok) return;   // (units, stage count and word format were checked for the plain tables)
  const int D = p->D, S = p->S, m = p->m;
  const std::vector<int32_t>& I = p->host_ints;
  const DevTables& T = p->tables;
  if ((int64_t)D * p->max_stride * (p->max_dur + max_lat) >= (1ll << 24) || max_lat >= (1ll << 16)) return;
  struct In { int from, lat, cls; };
  std::vector<std::vector<In>> fwd_in(S), bwd_in(S);
  std::vector<std::vector<int>> fwd_out(S), bwd_out(S), partners(S);
  // classes of the DAG's edges: chains, as for the plain tables
  std::vector<std::vector<int>> out_cls(S);
  int n_classes = 0;
  {
    std::vector<int> indeg(S, 0), order;
    std::vector<std::vector<int>> arriving(S);
    for (int s = 0; s < S; ++s) indeg[s] = I[T.off_pred_off + s + 1] - I[T.off_pred_off + s];
    for (int s = 0; s < S; ++s) if (!indeg[s]) order.push_back(s);
    for (size_t i = 0; i < order.size(); ++i) {
      const int s = order[i];
      size_t used = 0;
      for (int e = I[T.off_succ_off + s]; e < I[T.off_succ_off + s + 1]; ++e) {
        const int v = I[T.off_succ_stage + e], lat = I[T.off_succ_comm + e];
        const int cls = used < arriving[s].size() ? arriving[s][used++] : n_classes++;
        arriving[v].push_back(cls);
        fwd_out[s].push_back(cls); fwd_in[v].push_back(In{s, lat, cls});
        bwd_in[s].push_back(In{v, lat, cls}); bwd_out[v].push_back(cls);
        partners[s].push_back(v); partners[v].push_back(s);
        if (--indeg[v] == 0) order.push_back(v);
      }
    }
  }
  for (int i = 0; i < n_pairs; ++i) {
    const fpsched_dependency& q = pairs[i];
    const int a = q.stage_from, b = q.stage_to;
    const int lat = p->stage_device[a] != p->stage_device[b] ? q.latency : 0;
    const int cls = n_classes++;
    if (q.kind_from == FPSCHED_F && q.kind_to == FPSCHED_F) {
      fwd_out[a].push_back(cls); fwd_in[b].push_back(In{a, lat, cls});
    } else if (q.kind_from == FPSCHED_B && q.kind_to == FPSCHED_B) {
      bwd_out[a].push_back(cls); bwd_in[b].push_back(In{a, lat, cls});
    } else {
      return;   // a pair the mail slots cannot carry
    }
    partners[a].push_back(b); partners[b].push_back(a);
  }
  if (n_classes == 0) n_classes = 1;
  bool deg2 = false;
  for (int s = 0; s < S; ++s) {
    const size_t most = std::max({fwd_in[s].size(), fwd_out[s].size(), bwd_in[s].size(), bwd_out[s].size()});
    if (most > 2) return;
    if (most > 1) deg2 = true;
    if (grp[s] > 1)
      for (int t : partners[s]) if (grp[t] != 1) return;
  }
  if (p->lists_ok && !p->lists_wide && !getenv("FPSCHED_SYNC_SLOTS")) {
    // the two-pass evaluation's form, where no stage has more than two edge slots in a direction
    // (classes numbered per direction: a pair has slots in one only)
    std::vector<StageEdges> edges(S);
    std::vector<int> number[2];
    int n_of[2] = {0, 0};
    for (int dir = 0; dir < 2; ++dir) {
      number[dir].assign(n_classes, -1);
      auto numbered = [&](int cls) {
        if (number[dir][cls] < 0) number[dir][cls] = n_of[dir]++;
        return number[dir][cls];
      };
      for (int s = 0; s < S; ++s) {
        for (const In& in : dir == 0 ? fwd_in[s] : bwd_in[s]) edges[s].in[dir].push_back(StageEdge{numbered(in.cls), in.from, in.lat});
        for (int cls : dir == 0 ? fwd_out[s] : bwd_out[s]) edges[s].out[dir].push_back(StageEdge{numbered(cls), 0, 0});
      }
    }
    ListTables LT;
    bool two = false;
    std::vector<int32_t> image;
    if (fill_list_image(p, edges, n_of[0], n_of[1], false, true, items, &LT, &two, &image)) {
      // items of groups: rows that never issue and name two rows behind the timing rows (device_tables.h)
      std::vector<int32_t> rows;
      const int32_t old_ints = LT.n_time_ints;
      for (int kind : {(int)kF, (int)kFD, (int)kB})
        for (int d = 0; d < D; ++d)
          for (int c = 0; c < p->n_chunks[d]; ++c) {
            const int s = p->local_stage[(size_t)d * kMaxChunks + c], dir = kind == kB ? 1 : 0;
            const std::vector<EdgeSlot> slots = edge_slots(edges[s], dir);
            if (grp[s] <= 1 || slots.empty()) continue;   // (no slots: the device's own word)
            int32_t* t = &image[((kind * kMaxChunks + c) * D + (d & 1) * ((D + 1) / 2) + d / 2) * 4];
            int32_t of_group[8] = {0, (int32_t)((uint32_t)p->host_ints[p->tables.off_dur + kind * S + s] << 8 | (uint32_t)s), grp[s], 0, 0, 0, 0, 0};
            for (size_t e = 0; e < slots.size(); ++e) {
              const StageEdge* in = slots[e].in;
              of_group[4 * e] = in ? (int32_t)(((uint32_t)in->latency << 8) - (uint32_t)in->tag) : 0;
              of_group[4 * e + 2] |= (in ? (int32_t)kGroupIn : 0) | (slots[e].out ? (int32_t)kGroupOut : 0);
              of_group[4 * e + 3] = 4 * (list_slots_at(D) + (dir == 0 ? n_of[1] * m : 0) + slots[e].cls * m);
            }
            t[0] = 1; t[1] = (int32_t)kGroupRow;
            t[2] = (int32_t)((uint32_t)((old_ints + (int)rows.size()) / 4) << 18);
            t[3] = 4 * d;
            rows.insert(rows.end(), of_group, of_group + 8);
          }
      rows.resize((rows.size() + 7) & ~(size_t)7, 0);
      take_check_place(p->ltab, &LT);   // (the order pass is launched as for the plain model)
      LT.off_sync = old_ints;
      LT.n_time_ints += (int32_t)rows.size();
      LT.off_check += (int32_t)rows.size();
      LT.off_dev += (int32_t)rows.size();
      image.insert(image.begin() + old_ints, rows.begin(), rows.end());
      if (install_list_variant(p, LT, image, two, 1, &p->lists_sync) == FPSCHED_OK) {
        p->sync_slots_ok = true;
        return;
      }
      (void)hipGetLastError();
    }
  }
  const int V = p->slot_v, lpc = T.lanes_per_cand;
  const int slot_stride = ((2 * n_classes + 1) * m + 7) & ~7;
  if (4ll * slot_stride > 0xffff) return;
  const int64_t unit_scale = p->stab.unit_scale;
  const int n_meta = kNKinds * kMaxChunks * lpc * 4;
  const int n_meta2 = deg2 ? (2 * kMaxChunks + 1) * lpc * 2 : 0;
  const int n_shared = (n_meta + n_meta2 + 511) & ~511;
  const unsigned dump_bytes = (unsigned)(2 * n_classes * m) * 4u;
  const int dev_ints = 2 + 5 * V;
  const int words_per_chunk = (m + 7) / 8;
  const int state_words = V * words_per_chunk;
  std::vector<int32_t> J((size_t)n_shared + (size_t)lpc * dev_ints + (size_t)lpc * state_words, 0);
  static const int need_of[kNKinds] = {15, kAbsent, kRes, kBDone, kDisc, kRes, kOff, kAbsent};
  static const int next_of[kNKinds] = {0, kRes, kBDone, kDone, kRes, kOff, kRes, kDisc};
  auto fwd_slot = [&](int cls) { return (unsigned)((n_classes + cls) * m) * 4u; };
  auto bwd_slot = [&](int cls) { return (unsigned)(cls * m) * 4u; };
  for (int kind = 0; kind < kNKinds; ++kind)
    for (int c = 0; c < kMaxChunks; ++c)
      for (int d = 0; d < lpc; ++d) {
        int32_t* e = &J[(((size_t)kind * kMaxChunks + c) * lpc + d) * 4];
        e[2] = (int32_t)(15u | (dump_bytes << 16));
        if (d >= D || c >= p->n_chunks[d] || kind == kEnd || (kind == kW && !p->has_w)) continue;
        const int st = p->local_stage[(size_t)d * kMaxChunks + c];
        const unsigned units = (unsigned)(I[T.off_mem_units + st] / unit_scale);
        const bool allocs = kind == kF || kind == kFD || kind == kR || kind == kL;
        const bool frees = kind == kFD || kind == kO || kind == (p->has_w ? kW : kB);
        unsigned has_in = 0, tag = 0, prod = dump_bytes, comm = 0;
        if (kind == kF || kind == kFD) {
          if (!fwd_in[st].empty()) { has_in = 0xffu; tag = (unsigned)fwd_in[st][0].from; comm = (unsigned)fwd_in[st][0].lat; }
          if (!fwd_out[st].empty()) prod = fwd_slot(fwd_out[st][0]);
        } else if (kind == kB) {
          if (!bwd_in[st].empty()) { has_in = 0xffu; tag = (unsigned)bwd_in[st][0].from; comm = (unsigned)bwd_in[st][0].lat; }
          if (!bwd_out[st].empty()) prod = bwd_slot(bwd_out[st][0]);
        }
        e[0] = (int32_t)((unsigned)I[T.off_dur + kind * S + st] << 8);
        e[1] = (int32_t)((comm << 8) - tag);
        e[2] = (int32_t)((unsigned)need_of[kind] | ((unsigned)(need_of[kind] ^ next_of[kind]) << 8) | (prod << 16));
        e[3] = (int32_t)((allocs ? units : 0u) | ((frees ? units : 0u) << 8) | ((unsigned)st << 16) | (has_in << 24));
      }
  for (int dir = 0; dir < 2 && deg2; ++dir)
    for (int c = 0; c < kMaxChunks; ++c)
      for (int d = 0; d < D; ++d) {
        if (c >= p->n_chunks[d]) continue;
        const int st = p->local_stage[(size_t)d * kMaxChunks + c];
        int32_t* e = &J[(size_t)n_meta + (((size_t)dir * kMaxChunks + c) * lpc + d) * 2];
        const std::vector<In>& in = dir == 0 ? fwd_in[st] : bwd_in[st];
        const std::vector<int>& out = dir == 0 ? fwd_out[st] : bwd_out[st];
        unsigned y = 0;
        if (in.size() > 1) { y |= kMetaHasCons; e[0] = (int32_t)(((unsigned)in[1].lat << 8) - (unsigned)in[1].from); }
        if (out.size() > 1) y |= kMetaHasProd | (dir == 0 ? fwd_slot(out[1]) : bwd_slot(out[1]));
        e[1] = (int32_t)y;
      }
  for (int d = 0; d < D; ++d) {
    // state words of device d once every item placed on it is consumed
    int32_t* x = &J[(size_t)n_shared + (size_t)lpc * dev_ints + (size_t)d * state_words];
    const unsigned terminal = p->has_w ? kDone : kBDone;
    for (int c = 0; c < p->n_chunks[d]; ++c) {
      const int st = p->local_stage[(size_t)d * kMaxChunks + c];
      for (int g = 0; g < items[st]; ++g) x[c * words_per_chunk + (g >> 3)] |= (int32_t)(terminal << ((g & 7) * 4));
    }
    int32_t* e = &J[(size_t)n_shared + (size_t)d * dev_ints];
    e[0] = p->n_chunks[d];
    e[1] = (int32_t)(I[T.off_mem_cap + d] / unit_scale);
    for (int c = 0; c < p->n_chunks[d]; ++c) {
      const int st = p->local_stage[(size_t)d * kMaxChunks + c];
      e[2 + c] = !fwd_in[st].empty() ? (n_classes + fwd_in[st][0].cls) * m : 0;
      e[2 + V + c] = !bwd_in[st].empty() ? bwd_in[st][0].cls * m : 0;
      e[2 + 2 * V + c] = fwd_in[st].size() > 1 ? (n_classes + fwd_in[st][1].cls) * m : 0;
      e[2 + 3 * V + c] = bwd_in[st].size() > 1 ? bwd_in[st][1].cls * m : 0;
      e[2 + 4 * V + c] = grp[st] | (items[st] << 16);
    }
    for (int c = p->n_chunks[d]; c < V; ++c) e[2 + 4 * V + c] = 1;   // (no such chunk: no item is valid)
  }
  SlotTables ST = p->stab;
  ST.n_classes = n_classes;
  ST.slots_per_cand = slot_stride;
  ST.state_words = state_words;
  ST.n_shared_ints = n_shared;
  ST.off_meta2 = n_meta;
  ST.off_dev = n_shared;
  ST.dev_ints = dev_ints;
  ST.off_expect = n_shared + lpc * dev_ints;
  ST.link_words = 0; ST.copy_depth = 0;
  const SlotGeometry geo = slot_geometry(n_shared, lpc, state_words, slot_stride, p->max_lds);
  if (geo.waves < 1) return;
  ST.cands_per_wave = geo.cands_per_wave;
  ST.wave_ints = geo.wave_ints;
  DeviceGuard g(p->device_id);
  if (!g.ok) return;
  if (J.size() > p->sync_slot_image_ints) {
    if (p->d_sync_slot_image) (void)hipFree(p->d_sync_slot_image);
    p->d_sync_slot_image = nullptr;
    p->sync_slot_image_ints = 0;
    if (hipMalloc(&p->d_sync_slot_image, J.size() * sizeof(int32_t)) != hipSuccess) { (void)hipGetLastError(); p->d_sync_slot_image = nullptr; return; }
    p->sync_slot_image_ints = J.size();
  }
  if (hipMemcpy(p->d_sync_slot_image, J.data(), J.size() * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess ||
      hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotSync>(V, deg2, n_classes == 1)),
                          hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  ST.ints = p->d_sync_slot_image;
  p->stab_sync = ST;
  p->sync_deg2 = deg2;
  p->sync_slot_waves = geo.waves;
  p->sync_slot_grid = p->n_cu * geo.groups;
  p->sync_slot_lds_bytes = (int32_t)(4ll * (n_shared + (int64_t)geo.waves * geo.wave_ints));
  p->sync_slots_ok = true;
  if (getenv("FPSCHED_VERBOSE"))
    fprintf(stderr, "[fpsched] slot kernel, synchronisation: %d x %d wavefronts per compute unit, %d candidates each\n", geo.groups, geo.waves, geo.cands_per_wave);
}

int fpsched_problem_set_sync(fpsched_problem* p, const int32_t* group, int32_t n_pairs,
                             const fpsched_dependency* pairs) {
  if (!p || n_pairs < 0 || (n_pairs > 0 && !pairs)) return FPSCHED_EINVAL;
  const int D = p->D, S = p->S, m = p->m;
  bool trivial = n_pairs == 0;
  for (int s = 0; s < S && group; ++s) {
    if (group[s] < 1) return FPSCHED_EINVAL;
    if (group[s] != 1) trivial = false;
  }
  if (trivial) {   // back to the plain model; the table stays allocated for the next call
    if (p->sync_on) p->sync_items.assign(S, m);
    p->sync_on = false;
    return FPSCHED_OK;
  }
  if (p->mb_set || p->links_on || p->copy_depth > 0) return FPSCHED_EUNSUPPORTED;
  int64_t max_lat = p->max_comm;
  bool wants_w = false;
  for (int i = 0; i < n_pairs; ++i) {
    const fpsched_dependency& q = pairs[i];
    if (q.kind_from != FPSCHED_F && q.kind_from != FPSCHED_B && q.kind_from != FPSCHED_W) return FPSCHED_EINVAL;
    if (q.kind_to <= FPSCHED_END || q.kind_to >= FPSCHED_NKINDS) return FPSCHED_EINVAL;
    if ((q.kind_from == FPSCHED_W || q.kind_to == FPSCHED_W) && !p->has_w) return FPSCHED_EINVAL;
    if (q.stage_from < 0 || q.stage_from >= S || q.stage_to < 0 || q.stage_to >= S || q.latency < 0) return FPSCHED_EINVAL;
    if (q.stage_from == q.stage_to && (q.kind_from == q.kind_to || (q.kind_from == FPSCHED_F && q.kind_to == FPSCHED_FD)))
      return FPSCHED_EINVAL;
    max_lat = std::max<int64_t>(max_lat, q.latency);
    wants_w = wants_w || q.kind_from == FPSCHED_W;
  }
  if ((int64_t)D * p->max_stride * (p->max_dur + max_lat) >= (int64_t)1 << 31) return FPSCHED_EOVERFLOW;
  std::vector<int32_t> grp(S, 1), items(S, m);
  for (int s = 0; s < S; ++s) {
    grp[s] = group ? std::min(group[s], m) : 1;
    items[s] = (m + grp[s] - 1) / grp[s];
  }
  if (p->device_id >= 0) {
    const int rc = install_table_model(p, grp, items, n_pairs, pairs, wants_w, 0);
    if (rc != FPSCHED_OK) return rc;
    build_sync_slot_tables(p, grp, items, n_pairs, pairs, max_lat);
  }
  p->sync_items = items;
  p->sync_on = true;
  return FPSCHED_OK;
}

int fpsched_problem_set_copy_engine(fpsched_problem* p, int32_t depth) {
  if (!p || depth < 0 || depth > FPSCHED_MAX_COPY_DEPTH) return FPSCHED_EINVAL;
  if (depth == 0) {
    p->copy_depth = 0;
    return FPSCHED_OK;
  }
  if (p->mb_set || p->links_on || p->sync_on) return FPSCHED_EUNSUPPORTED;
  // a transfer takes time: with a cost of zero any number of them could end at one instant
  const std::vector<int32_t>& I = p->host_ints;
  for (int s = 0; s < p->S; ++s)
    if (I[p->tables.off_dur + kO * p->S + s] < 1 || I[p->tables.off_dur + kL * p->S + s] < 1) return FPSCHED_EINVAL;
  if (p->device_id >= 0) {
    const std::vector<int32_t> grp(p->S, 1), items(p->S, p->m);
    const int rc = install_table_model(p, grp, items, 0, nullptr, false, depth);
    if (rc != FPSCHED_OK) return rc;
    // the slot kernel has a form of this model too: the plain tables, 32 more dwords of LDS per lane for
    // the rings of the copy timeline
    p->copy_slots_ok = false;
    // the two-pass evaluation takes it where times fit 24 bits, at every depth (without its tables the slot kernel stays in use)
    p->copy_lists(depth).ok = false;
    if (p->slots_ok && build_copy_variant(p, depth) != FPSCHED_OK) (void)hipGetLastError();
    if (p->slots_ok) {
      const SlotTables& PT = p->stab;
      const SlotGeometry geo = slot_geometry(PT.n_shared_ints, PT.lanes_per_cand, PT.state_words + kSlotCopyWords,
                                             PT.slots_per_cand, p->max_lds, PT.cands_per_wave);
      DeviceGuard g(p->device_id);
      if (g.ok && geo.waves >= 1 && geo.cands_per_wave == PT.cands_per_wave &&
          hipFuncSetAttribute(reinterpret_cast<const void*>(slot_kernel_of<kSlotCopy>(p->slot_v, p->slot_deg2, PT.n_classes == 1)),
                              hipFuncAttributeMaxDynamicSharedMemorySize, p->max_lds) == hipSuccess) {
        p->stab_copy = PT;
        p->stab_copy.link_words = kSlotCopyWords;
        p->stab_copy.copy_depth = depth;
        p->stab_copy.wave_ints = geo.wave_ints;
        p->copy_waves = geo.waves;
        p->copy_grid = p->n_cu * geo.groups;
        p->copy_lds_bytes = (int32_t)(4ll * (PT.n_shared_ints + (int64_t)geo.waves * geo.wave_ints));
        p->copy_slots_ok = true;
        if (getenv("FPSCHED_VERBOSE"))
          fprintf(stderr, "[fpsched] slot kernel, copy engine: %d x %d wavefronts per compute unit, %d candidates each\n", geo.groups, geo.waves, geo.cands_per_wave);
      }
    }
  }
  p->copy_depth = depth;
  return FPSCHED_OK;
}

using GenKernel = void (*)(DevTables, const int32_t*, const int32_t*, const long long*, long long, long long, int, int, uint16_t*,
                           int32_t*, unsigned char*, unsigned long long*, GenResults);

// about how many draws from one counter a set's steps last as long as (about 1 us and 100 draws each; order_sets)
static int64_t gen_steps(const fpsched_problem* p) {
  const int64_t chunks = std::max(max_chunks_of(p), 1);
  return 15 * (p->has_w ? 3 : 2) * chunks * p->m * (1 + chunks);
}

// How the segments of a generator launch come by their sets.  No more sets than segments: each has its own (returns 0).
// Else a counter hands out those behind the segments' first ones (returns 1), or, for long sets, all of them class by class,
// the ones with many steps first (generate_order_kernel; returns the number of classes).  The classes keep a batch from
// ending on a few sets that were begun late; they cost four draws per set from one counter, some 1e8 a second, where the plain
// order costs at most one per set.  So they pay where a set's steps, about items per actor x (1 + stages per actor) / 2 at
// about 1 us each, last as long as the draws of one set per segment, and where a segment has two sets or more
// (results only: 1.25 or more, if the steps last half as long again).
// Measured over 2 to 32 devices, 16 to 128 micro-batches, 1 to 4 stages per device, classes and plain order: 36,864 sets of
// 32 x 64 x 2: 3.92 and 4.66 ms (lists), 16,588 of 32 x 128 x 2, sliding: 5.03 and 6.40 ms, 15,974 of 16 x 128 x 2 (1.3 per
// segment), sliding: 2.86 and 3.11 ms.  On the other side of the line 55,296 sets of 20 x 30 x 2: 2.57 and 1.86 ms,
// 65,536 of 8 x 8 x 1: 0.97 and 0.30 ms, 15,974 of 16 x 64 x 2: 1.60 and 1.30 ms (lists), 1.89 and 1.64 ms (sliding).  At the
// line 33,177 of 16 x 64 x 2: 1.92 and 1.96 ms.
static int order_sets(const fpsched_problem* p, const int32_t* d_inflight, const int64_t* d_select, int64_t n_src, int64_t n_sets,
                      int64_t n_segments, bool lists, uint8_t* d_status, unsigned long long* counter, hipStream_t st) {
  if (n_sets <= n_segments) return 0;
  const int64_t steps = gen_steps(p);
  const bool by_class = steps >= n_segments && (n_sets >= 2 * n_segments || (!lists && 2 * steps >= 3 * n_segments && 4 * n_sets >= 5 * n_segments));
  if (!by_class) {
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, st, counter, (unsigned long long)n_segments, 0ull);
    return hipGetLastError() == hipSuccess ? 1 : FPSCHED_EHIP;
  }
  if (n_sets >= (1ll << 33)) return FPSCHED_EINVAL;   // (more workgroups than a launch has)
  hipLaunchKernelGGL(generate_order_kernel, dim3((unsigned)((n_sets + 3) / 4)), dim3(256), 0, st, p->tables, d_inflight,
                     reinterpret_cast<const long long*>(d_select), (long long)n_src, (long long)n_sets,
                     2 * std::max(max_chunks_of(p), 1) * p->m, d_status, counter);
  return hipGetLastError() == hipSuccess ? kGenClasses : FPSCHED_EHIP;
}

// Launch shape of the generator: workgroups of one wavefront per SIMD, as many per compute unit as asked for and as LDS
// holds.  (In larger ones the sets with most steps, which are drawn first, go to all wavefronts of a few compute units; those
// of one wavefront come to the SIMDs unevenly.  16,384 sets of 32 x 128 x 2, eight wavefronts per compute unit as one
// workgroup, two, eight: results only 4.57, 3.40 and 3.52 ms, lists 4.36, 2.94 and 3.21.)
//
// Wavefronts per compute unit: with more of them the sets with most steps advance more slowly and are what the launch ends
// on, with fewer the SIMDs are idle between steps.  Short sets are drawn in plain order: 16 (65,536 sets of 4 x 16 x 2, sliding,
// with 8, 12 and 16: 313, 280 and 179 us; of 8 x 32 x 2: 892, 823 and 802; but of 16 x 128 x 1 16,384 sets 899, 737 and 844).
// Else eight while the sets with most steps take longer than all steps shared out over the segments, that is up to about
// 1.3 times as many sets per segment as the longest set has steps of the mean one's, and twelve beyond.  The longest set's
// steps over the mean's are about 1 + D / 8 with one stage per device, 1 + D / 13 with two, 1 + D / 10 with more (sets as the
// tuner's grid and `policy_sets` have them; 32 x 128 x 1 5.05, 16 x 128 x 1 3.2, 8 x 128 x 1 2.1; 32 x 128 x 2 3.34, 16 x 64 x 2 2.27,
// 4 x 128 x 2 1.47; 32 x 48 x 3 3.7, 24 x 48 x 4 3.3, 6 x 100 x 3 1.64).  Sets per segment of eight where twelve become as good:
// 32 x 128 x 2 4.3, 24 x 80 x 2 3.5, 16 x 64 x 2 2.7, 10 x 120 x 2 2.3, 32 x 48 x 3 5.1, 24 x 48 x 4 4.6, 28 x 100 x 1 6.  Over 20 shapes
// with 1 to 8 sets per segment, three forms each, this is 1.2 % off the best of 8, 12 and 16 on average (20 % at worst: 49,152
// sets of 5 x 128 x 4, lists; factors of 1.2 to 1.4 are as good); always eight 7 %, always twelve 5 %, always sixteen 9 %.
struct GenShape { int waves, resident; int64_t blocks, lds_bytes; };   // resident: wavefronts that a compute unit has room for
static GenShape gen_shape(const fpsched_problem* p, int64_t n_sets, int64_t sets_per_wave, int64_t shared_ints, int64_t wave_ints) {
  const int64_t lds_ints = p->max_lds / 4, segments_of_8 = 8ll * p->n_cu * sets_per_wave;
  int want = 16;
  if (2 * gen_steps(p) >= 3 * segments_of_8) {
    const int chunks = max_chunks_of(p);
    const double longest = 1.0 + p->D / (chunks <= 1 ? 8.0 : chunks == 2 ? 13.0 : 10.0);
    want = (double)n_sets < 1.3 * longest * (double)segments_of_8 ? 8 : 12;
  }
  // tuning knob: FPSCHED_GEN_WAVES = resident wavefronts per compute unit
  if (const char* env = getenv("FPSCHED_GEN_WAVES")) {
    const int v = atoi(env);
    if (v >= 1 && v <= 32) want = v;
  }
  int best_waves = 1, best_groups = 1;
  for (int groups = 1; groups <= 8; ++groups) {
    int wv = (int)std::min<int64_t>((lds_ints / groups - shared_ints - 64) / wave_ints, kGenThreads / 64);
    wv = std::min(wv, want / groups);
    if (wv >= 1 && wv * groups > best_waves * best_groups) { best_waves = wv; best_groups = groups; }
  }
  // (a small batch is spread over the compute units: fewer wavefronts per workgroup)
  const int64_t wavefronts = (n_sets + sets_per_wave - 1) / sets_per_wave;
  const int resident = best_waves * best_groups;
  best_waves = (int)std::clamp<int64_t>((wavefronts + p->n_cu - 1) / p->n_cu, 1, best_waves);
  return GenShape{best_waves, resident, std::min<int64_t>((wavefronts + best_waves - 1) / best_waves, (int64_t)p->n_cu * best_groups),
                  4 * (shared_ints + best_waves * wave_ints)};
}

// What a device's two stages wait for, forward and backward, is on one other device each (kGenOneNeighbour): a chain laid round the
// devices, but not up and down again.  (Its counters are by device in the place of those by stage: no more devices than stages.)
static bool one_neighbour(const fpsched_problem* p) {
  if (max_chunks_of(p) != 2 || p->max_degree > 1 || p->D > p->S) return false;
  const std::vector<int32_t>& I = p->host_ints;
  const DevTables& G = p->tables;
  for (int d = 0; d < p->D; ++d)
    for (int dir = 0; dir < 2; ++dir) {
      int other = -1;
      for (int c = 0; c < p->n_chunks[d]; ++c) {
        const int off = dir == 0 ? G.off_pred_off : G.off_succ_off, s = p->local_stage[(size_t)d * kMaxChunks + c];
        if (I[off + s] >= I[off + s + 1]) continue;
        const int of = p->stage_device[I[(dir == 0 ? G.off_pred_stage : G.off_succ_stage) + I[off + s]]];
        if (other >= 0 && other != of) return false;
        other = of;
      }
    }
  return true;
}

static int run_generate(const fpsched_problem* p, const fpsched_actor_policy* d_policy, const int32_t* d_inflight,
                 const int64_t* d_select, int64_t n_src, int64_t n_sets, int32_t stride_words, uint16_t* d_ops, int32_t* d_steps,
                 uint8_t* d_status, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p || n_sets < 0) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (n_sets == 0) return FPSCHED_OK;
  if (!d_policy || !d_inflight || !d_ops || !d_steps || !d_status) return FPSCHED_EINVAL;
  if (p->sync_on) return FPSCHED_EUNSUPPORTED;   // the generator schedules one item per micro-batch
  const int max_chunks = max_chunks_of(p);
  const int64_t longest = (int64_t)max_chunks * p->m * (p->has_w ? 3 : 2);
  if (stride_words < 8 || (stride_words & 7) || stride_words < longest) return FPSCHED_EINVAL;
  if (reinterpret_cast<uintptr_t>(d_ops) & 15) return FPSCHED_EINVAL;
  // the first 8 bytes of the workspace hold the counter the segments draw parameter sets from
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < 256) return FPSCHED_ENOMEM;
  const int deg = p->max_degree <= 1 ? 1 : (p->max_degree == 2 ? 2 : 0);
  // tables (if walked), counters and the constant word (a multiple of four), the staging dwords
  const int64_t shared_ints = deg == 0 ? p->tables.n_table_ints : 0, lds_ints = p->max_lds / 4;
  auto wave_ints_of = [&](int64_t sets) { return ((sets * 2 * p->S + 2 + 3) & ~3ll) + kGenStagingWords * 64; };
  int cpw = 64 / p->D;
  while (cpw > 1 && shared_ints + wave_ints_of(cpw) > lds_ints) --cpw;
  const int64_t wave_ints = wave_ints_of(cpw);
  if (shared_ints + wave_ints > lds_ints) return FPSCHED_EUNSUPPORTED;
  DevTables tables = p->tables;
  tables.gen_sets = cpw;
  const GenShape shape = gen_shape(p, n_sets, cpw, shared_ints, wave_ints);
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  const int V = max_chunks <= 1 ? 1 : (max_chunks <= 2 ? 2 : 4);
  static const GenKernel table[3][3] = {
      {&generate_kernel<1, 0, kGenPlain>, &generate_kernel<1, 1, kGenPlain>, &generate_kernel<1, 2, kGenPlain>},
      {&generate_kernel<2, 0, kGenPlain>, &generate_kernel<2, 1, kGenPlain>, &generate_kernel<2, 2, kGenPlain>},
      {&generate_kernel<4, 0, kGenPlain>, &generate_kernel<4, 1, kGenPlain>, &generate_kernel<4, 2, kGenPlain>}};
  const GenKernel kernel = one_neighbour(p) ? &generate_kernel<2, kGenOneNeighbour, kGenPlain> : table[V == 1 ? 0 : (V == 2 ? 1 : 2)][deg];
  if (shape.lds_bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                          p->max_lds) != hipSuccess)
    return FPSCHED_EHIP;
  unsigned long long* counter = static_cast<unsigned long long*>(d_workspace);
  const int n_classes = order_sets(p, d_inflight, d_select, n_src, n_sets, shape.blocks * shape.waves * cpw, true, d_status, counter, static_cast<hipStream_t>(hip_stream));
  if (n_classes < 0) return n_classes;
  hipLaunchKernelGGL(kernel, dim3((unsigned)shape.blocks), dim3(64 * shape.waves), (size_t)shape.lds_bytes,
                     static_cast<hipStream_t>(hip_stream), tables, reinterpret_cast<const int32_t*>(d_policy),
                     d_inflight, reinterpret_cast<const long long*>(d_select), (long long)n_src, (long long)n_sets,
                     n_classes, (int)stride_words, d_ops, d_steps, d_status, counter, GenResults{nullptr, nullptr, nullptr, nullptr});
  return check_hip(hipGetLastError());
}

int fpsched_generate(const fpsched_problem* p, const fpsched_actor_policy* d_policy, const int32_t* d_inflight,
                     int64_t n_sets, int32_t stride_words, uint16_t* d_ops, int32_t* d_steps, uint8_t* d_status,
                     void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  return run_generate(p, d_policy, d_inflight, nullptr, n_sets, n_sets, stride_words, d_ops, d_steps, d_status, d_workspace,
                      workspace_bytes, hip_stream);
}

int fpsched_generate_selected(const fpsched_problem* p, const fpsched_actor_policy* d_policy,
                              const int32_t* d_inflight, int64_t n_sets, const int64_t* d_select, int64_t n_selected,
                              int32_t stride_words, uint16_t* d_ops, int32_t* d_steps, uint8_t* d_status,
                              void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (n_sets < 0 || (n_selected > 0 && !d_select)) return FPSCHED_EINVAL;
  return run_generate(p, d_policy, d_inflight, d_select, n_sets, n_selected, stride_words, d_ops, d_steps, d_status,
                      d_workspace, workspace_bytes, hip_stream);
}

// generator and evaluator in one kernel; slide: with the weight-gradient sliding pass in it
static int run_generate_evaluate(const fpsched_problem* p, const fpsched_actor_policy* d_policy,
                                 const int32_t* d_inflight, int64_t n_sets, fpsched_results out, int32_t* d_steps,
                                 uint8_t* d_status, void* d_workspace, size_t workspace_bytes, void* hip_stream,
                                 bool slide) {
  if (!p || n_sets < 0) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (slide && !p->has_w) return FPSCHED_EINVAL;
  if (n_sets == 0) return FPSCHED_OK;
  if (!d_policy || !d_inflight || !d_steps || !d_status || !out.makespan || !out.idle || !out.peak || !out.flags)
    return FPSCHED_EINVAL;
  // the plain cost model only: one cost per (type, stage), transfers as latencies
  if (p->sync_on || p->copy_depth > 0 || p->mb_set || p->links_on) return FPSCHED_EUNSUPPORTED;
  if (p->tables.off_gen_rows < 0) return FPSCHED_EUNSUPPORTED;
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < 256) return FPSCHED_ENOMEM;
  // finish times stay below 2^30: every item starts at most (items before it) * (largest cost + latency) late
  if (3ll * p->S * p->m * (p->max_dur + p->max_comm) >= (1ll << 30)) return FPSCHED_EOVERFLOW;
  const int V = p->tables.gen_row_chunks;
  const int deg = p->max_degree <= 1 ? 1 : 2;
  // cost rows shared by the workgroup (the sliding form on a DAG of degree one needs the first halves only); per wavefront
  // its counters and its sets' slots, sliding: the rings of items and the queues (one bit per W item of a device at two
  // stages per device, two at four, none at one)
  const int64_t shared_ints = 3ll * V * p->D * (slide && deg == 1 ? 4 : 8);
  DevTables tables = p->tables;
  tables.gen_events = kGenFewEvents;
  // (one word more: the word of the next entry is written when all are in as well)
  tables.gen_queue_words = slide && V > 1 ? (int)((int64_t)V * p->m * (V == 2 ? 1 : 2) / 32) + 1 : 0;
  auto wave_ints_of = [&](int64_t sets) {
    return ((sets * 2 * p->S + 2 + 3) & ~3ll) + sets * p->tables.gen_slot_words +
           (slide ? 64ll * (tables.gen_events + tables.gen_queue_words) : 0ll);
  };
  const int64_t lds_ints = p->max_lds / 4;
  int cpw = 64 / p->D;
  while (cpw > 1 && shared_ints + wave_ints_of(cpw) + 64 > lds_ints) --cpw;
  // Sliding: the rounds in which items are settled are made for all lanes when some lane's ring is full, so a set is done sooner the
  // fewer others its wavefront has; up to two sets per SIMD there is a wavefront for each SIMD's share.  Full wavefronts and these, 32
  // to 1,024 sets: 2 x 32 x 2 124 and 102 to 110 us, 8 x 32 x 2 230 to 244 and 189 to 207, 8 x 48 x 1 121 to 135 and 103 to 115, 16 x 64 x 2
  // 628 to 658 and 560 to 615, 16 x 32 x 4 1270 to 1321 and 1190 to 1297, 32 x 128 x 2 2023 to 2220 and 1937 to 2101 (at 512 sets 2075
  // and 2101); 2,048 sets: 8 x 32 x 2 243 and 226, 16 x 64 x 2 704 and 650, 2 x 32 x 2 124 and 125; 4,096 (as many, so four each) 8 x 32 x
  // 2 258 and 241, but 4 x 24 x 1 57.5 and 59.2, 2 x 32 x 2 124 and 127.  (Results without sliding: no difference.)
  const int64_t n_simds = 4ll * p->n_cu;
  if (slide && n_sets <= 2 * n_simds) cpw = (int)std::clamp<int64_t>((n_sets + n_simds - 1) / n_simds, 1, cpw);
  if (shared_ints + wave_ints_of(cpw) > lds_ints) return FPSCHED_EUNSUPPORTED;
  tables.gen_sets = cpw;
  GenShape shape = gen_shape(p, n_sets, cpw, shared_ints, wave_ints_of(cpw));
  // A larger ring of items evens out lanes whose items come in bursts; but a set that ends has its ring emptied while the
  // other sets of its wavefront wait.  So it pays where a set has many items per actor and a wavefront few sets.  Items
  // per actor / sets per wavefront, rings of 16 and 32: 4 (65,536 sets of 4 x 16 x 2) 183 and 280 us, 16 (of 8 x 32 x 2) 800 and
  // 820, 16 (of 4 x 128 x 1) 533 and 621, 32 (of 16 x 64 x 1) 916 and 933, 48 (30,000 of 12 x 40 x 3) 2439 and 2385, 60
  // (16,384 of 6 x 100 x 3) 2360 and 2169, 64 (32,768 of 16 x 64 x 2) 1985 and 1960, 80 (16,384 of 10 x 120 x 2) 2167 and
  // 1425, 256 (of 32 x 128 x 2) 4138 and 3970.  (64: 4735 on the last, whose wavefronts then do not all find room.)  And it
  // must not cost wavefronts: 65,536 of 32 x 128 x 2 14,353 us with 8 per compute unit and rings of 32, 11,607 with 12
  // and 16; 32,768 of 20 x 100 x 2 3419 and 3200.
  if (slide && 2 * max_chunks_of(p) * p->m >= 40 * (64 / p->D)) {
    tables.gen_events = kGenMoreEvents;
    const int64_t more_ints = wave_ints_of(cpw);
    const GenShape other = gen_shape(p, n_sets, cpw, shared_ints, more_ints);
    if (shared_ints + more_ints + 64 <= lds_ints && other.resident >= shape.resident) shape = other;
    else tables.gen_events = kGenFewEvents;
  }
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  static const GenKernel table[2][3][2] = {
      {{&generate_kernel<1, 1, kGenTimed>, &generate_kernel<1, 2, kGenTimed>},
       {&generate_kernel<2, 1, kGenTimed>, &generate_kernel<2, 2, kGenTimed>},
       {&generate_kernel<4, 1, kGenTimed>, &generate_kernel<4, 2, kGenTimed>}},
      {{&generate_kernel<1, 1, kGenSlide>, &generate_kernel<1, 2, kGenSlide>},
       {&generate_kernel<2, 1, kGenSlide>, &generate_kernel<2, 2, kGenSlide>},
       {&generate_kernel<4, 1, kGenSlide>, &generate_kernel<4, 2, kGenSlide>}}};
  const GenKernel kernel = V == 2 && one_neighbour(p) ? (slide ? &generate_kernel<2, kGenOneNeighbour, kGenSlide> : &generate_kernel<2, kGenOneNeighbour, kGenTimed>)
                                                      : table[slide ? 1 : 0][V == 1 ? 0 : (V == 2 ? 1 : 2)][deg - 1];
  if (shape.lds_bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                          p->max_lds) != hipSuccess)
    return FPSCHED_EHIP;
  unsigned long long* counter = static_cast<unsigned long long*>(d_workspace);
  const int n_classes = order_sets(p, d_inflight, nullptr, n_sets, n_sets, shape.blocks * shape.waves * cpw, false, d_status, counter,
                                   static_cast<hipStream_t>(hip_stream));
  if (n_classes < 0) return n_classes;
  hipLaunchKernelGGL(kernel, dim3((unsigned)shape.blocks), dim3(64 * shape.waves), (size_t)shape.lds_bytes,
                     static_cast<hipStream_t>(hip_stream), tables, reinterpret_cast<const int32_t*>(d_policy),
                     d_inflight, nullptr, (long long)n_sets, (long long)n_sets, n_classes, 0, nullptr, d_steps, d_status, counter,
                     GenResults{reinterpret_cast<long long*>(out.makespan), reinterpret_cast<long long*>(out.idle),
                                out.peak, out.flags});
  return check_hip(hipGetLastError());
}

int fpsched_generate_evaluate(const fpsched_problem* p, const fpsched_actor_policy* d_policy,
                              const int32_t* d_inflight, int64_t n_sets, fpsched_results out, int32_t* d_steps,
                              uint8_t* d_status, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  return run_generate_evaluate(p, d_policy, d_inflight, n_sets, out, d_steps, d_status, d_workspace, workspace_bytes,
                               hip_stream, false);
}

int fpsched_generate_slide_evaluate(const fpsched_problem* p, const fpsched_actor_policy* d_policy,
                                    const int32_t* d_inflight, int64_t n_sets, fpsched_results out, int32_t* d_steps,
                                    uint8_t* d_status, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  return run_generate_evaluate(p, d_policy, d_inflight, n_sets, out, d_steps, d_status, d_workspace, workspace_bytes,
                               hip_stream, true);
}

// The order in which a top-k workgroup walks its batches of elements: every `step`-th of them, about 0.62 of all, so that
// the first few are spread over the part wherever they stop.
static unsigned batch_step(unsigned batches) {
  unsigned step = std::max(1u, batches * 5u / 8u);
  while (std::gcd(step, batches) != 1u) ++step;
  return step;   // (at most batches - 1, or 1: no common divisor)
}

// k smallest (key, index) among the entries whose flag byte is 0: parts, then parts of the parts' survivors, at last one
// workgroup.  key_buffers: as fpsched_workspace_bytes lays them out.
static int run_topk(const long long* keys, const unsigned char* flags, int64_t n_cand, int32_t k, bool wide_values,
                    int64_t* d_idx, int64_t* d_key, int32_t* d_count, char* key_buffers, hipStream_t st) {
  long long* f_idx = reinterpret_cast<long long*>(d_idx);
  long long* f_ms = reinterpret_cast<long long*>(d_key);
  Key* buffer[2] = {reinterpret_cast<Key*>(key_buffers), nullptr};
  buffer[1] = buffer[0] + std::max<int64_t>(1, (n_cand + kTile - 1) / kTile) * k;
  // Elements a workgroup sorts at a time: twice k at least, so that a sort makes room for as many as there are threads;
  // no more than 1024 unless k needs it (a sort of 2048 takes twice as long), no more than there are.
  auto room_for = [&](int64_t n) {
    int64_t room = 128;
    while (room < 2 * (int64_t)k || (room < n && room < 1024)) room <<= 1;
    return room;
  };
  const Key* in = nullptr;
  int64_t n = n_cand;
  for (int level = 0;; ++level) {
    // Parts: one while a workgroup needs but a few sorts; else as many as leave the next launch about 2048 survivors, but
    // enough that none is longer than kTopkPartRooms sorts' worth (more launches instead of longer ones: each level has
    // at most 1/16 of the elements of the one before).  At most one part per kTile elements: a level's survivors then fit
    // their buffer, k per kTile elements.
    const int64_t most = kTopkPartRooms * room_for(n), tiles = (n + kTile - 1) / kTile;
    int64_t parts = 1;
    if (level == 0 ? n > kTile : n > most) parts = std::max(std::min(std::clamp<int64_t>(2048 / k, 8, 64), tiles), (n + most - 1) / most);
    const int64_t n_part = std::max<int64_t>((n + parts - 1) / parts, 1);
    parts = std::max<int64_t>((n + n_part - 1) / n_part, 1);
    if (parts > 0x7fffffffll) return FPSCHED_EINVAL;
    const unsigned threads = (unsigned)(room_for(n_part) / 2), batches = (unsigned)((n_part + threads - 1) / threads);
    const bool last = parts == 1;
    Key* out = buffer[level & 1];
    hipLaunchKernelGGL(topk_kernel, dim3((unsigned)parts), dim3(threads), threads * 24u, st, keys, flags, in, (long long)n,
                       (long long)n_part, batches, batch_step(batches), (int)k, (int)wide_values, last ? (Key*)nullptr : out,
                       last ? f_idx : (long long*)nullptr, last ? f_ms : (long long*)nullptr, last ? d_count : (int*)nullptr);
    if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
    if (last) return FPSCHED_OK;
    in = out;
    n = parts * k;
  }
}

int fpsched_topk(const fpsched_problem* p, fpsched_results in, int64_t n_cand, int32_t k,
                 int64_t* d_idx, int64_t* d_makespan, int32_t* d_count, void* d_workspace,
                 size_t workspace_bytes, void* hip_stream) {
  if (!p || n_cand < 0 || k < 1 || k > 1024 || !d_idx || !d_makespan || !d_count) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (n_cand > 0 && (!in.makespan || !in.flags)) return FPSCHED_EINVAL;
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < fpsched_workspace_bytes(p, n_cand, k)) return FPSCHED_ENOMEM;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  return run_topk(reinterpret_cast<const long long*>(in.makespan), in.flags, n_cand, k, false, d_idx, d_makespan, d_count,
                  static_cast<char*>(d_workspace) + 256, static_cast<hipStream_t>(hip_stream));
}

size_t fpsched_static_scratch_bytes(void) { return kStaticScratchBytes; }

int fpsched_evaluate_topk_static(const fpsched_problem* p, const uint16_t* d_ops, int64_t n_cand,
                                 int32_t stride_words, fpsched_results out, int32_t k, int64_t* d_idx,
                                 int64_t* d_makespan, int32_t* d_count, void* hip_stream) {
  if (!p || n_cand < 0 || k < 1 || k > 1024) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (!p->d_static_scratch) return FPSCHED_EHIP;
  // the same layout as a caller's workspace: [256 bytes: work counter][top-k key buffers]
  if (fpsched_workspace_bytes(p, n_cand, k) > kStaticScratchBytes) return FPSCHED_ESCRATCH;
  // (the counter is preset by a kernel and every key that is read was written by the level before: nothing
  // of an earlier call's contents is ever looked at)
  const int rc = fpsched_evaluate(p, d_ops, n_cand, stride_words, out, p->d_static_scratch, kStaticScratchBytes,
                                  hip_stream);
  if (rc != FPSCHED_OK) return rc;
  return fpsched_topk(p, out, n_cand, k, d_idx, d_makespan, d_count, p->d_static_scratch, kStaticScratchBytes,
                      hip_stream);
}

size_t fpsched_rank_workspace_bytes(const fpsched_problem* p, int64_t n_cand, int32_t k) {
  if (!p || n_cand < 0) return 0;
  const size_t base = (fpsched_workspace_bytes(p, n_cand, k) + 15) & ~(size_t)15;
  return base + (size_t)n_cand * 8 + (((size_t)n_cand + 15) & ~(size_t)15);
}

int fpsched_rank(const fpsched_problem* p, fpsched_results in, int64_t n_cand, int32_t k, int32_t mode,
                 int32_t include_over_cap, int64_t* d_idx, int64_t* d_key, int32_t* d_count, void* d_workspace,
                 size_t workspace_bytes, void* hip_stream) {
  if (!p || n_cand < 0 || k < 1 || k > 1024 || !d_idx || !d_key || !d_count) return FPSCHED_EINVAL;
  if (mode < FPSCHED_RANK_MAKESPAN || mode > FPSCHED_RANK_IDLE) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (n_cand > 0 && (!in.makespan || !in.idle || !in.peak || !in.flags)) return FPSCHED_EINVAL;
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < fpsched_rank_workspace_bytes(p, n_cand, k)) return FPSCHED_ENOMEM;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const size_t base = (fpsched_workspace_bytes(p, n_cand, k) + 15) & ~(size_t)15;
  long long* keys = reinterpret_cast<long long*>(static_cast<char*>(d_workspace) + base);
  unsigned char* excluded = reinterpret_cast<unsigned char*>(keys + n_cand);
  if (n_cand > 0) {
    const int64_t blocks = (n_cand + 255) / 256;
    if (blocks > 0x7fffffffll) return FPSCHED_EINVAL;
    hipLaunchKernelGGL(rank_keys_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       reinterpret_cast<const long long*>(in.makespan), reinterpret_cast<const long long*>(in.idle),
                       in.peak, in.flags, (long long)n_cand, (int)p->D, (int)mode, (int)(include_over_cap != 0), keys,
                       excluded);
    if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  }
  return run_topk(keys, excluded, n_cand, k, mode == 1 || mode == 2, d_idx, d_key, d_count, static_cast<char*>(d_workspace) + 256, st);
}

// workspace of the sliding pass: [256 bytes: candidate counter][low halves of the start times: 16 bits per op
// word and lane of a candidate][escape lists: escape_cap dwords per row][stop positions: int32 per row]
// [flags of the timing pass: one byte per candidate]
static size_t wslide_starts_bytes(const fpsched_problem* p, int64_t n_cand, int32_t stride_words) {
  return (size_t)n_cand * p->tables.lanes_per_cand * (size_t)stride_words * sizeof(uint16_t);
}
// entries of a row's escape list: an op that waits 2^16 time units or more for its inputs; each such wait
// uses up 2^16 of the largest possible finish time (links: two transfers per op at most), plus the end mark
static int wslide_escape_cap(const fpsched_problem* p) {
  const int64_t bound = (int64_t)p->D * p->max_stride * (p->max_dur + 2 * p->max_comm);
  return (int)std::min<int64_t>(bound >> 16, 255) + 2;
}
static size_t wslide_escape_bytes(const fpsched_problem* p, int64_t n_cand) {
  return (((size_t)n_cand * p->D * wslide_escape_cap(p) * sizeof(uint32_t)) + 15) & ~(size_t)15;
}

size_t fpsched_wslide_workspace_bytes(const fpsched_problem* p, int64_t n_cand, int32_t stride_words) {
  if (!p || n_cand < 0 || stride_words < 8) return 0;
  const size_t rows = (size_t)n_cand * p->D;
  return 256 + wslide_starts_bytes(p, n_cand, stride_words) + wslide_escape_bytes(p, n_cand) +
         ((rows * sizeof(int32_t) + 15) & ~(size_t)15) + (((size_t)n_cand + 15) & ~(size_t)15);
}

int fpsched_wslide(const fpsched_problem* p, const uint16_t* d_ops, int64_t n_cand, int32_t stride_words,
                   uint16_t* d_ops_out, int32_t stride_out_words, fpsched_results out, void* d_workspace,
                   size_t workspace_bytes, void* hip_stream) {
  if (!p || n_cand < 0) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (!p->has_w) return FPSCHED_EINVAL;
  // the pass knows one cost per (type, stage)
  if (!p->slide_ok || p->mb_set || p->sync_on || p->copy_depth > 0 || (p->links_on && !p->links_slide_ok)) return FPSCHED_EUNSUPPORTED;
  if (n_cand == 0) return FPSCHED_OK;
  if (!d_ops || !d_ops_out || !out.makespan || !out.idle || !out.peak || !out.flags) return FPSCHED_EINVAL;
  if (stride_words < 8 || (stride_words & 7) || stride_words > p->max_stride) return FPSCHED_EINVAL;
  if (stride_out_words < 8 || (stride_out_words & 7) || stride_out_words > p->max_stride) return FPSCHED_EINVAL;
  if ((reinterpret_cast<uintptr_t>(d_ops) & 15) || (reinterpret_cast<uintptr_t>(d_ops_out) & 15)) return FPSCHED_EINVAL;
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < fpsched_wslide_workspace_bytes(p, n_cand, stride_words)) return FPSCHED_ENOMEM;
  const int lpc = p->stab.lanes_per_cand;
  // wavefronts per workgroup: as many workgroups of a compute unit's LDS as leave it full (rows differ in length, and a
  // workgroup's LDS is free when its last wavefront is done)
  const int64_t place_rows_bytes = (int64_t)kNKinds * kMaxChunks * lpc * 8;
  int place_waves = 1, place_groups = 1;
  for (int groups = 1; groups <= 8; ++groups) {
    const int wv = (int)std::min<int64_t>((p->max_lds / groups - place_rows_bytes) / kSlideWaveLdsBytes, kSlideThreads / 64);
    if (wv >= 1 && wv * groups >= place_waves * place_groups) { place_waves = wv; place_groups = groups; }
  }
  // (a small batch is spread over the compute units: fewer wavefronts per workgroup)
  const int64_t place_waves_all = (n_cand * lpc + 63) / 64;
  const int place_threads = 64 * (int)std::clamp<int64_t>((place_waves_all + std::max(p->n_cu, 1) - 1) / std::max(p->n_cu, 1),
                                                          1, place_waves);
  const int64_t place_blocks = (n_cand * lpc + place_threads - 1) / place_threads;
  if (place_blocks > 0x7fffffffll) return FPSCHED_EINVAL;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(d_workspace);
  unsigned long long* counter = reinterpret_cast<unsigned long long*>(ws);
  uint32_t* starts = reinterpret_cast<uint32_t*>(ws + 256);
  uint32_t* escapes = reinterpret_cast<uint32_t*>(ws + 256 + wslide_starts_bytes(p, n_cand, stride_words));
  const int escape_cap = wslide_escape_cap(p);
  int32_t* stops = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(escapes) + wslide_escape_bytes(p, n_cand));
  unsigned char* timed_flags = reinterpret_cast<unsigned char*>(stops) + (((size_t)n_cand * p->D * sizeof(int32_t) + 15) & ~(size_t)15);
  // pass 1: the lists without their W items, timed by the evaluation kernel (launched as in fpsched_evaluate)
  // (under the link model: that model's tables and workgroup shape; W items send nothing, so the second
  // pass is the same)
  const bool links = p->links_on;
  if (!links && p->lists_times.ok && stride_words <= kTimeMaxStride) {
    const fpsched_results timed{out.makespan, out.idle, out.peak, timed_flags};   // (what the order pass leaves stands in the results until pass 2)
    const StartTimes left{starts, escapes, stops, escape_cap, lpc};
    const int rc = run_list_evaluation(p, &p->lists_times, d_ops, n_cand, stride_words, timed, counter, st, &left);
    if (rc != FPSCHED_OK) return rc;
  } else {
    const SlotTables& times_tab = links ? p->stab_times_links : p->stab_times;
    const int waves = links ? p->links_waves : p->slot_waves;
    const int grid = links ? p->links_grid : p->slot_grid;
    const size_t times_lds = (size_t)(links ? p->links_lds_bytes : p->slot_lds_bytes) + 16;
    const SlotLaunch L = slot_launch(times_tab, waves, grid, times_lds, n_cand);
    const int per_block = times_tab.cands_per_wave * L.waves;
    const int64_t blocks = L.blocks;
    const int64_t row_words = (int64_t)p->D * stride_words;
    const int draw_block = (int)std::clamp<int64_t>((12288 + row_words - 1) / row_words, 1, times_tab.cands_per_wave);
    const bool one_class = p->stab.n_classes == 1;
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, st, counter, (unsigned long long)(blocks * per_block), 0ull);
    hipLaunchKernelGGL(links ? slot_kernel_of<kSlotTimesLinks>(p->slot_v, p->slot_deg2, one_class)
                             : slot_kernel_of<kSlotTimes>(p->slot_v, p->slot_deg2, one_class),
                       dim3((unsigned)blocks), dim3(64 * L.waves), L.lds_bytes, st, times_tab, d_ops, (long long)n_cand,
                       (int)stride_words, (long long*)nullptr, (long long*)nullptr, (int*)nullptr, timed_flags, counter,
                       draw_block, starts, stops, (const int32_t*)nullptr, escapes, escape_cap);
    if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  }
  // pass 2: every row places its W items on its own, by a lane, whose steps wait for each other, or by a wavefront, of which
  // a compute unit has few: so where rows are few, and the more so the longer they are.  Both passes, a lane / a wavefront per
  // row, 28 shapes, at 8,192, 12,288, 16,384 and 24,576 rows:
  //   up to 120 items 1.03 to 1.16, 0.91 (20 x 10 x 1) to 1.09 (12 x 30 x 1; 16 x 8 x 2 93 and 95 us), 0.84 to 1.03, 0.74 to 0.92; on four
  //   devices 1.17, 1.10, 0.99, 0.88;
  //   144 to 384 items on more than eight devices 1.01 (24 x 24 x 2, 30 x 60 x 1) to 1.14, 0.97 to 1.03 (16 x 64 x 2 545 and 541), 0.90 to 0.96
  //   (16 x 64 x 2 546 and 598), 0.78 to 0.86; on five and eight 1.19 and 1.20, 1.07 and 1.09 (8 x 32 x 2 220 and 202), 0.95 and 1.00, 0.77 and 0.87;
  //   on two and three 1.67 and 1.27, 1.58 and 1.13, 1.51 and 1.05, 1.41 and 0.88;
  //   450 items and more 1.23 to 1.89, 1.10 to 1.72, 1.05 (20 x 50 x 3) to 1.54, 0.94 (20 x 50 x 3; 32 x 50 x 3 1.00) to 1.35 (32 x 128 x
  //   2 2104 and 1851 us), at 32,768 0.82 to 1.16 (32 x 128 x 2 1.02).
  const int stash = (int)std::min<int64_t>((int64_t)max_chunks_of(p) * p->m, stride_words);
  const int64_t rows_shared = place_rows_bytes + 4ll * 4 * kMaxDevices, rows_wave = slide_rows_wave_bytes(stride_out_words, stash);
  const int64_t rows_waves = std::min<int64_t>({(p->max_lds - rows_shared) / rows_wave, kSlideThreads / 64, p->D});
  const int64_t items = 3ll * max_chunks_of(p) * p->m, few_rows = items >= 448 ? 24576 : p->D <= (items >= 128 ? 8 : 4) ? 16384 : 12288;
  if (n_cand * p->D <= few_rows && rows_waves >= std::min(p->D, 4)) {
    hipLaunchKernelGGL(wslide_place_rows_kernel, dim3((unsigned)n_cand), dim3(64 * (unsigned)rows_waves),
                       (size_t)(rows_shared + rows_waves * rows_wave), st, p->stab, d_ops, (int)stride_words, starts, escapes,
                       escape_cap, stops, timed_flags, d_ops_out, (int)stride_out_words, stash,
                       reinterpret_cast<long long*>(out.makespan), reinterpret_cast<long long*>(out.idle), out.peak, out.flags);
    return check_hip(hipGetLastError());
  }
  hipLaunchKernelGGL(p->slot_v > 2 ? wslide_place_kernel<true> : wslide_place_kernel<false>, dim3((unsigned)place_blocks), dim3(place_threads),
                     (size_t)place_rows_bytes + (place_threads / 64) * kSlideWaveLdsBytes, st, p->stab, d_ops,
                     (long long)n_cand, (int)stride_words,
                     starts, escapes, escape_cap, stops, timed_flags, d_ops_out, (int)stride_out_words,
                     reinterpret_cast<long long*>(out.makespan), reinterpret_cast<long long*>(out.idle), out.peak,
                     out.flags);
  return check_hip(hipGetLastError());
}

int fpsched_wslide_evaluate(const fpsched_problem* p, const uint16_t* d_ops, int64_t n_cand, int32_t stride_words,
                            fpsched_results out, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p || n_cand < 0) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (!p->has_w) return FPSCHED_EINVAL;
  if (!p->slide_eval_ok || p->mb_set || p->sync_on || p->copy_depth > 0 || (p->links_on && !p->links_slide_eval_ok))
    return FPSCHED_EUNSUPPORTED;
  if (n_cand == 0) return FPSCHED_OK;
  if (!d_ops || !out.makespan || !out.idle || !out.peak || !out.flags) return FPSCHED_EINVAL;
  if (stride_words < 8 || (stride_words & 7) || stride_words > p->max_stride) return FPSCHED_EINVAL;
  if (reinterpret_cast<uintptr_t>(d_ops) & 15) return FPSCHED_EINVAL;
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < 256) return FPSCHED_ENOMEM;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  unsigned long long* counter = static_cast<unsigned long long*>(d_workspace);
  // launched as fpsched_evaluate launches the plain form, or the link form (same workgroup shape; 16 bytes of LDS more)
  const bool links = p->links_on;
  const SlotTables& tab = links ? p->stab_slide_links : p->stab_slide;
  const SlotLaunch L = slot_launch(tab, links ? p->links_waves : p->slot_waves, links ? p->links_grid : p->slot_grid,
                                   (size_t)(links ? p->links_lds_bytes : p->slot_lds_bytes) + 16, n_cand);
  const int per_block = tab.cands_per_wave * L.waves;
  const int64_t blocks = L.blocks;
  const int64_t row_words = (int64_t)p->D * stride_words;
  const int draw_block = (int)std::clamp<int64_t>((12288 + row_words - 1) / row_words, 1, tab.cands_per_wave);
  hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, st, counter, (unsigned long long)(blocks * per_block), 0ull);
  hipLaunchKernelGGL(links ? slot_kernel_of<kSlotSlideLinks>(p->slot_v, p->slot_deg2, tab.n_classes == 1)
                           : slot_kernel_of<kSlotSlide>(p->slot_v, p->slot_deg2, tab.n_classes == 1), dim3((unsigned)blocks),
                     dim3(64 * L.waves), L.lds_bytes, st, tab, d_ops, (long long)n_cand,
                     (int)stride_words, reinterpret_cast<long long*>(out.makespan), reinterpret_cast<long long*>(out.idle),
                     out.peak, out.flags, counter, draw_block, (uint32_t*)nullptr, (int32_t*)nullptr,
                     (const int32_t*)nullptr, (uint32_t*)nullptr, 0);
  return check_hip(hipGetLastError());
}

static int64_t pareto_tiles(int64_t n_cand) { return (n_cand + kTile - 1) / kTile; }

size_t fpsched_pareto_workspace_bytes(const fpsched_problem* p, int64_t n_cand) {
  if (!p || n_cand < 0) return 0;
  const size_t tiles = (size_t)pareto_tiles(n_cand);
  // [256 reserved][tile fronts: Key, then peak, kTile entries per tile][entries per tile front]
  return 256 + tiles * kTile * (sizeof(Key) + sizeof(int32_t)) + ((tiles * sizeof(int32_t) + 15) & ~(size_t)15);
}

int fpsched_pareto(const fpsched_problem* p, fpsched_results in, int64_t n_cand, int32_t kmax, int64_t* d_idx,
                   int64_t* d_makespan, int32_t* d_peak, int32_t* d_count, void* d_workspace,
                   size_t workspace_bytes, void* hip_stream) {
  if (!p || n_cand < 0 || kmax < 1 || kmax > 1024 || !d_idx || !d_makespan || !d_peak || !d_count)
    return FPSCHED_EINVAL;
  if (pareto_tiles(n_cand) > kParetoMaxTiles) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (n_cand > 0 && (!in.makespan || !in.peak || !in.flags)) return FPSCHED_EINVAL;
  if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) & 15)) return FPSCHED_EINVAL;
  if (workspace_bytes < fpsched_pareto_workspace_bytes(p, n_cand)) return FPSCHED_ENOMEM;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int64_t tiles = pareto_tiles(n_cand);
  Key* front_keys = reinterpret_cast<Key*>(static_cast<char*>(d_workspace) + 256);
  int* front_peak = reinterpret_cast<int*>(front_keys + tiles * kTile);
  int* tile_count = front_peak + tiles * kTile;
  if (tiles > 0) {
    hipLaunchKernelGGL(pareto_tile_kernel, dim3((unsigned)tiles), dim3(kTile / 2), 0, st,
                       reinterpret_cast<const long long*>(in.makespan), in.peak, in.flags, (long long)n_cand,
                       (int)p->D, front_keys, front_peak, tile_count);
    if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  }
  hipLaunchKernelGGL(pareto_merge_kernel, dim3(1), dim3(kParetoMergeThreads), 0, st, front_keys, front_peak,
                     tile_count, (int)tiles, (int)kmax, reinterpret_cast<long long*>(d_idx),
                     reinterpret_cast<long long*>(d_makespan), d_peak, d_count);
  if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  return FPSCHED_OK;
}

int fpsched_apply_caps(const fpsched_problem* p, const int32_t* d_peak, const int32_t* d_caps,
                       int32_t per_candidate, int64_t n_cand, uint8_t* d_flags, void* hip_stream) {
  if (!p || n_cand < 0 || !d_caps) return FPSCHED_EINVAL;
  if (p->device_id < 0) return FPSCHED_ENODEV;
  if (n_cand == 0) return FPSCHED_OK;
  if (!d_peak || !d_flags) return FPSCHED_EINVAL;
  const int64_t blocks = (n_cand + 255) / 256;
  if (blocks > 0x7fffffffll) return FPSCHED_EINVAL;
  DeviceGuard g(p->device_id);
  if (!g.ok) return FPSCHED_EHIP;
  hipLaunchKernelGGL(apply_caps_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                     d_peak, d_caps, (int)(per_candidate != 0), (long long)n_cand, (int)p->D, d_flags);
  if (hipGetLastError() != hipSuccess) return FPSCHED_EHIP;
  return FPSCHED_OK;
}

int fpsched_encode(const fpsched_problem* p, const int32_t* ksm, int32_t device, int32_t n,
                   uint16_t* out_words) {
  if (!p || n < 0 || device < 0 || device >= p->D || (n > 0 && (!ksm || !out_words))) return FPSCHED_EINVAL;
  for (int i = 0; i < n; ++i) {
    const int kind = ksm[3 * i], s = ksm[3 * i + 1], j = ksm[3 * i + 2];
    if (kind <= FPSCHED_END || kind >= FPSCHED_NKINDS || s < 0 || s >= p->S || j < 0 || j >= p->sync_items[s])
      return FPSCHED_EINVAL;
    if (p->stage_device[s] != device) return FPSCHED_EINVAL;
    if (kind == FPSCHED_W && !p->has_w) return FPSCHED_EINVAL;
    out_words[i] = FPSCHED_WORD(kind, p->stage_chunk[s], j);
  }
  return FPSCHED_OK;
}

int64_t fpsched_validate(const fpsched_problem* p, const uint16_t* h_ops, int64_t n_cand,
                         int32_t stride_words) {
  if (!p || n_cand < 0 || stride_words < 1 || (n_cand > 0 && !h_ops)) return FPSCHED_EINVAL;
  int64_t bad = 0;
  for (int64_t c = 0; c < n_cand; ++c) {
    bool cand_bad = false;
    for (int d = 0; d < p->D && !cand_bad; ++d) {
      const uint16_t* row = h_ops + ((size_t)c * p->D + d) * stride_words;
      for (int i = 0; i < stride_words; ++i) {
        const unsigned w = row[i];
        const int kind = w >> 13;
        if (kind == FPSCHED_END) break;
        const int c = (int)((w >> 11) & 3);
        if (c >= p->n_chunks[d] || (int)(w & 0x7ff) >= p->sync_items[p->local_stage[(size_t)d * kMaxChunks + c]] ||
            (kind == FPSCHED_W && !p->has_w)) { cand_bad = true; break; }
      }
    }
    bad += cand_bad;
  }
  return bad;
}

}  // extern "C"
