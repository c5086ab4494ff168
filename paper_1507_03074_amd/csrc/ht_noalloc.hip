// ht_noalloc.hip -- ht_fill_peaks_noalloc: the fused fill and peak search of one event with all
// of the library's device scratch in one fixed array of this file, so the call allocates no
// device memory.
//
// The array `scratch` (kNoAllocBytes, 256-byte aligned, zero when the code object is loaded)
// holds, on each device the library runs on:
//   [0, kCounterBytes)            the pair of slab-counter arrays (one counts, one is cleared)
//   [kTabOff, kTabOff + kTabBytes) the bin-rule tables of the grid last used on the device
//   [kEvOff, kNoAllocBytes)       the event scratch (slab lists, survivor masks, peak counts)
// Host code never passes the array's name to a kernel or a copy: its host-side symbol is only
// a stand-in. The device address of each device's copy is looked up once, with that device
// current, and kept in g_ptr[device].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "ht_internal.h"

// 64 MiB: the largest event scratch of the call (see kNoAllocBytes below)
static __device__ __align__(256) unsigned char scratch[(size_t)64 << 20];

namespace ht {
namespace {

constexpr size_t kNoAllocBytes = (size_t)64 << 20;
constexpr int kNoAllocMaxDevices = 64;
// tables: a2 up to kNoAllocMaxA floats, phi up to 4 * 4096, theta up to 2 * (2 * 4096 + 1)
constexpr size_t kNoAllocMaxA = 16384;
constexpr size_t kTabOff = (kCounterBytes + 255) & ~(size_t)255;
constexpr size_t kEvOff = 295424;  // the limit below is what the array holds past it
constexpr size_t kTabBytes = kEvOff - kTabOff;
static_assert(4 * (kNoAllocMaxA + 4 * kMaxSlabs + 2 * (2 * kMaxSlabs + 1)) + 3 * 256 <= kTabBytes,
              "the largest tables fit their region");

static_assert(sizeof(scratch) == kNoAllocBytes, "the array is kNoAllocBytes long");

std::mutex g_na_mu;
char* g_ptr[kNoAllocMaxDevices];          // device address of each device's scratch, or null
uint8_t g_parity[kNoAllocMaxDevices];     // which counter array the next call counts into
bool g_tab_valid[kNoAllocMaxDevices];     // the table region holds the tables of g_tab_grid
ht_grid g_tab_grid[kNoAllocMaxDevices];
float g_inv_db[kNoAllocMaxDevices];       // and their 1 / (width of a B bin)
// host staging of the tables (a fixed array, so no host allocation either)
float g_tab_host[kTabBytes / 4];

bool same_tables(const ht_grid& a, const ht_grid& b)
{
  return a.n_theta == b.n_theta && a.n_phi == b.n_phi && a.n_a == b.n_a && a.n_b == b.n_b &&
         std::memcmp(&a.a_min, &b.a_min, 4) == 0 && std::memcmp(&a.a_max, &b.a_max, 4) == 0 &&
         std::memcmp(&a.b_min, &b.b_min, 4) == 0 && std::memcmp(&a.b_max, &b.b_max, 4) == 0;
}

size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

// The call's size limit, in bytes: what it accepts is part of its contract, so it is an arithmetic
// of its own and not what the layout of the day takes. The slab lists, 16 bytes per tile of the
// reported launch shape, and for a crowded event (of at least the reported dense_hits hits) the
// stencil's peak words, for any other nine bytes per entry of a candidate list of cand_cap cells per
// tile, or of a quarter of the bound 4 n_hits n_a / threshold on the cells that can reach the
// threshold where that is more.
size_t limit_bytes(const DevGrid& g, const Tiling& tl, int64_t n, bool direct)
{
  const size_t t = (size_t)tl.n_tiles;
  size_t b = event_scratch_bytes(g, n, direct, 0) + 4 * al256(4 * t) +
             al256(4 * ((t + tl.group_tiles - 1) / tl.group_tiles));
  if (g.lds_fill && tl.dense_hits > 0 && n >= tl.dense_hits) return b + al256(mask_bytes(g));  // crowded
  const size_t cells = (size_t)g.n_theta * g.n_phi * g.n_a * g.n_b;
  const size_t bound = (size_t)n * (g.phi_sectors ? 2 : 4) * (size_t)g.n_a / (size_t)g.threshold;
  const size_t pool = std::min<size_t>(std::max(t * (size_t)tl.cand_cap, std::min(cells, bound / 4)), 0xfffffff0u);
  return b + al256(8 * pool) + al256(pool);
}

int check_tables(const ht_grid& grid)
{
  if ((size_t)grid.n_a > kNoAllocMaxA)
    return fail(HT_EINVAL, "ht_fill_peaks_noalloc: n_a = %d exceeds its table limit of %zu A bins",
                grid.n_a, kNoAllocMaxA);
  return HT_OK;
}

}  // namespace

int plan_noalloc(const ht_grid& grid, const Tiling& tl, const DevGrid& g, int64_t n, NoallocPlan* plan)
{
  if (int rc = check_tables(grid)) return rc;
  const size_t room = kNoAllocBytes - kEvOff;
  const bool can_direct = direct_lists(g, n);
  const size_t need = limit_bytes(g, tl, n, can_direct && limit_bytes(g, tl, n, true) <= room);
  if (need > room)
    return fail(HT_EINVAL,
                "ht_fill_peaks_noalloc: this event needs %zu bytes of scratch; the fixed scratch "
                "holds %zu (use ht_fill_peaks)", need, room);
  // the layout: direct slab lists where they fit with the search's scratch, else the counting sort
  auto fits = [&](bool direct, int peaks) { return event_scratch_bytes(g, n, direct, peaks) <= room; };
  auto either = [&](int peaks) { return (can_direct && fits(true, peaks)) || fits(false, peaks); };
  // survivors that do not fit beside the lists of an event that the limit takes for a crowded one
  // leave it to the stencil
  const bool crowded = g.lds_fill && tl.dense_hits > 0 && n >= tl.dense_hits;
  plan->dense = g.lds_fill && (dense_peaks(g, n) || (crowded && !either(kPeakBands)));
  const int search = batch_shape(g, 1, n, plan->dense, 1).few ? kPeakFew : kPeakBands;
  plan->sliced = !plan->dense && !either(search);
  const int layout = plan->sliced ? 0 : plan->dense ? kPeakMask : search;
  plan->layout = layout;
  plan->direct = can_direct && fits(true, layout);
  plan->scratch_bytes = event_scratch_bytes(g, n, plan->direct, layout);
  plan->slice_groups = 0;
  if (plan->sliced) {
    // The survivors do not fit beside the slab lists: the peaks are searched in the written matrix,
    // as many groups of job rows at a time as fit the whole event scratch (the lists are done with
    // then), each slice counting on from the one before.
    DevGrid sg = g;
    set_jobs(&sg, 0, 1);
    const size_t fixed = 256 + al256(4 * (size_t)sg.j.n_groups * sg.j.pk_step) + al256(4 * (size_t)sg.j.n_groups) + surv_bytes(sg, n, kPeakBands) + 6 * 256;
    const size_t per = (size_t)(1 + 64 * sg.j.elem_bytes) * sg.j.group_jobs + 8 * (size_t)sg.j.seg;
    const size_t fit = fixed < room ? (room - fixed) / per : 0;
    if (fit == 0) return fail(HT_EINVAL, "ht_fill_peaks_noalloc: one group of rows needs %zu bytes of scratch", per);
    plan->slice_groups = (uint32_t)std::min<size_t>(fit, sg.j.n_groups);
    plan->scratch_bytes = room;
  }
  if (plan->scratch_bytes > room)
    return fail(HT_EINVAL, "ht_fill_peaks_noalloc: this event needs %zu bytes of scratch; the fixed scratch holds %zu",
                plan->scratch_bytes, room);
  return HT_OK;
}

}  // namespace ht

using namespace ht;

extern "C" int ht_fill_peaks_noalloc(const ht_grid* grid, const float* x, const float* y,
                                     const float* z, int64_t n_hits, uint32_t* acc, ht_peak* out,
                                     int64_t capacity, int64_t* n_found, void* stream)
{
  if (n_hits < 0) return fail(HT_EINVAL, "n_hits < 0");
  if (!acc) return fail(HT_EINVAL, "acc is NULL");
  if (n_hits > 0 && (!x || !y || !z)) return fail(HT_EINVAL, "hit arrays are NULL");
  if (capacity < 0 || !n_found || (capacity > 0 && !out))
    return fail(HT_EINVAL, "peak output arguments are invalid");
  if (n_hits > ((int64_t)1 << 28)) return fail(HT_EINVAL, "n_hits must be <= 2^28");
  int rc = validate_grid(grid);
  if (rc) return rc;
  if ((rc = check_tables(*grid))) return rc;
  if ((rc = check_accessible(out, "out")) || (rc = check_accessible(n_found, "n_found"))) return rc;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  if (dev < 0 || dev >= kNoAllocMaxDevices)
    return fail(HT_EINVAL, "ht_fill_peaks_noalloc supports device ordinals below %d", kNoAllocMaxDevices);
  hipStream_t s = (hipStream_t)stream;

  // an event that does not fit is refused before any device work
  const Tiling tl = choose_tiling(*grid);
  DevGrid g = make_devgrid(*grid, DevTables(), tl, 1, n_hits);
  NoallocPlan plan;
  if ((rc = plan_noalloc(*grid, tl, g, n_hits, &plan))) return rc;
  const bool atomic = !g.lds_fill, dense = plan.dense, direct = plan.direct, sliced = plan.sliced;

  std::lock_guard<std::mutex> lk(g_na_mu);
  if (!g_ptr[dev]) {
    // once per device, with the device current: the address of this device's copy
    void* ptr = nullptr;
    if ((e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) != hipSuccess)
      return fail_hip(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) return fail(HT_EDEVICE, "hipGetSymbolAddress(scratch) returned NULL");
    g_ptr[dev] = (char*)ptr;
  }
  char* base = g_ptr[dev];
  // bin-rule tables: uploaded when the grid differs from the one whose tables the region holds
  // (a synchronous copy on the caller's stream)
  const size_t a2_off = 0;
  const size_t phi_off = al256(4 * a2_floats(*grid));
  const size_t th_off = phi_off + al256(4 * phi_floats(*grid));
  const size_t tab_bytes = th_off + 4 * th_floats(*grid);
  if (!g_tab_valid[dev] || !same_tables(g_tab_grid[dev], *grid)) {
    g_tab_valid[dev] = false;
    host_tables_into(*grid, g_tab_host + a2_off / 4, &g_inv_db[dev], g_tab_host + phi_off / 4,
                     g_tab_host + th_off / 4);
    if ((e = hipMemcpyAsync(base + kTabOff, g_tab_host, tab_bytes, hipMemcpyHostToDevice, s)) != hipSuccess)
      return fail_hip(e, "hipMemcpyAsync(tables)");
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail_hip(e, "hipStreamSynchronize(tables)");
    g_tab_grid[dev] = *grid;
    g_tab_valid[dev] = true;
  }
  DevTables t;
  t.a2 = (float*)(base + kTabOff + a2_off);
  t.phi = (float*)(base + kTabOff + phi_off);
  t.th = (float*)(base + kTabOff + th_off);
  t.inv_db = g_inv_db[dev];
  g = make_devgrid(*grid, t, tl, 1, n_hits);

  EvDesc ev;
  std::memset(&ev, 0, sizeof(ev));
  carve_event_scratch(g, n_hits, direct, base + kEvOff, &ev, plan.layout);
  ev.dense = dense ? 1 : 0;
  if (plan.layout == kPeakBands && !atomic && !use_lists(g, 1, n_hits, n_hits)) ev.lists = 0;
  uint32_t* pair = (uint32_t*)base;
  ev.slab_cnt = pair + (g_parity[dev] ? kCounterWords : 0);
  ev.slab_cnt_next = pair + (g_parity[dev] ? 0 : kCounterWords);
  ev.x = x;
  ev.y = y;
  ev.z = z;
  ev.n_hits = n_hits;
  ev.acc = acc;
  ev.out = out;
  ev.cap = capacity;
  ev.n_found = n_found;
  bool used = false;
  rc = enqueue_event(g, ev, n_hits, direct, atomic, true, !sliced, false, s, &used);
  if (used) g_parity[dev] ^= 1;
  if (rc || !sliced) return rc;
  set_jobs(&g, 0, 1);
  int64_t* carry = (int64_t*)(base + kEvOff);
  for (uint32_t g0 = 0, k = 0; g0 < g.j.n_groups; ++k) {
    const uint32_t n_grp = std::min<uint32_t>(plan.slice_groups, g.j.n_groups - g0);
    carve_peak_scratch(g, n_hits, base + kEvOff + 256, &ev, kPeakBands, g0, n_grp);
    ev.carry_in = k > 0 ? carry + (k & 1) : nullptr;
    ev.carry_out = carry + ((k + 1) & 1);
    ev.slab_cnt = pair + (g_parity[dev] ? kCounterWords : 0);
    ev.slab_cnt_next = pair + (g_parity[dev] ? 0 : kCounterWords);
    if ((e = launch_scan(g, ev, nullptr, 1, n_grp, true, s)) != hipSuccess) return fail_hip(e, "candidate launch");
    g_parity[dev] ^= 1;
    if ((e = launch_peaks(g, ev, nullptr, 1, n_grp, s)) != hipSuccess) return fail_hip(e, "peak launch");
    g0 += n_grp;
  }
  return HT_OK;
}
