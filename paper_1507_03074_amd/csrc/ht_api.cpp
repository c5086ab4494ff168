// ht_api.cpp -- C ABI of libht.so: validation, bin-rule tables, tiling, scratch, launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "ht_debug.h"
#include "ht_internal.h"

namespace ht {
hipError_t launch_debug_hits(const DevGrid& g, const float* x, const float* y, const float* z,
                             int64_t n, int32_t* info, float* vals, int32_t* slabs, hipStream_t s);
hipError_t launch_debug_unary(const float* v, float* root, float* inv2, int64_t n, hipStream_t s);

thread_local std::string g_err;

int fail(int code, const char* fmt, ...)
{
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int fail_hip(hipError_t e, const char* what)
{
  return fail(e == hipErrorOutOfMemory ? HT_ENOMEM : HT_EDEVICE, "%s: %s", what,
              hipGetErrorString(e));
}

static const int64_t kBlockJobs = 256;  // job flags that a workgroup of the peak test loads at once
static const double kPi = 3.14159265358979323846;

int validate_grid(const ht_grid* g)
{
  if (!g) return fail(HT_EINVAL, "grid is NULL");
  if (g->phi_sectors != 0 && g->phi_sectors != 1) return fail(HT_EINVAL, "phi_sectors must be 0 or 1");
  if (g->n_theta < 1 || g->n_phi < (g->phi_sectors ? 1 : 3) || g->n_a < 1 || g->n_b < 1)
    return fail(HT_EINVAL, "grid needs n_theta >= 1, n_phi >= 3 (>= 1 with phi sectors), n_a >= 1, n_b >= 1");
  if (g->n_a > (1 << 24) || g->n_b > (1 << 24)) return fail(HT_EINVAL, "n_a and n_b must be <= 2^24");
  if ((int64_t)g->n_theta * g->n_phi > kMaxSlabs) return fail(HT_EINVAL, "n_theta*n_phi must be <= 4096");
  if (!std::isfinite(g->a_min) || !std::isfinite(g->a_max) || !std::isfinite(g->b_min) ||
      !std::isfinite(g->b_max))
    return fail(HT_EINVAL, "grid ranges must be finite");
  if (!(g->a_min < g->a_max) || !(g->b_min < g->b_max))
    return fail(HT_EINVAL, "grid ranges need min < max");
  if (g->threshold < 1) return fail(HT_EINVAL, "threshold must be >= 1");
  const double cells = (double)g->n_theta * g->n_phi * (double)g->n_a * (double)g->n_b;
  if (cells > 4294967296.0) return fail(HT_EINVAL, "more than 2^32 cells");
  return HT_OK;
}

uint64_t n_cells(const ht_grid& g) { return (uint64_t)g.n_theta * g.n_phi * g.n_a * g.n_b; }

// Bin-rule tables, computed in double and rounded once to float.
void host_tables_into(const ht_grid& g, float* a2, float* inv_db, float* phi, float* th)
{
  const double da = ((double)g.a_max - (double)g.a_min) / (double)g.n_a;
  for (int32_t i = 0; i < g.n_a; ++i)
    a2[i] = (float)(2.0 * (double)g.a_min + (double)(2 * (int64_t)i + 1) * da);
  *inv_db = (float)((double)g.n_b / ((double)g.b_max - (double)g.b_min));
  for (int32_t m = 0; m < 2 * g.n_phi; ++m) {
    const double ang = ((double)m * kPi) / (double)g.n_phi;
    phi[2 * m] = (float)std::cos(ang);
    phi[2 * m + 1] = (float)std::sin(ang);
  }
  for (int32_t m = 0; m <= 2 * g.n_theta; ++m) {
    const double ang = ((double)m * kPi) / (double)(2 * g.n_theta);
    th[2 * m] = (float)std::cos(ang);
    th[2 * m + 1] = (float)std::sin(ang);
  }
}

void host_tables(const ht_grid& g, std::vector<float>& a2, float& inv_db, std::vector<float>& phi,
                 std::vector<float>& th)
{
  a2.resize(a2_floats(g));
  phi.resize(phi_floats(g));
  th.resize(th_floats(g));
  host_tables_into(g, a2.data(), &inv_db, phi.data(), th.data());
}

// ---------------------------------------------------------------------------------------------
// Tiling
// ---------------------------------------------------------------------------------------------
static int env_int(const char* name, int def)
{
  const char* v = std::getenv(name);
  return v && *v ? std::atoi(v) : def;
}

// Largest power-of-two row count (<= 64) whose u32 tile fits the LDS budget.
// Per-grid launch shapes set through ht_set_tuning (keyed by dimensions and ranges).
typedef std::tuple<int32_t, int32_t, int32_t, int32_t, uint32_t, uint32_t, uint32_t, uint32_t> TuneKey;
static std::mutex g_tune_mu;
static std::map<TuneKey, ht_tuning> g_tune;

static uint32_t fbits(float f);

static TuneKey tune_key(const ht_grid& g)
{
  return TuneKey{g.n_theta, g.n_phi, g.n_a, g.n_b, fbits(g.a_min), fbits(g.a_max), fbits(g.b_min),
                 fbits(g.b_max)};
}

static const int64_t kLdsTileMax = 65536 - 8192;  // bytes of an LDS tile (leaves room for the small scratch words)

Tiling choose_tiling(const ht_grid& g)
{
  Tiling t;
  const int64_t row_bytes = (int64_t)g.n_b * 4;
  const int64_t budget = env_int("HT_FILL_LDS_BYTES", 32768);
  const int64_t lds_max = kLdsTileMax;
  t.lds_fill = row_bytes <= lds_max ? 1 : 0;
  int rows = 1;
  if (t.lds_fill) {
    while (rows < 64 && (int64_t)(rows * 2) * row_bytes <= std::max<int64_t>(budget, row_bytes) &&
           rows < g.n_a)
      rows *= 2;
    const int forced = env_int("HT_FILL_ROWS", 0);
    if (forced > 0 && (forced & (forced - 1)) == 0 && forced <= 64 &&
        (int64_t)forced * row_bytes <= lds_max)
      rows = forced;
  }
  // keep the tile count inside a 32-bit grid dimension
  while (rows < 64 && (int64_t)g.n_theta * g.n_phi * ((g.n_a + rows - 1) / rows) > 0x7fffffffLL) rows *= 2;
  t.rows = rows;
  t.tiles_per_slab = (g.n_a + rows - 1) / rows;
  t.n_tiles = g.n_theta * g.n_phi * t.tiles_per_slab;
  const int64_t tile_cells = (int64_t)rows * g.n_b;
  int cap = 64;
  while (cap < 1024 && cap * 32 < tile_cells) cap *= 2;
  const int forced_cap = env_int("HT_CAND_CAP", 0);
  if (forced_cap >= 2 && forced_cap <= 4096 && (forced_cap & (forced_cap - 1)) == 0) cap = forced_cap;
  t.cand_cap = cap;
  // peak-search groups: small groups spread clustered candidates over more workgroups; the
  // write kernel sums the earlier groups' totals, so keep the group count moderate
  int gt = 16;
  while (gt < 64 && ((int64_t)t.n_tiles + gt - 1) / gt > 2048) gt *= 2;
  const int forced_gt = env_int("HT_GROUP_TILES", 0);
  if (forced_gt == 16 || forced_gt == 32 || forced_gt == 64) gt = forced_gt;
  t.group_tiles = gt;
  t.nt_store = std::min(2, std::max(0, env_int("HT_FILL_NT", 0)));
  t.auto_nt = env_int("HT_FILL_NT", -1) < 0 ? 1 : 0;
  t.auto_rows = env_int("HT_FILL_ROWS", 0) <= 0 && env_int("HT_FILL_LDS_BYTES", 0) <= 0 ? 1 : 0;
  // fill tiles per workgroup: one by default (measured fastest on the paper grid: many short
  // workgroups hide the record-load latency better than fewer workgroups looping over tiles)
  int ft = 1;
  const int forced_ft = env_int("HT_FILL_TILES", 0);
  if (forced_ft > 0 && forced_ft <= 64 && (forced_ft & (forced_ft - 1)) == 0) ft = forced_ft;
  t.fill_tiles = ft;
  // HT_PACKED_LISTS=1: every event takes the counting sort into packed slab lists, the layout
  // that large batches and very large events use, so that tests reach it on small grids
  t.packed_lists = env_int("HT_PACKED_LISTS", 0) != 0 ? 1 : 0;
  ht_tuning tu;
  std::memset(&tu, 0, sizeof(tu));
  bool have = false;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune.find(tune_key(g));
    if (it != g_tune.end()) {
      tu = it->second;
      have = true;
    }
  }
  // A field set to its reported default is as good as unset: setting what ht_get_tuning returned
  // changes nothing, and a shape pins only what it changes.
  if (have) {
    if (tu.rows > 0 && tu.rows != t.rows && t.lds_fill) {
      t.rows = tu.rows;
      t.auto_rows = 0;
    }
    if (tu.group_tiles > 0) t.group_tiles = tu.group_tiles;
    if (tu.cand_cap > 0) t.cand_cap = tu.cand_cap;
    if (tu.nt_store >= 0 && tu.nt_store != t.nt_store) {
      t.nt_store = tu.nt_store;
      t.auto_nt = 0;
    }
    if (tu.tiles_per_block > 0) t.fill_tiles = tu.tiles_per_block;
    t.tiles_per_slab = (g.n_a + t.rows - 1) / t.rows;
    t.n_tiles = g.n_theta * g.n_phi * t.tiles_per_slab;
  }
  // Stencil peak search of crowded events: a workgroup holds kChunkCells B columns of every
  // slab, one wave per phi cell with every theta cell in its registers (so at most 16 phi cells
  // and 4 theta cells), and walks dense_rows A rows (a multiple of 12, its unrolled step loop).
  // It needs LDS tiles for the fill (whose candidate pass it replaces). By default the segments
  // are as long as lets every workgroup run at once, two per CU (256 CUs).
  // One buffer resource spans a row of every theta cell's slab: under 2^31 bytes.
  const bool st_offsets = ((uint64_t)(g.n_theta - 1) * g.n_phi * g.n_a + 1) * g.n_b * 4 < (1ull << 31);
  t.dense_w = (t.lds_fill && g.n_theta <= 4 && g.n_phi <= 16 && st_offsets) ? 1 : 0;
  {
    const int n_chunks = (g.n_b + kChunkCells - 1) / kChunkCells;
    const int segs = std::max(1, 512 / n_chunks);
    int s_rows = (g.n_a + segs - 1) / segs;
    const int forced = env_int("HT_DENSE_ROWS", 0);
    if (forced > 0) s_rows = std::min(forced, 4096);
    t.dense_rows = std::max(12, ((s_rows + 11) / 12) * 12);
  }
  // The reported default, n_slabs n_b / 4 hits (a quarter of a hit per (theta, phi, B) cell), is
  // where one pass over the matrix beats a test of every candidate. The survivors are a quarter of
  // them, so unless the caller sets a threshold the stencil starts later: at twice that for peaks of
  // seven votes or more, 2.5 times (nine votes) in matrices of 128 MiB or more, where a pass is long.
  // Peaks of fewer votes have many more survivors, and the stencil's time does not depend on them.
  // Whole calls, survivors against stencil, in us, by the threshold T and multiples of the default:
  // 4x16x1024x1024 T 9: x2 104 / 129, x2.5 127 / 136; T 8: x2 111 / 130, x2.5 145 / 136; T 7: x1.5
  // 108 / 129, x2 122 / 130, x2.5 187 / 137; T 6: x1.5 118 / 130, x2 143 / 131; T 5: x1.05 116 / 130,
  // x1.5 139 / 130; T 4: x1.05 131 / 131; T 3: x1.1 210 / 131. 4x16x512x512 T 8: x2 52 / 52, x2.5
  // 64 / 54; T 7: x2 54 / 53, x2.5 67 / 54; T 5: x1.05 54 / 50, x1.5 65 / 53. 4x16x256x256 T 8: x2
  // 34 / 42, x2.5 48 / 44; T 7: x2 36 / 43; T 6: x1.5 42 / 42, x2 49 / 44; T 5, x1.1 62 / 42. At x2 and T 8 on 2x8x512x512 30 / 34,
  // 3x7x501x333 31 / 33, 3x12x900x200 42 / 41, 2x16x300x900 36 / 45, 1x3x256x256 22 / 23, sectors
  // 4x4x1024x1024 38 / 42; sixteen events of 4x16x256x256 160 / 154, 4x16x128x128 68 / 67. -1: never
  const int64_t def = ((int64_t)g.n_theta * g.n_phi * g.n_b + 3) / 4;
  const int64_t bytes = 4 * (int64_t)g.n_theta * g.n_phi * g.n_a * g.n_b;
  const int64_t T = std::min<int64_t>(g.threshold, 16);
  int64_t dh = def, from = bytes >= ((int64_t)128 << 20) ? std::min(def * (T - 1) / 3, def * 5 / 2)
                                                         : std::min(def * (T - 3) / 2, def * 2);
  from = std::max(from, def);
  const int forced_dh = env_int("HT_DENSE_HITS", 0);
  if (forced_dh != 0) dh = from = forced_dh;
  auto reported = [&](int64_t hits) { return t.dense_w > 0 && hits > 0 ? (int32_t)std::min<int64_t>(hits, 1 << 28) : 0; };
  const int32_t unset = reported(dh);
  if (have && tu.dense_hits != 0 && tu.dense_hits != (unset > 0 ? unset : -1)) dh = from = tu.dense_hits;
  t.dense_hits = reported(dh);
  const bool on = t.dense_hits > 0;
  t.dense_from = on ? (int32_t)std::min<int64_t>(from, 1 << 28) : 0;
  return t;
}

int check_tuning(const ht_grid& g, const ht_tuning& tu)
{
  auto pow2 = [](int v) { return v > 0 && (v & (v - 1)) == 0; };
  if (tu.rows < 0 || (tu.rows > 0 && (!pow2(tu.rows) || tu.rows > 64 ||
                                      (int64_t)tu.rows * g.n_b * 4 > kLdsTileMax)))
    return fail(HT_EINVAL, "tuning.rows must be a power of two <= 64 with rows*n_b*4 <= %lld",
                (long long)kLdsTileMax);
  if ((int64_t)g.n_theta * g.n_phi * ((g.n_a + std::max(tu.rows, 1) - 1) / std::max(tu.rows, 1)) >
      0x7fffffffLL)
    return fail(HT_EINVAL, "tuning.rows gives too many tiles");
  if (tu.group_tiles != 0 && tu.group_tiles != 16 && tu.group_tiles != 32 && tu.group_tiles != 64)
    return fail(HT_EINVAL, "tuning.group_tiles must be 16, 32 or 64");
  if (tu.cand_cap < 0 || (tu.cand_cap > 0 && (!pow2(tu.cand_cap) || tu.cand_cap > 4096)))
    return fail(HT_EINVAL, "tuning.cand_cap must be a power of two <= 4096");
  if (tu.nt_store < -1 || tu.nt_store > 2) return fail(HT_EINVAL, "tuning.nt_store must be -1, 0, 1 or 2");
  if (tu.tiles_per_block < 0 || (tu.tiles_per_block > 0 && (!pow2(tu.tiles_per_block) || tu.tiles_per_block > 64)))
    return fail(HT_EINVAL, "tuning.tiles_per_block must be a power of two <= 64");
  if (tu.dense_hits < -1) return fail(HT_EINVAL, "tuning.dense_hits must be -1, 0 or a hit count");
  return HT_OK;
}

// ---------------------------------------------------------------------------------------------
// Device tables, cached per (device, grid)
// ---------------------------------------------------------------------------------------------
static std::mutex g_mu;
typedef std::tuple<int, int32_t, int32_t, int32_t, int32_t, uint32_t, uint32_t, uint32_t, uint32_t>
    TabKey;
static std::map<TabKey, DevTables> g_tables;

static uint32_t fbits(float f)
{
  uint32_t u;
  std::memcpy(&u, &f, 4);
  return u;
}

int get_tables(const ht_grid& g, int dev, DevTables* out)
{
  TabKey key{dev, g.n_theta, g.n_phi, g.n_a, g.n_b, fbits(g.a_min), fbits(g.a_max), fbits(g.b_min),
             fbits(g.b_max)};
  std::lock_guard<std::mutex> lk(g_mu);
  auto it = g_tables.find(key);
  if (it != g_tables.end()) {
    *out = it->second;
    return HT_OK;
  }
  std::vector<float> a2, phi, th;
  DevTables t;
  host_tables(g, a2, t.inv_db, phi, th);
  hipError_t e;
  if ((e = hipMalloc(&t.a2, a2.size() * 4)) != hipSuccess) return fail_hip(e, "hipMalloc(tables)");
  if ((e = hipMalloc(&t.phi, phi.size() * 4)) != hipSuccess) return fail_hip(e, "hipMalloc(tables)");
  if ((e = hipMalloc(&t.th, th.size() * 4)) != hipSuccess) return fail_hip(e, "hipMalloc(tables)");
  if ((e = hipMemcpy(t.a2, a2.data(), a2.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(t.phi, phi.data(), phi.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(t.th, th.data(), th.size() * 4, hipMemcpyHostToDevice)) != hipSuccess)
    return fail_hip(e, "hipMemcpy(tables)");
  g_tables[key] = t;
  *out = t;
  return HT_OK;
}

// The rows per tile and the store kind of a launch of n_ev events of up to max_hits hits, where
// the caller set none (the tiling's are those of crowded events).
static void shape_launch(DevGrid* d, const Tiling& tl, int n_ev, int64_t max_hits)
{
  const int rows = d->rows;
  if (tl.auto_rows && tl.lds_fill) {
    // Long slab lists: 32 KiB tiles of up to eight rows, as the long-list fill takes (14k hits on
    // 512x512 planes: 54.6 us with eight rows, 64.8 with sixteen, which go to the other fill).
    // Short ones: tiles of 16 KiB, twice the workgroups per CU (paper event, 4 against 8 rows: 62.3
    // and 66.5 us; at 512 and 256 columns the 16 KiB tile is the fastest of three as well), but
    // four rows, a whole band. Launches of fewer tiles than the chip has CUs take lower ones (a
    // hundred events of 250 hits on 4x16x64x64: 64 rows, 64 us, 16 rows 85).
    // Where 16 KiB hold more than eight rows, eight of them are a small tile for a long list, which
    // large launches pay for more often: whole calls, eight rows and 16 KiB, in us: 30k hits on
    // 4x16x1024x256 (8192 tiles of eight rows) 73 and 75, 18k on 4x16x256x256 (2048) 40 and 44, forty
    // events of 4000-8000 on 2x8x200x100 (16000) 109 and 100, 41k hits on 8x27x1604x100 (43k) 288 and
    // 214, eight events of 15k on 4x16x1024x256 (65k) 449 and 314.
    int low = rows;
    while (low > 4 && (int64_t)low * d->n_b * 4 > 16384) low /= 2;
    const bool many = (int64_t)d->n_slabs * ((d->n_a + 7) / 8) * n_ev > 10000;
    d->rows = std::min(rows, 8);
    if ((low > 8 && many) || !long_lists(*d, n_ev, max_hits)) {
      d->rows = low;
      while (d->rows > 8 && (int64_t)d->n_slabs * ((d->n_a + d->rows - 1) / d->rows) * n_ev < 256) d->rows /= 2;
    }
    d->tiles_per_slab = (d->n_a + d->rows - 1) / d->rows;
    d->n_tiles = d->n_slabs * d->tiles_per_slab;
  }
  const bool long_l = tl.lds_fill && long_lists(*d, n_ev, max_hits);
  if (tl.auto_nt) {
    // Non-temporal stores where the launch writes more than the 256 MiB last-level cache holds (100
    // paper events: 4.5 and 5.3 ms), or the fill is not what waits for its stores: long lists and
    // the stencil (14k hits: 72.6 and 81.5 us; 40k hits with the stencil: 137 and 161 us). A single
    // ordinary event's matrix stays in the cache for its peak test and for the next event in the
    // same matrix (paper event in one matrix: 56.7 us, non-temporal 61.6; in three by turns 64.0
    // and 62.3). Below 128 MiB the stencil reads what the cache kept (512x512 planes: 46.9 and
    // 51.9 us); below 4 MiB the L2 does (17.0 and 18.8 us).
    const int64_t bytes = (int64_t)n_ev * 4 * d->n_slabs * d->n_a * d->n_b;
    const bool dense = dense_peaks(*d, max_hits);
    d->nt_store = bytes > ((int64_t)256 << 20) || (dense && bytes >= ((int64_t)128 << 20)) ||
                  (long_l && !dense && bytes >= ((int64_t)4 << 20));
  }
}

int32_t stencil_from(const Tiling& tl, int n_ev, int64_t max_hits)
{
  // A batch that has the stencil's launches anyway, as one of its events reaches its threshold, takes
  // it for its events from the reported one on (six events of 3050-15250 hits on 4x16x532x171, both
  // searches: 145 us)
  return n_ev > 1 && tl.dense_from > 0 && max_hits >= tl.dense_from ? tl.dense_hits : tl.dense_from;
}

DevGrid make_devgrid(const ht_grid& g, const DevTables& t, const Tiling& tl, int n_ev, int64_t max_hits, bool search)
{
  DevGrid d;
  std::memset(&d, 0, sizeof(d));  // padding too: the bytes key the graph cache
  d.n_theta = g.n_theta;
  d.n_phi = g.n_phi;
  d.n_a = g.n_a;
  d.n_b = g.n_b;
  d.b_min = g.b_min;
  d.inv_db = t.inv_db;
  d.nb_f = (float)g.n_b;
  d.threshold = g.threshold;
  d.n_slabs = g.n_theta * g.n_phi;
  d.rows = tl.rows;
  d.tiles_per_slab = tl.tiles_per_slab;
  d.n_tiles = tl.n_tiles;
  d.lds_fill = tl.lds_fill;
  d.group_tiles = tl.group_tiles;
  d.nt_store = tl.nt_store;
  d.fill_tiles = tl.fill_tiles;
  d.phi_sectors = g.phi_sectors;
  d.packed_lists = tl.packed_lists;
  // |A2| <= 2^60 and a hit's |x| < 2^64 (r2 is finite): A2 x is finite, r2 - A2 x no NaN; 1/(2y) is
  // finite and not 0, so B is no NaN; and neither is (B - b_min) inv_db while inv_db is finite
  d.finite_votes = std::max(std::fabs((double)g.a_min), std::fabs((double)g.a_max)) <= std::ldexp(1.0, 59) &&
                   std::isfinite((float)((double)g.n_b / ((double)g.b_max - (double)g.b_min))) ? 1 : 0;
  d.search = search ? 1 : 0;
  d.dense_w = tl.dense_w;
  d.dense_rows = tl.dense_rows;
  d.dense_hits = stencil_from(tl, n_ev, max_hits);
  d.a2 = t.a2;
  d.phi_cs = t.phi;
  d.th_cs = t.th;
  shape_launch(&d, tl, n_ev, max_hits);
  set_jobs(&d, tl.lds_fill ? d.rows : 0, n_ev);
  return d;
}

void set_jobs(DevGrid* g, int tile_rows, int n_ev)
{
  JobGeom& j = g->j;
  j.units = (g->n_b + 3) / 4;
  j.ch = tile_rows ? std::min(tile_rows, 4) : (j.units > 64 * 64 ? 1 : 4);
  j.sub = 1;
  while (j.sub * 2 * (int64_t)j.units <= 64 && (!tile_rows || j.sub * 2 <= tile_rows / j.ch)) j.sub *= 2;
  j.strips = (j.units + 63) / 64;
  j.tile_rows = tile_rows ? tile_rows : j.ch * j.sub;
  j.tiles_per_slab = (g->n_a + j.tile_rows - 1) / j.tile_rows;
  j.tile_jobs = j.tile_rows / (j.ch * j.sub) * j.strips;
  j.elem_bytes = j.ch == 4 ? 2 : 1;
  j.n_jobs = (uint32_t)g->n_slabs * (uint32_t)j.tiles_per_slab * (uint32_t)j.tile_jobs;
  j.row_jobs = j.ch * j.sub == 1 ? 1 : j.strips;
  // Groups of the peak test, one workgroup each: 32 jobs a group (2048 groups on the paper grid; a
  // 14k-hit event's test takes 22.8 us, 26.6 us with 64 jobs, 25.2 us with 16); smaller events get
  // smaller groups, down to 8 jobs, to use more CUs (24.6k hits on 512x512 planes: 61 us whole,
  // 100 us with a quarter of the groups), batches of them fewer (100 small events: 62.6 and 66.7
  // us); launches of many groups get larger ones, which pay a workgroup's start once for more jobs
  // (its flags come 256 jobs at a time).
  int64_t gj = 32;
  const int64_t all = (int64_t)j.n_jobs * n_ev;
  while (gj > 8 && all / gj < (n_ev > 1 ? 512 : 2048)) gj /= 2;
  while (gj < kBlockJobs / 2 && all / gj > 65536) gj *= 2;
  while (j.n_jobs / gj > 16384) gj *= 2;
  gj = std::max<int64_t>(1, gj / j.row_jobs) * j.row_jobs;
  j.group_jobs = (int32_t)gj;
  j.n_groups = (uint32_t)((j.n_jobs + gj - 1) / gj);
  // The test adds its peaks to the counts with atomics, which take 10 ns each on one cache line (32
  // words), and peaks cluster: the counts of up to 16384 words are spread out.
  j.pk_step = 1;
  while (j.pk_step < 32 && (int64_t)j.n_groups * j.pk_step * 2 <= 16384) j.pk_step *= 2;
  // one peak per 64 cells: uncorrelated counts give one local maximum per 81
  j.seg = (int32_t)std::min<int64_t>(kSegMax, std::max<int64_t>(128, 16 * gj));
}

// ---------------------------------------------------------------------------------------------
// Per-event scratch
// ---------------------------------------------------------------------------------------------
static size_t al(size_t v) { return (v + 255) & ~(size_t)255; }

bool dense_peaks(const DevGrid& g, int64_t n)
{
  return g.dense_w > 0 && g.dense_hits > 0 && n >= g.dense_hits;
}

bool direct_lists(const DevGrid& g, int64_t n)
{
  return g.lds_fill && !g.packed_lists &&
         (size_t)g.n_slabs * (size_t)std::max<int64_t>(n, 1) * 16 <= kDirectListMax;
}

size_t mask_bytes(const DevGrid& g)
{
  // one 64-bit word per (slab, row, chunk of kChunkCells columns), rows padded to whole segments
  // of dense_rows (the stencil's waves store their segments whole)
  const size_t n_chunks = ((size_t)g.n_b + kChunkCells - 1) / kChunkCells;
  const size_t rows = (((size_t)g.n_a + g.dense_rows - 1) / g.dense_rows) * g.dense_rows;
  return 8 * (size_t)g.n_slabs * rows * n_chunks;
}

// peaks per group: of job rows (the fill's survivors), of tiles (the stencil)
static size_t group_words(const DevGrid& g, int peaks)
{
  return std::max<size_t>((peaks & kPeakBands) ? (size_t)g.j.n_groups * g.j.pk_step : 0, (peaks & kPeakMask) ? (size_t)n_groups(g) : 0);
}

// Entries of a survivor list of an event of up to n hits (below 0: unknown). Of few cells all fit the
// one list. Else the lists hold one in 32 of the matrix's cells in all, or a quarter of those that can
// reach the threshold where that is more, and none more than can; past that, and past kListCap a
// list, the search works from the masks.
static uint32_t surv_cap(const DevGrid& g, int64_t n, int peaks)
{
  const int64_t cells = (int64_t)g.n_slabs * g.n_a * g.n_b;
  const int64_t bound = n < 0 ? cells : std::min(cells, cells_bound(g, n));
  if (peaks & kPeakFew) return (uint32_t)std::max<int64_t>(1, std::min<int64_t>(bound, kFewCells));
  const int64_t share = std::max(cells / 32, bound / 4) / kLists;
  return (uint32_t)std::max<int64_t>(8, std::min<int64_t>(std::min(bound, share), kListCap));
}

size_t surv_bytes(const DevGrid& g, int64_t n, int peaks)
{
  return al(16 * (size_t)(peaks & kPeakFew ? 1 : kLists) * surv_cap(g, n, peaks));
}

size_t event_scratch_bytes(const DevGrid& g, int64_t n, bool direct, int peaks)
{
  const size_t nn = (size_t)std::max<int64_t>(n, 0);
  size_t b = 0;
  b += al(4 * ((size_t)g.n_slabs + 1));       // slab_off
  if (direct) {
    b += al(16 * (size_t)g.n_slabs * std::max<size_t>(nn, 1));  // list
  } else {
    b += al(16 * nn);                         // hit_slab
    b += al(16 * nn);                         // hit_pos
    b += al(16 * nn);                         // hit_rec
    b += al(64 * nn + 16);                    // list (+1 record of slack for the fill)
  }
  if (peaks & (kPeakBands | kPeakMask)) b += al(4 * group_words(g, peaks));  // group_pk
  if (peaks & kPeakBands) {
    b += al(4 * kSuperStep * (((size_t)g.j.n_groups + 63) / 64));  // super_pk
    b += al(8 * (size_t)g.j.seg * g.j.n_groups);                   // seg
  }
  if (peaks & (kPeakBands | kPeakFew)) b += al(g.j.n_jobs) + al((size_t)64 * g.j.elem_bytes * g.j.n_jobs) + surv_bytes(g, n, peaks);
  if (peaks & kPeakMask) b += al(mask_bytes(g));  // pk_mask
  return b;
}

void carve_event_scratch(const DevGrid& g, int64_t n, bool direct, char* p, EvDesc* ev, int peaks)
{
  const size_t nn = (size_t)std::max<int64_t>(n, 0);
  auto take = [&p](size_t bytes) {
    char* r = p;
    p += al(bytes);
    return r;
  };
  ev->slab_off = (uint32_t*)take(4 * ((size_t)g.n_slabs + 1));
  if (direct) {
    ev->list_cap = (int64_t)std::max<size_t>(nn, 1);
    ev->list = (float4*)take(16 * (size_t)g.n_slabs * (size_t)ev->list_cap);
    ev->hit_slab = nullptr;
    ev->hit_pos = nullptr;
    ev->hit_rec = nullptr;
  } else {
    ev->list_cap = 0;
    ev->hit_slab = (int32_t*)take(16 * nn);
    ev->hit_pos = (uint32_t*)take(16 * nn);
    ev->hit_rec = (float4*)take(16 * nn);
    ev->list = (float4*)take(64 * nn + 16);
  }
  carve_peak_scratch(g, n, p, ev, peaks, 0, g.j.n_groups);
}

void carve_peak_scratch(const DevGrid& g, int64_t n_hits, char* p, EvDesc* ev, int peaks, uint32_t grp0, uint32_t n_grp)
{
  auto take = [&p](size_t bytes) {
    char* r = p;
    p += al(bytes);
    return r;
  };
  const size_t n = std::min<size_t>((size_t)n_grp * g.j.group_jobs, g.j.n_jobs);
  ev->grp0 = grp0;
  ev->n_grp = n_grp;
  ev->clear_n16 = 0;
  ev->lists = 0;
  if (peaks & kPeakBands) ev->super_pk = (uint32_t*)take(4 * kSuperStep * (((size_t)n_grp + 63) / 64));
  if (peaks & (kPeakBands | kPeakMask)) ev->group_pk = (uint32_t*)take(4 * group_words(g, peaks));
  if (peaks & (kPeakBands | kPeakFew)) {
    ev->job_any = (uint8_t*)take(n);
    ev->masks = (uint8_t*)take((size_t)64 * g.j.elem_bytes * n);
  }
  if (peaks & kPeakBands) {
    ev->clear = ev->super_pk;
    ev->clear_n16 = (uint32_t)((ev->masks - (uint8_t*)ev->super_pk) / 16);
    ev->seg = (uint2*)take(8 * (size_t)g.j.seg * n_grp);
  }
  if (peaks & (kPeakBands | kPeakFew)) {
    ev->surv = (uint4*)take(surv_bytes(g, n_hits, peaks));
    ev->lists = (peaks & kPeakFew ? 0u : (kLists - 1u) << kListShift) | surv_cap(g, n_hits, peaks);
  }
  if (peaks & kPeakMask) ev->pk_mask = (uint8_t*)take(mask_bytes(g));
  if (peaks == kPeakMask) clear_groups(g, ev);
}

void clear_groups(const DevGrid& g, EvDesc* ev)
{
  ev->clear = ev->group_pk;
  ev->clear_n16 = (uint32_t)(al(4 * (size_t)n_groups(g)) / 16);
}

// Scratch owned by the library, one per (device, stream). Calls on one stream are ordered on
// the device, so they may reuse the same scratch; growing it waits for the stream first.
struct Workspace {
  char* dev = nullptr;
  size_t bytes = 0;
  uint32_t* ctr = nullptr;  // zeroed slab counter pairs, kCounterBytes per event slot
  int ctr_events = 0;
  std::vector<uint8_t> parity;  // which array of each pair the next call counts into
  // Pinned staging of batch descriptors, two by turns: a call writes its own while the batch
  // before it is still running (its launches then follow without a gap), and waits only for the
  // one before that. Their copy on the device is fetched in stream order, so it needs no second.
  EvDesc* h_ev[2] = {};
  hipEvent_t ev_read[2] = {};  // the launches that read each staging are done
  int turn = 0;
  EvDesc* d_ev = nullptr;
  int ev_cap = 0;
  hipStream_t capture = nullptr;  // private stream used only to capture batch graphs
  hipStream_t side = nullptr;     // side stream of split batches (eager launches)
  hipStream_t capture_side = nullptr;  // side stream of split batches under capture
  hipEvent_t split_ev[kMaxPieces + 1] = {};
  struct Graph {
    std::vector<unsigned char> key;
    hipGraphExec_t exec;
  };
  std::vector<Graph> graphs;
};

static std::map<std::pair<int, hipStream_t>, Workspace*> g_ws;

int get_workspace(int dev, hipStream_t s, size_t bytes, Workspace** out)
{
  Workspace* w;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    Workspace*& slot = g_ws[{dev, s}];
    if (!slot) slot = new Workspace();
    w = slot;
  }
  if (bytes > w->bytes) {
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
    if (w->dev) (void)hipFree(w->dev);
    w->dev = nullptr;
    w->bytes = 0;
    const size_t want = std::max(bytes, (size_t)1 << 20);
    if ((e = hipMalloc(&w->dev, want)) != hipSuccess) return fail_hip(e, "hipMalloc(scratch)");
    w->bytes = want;
  }
  *out = w;
  return HT_OK;
}

int ensure_counters(Workspace* w, int n_ev, hipStream_t s)
{
  if (n_ev <= w->ctr_events) return HT_OK;
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  if (w->ctr) (void)hipFree(w->ctr);
  w->ctr = nullptr;
  w->ctr_events = 0;
  const int want = std::max(n_ev, 16);
  if ((e = hipMalloc((void**)&w->ctr, kCounterBytes * want)) != hipSuccess)
    return fail_hip(e, "hipMalloc(counters)");
  if ((e = hipMemset(w->ctr, 0, kCounterBytes * want)) != hipSuccess) return fail_hip(e, "hipMemset(counters)");
  w->ctr_events = want;
  w->parity.assign(want, 0);
  return HT_OK;
}

// Counter arrays of event slot i for this call: count into the zero one, clear the other.
void use_counters(Workspace* w, int i, EvDesc* d)
{
  uint32_t* pair = w->ctr + (size_t)i * (kCounterBytes / 4);
  d->slab_cnt = pair + (w->parity[i] ? kCounterWords : 0);
  d->slab_cnt_next = pair + (w->parity[i] ? 0 : kCounterWords);
}

void flip_counters(Workspace* w, int n) { for (int i = 0; i < n; ++i) w->parity[i] ^= 1; }

// Makes w->h_ev[w->turn] free for n_ev descriptors of a new call.
int ensure_ev_staging(Workspace* w, int n_ev, hipStream_t s)
{
  w->turn ^= 1;
  hipError_t e;
  if (n_ev <= w->ev_cap) {
    if ((e = hipEventSynchronize(w->ev_read[w->turn])) != hipSuccess) return fail_hip(e, "hipEventSynchronize");
    return HT_OK;
  }
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  if (w->d_ev) (void)hipFree(w->d_ev);
  w->d_ev = nullptr;
  w->ev_cap = 0;
  int cap = std::max(n_ev, 16);
  for (int k = 0; k < 2; ++k) {
    if (w->h_ev[k]) (void)hipHostFree(w->h_ev[k]);
    w->h_ev[k] = nullptr;
    if ((e = hipHostMalloc((void**)&w->h_ev[k], sizeof(EvDesc) * cap, hipHostMallocDefault)) != hipSuccess)
      return fail_hip(e, "hipHostMalloc(descriptors)");
    if (!w->ev_read[k] && (e = hipEventCreateWithFlags(&w->ev_read[k], hipEventDisableTiming)) != hipSuccess)
      return fail_hip(e, "hipEventCreate");
  }
  if ((e = hipMalloc((void**)&w->d_ev, sizeof(EvDesc) * cap)) != hipSuccess)
    return fail_hip(e, "hipMalloc(descriptors)");
  w->ev_cap = cap;
  return HT_OK;
}

int make_device_grid(const ht_grid& g, int dev, int n_ev, int64_t max_hits, DevGrid* out, Tiling* tl, bool search)
{
  int rc = validate_grid(&g);
  if (rc) return rc;
  DevTables t;
  if ((rc = get_tables(g, dev, &t))) return rc;
  const Tiling tiling = choose_tiling(g);
  if (tl) *tl = tiling;
  *out = make_devgrid(g, t, tiling, n_ev, max_hits, search);
  return HT_OK;
}

// ---------------------------------------------------------------------------------------------
// Stage profiler: HIP events recorded on the launch stream around each stage.
// ---------------------------------------------------------------------------------------------
struct ProfRec {
  const char* name;
  hipEvent_t a, b;
};
static std::mutex g_prof_mu;
static int g_prof_mode = 0;  // 0 off, 1 every stage, 2 the fill stages only
static std::vector<ProfRec> g_prof;
static std::vector<hipEvent_t> g_prof_pool;

static thread_local bool t_capturing = false;

static hipEvent_t prof_event()
{
  if (!g_prof_pool.empty()) {
    hipEvent_t e = g_prof_pool.back();
    g_prof_pool.pop_back();
    return e;
  }
  // timing events without the system-scope fence: they order nothing for the host, and the
  // fence (a cache writeback) would add to what they measure
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
  return e;
}

struct StageTimer {
  const char* name;
  hipStream_t s;
  hipEvent_t a = nullptr;
  StageTimer(const char* n, hipStream_t st) : name(n), s(st)
  {
    if (!name) return;  // untimed call
    std::lock_guard<std::mutex> lk(g_prof_mu);
    if (g_prof_mode == 0 || t_capturing) return;
    if (g_prof_mode == 2 && std::strncmp(name, "fill", 4) != 0) return;
    a = prof_event();
    if (a) (void)hipEventRecord(a, s);
  }
  ~StageTimer()
  {
    std::lock_guard<std::mutex> lk(g_prof_mu);
    if (!a) return;
    hipEvent_t b = prof_event();
    if (!b) return;
    (void)hipEventRecord(b, s);
    g_prof.push_back({name, a, b});
  }
};

struct Prepared {
  DevGrid g;
  int dev;
  hipStream_t s;
};

int prepare(const ht_grid* grid, void* stream, Prepared* p, int n_ev, int64_t max_hits, bool search = true)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  hipError_t e = hipGetDevice(&p->dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  if ((rc = make_device_grid(*grid, p->dev, n_ev, max_hits, &p->g, nullptr, search))) return rc;
  p->s = (hipStream_t)stream;
  return HT_OK;
}

int check_launch(hipError_t e, const char* what)
{
  if (e != hipSuccess) return fail_hip(e, what);
  return HT_OK;
}

// Failure injection for tests of the error paths: with HT_TEST_FAIL_STAGE set to a stage name
// ("prep", "fill" or "peaks"), that stage's launch is not made and the call fails as a failed
// launch would (HT_EDEVICE), with the earlier stages already on the stream.
int injected_failure(const char* stage)
{
  const char* v = std::getenv("HT_TEST_FAIL_STAGE");
  if (v && std::strcmp(v, stage) == 0)
    return fail(HT_EDEVICE, "injected failure before the %s launch (HT_TEST_FAIL_STAGE)", stage);
  return HT_OK;
}

size_t slot_scratch_bytes(const DevGrid& g, const Tiling& tl, int max_batch, int64_t max_hits, int* layout)
{
  const bool direct = direct_lists(g, max_hits), crowded = tl.dense_from > 0 && max_hits >= tl.dense_from;
  if (!crowded && batch_shape(g, max_batch, max_hits, false, 1).few) {  // and so are smaller batches
    *layout = kPeakFew;
    return event_scratch_bytes(g, max_hits, direct, kPeakFew);
  }
  *layout = kPeakBands | (crowded ? kPeakMask : 0);
  return std::max(event_scratch_bytes(g, max_hits, direct, *layout), event_scratch_bytes(g, max_hits, direct, kPeakFew));
}

BatchShape batch_shape(const DevGrid& g, int n_ev, int64_t max_hits, bool any_dense, int pieces)
{
  BatchShape b;
  b.prep_hits = max_hits;
  b.long_l = g.lds_fill && long_lists(g, n_ev, max_hits);
  b.tiny = !any_dense && pieces == 1 && tiny_launch(g, n_ev, max_hits);
  b.few = b.tiny || (!any_dense && pieces == 1 && g.lds_fill && few_cells(g, max_hits) && use_lists(g, n_ev, max_hits, max_hits));
  return b;
}

int launch_batch(const DevGrid& g, const EvDesc* d_ev, int n_ev, const BatchShape& bs, bool direct,
                 bool any_bands, bool any_dense, hipStream_t s, bool* prep_enqueued, const BatchSplit* split)
{
  EvDesc none;
  std::memset(&none, 0, sizeof(none));
  int rc;
  *prep_enqueued = false;
  const int pieces = split && g.lds_fill ? std::min(split->pieces, n_ev) : 1;
  if (bs.tiny) {
    if ((rc = injected_failure("prep")) || (rc = injected_failure("fill"))) return rc;
    {
      StageTimer t("fill", s);
      if ((rc = check_launch(launch_tiny_fill(g, none, d_ev, n_ev, s), "fill launch"))) return rc;
      *prep_enqueued = true;
    }
    if ((rc = injected_failure("peaks"))) return rc;
    StageTimer t("peaks", s);
    return check_launch(launch_few_peaks(g, none, d_ev, n_ev, s), "peak launch");
  }
  {
    StageTimer t("prep", s);
    if ((rc = injected_failure("prep")) ||
        (rc = check_launch(launch_prep(g, none, d_ev, n_ev, bs.prep_hits, direct && g.lds_fill, s), "prep launch")))
      return rc;
    *prep_enqueued = true;
  }
  if ((rc = injected_failure("fill"))) return rc;
  if (pieces > 1) {
    // The batch in `pieces` runs of consecutive events: the fill of run i + 1 (on s) overlaps
    // the peak search of run i (on the side stream, after an event recorded when run i's fill
    // is done): the fill is bound by HBM writes, the peak test by memory latency. s waits
    // for the side stream at the end, so the call's completion on s covers everything.
    hipError_t e;
    for (int i = 0; i < pieces; ++i) {
      const int e0 = (int)((int64_t)n_ev * i / pieces), e1 = (int)((int64_t)n_ev * (i + 1) / pieces);
      if ((rc = check_launch(launch_fill(g, none, d_ev + e0, e1 - e0, any_bands, bs.long_l, s), "fill launch")))
        return rc;
      if ((e = hipEventRecord(split->filled[i], s)) != hipSuccess) return fail_hip(e, "hipEventRecord");
      if ((e = hipStreamWaitEvent(split->side, split->filled[i], 0)) != hipSuccess)
        return fail_hip(e, "hipStreamWaitEvent");
      if (i == 0 && (rc = injected_failure("peaks"))) return rc;
      if (any_bands && (rc = check_launch(launch_peaks(g, none, d_ev + e0, e1 - e0, g.j.n_groups, split->side), "peak launch")))
        return rc;
      if (any_dense &&
          (rc = check_launch(launch_peaks_dense(g, none, d_ev + e0, e1 - e0, split->side), "stencil peak launch")))
        return rc;
    }
    if ((e = hipEventRecord(split->done, split->side)) != hipSuccess) return fail_hip(e, "hipEventRecord");
    if ((e = hipStreamWaitEvent(s, split->done, 0)) != hipSuccess) return fail_hip(e, "hipStreamWaitEvent");
    return HT_OK;
  }
  if (g.lds_fill) {
    StageTimer t("fill", s);
    if ((rc = check_launch(launch_fill(g, none, d_ev, n_ev, any_bands, bs.long_l, s), "fill launch"))) return rc;
  } else {
    {
      StageTimer t("fill_atomic", s);
      if ((rc = check_launch(launch_fill_atomic(g, none, d_ev, n_ev, bs.prep_hits, s), "fill launch")))
        return rc;
    }
    StageTimer t("candidates", s);
    if ((rc = check_launch(launch_scan(g, none, d_ev, n_ev, g.j.n_groups, false, s), "candidate launch"))) return rc;
  }
  if ((rc = injected_failure("peaks"))) return rc;
  StageTimer t("peaks", s);
  if (bs.few) return check_launch(launch_few_peaks(g, none, d_ev, n_ev, s), "peak launch");
  if (any_bands && (rc = check_launch(launch_peaks(g, none, d_ev, n_ev, g.j.n_groups, s), "peak launch"))) return rc;
  if (any_dense && (rc = check_launch(launch_peaks_dense(g, none, d_ev, n_ev, s), "stencil peak launch")))
    return rc;
  return HT_OK;
}

// Outputs (peak list, count) may live in device memory or in pinned host memory that is
// mapped into the device's address space; anything else would fault on the device, so it is
// rejected here, on the host, before any launch.
// 0: not usable by a kernel; 1: device memory; 2: host memory mapped into the device; 3: managed.
// Only what the runtime positively reports as device-accessible is accepted: unregistered host
// memory (malloc, numpy, unpinned tensors) is reported as a successful query of type
// hipMemoryTypeUnregistered and must be refused.
int pointer_kind(const void* ptr)
{
  hipPointerAttribute_t attr;
  std::memset(&attr, 0, sizeof(attr));
  hipError_t e = hipPointerGetAttributes(&attr, ptr);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  if (attr.type == hipMemoryTypeDevice) return 1;
  if (attr.type == hipMemoryTypeHost && attr.devicePointer) return 2;
  if (attr.type == hipMemoryTypeManaged) return 3;
  return 0;
}

int check_accessible(const void* ptr, const char* what)
{
  if (!ptr) return HT_OK;
  if (pointer_kind(ptr) == 0)
    return fail(HT_EINVAL, "%s is neither device memory nor mapped pinned host memory", what);
  return HT_OK;
}

// The event size that a captured batch's preparation is made for: a power-of-two bucket of
// workgroups, so that batches of one size share a graph (workgroups past an event's hits return at
// once).
int64_t batch_hits(int64_t max_hits)
{
  int64_t blocks = 1;
  while (blocks * 256 < max_hits) blocks *= 2;
  return max_hits > 0 ? blocks * 256 : 0;
}

// Scratch layout of a batch: direct slab lists for every event when each event allows them and
// their scratch totals at most 8 GiB, else the counting sort for all (the 16-event batch of
// 105600-hit events on the 8x32x2048x2048 grid takes the counting sort). Returns whether the
// lists are direct; offs[i] is event i's scratch offset, *total the bytes of all of them.
bool plan_batch(const DevGrid& g, const ht_event* events, int n_events, bool few, std::vector<size_t>* offs,
                size_t* total)
{
  auto layout = [&g, few](int64_t n) { return dense_peaks(g, n) ? kPeakMask : few ? kPeakFew : kPeakBands; };
  bool direct = g.lds_fill != 0;
  size_t direct_bytes = 0;
  for (int i = 0; i < n_events; ++i) {
    direct = direct && direct_lists(g, events[i].n_hits);
    direct_bytes += event_scratch_bytes(g, events[i].n_hits, true, layout(events[i].n_hits));
  }
  if (direct_bytes > kBatchDirectMax) direct = false;
  offs->assign((size_t)n_events, 0);
  *total = 0;
  for (int i = 0; i < n_events; ++i) {
    (*offs)[i] = *total;
    *total += event_scratch_bytes(g, events[i].n_hits, direct, layout(events[i].n_hits));
  }
  return direct;
}

int enqueue_event(const DevGrid& g, const EvDesc& ev, int64_t nh, bool direct, bool atomic,
                  bool do_fill, bool do_peaks, bool timed, hipStream_t s, bool* counters_used)
{
  // stage timers only where asked for (they may create HIP events); a null name times nothing
#define HT_STAGE(var, name) StageTimer var(timed ? name : nullptr, s)
  int rc;
  *counters_used = false;
  const bool few = do_fill && do_peaks && ev.lists != 0 && ev.lists >> kListShift == 0;
  if (few && tiny_launch(g, 1, nh)) {
    if ((rc = injected_failure("prep")) || (rc = injected_failure("fill"))) return rc;
    {
      HT_STAGE(t, "fill");
      if ((rc = check_launch(launch_tiny_fill(g, ev, nullptr, 1, s), "fill launch"))) return rc;
      *counters_used = true;
    }
    if ((rc = injected_failure("peaks"))) return rc;
    HT_STAGE(t, "peaks");
    return check_launch(launch_few_peaks(g, ev, nullptr, 1, s), "peak launch");
  }
  if (do_fill) {
    {
      HT_STAGE(t, "prep");
      if ((rc = injected_failure("prep")) ||
          (rc = check_launch(launch_prep(g, ev, nullptr, 1, nh, direct, s), "prep launch")))
        return rc;
      *counters_used = true;
    }
    if ((rc = injected_failure("fill"))) return rc;
    if (atomic) {
      HT_STAGE(t, "fill_atomic");
      if ((rc = check_launch(launch_fill_atomic(g, ev, nullptr, 1, nh, s), "fill launch"))) return rc;
    } else {
      HT_STAGE(t, "fill");
      if ((rc = check_launch(launch_fill(g, ev, nullptr, 1, do_peaks && !ev.dense, long_lists(g, 1, nh), s), "fill launch"))) return rc;
    }
  }
  if (do_peaks) {
    if (!do_fill || atomic) {
      HT_STAGE(t, "candidates");
      if ((rc = check_launch(launch_scan(g, ev, nullptr, 1, ev.n_grp, !do_fill, s), "candidate launch"))) return rc;
      *counters_used = true;
    }
    if ((rc = injected_failure("peaks"))) return rc;
    HT_STAGE(t, "peaks");
    if (ev.dense) {
      if ((rc = check_launch(launch_peaks_dense(g, ev, nullptr, 1, s), "stencil peak launch"))) return rc;
    } else if (few) {
      if ((rc = check_launch(launch_few_peaks(g, ev, nullptr, 1, s), "peak launch"))) return rc;
    } else if ((rc = check_launch(launch_peaks(g, ev, nullptr, 1, ev.n_grp, s), "peak launch"))) {
      return rc;
    }
  }
#undef HT_STAGE
  return HT_OK;
}

int run_event(const ht_grid* grid, const float* x, const float* y, const float* z, int64_t n,
              uint32_t* acc, ht_peak* out, int64_t cap, int64_t* n_found, void* stream,
              bool do_fill, bool do_peaks, bool force_atomic)
{
  if (n < 0) return fail(HT_EINVAL, "n_hits < 0");
  if (!acc) return fail(HT_EINVAL, "acc is NULL");
  if (do_fill && n > 0 && (!x || !y || !z)) return fail(HT_EINVAL, "hit arrays are NULL");
  if (do_peaks && (cap < 0 || !n_found || (cap > 0 && !out)))
    return fail(HT_EINVAL, "peak output arguments are invalid");
  if (n > ((int64_t)1 << 28)) return fail(HT_EINVAL, "n_hits must be <= 2^28");
  Prepared p;
  int rc = prepare(grid, stream, &p, 1, do_fill ? n : 0, do_peaks);
  if (rc) return rc;
  if (do_peaks && ((rc = check_accessible(out, "out")) || (rc = check_accessible(n_found, "n_found"))))
    return rc;
  const int64_t nh = do_fill ? n : 0;
  const bool atomic = force_atomic || !p.g.lds_fill;
  const bool direct = !atomic && direct_lists(p.g, nh);
  // crowded events of the fused call: peaks from the stencil over the written matrix
  const bool dense = do_fill && do_peaks && !atomic && dense_peaks(p.g, nh);
  const bool few = do_fill && do_peaks && !atomic && batch_shape(p.g, 1, nh, dense, 1).few;
  const int layout = !do_peaks ? 0 : dense ? kPeakMask : few ? kPeakFew : kPeakBands;
  const int64_t hits = do_fill ? nh : -1;  // for the scratch
  if (do_peaks && (!do_fill || atomic)) set_jobs(&p.g, 0, 1);  // the survivors come from a scan
  Workspace* w;
  if ((rc = get_workspace(p.dev, p.s, event_scratch_bytes(p.g, hits, direct, layout), &w))) return rc;
  if ((rc = ensure_counters(w, 1, p.s))) return rc;
  EvDesc ev;
  std::memset(&ev, 0, sizeof(ev));
  carve_event_scratch(p.g, hits, direct, w->dev, &ev, layout);
  ev.dense = dense ? 1 : 0;
  if (layout == kPeakBands && do_fill && !atomic && !use_lists(p.g, 1, nh, nh)) ev.lists = 0;
  use_counters(w, 0, &ev);
  ev.x = x;
  ev.y = y;
  ev.z = z;
  ev.n_hits = nh;
  ev.acc = acc;
  ev.out = out;
  ev.cap = cap;
  ev.n_found = n_found;
  bool used = false;
  rc = enqueue_event(p.g, ev, nh, direct, atomic, do_fill, do_peaks, true, p.s, &used);
  // the next call counts into the other array only if a kernel of this call counts into this
  // one and clears that one (a launch that failed before it leaves both as they were)
  if (used) flip_counters(w, 1);
  return rc;
}

}  // namespace ht

using namespace ht;

extern "C" {

int ht_tables(const ht_grid* grid, float* a2, float* inv_db, float* phi_cs, float* th_cs)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  if (!a2 || !inv_db || !phi_cs || !th_cs) return fail(HT_EINVAL, "table pointers are NULL");
  host_tables_into(*grid, a2, inv_db, phi_cs, th_cs);
  return HT_OK;
}

int ht_tiling(const ht_grid* grid, int32_t* rows, int32_t* n_tiles, int32_t* cand_cap,
              int32_t* lds_fill)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  Tiling t = choose_tiling(*grid);
  if (rows) *rows = t.rows;
  if (n_tiles) *n_tiles = t.n_tiles;
  if (cand_cap) *cand_cap = t.cand_cap;
  if (lds_fill) *lds_fill = t.lds_fill;
  return HT_OK;
}

int ht_fill(const ht_grid* grid, const float* x, const float* y, const float* z, int64_t n_hits,
            uint32_t* acc, void* stream)
{
  return run_event(grid, x, y, z, n_hits, acc, nullptr, 0, nullptr, stream, true, false, false);
}

int ht_fill_atomic(const ht_grid* grid, const float* x, const float* y, const float* z,
                   int64_t n_hits, uint32_t* acc, void* stream)
{
  return run_event(grid, x, y, z, n_hits, acc, nullptr, 0, nullptr, stream, true, false, true);
}

int ht_peaks(const ht_grid* grid, const uint32_t* acc, ht_peak* out, int64_t capacity,
             int64_t* n_found, void* stream)
{
  return run_event(grid, nullptr, nullptr, nullptr, 0, const_cast<uint32_t*>(acc), out, capacity,
                   n_found, stream, false, true, false);
}

int ht_fill_peaks(const ht_grid* grid, const float* x, const float* y, const float* z,
                  int64_t n_hits, uint32_t* acc, ht_peak* out, int64_t capacity,
                  int64_t* n_found, void* stream)
{
  return run_event(grid, x, y, z, n_hits, acc, out, capacity, n_found, stream, true, true, false);
}

int ht_fill_peaks_batch(const ht_grid* grid, const ht_event* events, int32_t n_events,
                        const float* x, const float* y, const float* z, uint32_t* acc,
                        ht_peak* out, int64_t* n_found, void* stream)
{
  if (n_events < 0 || n_events > 65535) return fail(HT_EINVAL, "n_events must be in [0, 65535]");
  if (n_events == 0) return HT_OK;
  if (!events || !acc || !n_found) return fail(HT_EINVAL, "NULL batch argument");
  int64_t max_hits = 0;
  int rc = validate_grid(grid);
  if (rc) return rc;
  for (int32_t i = 0; i < n_events; ++i) {
    const ht_event& ev = events[i];
    if (ev.n_hits < 0 || ev.n_hits > ((int64_t)1 << 28) || ev.hit_offset < 0 || ev.peak_capacity < 0 ||
        ev.peak_offset < 0)
      return fail(HT_EINVAL, "event %d has invalid offsets or sizes", i);
    max_hits = std::max(max_hits, ev.n_hits);
    if (ev.n_hits > 0 && (!x || !y || !z)) return fail(HT_EINVAL, "hit arrays are NULL");
    if (ev.peak_capacity > 0 && !out) return fail(HT_EINVAL, "out is NULL");
  }
  Prepared p;
  if ((rc = prepare(grid, stream, &p, n_events, max_hits))) return rc;
  if ((rc = check_accessible(out, "out")) || (rc = check_accessible(n_found, "n_found"))) return rc;
  // overlap of the peak searches with the fills of later events: the batch in `pieces` runs
  const int pieces = std::max(1, std::min(std::min(env_int("HT_BATCH_PIECES", 1), kMaxPieces), (int)n_events));
  bool any_bands = false, any_dense = false;
  for (int32_t i = 0; i < n_events; ++i) {
    const bool dense = p.g.lds_fill && dense_peaks(p.g, events[i].n_hits);
    any_bands = any_bands || !dense;
    any_dense = any_dense || dense;
  }
  BatchShape shape = batch_shape(p.g, n_events, max_hits, any_dense, pieces);
  std::vector<size_t> offs;
  size_t total_scratch = 0;
  const bool direct = plan_batch(p.g, events, n_events, shape.few, &offs, &total_scratch);
  Workspace* w;
  if ((rc = get_workspace(p.dev, p.s, total_scratch, &w))) return rc;
  if ((rc = ensure_ev_staging(w, n_events, p.s))) return rc;
  if ((rc = ensure_counters(w, n_events, p.s))) return rc;
  EvDesc* const h_ev = w->h_ev[w->turn];
  const uint64_t cells = n_cells(*grid);
  for (int32_t i = 0; i < n_events; ++i) {
    const ht_event& ev = events[i];
    EvDesc& d = h_ev[i];
    std::memset(&d, 0, sizeof(d));
    const bool dense = p.g.lds_fill && dense_peaks(p.g, ev.n_hits);
    carve_event_scratch(p.g, ev.n_hits, direct, w->dev + offs[i], &d, dense ? kPeakMask : shape.few ? kPeakFew : kPeakBands);
    d.dense = dense ? 1 : 0;
    if (!shape.few && p.g.lds_fill && !use_lists(p.g, n_events, max_hits, ev.n_hits)) d.lists = 0;
    use_counters(w, i, &d);
    d.x = x ? x + ev.hit_offset : nullptr;
    d.y = y ? y + ev.hit_offset : nullptr;
    d.z = z ? z + ev.hit_offset : nullptr;
    d.n_hits = ev.n_hits;
    d.acc = acc + (size_t)i * cells;
    d.out = out ? out + ev.peak_offset : nullptr;
    d.cap = ev.peak_capacity;
    d.n_found = n_found + i;
  }
  hipError_t e;
  BatchSplit split;
  std::memset(&split, 0, sizeof(split));
  split.pieces = pieces;
  // The launches go to the stream one by one: five kernels cost the host what one graph launch
  // costs, and a graph starts 8 us after the work before it (100 events of 250 hits: 44.7 us a
  // batch, 52.8 as a graph; 100 paper events 4457 and 4465). HT_BATCH_GRAPH=1 captures the batch
  // once per shape and replays it; so does a caller's stream under capture, as the descriptors
  // are staged anew on each call.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  const int graph_env = env_int("HT_BATCH_GRAPH", -1);
  if (graph_env < 0 && hipStreamIsCapturing(p.s, &cap) != hipSuccess) {  // the default stream beside a capture
    (void)hipGetLastError();
    cap = hipStreamCaptureStatusActive;
  }
  const bool graph_mode = graph_env < 0 ? cap != hipStreamCaptureStatusNone : graph_env != 0;
  if (pieces > 1) {
    hipStream_t& side = graph_mode ? w->capture_side : w->side;
    if (!side && (e = hipStreamCreateWithFlags(&side, hipStreamNonBlocking)) != hipSuccess)
      return fail_hip(e, "hipStreamCreate(side)");
    for (int i = 0; i <= kMaxPieces; ++i)
      if (!w->split_ev[i] && (e = hipEventCreateWithFlags(&w->split_ev[i], hipEventDisableTiming)) != hipSuccess)
        return fail_hip(e, "hipEventCreate(split)");
    split.side = side;
    for (int i = 0; i < kMaxPieces; ++i) split.filled[i] = w->split_ev[i];
    split.done = w->split_ev[kMaxPieces];
  }
  // The descriptors above hold this call's counter arrays. The next call switches to the other
  // arrays only once this call's preparation (which counts into these and clears those) is on
  // the stream; a call that fails before that leaves the counters as they were.
  if (!graph_mode) {
    if ((e = launch_fetch(w->d_ev, h_ev, n_events, p.s)) != hipSuccess) return fail_hip(e, "descriptor launch");
    if ((e = hipEventRecord(w->ev_read[w->turn], p.s)) != hipSuccess) return fail_hip(e, "hipEventRecord");
    bool prep_enqueued = false;
    rc = launch_batch(p.g, w->d_ev, n_events, shape, direct, any_bands, any_dense, p.s, &prep_enqueued,
                      pieces > 1 ? &split : nullptr);
    if (prep_enqueued) flip_counters(w, n_events);
    return rc;
  }
  // graph key: everything the captured launches depend on besides the descriptor contents
  shape.prep_hits = batch_hits(max_hits);
  std::vector<unsigned char> key(sizeof(DevGrid) + 4 * sizeof(int64_t) + 2 * sizeof(void*));
  {
    unsigned char* q = key.data();
    std::memcpy(q, &p.g, sizeof(DevGrid));
    q += sizeof(DevGrid);
    const int64_t ints[4] = {n_events, shape.prep_hits, p.dev,
                             (direct ? 1 : 0) | (any_bands ? 2 : 0) | (any_dense ? 4 : 0) | (shape.long_l ? 8 : 0) |
                                 (shape.tiny ? 16 : 0) | (shape.few ? 32 : 0) | (pieces << 6)};
    std::memcpy(q, ints, sizeof(ints));
    q += sizeof(ints);
    const void* ptrs[2] = {w->d_ev, h_ev};
    std::memcpy(q, ptrs, sizeof(ptrs));
  }
  hipGraphExec_t exec = nullptr;
  for (auto& gr : w->graphs)
    if (gr.key == key) exec = gr.exec;
  if (!exec) {
    if (!w->capture && (e = hipStreamCreateWithFlags(&w->capture, hipStreamNonBlocking)) != hipSuccess)
      return fail_hip(e, "hipStreamCreate(capture)");
    // the capture stream must not start before earlier work on the caller's stream is done
    // with the descriptor staging; capturing records work without running it
    if ((e = hipStreamBeginCapture(w->capture, hipStreamCaptureModeThreadLocal)) != hipSuccess)
      return fail_hip(e, "hipStreamBeginCapture");
    t_capturing = true;
    e = launch_fetch(w->d_ev, h_ev, n_events, w->capture);
    bool captured_prep = false;
    int lrc = e == hipSuccess
                  ? launch_batch(p.g, w->d_ev, n_events, shape, direct, any_bands, any_dense, w->capture,
                                 &captured_prep, pieces > 1 ? &split : nullptr)
                  : HT_EDEVICE;
    t_capturing = false;
    hipGraph_t graph = nullptr;
    hipError_t e2 = hipStreamEndCapture(w->capture, &graph);
    if (e != hipSuccess) return fail_hip(e, "descriptor launch (capture)");
    if (lrc != HT_OK) {
      if (graph) (void)hipGraphDestroy(graph);
      return lrc;
    }
    if (e2 != hipSuccess) return fail_hip(e2, "hipStreamEndCapture");
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return fail_hip(e, "hipGraphInstantiate");
    if (w->graphs.size() >= 32) {  // two per batch shape; the oldest may still be running
      if ((e = hipStreamSynchronize(p.s)) != hipSuccess) {
        (void)hipGraphExecDestroy(exec);
        return fail_hip(e, "hipStreamSynchronize");
      }
      (void)hipGraphExecDestroy(w->graphs.front().exec);
      w->graphs.erase(w->graphs.begin());
    }
    w->graphs.push_back({key, exec});
  }
  {
    StageTimer t("batch", p.s);
    if ((e = hipGraphLaunch(exec, p.s)) != hipSuccess) return fail_hip(e, "hipGraphLaunch");
  }
  flip_counters(w, n_events);
  if ((e = hipEventRecord(w->ev_read[w->turn], p.s)) != hipSuccess) return fail_hip(e, "hipEventRecord");
  return HT_OK;
}

int ht_set_tuning(const ht_grid* grid, const ht_tuning* tuning)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  if (!tuning) {
    g_tune.erase(tune_key(*grid));
    return HT_OK;
  }
  if ((rc = check_tuning(*grid, *tuning))) return rc;
  g_tune[tune_key(*grid)] = *tuning;
  return HT_OK;
}

int ht_get_tuning(const ht_grid* grid, ht_tuning* tuning)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  if (!tuning) return fail(HT_EINVAL, "tuning is NULL");
  Tiling t = choose_tiling(*grid);
  tuning->rows = t.rows;
  tuning->group_tiles = t.group_tiles;
  tuning->cand_cap = t.cand_cap;
  tuning->nt_store = t.nt_store;
  tuning->tiles_per_block = t.fill_tiles;
  tuning->dense_hits = t.dense_w > 0 && t.dense_hits > 0 ? t.dense_hits : -1;
  return HT_OK;
}

int ht_readout(const ht_grid* grid, const ht_peak* peaks, const int64_t* n_found, int64_t capacity,
               ht_track* tracks, void* stream)
{
  if (capacity < 0 || capacity > ((int64_t)1 << 31)) return fail(HT_EINVAL, "capacity out of range");
  if (!n_found || (capacity > 0 && (!peaks || !tracks))) return fail(HT_EINVAL, "NULL readout argument");
  Prepared p;
  int rc = prepare(grid, stream, &p, 1, 0);
  if (rc) return rc;
  if ((rc = check_accessible(peaks, "peaks")) || (rc = check_accessible(n_found, "n_found")) ||
      (rc = check_accessible(tracks, "tracks")))
    return rc;
  const double db = ((double)grid->b_max - (double)grid->b_min) / (double)grid->n_b;
  return check_launch(launch_readout(p.g, peaks, n_found, capacity, tracks, (double)grid->b_min, db, p.s),
                      "readout launch");
}

int ht_debug_pointer_kind(const void* ptr, int32_t* kind)
{
  if (!ptr || !kind) return fail(HT_EINVAL, "NULL argument");
  *kind = pointer_kind(ptr);
  return HT_OK;
}

int ht_debug_hit_values(const ht_grid* grid, const float* x, const float* y, const float* z,
                        int64_t n_hits, int32_t* info, float* vals, int32_t* slabs, void* stream)
{
  if (n_hits < 0) return fail(HT_EINVAL, "n_hits < 0");
  if (n_hits > 0 && (!x || !y || !z || !info || !vals || !slabs)) return fail(HT_EINVAL, "NULL pointer");
  Prepared p;
  int rc = prepare(grid, stream, &p, 1, 0);
  if (rc) return rc;
  return check_launch(launch_debug_hits(p.g, x, y, z, n_hits, info, vals, slabs, p.s), "debug launch");
}

int ht_debug_unary(const float* v, float* root, float* inv2, int64_t n, void* stream)
{
  if (n < 0) return fail(HT_EINVAL, "n < 0");
  if (n == 0) return HT_OK;
  if (!v || !root || !inv2) return fail(HT_EINVAL, "NULL pointer");
  if (pointer_kind(v) == 0 || pointer_kind(root) == 0 || pointer_kind(inv2) == 0)
    return fail(HT_EINVAL, "an array is not device-accessible memory");
  return check_launch(launch_debug_unary(v, root, inv2, n, (hipStream_t)stream), "debug launch");
}

int ht_debug_batch_plan(const ht_grid* grid, const ht_event* events, int32_t n_events,
                        int32_t* direct, int64_t* scratch_bytes)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  if (!events || !direct || !scratch_bytes || n_events < 1 || n_events > 65535)
    return fail(HT_EINVAL, "invalid batch-plan arguments");
  for (int32_t i = 0; i < n_events; ++i)
    if (events[i].n_hits < 0 || events[i].n_hits > ((int64_t)1 << 28))
      return fail(HT_EINVAL, "event %d has an invalid size", i);
  // the tiling alone decides the layout; the tables (device memory) are not needed
  int64_t max_hits = 0;
  for (int32_t i = 0; i < n_events; ++i) max_hits = std::max(max_hits, events[i].n_hits);
  const DevGrid g = make_devgrid(*grid, DevTables(), choose_tiling(*grid), n_events, max_hits);
  bool any_dense = false;
  for (int32_t i = 0; i < n_events; ++i) any_dense = any_dense || (g.lds_fill && dense_peaks(g, events[i].n_hits));
  std::vector<size_t> offs;
  size_t total = 0;
  *direct = plan_batch(g, events, n_events, batch_shape(g, n_events, max_hits, any_dense, 1).few, &offs, &total) ? 1 : 0;
  *scratch_bytes = (int64_t)total;
  return HT_OK;
}

int ht_debug_launch_plan(const ht_grid* grid, int32_t call, const int64_t* n_hits, int32_t n_events,
                         ht_launch_plan* plan)
{
  int rc = validate_grid(grid);
  if (rc) return rc;
  const bool serve = call == 3, batch = call == 1 || serve;
  if (!n_hits || !plan || call < 0 || call > 3 || n_events < (serve ? 2 : 1) || n_events > (batch ? 65535 : 1))
    return fail(HT_EINVAL, "invalid launch-plan arguments");
  std::vector<ht_event> events((size_t)n_events);
  int64_t max_hits = 0;
  for (int32_t i = 0; i < n_events; ++i) {
    if (n_hits[i] < 0 || n_hits[i] > ((int64_t)1 << 28)) return fail(HT_EINVAL, "event %d has an invalid size", i);
    events[i] = ht_event{0, n_hits[i], 0, 0};
    if (!serve || i > 0) max_hits = std::max(max_hits, n_hits[i]);
  }
  const Tiling tl = choose_tiling(*grid);
  const int64_t loop_hits = serve ? n_hits[0] : 0;
  if (serve) events.erase(events.begin());
  const int n_ev = (int)events.size();
  DevGrid g = make_devgrid(*grid, DevTables(), tl, n_ev, serve ? loop_hits : max_hits);
  if (serve) g.dense_hits = stencil_from(tl, n_ev, max_hits);
  std::memset(plan, 0, sizeof(*plan));
  NoallocPlan na;
  std::memset(&na, 0, sizeof(na));
  if (call == 2 && (rc = plan_noalloc(*grid, tl, g, max_hits, &na))) return rc;
  plan->rows = g.rows;
  plan->nt_store = g.nt_store;
  for (const ht_event& ev : events) {
    const bool dense = call == 2 ? na.dense : g.lds_fill && dense_peaks(g, ev.n_hits);
    plan->n_stencil += dense ? 1 : 0;
  }
  plan->sliced = na.sliced ? 1 : 0;
  const BatchShape b = batch_shape(g, n_ev, max_hits, plan->n_stencil > 0 || na.sliced, 1);
  for (const ht_event& ev : events)
    if (na.sliced || b.few || !g.lds_fill || use_lists(g, n_ev, max_hits, ev.n_hits))
      plan->n_lists += call == 2 ? !na.dense : !(g.lds_fill && dense_peaks(g, ev.n_hits));
  plan->long_lists = b.long_l ? 1 : 0;
  plan->tiny = b.tiny ? 1 : 0;
  plan->few = b.few ? 1 : 0;
  if (call == 2) {
    plan->direct = na.direct ? 1 : 0;
    plan->scratch_bytes = (int64_t)na.scratch_bytes;
    return HT_OK;
  }
  if (serve) {
    plan->direct = direct_lists(g, loop_hits) ? 1 : 0;
    int layout;
    plan->scratch_bytes = (int64_t)n_ev * (int64_t)slot_scratch_bytes(g, tl, n_ev, loop_hits, &layout);
    return HT_OK;
  }
  std::vector<size_t> offs;
  size_t total = 0;
  plan->direct = plan_batch(g, events.data(), n_ev, b.few, &offs, &total) ? 1 : 0;
  plan->scratch_bytes = (int64_t)total;
  return HT_OK;
}

int ht_profile_enable(int mode)
{
  if (mode < 0 || mode > 2) return fail(HT_EINVAL, "profile mode must be 0, 1 or 2");
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_mode = mode;
  return HT_OK;
}

int ht_profile_read(const char* name, double* total_ms, int64_t* count, int reset)
{
  if (!name || !total_ms || !count) return fail(HT_EINVAL, "NULL profile argument");
  std::lock_guard<std::mutex> lk(g_prof_mu);
  double tot = 0.0;
  int64_t n = 0;
  for (const ProfRec& r : g_prof) {
    if (std::strcmp(r.name, name) != 0) continue;
    hipError_t e = hipEventSynchronize(r.b);
    if (e != hipSuccess) return fail_hip(e, "hipEventSynchronize(profile)");
    float ms = 0.0f;
    if ((e = hipEventElapsedTime(&ms, r.a, r.b)) != hipSuccess) return fail_hip(e, "hipEventElapsedTime");
    tot += ms;
    ++n;
  }
  *total_ms = tot;
  *count = n;
  if (reset) {
    for (const ProfRec& r : g_prof) {
      (void)hipEventSynchronize(r.b);
      g_prof_pool.push_back(r.a);
      g_prof_pool.push_back(r.b);
    }
    g_prof.clear();
  }
  return HT_OK;
}

const char* ht_last_error(void) { return g_err.c_str(); }

}  // extern "C"
