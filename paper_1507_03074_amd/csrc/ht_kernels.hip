// ht_kernels.hip -- gfx950 kernels of the Hough-transform fill and peak search.
//
// Pipeline (paper section 2: every hit votes along its circles through the interaction point,
// then the local maxima above a threshold are the track candidates). Every kernel takes a batch
// of events (grid.y = event), so one launch per stage serves a single event or a whole batch:
//   k_prep_direct per hit: validity, r2, k = 1/(2y), theta/phi half-sectors and the 2-4
//                 (theta, phi) cells; the (hit, cell) records go to fixed-capacity per-slab lists
//                 (one slab = the A x B plane of one (theta, phi) cell), their positions reserved
//                 with LDS-aggregated atomics. Very large events use a counting sort instead:
//                 k_prep counts, then k_bucket scans the counts in LDS and scatters.
//   k_fill        one workgroup per (slab, tile of A rows): the slab's records vote into an LDS
//                 tile (ds_add), then every cell of the tile is written to HBM once with
//                 coalesced 16-byte stores (so the matrix needs no memset); the survivors, the
//                 cells >= threshold that no cell of the wave's own job beats, go to bit masks
//   k_peak_test   one workgroup per group of jobs: the survivors take the strict 3^4 test against
//                 their 80 neighbours (a cell below the threshold can never beat one at or above
//                 it, so only survivors need testing); the group's peaks, sorted, and their count
//   k_peak_write  per group: its output offset from the earlier groups' counts; its peaks go
//                 to the ordered list
//   crowded events (at least dense_hits hits) have no masks: the fill only writes
//   the matrix, k_peak_stencil tests every cell in one read of it (one wave per phi cell, the
//   theta cells in its registers, the phi neighbours through LDS) into 64-bit peak words, and
//   k_peak_write_dense writes the ordered peak list from them
//   k_few_peaks   both of these in one workgroup per event, where few cells can be peaks
//   k_tiny_fill   the preparation and the fill in one launch, for the smallest events
// ht_peaks on an arbitrary matrix replaces prep and fill with k_scan (one read of it).
// No kernel synchronises workgroups with each other: on this multi-XCD part an agent-scope
// release costs an L2 write-back, while a kernel boundary is cheap.
//
// Every floating-point step of the bin rule is one binary32 operation, rounded to nearest even,
// in the documented order: contraction is off for this file, sqrtf and the division are the
// correctly rounded forms.
#include <cmath>
#include <cstdlib>

#include "ht_device.h"

#pragma clang fp contract(off)

namespace ht {
namespace {

// ---------------------------------------------------------------------------------------------
// Per-hit preparation (validity, per-hit values, half-sectors, cells)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int half_plane(float c, float s, float vx, float vy)
{
  float lhs = c * vy;
  float rhs = s * vx;
  float d = lhs - rhs;
  return d >= 0.0f ? 1 : 0;
}

// The two correctly rounded operations of the per-hit values: r = sqrt(r2) and k = 1/(2y)
// (2y is exact). Shared by the preparation and by ht_debug_unary, which checks them against
// the host over every binary32 input.
__device__ __forceinline__ float hit_root(float r2) { return sqrtf(r2); }
__device__ __forceinline__ float hit_inv2(float y)
{
  float ty = y + y;
  return 1.0f / ty;
}

struct HitPrep {
  int n;  // number of (theta, phi) cells, 0 when the hit votes nothing
  int slab[4];
  int s_theta, s_phi;
  float x, r2, r, k;
};

// phi_cs, th_cs: the boundary tables (g.phi_cs, g.th_cs or a copy of them in LDS).
__device__ HitPrep prep_hit(const DevGrid& g, const float* phi_cs, const float* th_cs, float x,
                            float y, float z)
{
  HitPrep h;
  h.n = 0;
  h.s_theta = h.s_phi = 0;
  h.x = x;
  h.r2 = h.r = h.k = 0.0f;
  // one test of all three coordinates (no short cut), so the load of z is not held back until
  // x and y have been checked
  if (!(isfinite(x) & isfinite(y) & isfinite(z)) | (y == 0.0f)) return h;
  float xx = x * x;
  float yy = y * y;
  float r2 = xx + yy;
  if (!(r2 > 0.0f) || isinf(r2)) return h;
  float r = hit_root(r2);
  float k = hit_inv2(y);
  // the boundary counts, several table entries in flight (one after another they cost an LDS round
  // trip each: 6.0 us for the preparation of the paper event, 5.2 now); the phi boundaries of the half plane that holds the hit
  const int m0 = y > 0.0f ? 0 : g.n_phi;
  int s_phi = m0;
#pragma unroll 5
  for (int m = 1; m < g.n_phi; ++m) s_phi += half_plane(phi_cs[2 * (m0 + m)], phi_cs[2 * (m0 + m) + 1], x, y);
  int s_th = 0;
#pragma unroll 7
  for (int m = 1; m < 2 * g.n_theta; ++m) s_th += half_plane(th_cs[2 * m], th_cs[2 * m + 1], z, r);
  const int p0 = s_phi >> 1;
  const int p1 = (s_phi & 1) ? (p0 + 1 == g.n_phi ? 0 : p0 + 1) : (p0 == 0 ? g.n_phi - 1 : p0 - 1);
  const int t0 = s_th >> 1;
  const int t1 = (s_th & 1) ? t0 + 1 : t0 - 1;
  if (g.phi_sectors) {
    // section 4: the hit's own sector only
    h.slab[0] = t0 * g.n_phi + p0;
    h.n = 1;
    if (t1 >= 0 && t1 < g.n_theta) {
      h.slab[1] = t1 * g.n_phi + p0;
      h.n = 2;
    }
  } else {
    h.slab[0] = t0 * g.n_phi + p0;
    h.slab[1] = t0 * g.n_phi + p1;
    h.n = 2;
    if (t1 >= 0 && t1 < g.n_theta) {
      h.slab[2] = t1 * g.n_phi + p0;
      h.slab[3] = t1 * g.n_phi + p1;
      h.n = 4;
    }
  }
  h.s_theta = s_th;
  h.s_phi = s_phi;
  h.r2 = r2;
  h.r = r;
  h.k = k;
  return h;
}

// The boundary tables copied into LDS (dynamic shared memory): the sector counts then read
// them at LDS latency instead of one scalar load after another. The caller's next barrier makes
// the copy visible. Without LDS_TABLES (grids whose tables exceed kLdsTableBytes) the tables are
// read from global memory.
constexpr size_t kLdsTableBytes = 16384;

template <bool LDS_TABLES>
__device__ __forceinline__ void tables_to_lds(const DevGrid& g, float* s_tab, const float** tab_phi,
                                              const float** tab_th)
{
  if (!LDS_TABLES) {
    *tab_phi = g.phi_cs;
    *tab_th = g.th_cs;
    return;
  }
  const int n_phi = 4 * g.n_phi, n_th = 2 * (2 * g.n_theta + 1);
  for (int i = threadIdx.x; i < n_phi + n_th; i += kBlock)
    s_tab[i] = i < n_phi ? gp(g.phi_cs)[i] : gp(g.th_cs)[i - n_phi];
  *tab_phi = s_tab;
  *tab_th = s_tab + n_phi;
}

// Clears the event's peak counts and job flags, and the other counter array: all of it, since an
// earlier call on a grid with more slabs may have used entries past this grid's n_slabs (the
// preparation's workgroups share the work).
__device__ __forceinline__ void clear_jobs(const EvDesc& e)
{
  for (int i = (int)(blockIdx.x * kBlock + threadIdx.x); i < kCounterWords; i += (int)(gridDim.x * kBlock))
    gp(e.slab_cnt_next)[i] = 0u;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  GLOBAL u32x4* const p = (GLOBAL u32x4*)gp((uint32_t*)e.clear);
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < e.clear_n16; i += gridDim.x * kBlock) p[i] = zero;
}

// A batch's descriptors, fetched from pinned host memory by a kernel like the others: a copy command
// is a 3 us kernel too, and 4 us pass after it before the next kernel starts.
__global__ __launch_bounds__(kBlock) void k_fetch(u32x2* to, const u32x2* from, uint32_t n)
{
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) ((GLOBAL u32x2*)to)[i] = ((const GLOBAL u32x2*)from)[i];
}

// Direct lists: counts per slab in LDS per workgroup, one global atomic per (workgroup, slab)
// reserves the workgroup's range of each slab's fixed-capacity list, then the records are
// written there. slab_cnt is zero on entry and ends holding the list lengths; The workgroups
// clear the other counter array for the next call.
template <bool LDS_TABLES>
__global__ __launch_bounds__(kBlock) void k_prep_direct(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  __shared__ uint32_t lcnt[kMaxSlabs];
  extern __shared__ float s_tab[];
  EvDesc e = load_ev(ev0, evs);
  clear_jobs(e);
  if ((int64_t)blockIdx.x * kBlock >= e.n_hits) return;  // uniform: whole block idle
  const int64_t h = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  // the hit's coordinates are loaded first, so their round trip overlaps the table copy
  const int64_t hc = min(h, e.n_hits - 1);
  const float hx = gp(e.x)[hc], hy = gp(e.y)[hc], hz = gp(e.z)[hc];
  const float *tab_phi, *tab_th;
  tables_to_lds<LDS_TABLES>(g, s_tab, &tab_phi, &tab_th);
  for (int i = threadIdx.x; i < g.n_slabs; i += kBlock) lcnt[i] = 0u;
  lds_barrier();
  HitPrep p;
  p.n = 0;
  uint32_t local[4] = {0u, 0u, 0u, 0u};
  if (h < e.n_hits) {
    p = prep_hit(g, tab_phi, tab_th, hx, hy, hz);
    if (isinf(p.k)) p.n = 0;  // (2y subnormal) every B is infinite or NaN: it has no votes
    // constant indices keep p.slab and local in registers (a runtime index would put them in
    // scratch memory)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < p.n) local[q] = atomicAdd(&lcnt[p.slab[q]], 1u);
  }
  lds_barrier();
  for (int i = threadIdx.x; i < g.n_slabs; i += kBlock) {
    uint32_t c = lcnt[i];
    if (c) lcnt[i] = gatomic_add(e.slab_cnt + i, c);
  }
  lds_barrier();
  if (h < e.n_hits) {
    const float4 rec = make_float4(p.x, p.r2, p.k, 0.0f);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < p.n) st_rec(e.list, (size_t)p.slab[q] * (size_t)e.list_cap + lcnt[p.slab[q]] + local[q], rec);
  }
}

// Counting sort, first pass: counts per slab (LDS, then one global atomic per workgroup and
// slab) and each record's position within its slab. The workgroups clear the other counter array.
template <bool LDS_TABLES>
__global__ __launch_bounds__(kBlock) void k_prep(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  __shared__ uint32_t lcnt[kMaxSlabs];
  extern __shared__ float s_tab[];
  EvDesc e = load_ev(ev0, evs);
  clear_jobs(e);
  if ((int64_t)blockIdx.x * kBlock >= e.n_hits) return;  // uniform: whole block idle
  const int64_t h = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t hc = min(h, e.n_hits - 1);
  const float hx = gp(e.x)[hc], hy = gp(e.y)[hc], hz = gp(e.z)[hc];
  const float *tab_phi, *tab_th;
  tables_to_lds<LDS_TABLES>(g, s_tab, &tab_phi, &tab_th);
  for (int i = threadIdx.x; i < g.n_slabs; i += kBlock) lcnt[i] = 0u;
  lds_barrier();
  HitPrep p;
  p.n = 0;
  uint32_t local[4] = {0u, 0u, 0u, 0u};
  if (h < e.n_hits) {
    p = prep_hit(g, tab_phi, tab_th, hx, hy, hz);
    if (isinf(p.k)) p.n = 0;  // (2y subnormal) every B is infinite or NaN: it has no votes
    e.hit_rec[h] = make_float4(p.x, p.r2, p.k, 0.0f);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int s = q < p.n ? p.slab[q] : -1;
      e.hit_slab[4 * h + q] = s;
      if (s >= 0) local[q] = atomicAdd(&lcnt[s], 1u);
    }
  }
  lds_barrier();
  for (int i = threadIdx.x; i < g.n_slabs; i += kBlock) {
    uint32_t c = lcnt[i];
    if (c) lcnt[i] = atomicAdd(&e.slab_cnt[i], c);
  }
  lds_barrier();
  if (h < e.n_hits)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < p.n) e.hit_pos[4 * h + q] = lcnt[p.slab[q]] + local[q];
}

// Every workgroup scans the slab counts into LDS (they are few); workgroup 0 also publishes the
// offsets for the fill. Then each hit's records go to their slab lists.
__global__ __launch_bounds__(kBlock) void k_bucket(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  __shared__ uint32_t s_off[kMaxSlabs];
  __shared__ uint32_t smem[32];
  EvDesc e = load_ev(ev0, evs);
  if (blockIdx.x > 0 && (int64_t)blockIdx.x * kBlock >= e.n_hits) return;
  const int ns = g.n_slabs;
  const int per = (ns + kBlock - 1) / kBlock;
  const int beg = min(ns, (int)threadIdx.x * per);
  const int end = min(ns, beg + per);
  uint32_t sum = 0;
  for (int i = beg; i < end; ++i) sum += e.slab_cnt[i];
  uint32_t total;
  uint32_t run = block_excl_scan(sum, smem, &total);
  for (int i = beg; i < end; ++i) {
    const uint32_t c = e.slab_cnt[i];
    s_off[i] = run;
    if (blockIdx.x == 0) e.slab_off[i] = run;
    run += c;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) e.slab_off[ns] = total;
  lds_barrier();
  const int64_t h = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (h >= e.n_hits) return;
  const float4 rec = e.hit_rec[h];
  for (int q = 0; q < 4; ++q) {
    const int s = e.hit_slab[4 * h + q];
    if (s < 0) break;
    e.list[s_off[s] + e.hit_pos[4 * h + q]] = rec;
  }
}

// ---------------------------------------------------------------------------------------------
// Tiny events (tiny_launch: up to 1024 hits, 1024 tiles). Their calls were bound by the launches,
// four of them, of which each takes the host 2 us and the device 3 to 5: now two, 15.6 and 9.6 us
// for 250 hits on 4x16x64x64.
//
// The fill: every workgroup prepares all of the event's hits itself (170 instructions per thread
// and 256 hits, less than a round trip to a list), and keeps the records of its own slab in LDS;
// each wave then votes a quarter of the rows. Survivors go to the lists only.
// ---------------------------------------------------------------------------------------------
template <bool VEC, bool NT>
__global__ __launch_bounds__(kBlock) void k_tiny_fill(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  extern __shared__ uint32_t smem[];
  __shared__ float s_x[kTinyHits], s_r2[kTinyHits], s_k[kTinyHits];
  __shared__ uint32_t s_n;
  EvDesc e = load_ev(ev0, evs);
  const uint32_t nb = (uint32_t)g.n_b, ldr4 = (nb + 3u) / 4u, ldr = 4u * ldr4;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t tile_words = (uint32_t)g.rows * ldr;
  u32x4* const s4 = reinterpret_cast<u32x4*>(smem);
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  const int n_hits = (int)e.n_hits;
  // the first hits are loaded before anything else
  const int h0 = min((int)threadIdx.x, n_hits - 1);
  float hx = 0.0f, hy = 0.0f, hz = 0.0f;
  if (n_hits > 0) {  // uniform
    hx = gp(e.x)[h0];
    hy = gp(e.y)[h0];
    hz = gp(e.z)[h0];
  }
  const float *tab_phi, *tab_th;
  tables_to_lds<true>(g, reinterpret_cast<float*>(smem) + tile_words, &tab_phi, &tab_th);
  for (uint32_t i = threadIdx.x; i < tile_words / 4u; i += kBlock) s4[i] = zero4;
  if (threadIdx.x == 0) s_n = 0u;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < (uint32_t)kCounterWords; i += gridDim.x * kBlock)
    gp(e.slab_cnt_next)[i] = 0u;
  const int slab = (int)blockIdx.x / g.tiles_per_slab;
  const int a0 = ((int)blockIdx.x - slab * g.tiles_per_slab) * g.rows;
  const int rows = min(g.rows, g.n_a - a0);
  lds_barrier();
  for (int h = 0; h < n_hits; h += kBlock) {  // uniform
    if (h > 0) {
      const int i = min(h + (int)threadIdx.x, n_hits - 1);
      hx = gp(e.x)[i];
      hy = gp(e.y)[i];
      hz = gp(e.z)[i];
    }
    const HitPrep p = prep_hit(g, tab_phi, tab_th, hx, hy, hz);
    bool mine = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) mine |= q < p.n && p.slab[q] == slab;  // its cells are distinct
    if (mine && h + (int)threadIdx.x < n_hits) {
      const uint32_t i = atomicAdd(&s_n, 1u);
      s_x[i] = p.x;
      s_r2[i] = p.r2;
      s_k[i] = p.k;
    }
  }
  lds_barrier();
  const uint32_t n = s_n;
  for (uint32_t i0 = 0u; i0 < n; i0 += 64u) {  // uniform
    const uint32_t i = min(i0 + lane, n - 1u);
    const float x = s_x[i], r2 = s_r2[i], k = s_k[i];
#pragma unroll 4
    for (int r = (int)wave; r < rows; r += kBlock / 64) {
      const float ax = g.a2[a0 + r] * x;
      const float num = r2 - ax;
      const float Bv = num * k;
      const float d = Bv - g.b_min;
      const float f = d * g.inv_db;
      if (i0 + lane < n && f >= 0.0f && f < g.nb_f) atomicAdd(&smem[(uint32_t)r * ldr + (uint32_t)(int)f], 1u);
    }
  }
  lds_barrier();
  const uint32_t sub = g.j.sub > 1 ? lane / ldr4 : 0u;
  const uint32_t unit0 = g.j.sub > 1 ? lane - sub * ldr4 : lane;
  const uint32_t lmask = unit0 > 0u ? ~0u : 0u, rmask = g.j.sub > 1 && unit0 + 1u == ldr4 ? 0u : ~0u;
  const uint32_t cell0 = ((uint32_t)slab * (uint32_t)g.n_a + (uint32_t)a0) * nb;
  sweep_jobs<4, VEC, NT, false, kBlock / 64>(g, e.acc, s4, ldr4, ldr4, nb, cell0, rows, wave, lane, sub, unit0,
                                      [&](uint32_t job, uint32_t c0, const u32x4 (&v)[4]) {
    const uint32_t m = job_survivors<4>(v, g.threshold, lmask, rmask);
    if (__builtin_amdgcn_ballot_w64(m != 0u) == 0u) return;  // uniform
    list_survivors<4>(e, blockIdx.x * (uint32_t)g.j.tile_jobs + job, 0u, lane, m, c0, nb, v);
  });
}

// Where a job's cells are: its rows are a0 .. of `slab` (absent from row n_a and, in a fill tile,
// from the tile's end on), lane l's band starts at row a0 + sub * ch and its unit is u.
struct JobAt {
  uint32_t slab, a0, st;
};
__device__ __forceinline__ JobAt job_at(const DevGrid& g, uint32_t job)
{
  const uint32_t tile = job / (uint32_t)g.j.tile_jobs, k = job - tile * (uint32_t)g.j.tile_jobs;
  const uint32_t bg = k / (uint32_t)g.j.strips;
  JobAt j;
  j.slab = tile / (uint32_t)g.j.tiles_per_slab;
  j.a0 = (tile - j.slab * (uint32_t)g.j.tiles_per_slab) * (uint32_t)g.j.tile_rows +
         bg * (uint32_t)(g.j.sub * g.j.ch);
  j.st = k - bg * (uint32_t)g.j.strips;
  return j;
}

// Survivors of an arbitrary matrix: every job's cells read once, straight into registers, two
// jobs per wave in flight. Bound by the read of the matrix. Stores every job's flag, and clears
// the peak counts that the test adds to and (counters: no preparation came before) the other
// counter array.
template <bool VEC, int CH>
__global__ __launch_bounds__(kBlock) void k_scan(DevGrid g, EvDesc ev0, const EvDesc* evs, int counters)
{
  EvDesc e = load_ev(ev0, evs);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t nb = (uint32_t)g.n_b, units = (uint32_t)g.j.units, P = (uint32_t)g.j.sub;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < e.n_grp; i += gridDim.x * kBlock) {
    gp(e.group_pk)[i * (uint32_t)g.j.pk_step] = 0u;
    if (i < (e.n_grp + 63u) / 64u) gp(e.super_pk)[i * kSuperStep] = 0u;
  }
  if (counters)  // uniform
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < (uint32_t)kCounterWords; i += gridDim.x * kBlock)
      gp(e.slab_cnt_next)[i] = 0u;
  const uint32_t sub = P > 1u ? lane / units : 0u;
  const uint32_t unit0 = P > 1u ? lane - sub * units : lane;
  const uint32_t lmask = unit0 > 0u ? ~0u : 0u;
  const uint32_t rmask = P > 1u && unit0 + 1u == units ? 0u : ~0u;
  const uint32_t gj = (uint32_t)g.j.group_jobs;
  const uint64_t first = (uint64_t)e.grp0 * gj;
  const uint64_t n = min((uint64_t)g.j.n_jobs - first, (uint64_t)e.n_grp * gj);
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  u32x4 v[2][CH];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint64_t jl = (uint64_t)blockIdx.x * 8u + (uint32_t)h * 4u + wave;
#pragma unroll
    for (int q = 0; q < CH; ++q) v[h][q] = zero4;
    if (jl < n) {  // uniform
      const JobAt at = job_at(g, (uint32_t)(first + jl));
      const uint32_t u = P > 1u ? unit0 : at.st * 64u + lane;
      const uint32_t a = at.a0 + sub * CH;
      const bool in = u < units && sub < P;
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        if (in && a + (uint32_t)q < (uint32_t)g.n_a) {
          const GLOBAL uint32_t* src = gp((const uint32_t*)e.acc) + (at.slab * (uint32_t)g.n_a + a + (uint32_t)q) * nb + 4u * u;
          if (VEC) {
            v[h][q] = __builtin_nontemporal_load(reinterpret_cast<const GLOBAL u32x4*>(src));
          } else if (4u * u + 3u < nb) {
            v[h][q] = *reinterpret_cast<const GLOBAL u32x4_a4*>(src);
          } else {
#pragma unroll
            for (int k = 0; k < 3; ++k)
              if (4u * u + (uint32_t)k < nb) v[h][q][k] = src[k];
          }
        }
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint64_t jl = (uint64_t)blockIdx.x * 8u + (uint32_t)h * 4u + wave;
    if (jl >= n) return;  // uniform
    const uint32_t m = job_survivors<CH>(v[h], g.threshold, lmask, rmask);
    if (__builtin_amdgcn_ballot_w64(m != 0u) == 0u) {  // uniform
      if (lane == 0u) gp(e.job_any)[jl] = 0;
      continue;
    }
    put_mask<CH>(e, (uint32_t)jl, lane, m);
    const JobAt at = job_at(g, (uint32_t)(first + jl));
    const uint32_t c0 = (at.slab * (uint32_t)g.n_a + at.a0 + sub * CH) * nb + 4u * (P > 1u ? unit0 : at.st * 64u + lane);
    list_survivors<CH>(e, (uint32_t)jl, (uint32_t)jl / gj, lane, m, c0, nb, v[h]);
  }
}

// ---------------------------------------------------------------------------------------------
// Peak test: strict maximum under (votes, -index) over the 3^4 box, phi periodic.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void cell_coords(const DevGrid& g, uint32_t c, uint32_t* t, uint32_t* p,
                                            uint32_t* a, uint32_t* b)
{
  const uint32_t nb = (uint32_t)g.n_b, na = (uint32_t)g.n_a, np = (uint32_t)g.n_phi;
  *b = c % nb;
  uint32_t q = c / nb;
  *a = q % na;
  q /= na;
  *p = q % np;
  *t = q / np;
}


// A cell under test: its coordinates and the window of three columns that its neighbour rows are
// read through, which starts at min(max(b, 1) - 1, n_b - 3) so that it stays inside the row (grids
// with n_b < 3 read their one or two columns).
struct TestCell {
  uint32_t c, v, t, p, a, b, w0;
};
__device__ __forceinline__ TestCell test_cell(const DevGrid& g, uint32_t c, uint32_t v)
{
  TestCell x;
  x.c = c;
  x.v = v;
  cell_coords(g, c, &x.t, &x.p, &x.a, &x.b);
  x.w0 = min(max(x.b, 1u) - 1u, max((uint32_t)g.n_b, 3u) - 3u);
  return x;
}
// Neighbour row (dt, dp, da): its first window cell, or the cell's own window where the row is
// absent (outside theta or A, or a phi neighbour across sectors; *in false). Phi wraps.
__device__ __forceinline__ uint32_t row_window(const DevGrid& g, const TestCell& x, int dt, int dp, int da, bool* in)
{
  const uint32_t nb = (uint32_t)g.n_b, na = (uint32_t)g.n_a, np = (uint32_t)g.n_phi;
  const int tt = (int)x.t + dt, aa = (int)x.a + da;
  *in = tt >= 0 && tt < g.n_theta && aa >= 0 && aa < (int)na && !(g.phi_sectors && dp != 0);
  uint32_t pp = x.p;
  if (dp < 0) pp = x.p == 0u ? np - 1u : x.p - 1u;
  if (dp > 0) pp = x.p + 1u == np ? 0u : x.p + 1u;
  return (*in ? (((uint32_t)tt * np + pp) * na + (uint32_t)aa) * nb : x.c - x.b) + x.w0;
}
struct Row3 {
  uint32_t w[3];
};
// NARROW: rows of fewer than three cells; else one 12-byte load.
template <bool NARROW>
__device__ __forceinline__ Row3 load_row(const DevGrid& g, const uint32_t* acc, uint32_t at)
{
  const GLOBAL uint32_t* r = gp(acc) + at;
  Row3 o;
  o.w[0] = r[0];
  o.w[1] = !NARROW || g.n_b > 1 ? r[1] : 0u;
  o.w[2] = !NARROW ? r[2] : 0u;
  return o;
}
// Whether the row beats the cell under (votes, -index): a row other than the cell's own lies
// wholly before it (an equal count beats it) or after it. v >= 1, so zeros beat nothing. (Votes
// may be any 32-bit count: no + 1 here.)
__device__ __forceinline__ bool row_wins(const TestCell& x, const Row3& r, uint32_t at, bool own)
{
  bool beaten = false;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint32_t bb = x.w0 + (uint32_t)q;
    const bool near = bb + 1u >= x.b && bb <= x.b + 1u && !(own && bb == x.b);
    const bool before = own ? bb < x.b : at < x.c;
    beaten |= near && (r.w[q] > x.v || (before && r.w[q] == x.v));
  }
  return beaten;
}
// The nine neighbour rows of theta cell t + DT: whether one beats the cell, one cell per lane. With
// every lane at it, this is bound by the lines and the instructions of its rows. So three rows are
// in flight at a time, those of one phi cell (the nearest lines first), and a lane stops at the first
// that beats it; rows lie at constant distances (row_window takes three products for each); and a
// row counts by the maximum of its near columns, which beats the cell above v, or above v - 1 where
// the row lies before the cell. (With sectors the rows of the other phi cells are the same ones
// again: a branch around them costs the other grids 3%.) The test of a 40k-hit event takes 54 us; with the nine rows together
// 64 (whatever the occupancy, from three to eight waves), with two rows of either side first 65.
template <bool NARROW, int DT>
__device__ __forceinline__ bool slice_wins(const DevGrid& g, const uint32_t* acc, const TestCell& x)
{
  const uint32_t nb = (uint32_t)g.n_b, np = (uint32_t)g.n_phi, S = (uint32_t)g.n_a * nb;
  if (DT < 0 ? x.t == 0u : DT > 0 && x.t + 1u == (uint32_t)g.n_theta) return false;
  const uint32_t at0 = x.c - x.b + x.w0 + (uint32_t)DT * np * S;
  const bool first = x.b == 0u, last = x.b + 1u == nb;  // the window's third or first column is not near
  const uint32_t before = x.v - 1u;                     // x.v >= 1
  // the rows at A - 1 and A + 1; where there is none, the one at A again
  const uint32_t up = x.a > 0u ? 0u - nb : 0u, down = x.a + 1u < (uint32_t)g.n_a ? nb : 0u;
#pragma unroll
  for (int q = 0; q < 3; ++q) {  // phi cells p, p - 1, p + 1
    const bool wraps = q == 1 ? x.p == 0u : x.p + 1u == np;
    const uint32_t at = at0 + (q == 0 || g.phi_sectors ? 0u : q == 1 ? (wraps ? (np - 1u) * S : 0u - S) : (wraps ? 0u - (np - 1u) * S : S));
    Row3 r[3] = {load_row<NARROW>(g, acc, at + up), load_row<NARROW>(g, acc, at), load_row<NARROW>(g, acc, at + down)};
    // whole rows: the compiler would load a column that an edge drops by itself, and later
#pragma unroll
    for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(r[k].w[0]), "+v"(r[k].w[1]), "+v"(r[k].w[2]));
    uint32_t m[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      m[k] = max(max(!NARROW && last ? 0u : r[k].w[0], r[k].w[1]), first ? 0u : r[k].w[2]);
    if (DT == 0 && q == 0) {  // of the own row, the columns beside the cell
      const uint32_t left = first ? 0u : !NARROW && last ? r[1].w[1] : r[1].w[0];
      const uint32_t right = last ? 0u : first ? r[1].w[1] : r[1].w[2];
      if (max(left, up ? m[0] : 0u) > before || max(right, down ? m[2] : 0u) > x.v) return true;
    } else {
      const bool lies_before = DT < 0 || (DT == 0 && (q == 1) != wraps);
      if (max(max(m[0], m[1]), m[2]) > (lies_before ? before : x.v) && !(DT == 0 && g.phi_sectors)) return true;
    }
  }
  return false;
}

// Block b of a grid of G runs on XCD b % 8 (workgroups are dealt to the eight XCDs in turn); the
// number this returns is a bijection of [0, G) under which XCD x runs one contiguous range of
// numbers: the first G % 8 XCDs take ceil(G / 8) of them, the others floor(G / 8).
__device__ __forceinline__ uint32_t xcd_contiguous(uint32_t b, uint32_t G)
{
  const uint32_t x = b & 7u, i = b >> 3, q = G >> 3, r = G & 7u;
  return x < r ? x * (q + 1u) + i : r * (q + 1u) + (x - r) * q + i;
}

__device__ __forceinline__ void tile_range(const DevGrid& g, int tile, uint32_t* cell0, uint32_t* L)
{
  const int slab = tile / g.tiles_per_slab;
  const int a0 = (tile - slab * g.tiles_per_slab) * g.rows;
  const int rows = min(g.rows, g.n_a - a0);
  *cell0 = ((uint32_t)slab * (uint32_t)g.n_a + (uint32_t)a0) * (uint32_t)g.n_b;
  *L = (uint32_t)rows * (uint32_t)g.n_b;
}

// Peak test of the survivors. It is bound by the latency of its gather (27 rows of 12 bytes, each
// in a cache line of its own). Two forms:
//
// From the lists, when they are made and every survivor fits them (ordinary events: 2.7k
// survivors on the paper event): spread evenly over the grid whatever their groups, half a wave
// each, one lane per neighbour row, so the whole test is two memory round trips (the list, the
// rows) and a third for each peak's place in its group's segment. Survivors cluster (the
// fullest of the paper event's 1024 groups holds 157 of them, the mean group 2.7), and a
// workgroup per group waited 15 us for that one.
//
// Else from the masks, one workgroup per group of jobs. The flagged jobs' masks (64 jobs at a
// time, their loads in flight together) are turned into one list of survivors in LDS, shared by
// the four waves, so the tests run with full waves however the survivors lie in their jobs: up
// to kFew of them half a wave each, more a lane each, the nine rows of the own theta cell first
// (they beat most: adjacent phi cells hold the same circles), and those left, packed again into
// full waves, the rows of the two theta neighbours. The group's peaks are then sorted by rank in
// LDS and stored in the group's segment; the masks are written back as the peaks' masks, for
// groups whose peaks do not fit it.
constexpr uint32_t kList = 1024;  // four jobs have at most this many survivors (one per 2 x 2 cells)
constexpr uint32_t kFew = 64;
constexpr uint32_t kSuperGroups = 8192;
constexpr uint32_t kTestBlocks = 4 * kLists * 32 / kBlock;
constexpr uint32_t kTestGrid = 8192;
constexpr uint32_t kPassJobs = 64;

template <bool NARROW>
__global__ __launch_bounds__(kBlock) void k_peak_test(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  __shared__ uint32_t s_pos[kList];         // survivors: slot << 10 | lane << 4 | bit of the mask
  __shared__ uint32_t s_m[kPassJobs * 32];  // masks of the pass, 16 bits per lane
  __shared__ uint32_t s_slab[kPassJobs], s_a0[kPassJobs], s_st[kPassJobs];  // where its jobs are
  __shared__ __align__(16) uint32_t s_pc[kSegMax];
  __shared__ uint32_t s_pv[kSegMax];
  __shared__ uint16_t s_ids[kBlock];
  __shared__ uint32_t s_w[4], s_n, s_np;
  EvDesc e = load_ev(ev0, evs);
  if (e.dense) return;  // uniform: searched by the stencil
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool supers = e.n_grp > kSuperGroups;
  const uint32_t seg_cap = (uint32_t)g.j.seg;
  if (e.lists) {  // uniform
    // half wave h takes entries h / kLists, h / kLists + step, ... of list h % kLists, four of them
    // in flight (half waves past a multiple of kLists of them take none)
    const uint32_t hw = blockIdx.x * (kBlock / 32) + (threadIdx.x >> 5), k = threadIdx.x & 31u;
    const uint32_t l = hw % kLists, step = gridDim.x * (kBlock / 32) / kLists;
    const uint32_t cap = e.lists & kListEntries;
    const GLOBAL u32x4* const list = (const GLOBAL u32x4*)gp((const uint4*)e.surv) + l * cap;
    // the first entry is loaded before the list's length is known: one round trip for both
    u32x4 en[4];
    en[0] = list[min(hw / kLists, cap - 1u)];
    const uint32_t n = gp((const uint32_t*)e.slab_cnt)[kListLens + l * kListLine];
    if (gp((const uint32_t*)e.slab_cnt)[kListOver] == 0u) {  // uniform over the grid
      const int kk = (int)min(k, 26u), dt = kk / 9 - 1, dp = kk / 3 % 3 - 1, da = kk % 3 - 1;
      const uint32_t n_max = max((uint32_t)__builtin_amdgcn_readlane((int)n, 0), (uint32_t)__builtin_amdgcn_readlane((int)n, 32));
      const uint32_t i_wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(hw / kLists));  // the same in both halves
      if (i_wave >= step) return;
      for (uint32_t i0 = i_wave; i0 < n_max; i0 += 4u * step) {  // wave-uniform
        bool beaten[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
          const uint32_t i = i0 + q * step;
          if (i < n_max && i != i_wave) en[q] = list[min(i, cap - 1u)];
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
          const uint32_t i = i0 + q * step;
          beaten[q] = true;
          if (i < n) {
            const TestCell x = test_cell(g, en[q].x, en[q].y);
            bool in;
            const uint32_t at = row_window(g, x, dt, dp, da, &in);
            beaten[q] = row_wins(x, load_row<NARROW>(g, e.acc, at), at, kk == 13) && in && k < 27u;
          }
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
          const uint32_t hm = (uint32_t)(__builtin_amdgcn_ballot_w64(beaten[q]) >> (lane & 32u));
          if (k == 0u && hm == 0u) {
            const uint32_t o = gatomic_add(e.group_pk + en[q].z * (uint32_t)g.j.pk_step, 1u);
            if (supers) gatomic_add(e.super_pk + en[q].z / 64u * kSuperStep, 1u);
            const u32x2 pk = {en[q].x, en[q].y};
            if (o < seg_cap) ((GLOBAL u32x2*)gp(e.seg))[(size_t)en[q].z * seg_cap + o] = pk;
          }
        }
      }
      return;
    }
  }
  const bool two = g.j.elem_bytes == 2;
  const uint32_t* acc = e.acc;
  const uint32_t na = (uint32_t)g.n_a, nb = (uint32_t)g.n_b, np = (uint32_t)g.n_phi;
  const uint32_t P = (uint32_t)g.j.sub, ch = (uint32_t)g.j.ch, units = (uint32_t)g.j.units;
  uint16_t* const m16 = reinterpret_cast<uint16_t*>(s_m);
  // the survivor of a list entry
  auto cell_of = [&](uint32_t pos) {
    const uint32_t slot = pos >> 10, l = pos >> 4 & 63u, bit = pos & 15u;
    const uint32_t sub = P > 1u ? l / units : 0u;
    const uint32_t slab = s_slab[slot];
    TestCell x;
    x.a = s_a0[slot] + sub * ch + (bit >> 2);
    x.b = 4u * (P > 1u ? l - sub * units : s_st[slot] * 64u + l) + (bit & 3u);
    x.t = slab >> 16;
    x.p = slab & 0xffffu;
    x.c = ((x.t * np + x.p) * na + x.a) * nb + x.b;
    x.v = gp(acc)[x.c];
    x.w0 = min(max(x.b, 1u) - 1u, max(nb, 3u) - 3u);
    return x;
  };
  auto keep = [&](uint32_t pos, const TestCell& x) {
    atomicOr(&s_m[pos >> 5], 1u << (pos & 31u));
    const uint32_t i = atomicAdd(&s_np, 1u);
    if (i < seg_cap) {
      s_pc[i] = x.c;
      s_pv[i] = x.v;
    }
  };
  auto rank_of = [](uint64_t m, uint32_t from) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, from));
  };
  // Workgroups are dealt to the eight XCDs in turn (their number is a multiple of eight). Each XCD
  // takes pieces of four slabs' groups, so that the rows which neighbouring groups and phi cells
  // share are fetched into one L2, and the pieces go round the XCDs shifted by one each time, as
  // some phi and theta cells are more crowded than others. (One range of groups per XCD, a theta cell
  // each, took 506 us per event on 8x32x2048x2048 cells, this takes 310. The groups in plain turn are
  // as fast there, but a 40k-hit event on the paper grid takes 139 us with them and with pieces of
  // two slabs 135, with four 131.)
  const uint32_t piece = min((e.n_grp + 7u) / 8u, 4u * max(1u, e.n_grp / (uint32_t)g.n_slabs));
  const uint32_t rounds = (e.n_grp + 8u * piece - 1u) / (8u * piece);
  for (uint32_t sl = blockIdx.x; sl < rounds * 8u * piece; sl += gridDim.x) {  // uniform
    const uint32_t round = (sl >> 3) / piece;
    const uint32_t grp = (round * 8u + (((sl & 7u) - round) & 7u)) * piece + ((sl >> 3) - round * piece);
    if (grp >= e.n_grp) continue;
    const uint32_t gj = (uint32_t)g.j.group_jobs;
    const uint64_t first = (uint64_t)(e.grp0 + grp) * gj;
    const uint32_t nj = (uint32_t)min((uint64_t)gj, (uint64_t)g.j.n_jobs - first);
    const uint64_t l0 = (uint64_t)grp * gj;  // the group's first job in the event's arrays
    if (threadIdx.x == 0) s_np = 0u;
    for (uint32_t win = 0u; win < nj; win += kBlock) {  // uniform
      // the window's flagged jobs, in order
      const uint32_t j = win + threadIdx.x;
      uint32_t flag = 0u;
      if (j < nj) flag = gp(e.job_any)[l0 + j];
      const uint64_t fb = __builtin_amdgcn_ballot_w64(flag != 0u);
      if (lane == 0u) s_w[w] = (uint32_t)__builtin_popcountll(fb);
      lds_barrier();
      const uint32_t f1 = s_w[0], f2 = f1 + s_w[1], f3 = f2 + s_w[2], nf = f3 + s_w[3];
      if (flag) s_ids[rank_of(fb, w == 0u ? 0u : w == 1u ? f1 : w == 2u ? f2 : f3)] = (uint16_t)threadIdx.x;
      lds_barrier();
      for (uint32_t p0 = 0u; p0 < nf; p0 += kPassJobs) {  // uniform
        const uint32_t n_job = min(kPassJobs, nf - p0);
        // the pass's masks: slot w + 4 i is this wave's i-th job
        uint32_t m[kPassJobs / 4];
#pragma unroll
        for (uint32_t i = 0; i < kPassJobs / 4; ++i) {
          m[i] = 0u;
          if (w + 4u * i < n_job) {  // uniform
            const size_t at = (size_t)(l0 + win + s_ids[p0 + w + 4u * i]) * 64u + lane;
            m[i] = two ? ((const GLOBAL uint16_t*)gp((const uint8_t*)e.masks))[at]
                       : gp((const uint8_t*)e.masks)[at];
          }
        }
        if (threadIdx.x < n_job) {  // meanwhile, a lane per job: where it is
          const JobAt at = job_at(g, (uint32_t)(first + win + s_ids[p0 + threadIdx.x]));
          const uint32_t t = at.slab / np;
          s_slab[threadIdx.x] = t << 16 | (at.slab - t * np);
          s_a0[threadIdx.x] = at.a0;
          s_st[threadIdx.x] = at.st;
        }
        uint32_t cnt = 0u;
#pragma unroll
        for (uint32_t i = 0; i < kPassJobs / 4; ++i) {
          if (w + 4u * i < n_job) {  // uniform
            m16[(w + 4u * i) * 64u + lane] = (uint16_t)m[i];
            cnt += (uint32_t)__builtin_popcount(m[i]);
          }
        }
        cnt = wave_sum(cnt);
        if (lane == 0u) s_w[w] = cnt;
        if (threadIdx.x == 0) s_n = 0u;
        lds_barrier();
        // all the jobs' survivors at once where the list holds them, else four jobs at a time
        const uint32_t step = s_w[0] + s_w[1] + s_w[2] + s_w[3] <= kList ? kPassJobs / 4 : 1u;
        for (uint32_t i0 = 0u; 4u * i0 < n_job; i0 += step) {               // uniform
          for (uint32_t i = i0; i < i0 + step && w + 4u * i < n_job; ++i) {  // uniform
            const uint32_t slot = w + 4u * i;
            uint32_t mm = m16[slot * 64u + lane];
            m16[slot * 64u + lane] = 0;
            const uint32_t c = (uint32_t)__builtin_popcount(mm), incl = wave_incl_scan(c);
            uint32_t from = 0u;
            if (lane == 63u) from = atomicAdd(&s_n, incl);
            uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)from, 63) + incl - c;
            while (mm) {
              s_pos[at++] = (slot << 10) | (lane << 4) | (uint32_t)__builtin_ctz(mm);
              mm &= mm - 1u;
            }
          }
          lds_barrier();
          const uint32_t n = s_n;  // uniform
          if (n <= kFew) {
            const uint32_t half = threadIdx.x >> 5, k = threadIdx.x & 31u;
            const int kk = (int)min(k, 26u), dt = kk / 9 - 1, dp = kk / 3 % 3 - 1, da = kk % 3 - 1;
            for (uint32_t b0 = 0u; b0 < n; b0 += 32u) {  // uniform
              TestCell x[4];
              bool beaten[4];
#pragma unroll
              for (uint32_t q = 0; q < 4; ++q) {
                x[q] = cell_of(s_pos[min(b0 + half + 8u * q, n - 1u)]);
                bool in;
                const uint32_t at = row_window(g, x[q], dt, dp, da, &in);
                beaten[q] = row_wins(x[q], load_row<NARROW>(g, acc, at), at, kk == 13) && in && k < 27u;
              }
#pragma unroll
              for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t i = b0 + half + 8u * q;
                const uint32_t hm = (uint32_t)(__builtin_amdgcn_ballot_w64(beaten[q]) >> (lane & 32u));
                if (k == 0u && i < n && hm == 0u) keep(s_pos[i], x[q]);
              }
            }
          } else {
            uint32_t n2 = 0u;
            for (uint32_t b0 = 0u; b0 < n; b0 += kBlock) {  // uniform
              const uint32_t i = b0 + threadIdx.x;
              uint32_t pos = 0u;
              bool alive = false;
              if (i < n) {
                pos = s_pos[i];
                alive = !slice_wins<NARROW, 0>(g, acc, cell_of(pos));
              }
              const uint64_t b = __builtin_amdgcn_ballot_w64(alive);
              if (lane == 0u) s_w[w] = (uint32_t)__builtin_popcountll(b);
              lds_barrier();  // every wave has read its entries: the front of the list is free
              const uint32_t c1 = s_w[0], c2 = c1 + s_w[1], c3 = c2 + s_w[2];
              if (alive) s_pos[rank_of(b, n2 + (w == 0u ? 0u : w == 1u ? c1 : w == 2u ? c2 : c3))] = pos;
              n2 += c3 + s_w[3];
              lds_barrier();
            }
            for (uint32_t i = threadIdx.x; i < n2; i += kBlock) {
              const uint32_t pos = s_pos[i];
              const TestCell x = cell_of(pos);
              if (!slice_wins<NARROW, -1>(g, acc, x) && !slice_wins<NARROW, 1>(g, acc, x)) keep(pos, x);
            }
          }
          lds_barrier();
          if (threadIdx.x == 0) s_n = 0u;
          lds_barrier();
        }
        for (uint32_t i = 0u; i < kPassJobs / 4 && w + 4u * i < n_job; ++i) {  // uniform: the peaks' masks
          const uint32_t slot = w + 4u * i;
          const size_t at = (size_t)(l0 + win + s_ids[p0 + slot]) * 64u + lane;
          const uint32_t mm = m16[slot * 64u + lane];
          if (two) ((GLOBAL uint16_t*)gp(e.masks))[at] = (uint16_t)mm;
          else gp(e.masks)[at] = (uint8_t)mm;
        }
      }
    }
    lds_barrier();
    const uint32_t n = s_np;
    if (threadIdx.x == 0) {
      gp(e.group_pk)[grp * (uint32_t)g.j.pk_step] = n;
      if (n && supers) gatomic_add(e.super_pk + grp / 64u * kSuperStep, n);
    }
    if (n == 0u || n > seg_cap) {  // uniform
      lds_barrier();
      continue;
    }
    // pad to whole 16-byte reads with cells that rank after every peak's
    if (threadIdx.x < 4u && n + threadIdx.x < seg_cap) s_pc[n + threadIdx.x] = 0xffffffffu;
    lds_barrier();
    const u32x4* s4 = reinterpret_cast<const u32x4*>(s_pc);
    for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
      const uint32_t c = s_pc[i];
      uint32_t r = 0u;
      for (uint32_t k = 0u; k < (n + 3u) / 4u; ++k) {
        const u32x4 o = s4[k];
        r += (o.x < c ? 1u : 0u) + (o.y < c ? 1u : 0u) + (o.z < c ? 1u : 0u) + (o.w < c ? 1u : 0u);
      }
      const u32x2 pk = {c, s_pv[i]};
      ((GLOBAL u32x2*)gp(e.seg))[(size_t)grp * seg_cap + r] = pk;
    }
    lds_barrier();  // the next group clears what this one still reads
  }
}

// Peaks of an event of few cells (few_cells), whose one list holds all survivors, by one workgroup:
// half a wave each, one lane per neighbour row, four in flight; the peaks wait in LDS, and each is
// written at its rank. Bound by its three memory round trips (the list, the rows, the stores), where
// the test and the ordered write are two launches of two each. (One list, not eight: 100 events of 250
// hits 5.3 us before, 4.6 now, and the fill's reservations are too few to queue at its counter.)
template <bool NARROW>
__global__ __launch_bounds__(1024) void k_few_peaks(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  __shared__ __align__(16) uint32_t s_c[kFewCells + 4];
  __shared__ uint16_t s_v[kFewCells];  // votes: at most one per hit
  static_assert(kFewHits <= 0xffff, "the counts of an event with few cells have 16 bits");
  __shared__ uint32_t s_n;
  EvDesc e = load_ev(ev0, evs);
  const bool a8 = ((uintptr_t)e.out & 7u) == 0;
  const uint32_t lane = threadIdx.x & 63u, hw = threadIdx.x >> 5, k = threadIdx.x & 31u;
  constexpr uint32_t kStep = 1024 / 32;  // half waves
  const GLOBAL u32x4* const list = (const GLOBAL u32x4*)gp((const uint4*)e.surv);
  const uint32_t last = (e.lists & kListEntries) - 1u;
  if (threadIdx.x == 0) s_n = 0u;
  u32x4 en[4];
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) en[q] = list[min(hw + q * kStep, last)];  // before their number is known
  const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)gp((const uint32_t*)e.slab_cnt)[kListLens]);
  const int kk = (int)min(k, 26u), dt = kk / 9 - 1, dp = kk / 3 % 3 - 1, da = kk % 3 - 1;
  lds_barrier();
  for (uint32_t i0 = 0u; i0 < n; i0 += 4u * kStep) {  // uniform
    bool beaten[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q)
      if (i0 > 0u) en[q] = list[min(i0 + hw + q * kStep, last)];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      beaten[q] = true;
      if (i0 + hw + q * kStep < n) {
        const TestCell x = test_cell(g, en[q].x, en[q].y);
        bool in;
        const uint32_t at = row_window(g, x, dt, dp, da, &in);
        beaten[q] = row_wins(x, load_row<NARROW>(g, e.acc, at), at, kk == 13) && in && k < 27u;
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const uint32_t hm = (uint32_t)(__builtin_amdgcn_ballot_w64(beaten[q]) >> (lane & 32u));
      if (k == 0u && hm == 0u) {
        const uint32_t o = atomicAdd(&s_n, 1u);
        s_c[o] = en[q].x;
        s_v[o] = (uint16_t)en[q].y;
      }
    }
  }
  lds_barrier();
  const uint32_t np = s_n;
  if (threadIdx.x == 0) *gp(e.n_found) = (int64_t)np;
  if (threadIdx.x < 4u) s_c[np + threadIdx.x] = 0xffffffffu;  // whole 16-byte reads
  lds_barrier();
  const u32x4* s4 = reinterpret_cast<const u32x4*>(s_c);
  for (uint32_t i = threadIdx.x; i < np; i += 1024u) {
    const uint32_t c = s_c[i];
    uint32_t r = 0u;
    for (uint32_t j = 0u; j < (np + 3u) / 4u; ++j) {
      const u32x4 o = s4[j];
      r += (o.x < c ? 1u : 0u) + (o.y < c ? 1u : 0u) + (o.z < c ? 1u : 0u) + (o.w < c ? 1u : 0u);
    }
    if ((int64_t)r < e.cap) st_peak(e.out, r, c, s_v[i], a8);
  }
}

// Ordered peak list, one wave per group: its output offset is the sum of the earlier groups'
// counts (a workgroup's four waves share it: with 2048 groups a wave of its own took 6.2 us, four
// together 4.7), loaded together with its first 64 peaks, so an ordinary group is one memory
// round trip. Past kSuperGroups groups the counts are also kept per block of 64 groups, a cache line
// each (not below: a test's atomic additions to one cache line take 10 ns each, which cost 9 us on the
// paper event, and 80 us of a 23k-hit event's test on 7x29x573x923 cells, 3654 groups). Peaks found
// from the lists are in no order in their segment: each lane ranks its
// own among the group's. A group with more peaks than its segment holds is listed from its masks
// in LDS, in cell order (whole job rows: band by band, row by row, strip by strip, then lane and
// column), up to eight jobs' masks in flight; masks that the lists replaced still hold survivors,
// which are tested again.
template <bool NARROW>
__global__ __launch_bounds__(kBlock) void k_peak_write(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  __shared__ __align__(16) uint32_t s_all[kBlock / 64][kSegMax];
  __shared__ uint16_t s_m[kBlock / 64][8 * 64];
  __shared__ uint32_t s_sum[kBlock / 64];
  EvDesc e = load_ev(ev0, evs);
  if (e.dense) return;  // uniform: written by k_peak_write_dense
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t G = blockIdx.x * (kBlock / 64) + w;
  const bool a8 = ((uintptr_t)e.out & 7u) == 0;
  const uint32_t seg_cap = (uint32_t)g.j.seg;
  const bool live = G < e.n_grp;  // uniform in a wave
  const uint32_t Gl = live ? G : 0u;
  const GLOBAL u32x2* const seg = (const GLOBAL u32x2*)gp((const uint2*)e.seg) + (size_t)Gl * seg_cap;
  const u32x2 head = seg[lane];  // may hold no peaks yet
  // the test worked from the lists if they were made and none overflowed
  const bool sorted = !e.lists || gp((const uint32_t*)e.slab_cnt)[kListOver] != 0u;
  const uint32_t ps = (uint32_t)g.j.pk_step;
  const uint32_t G0 = blockIdx.x * (kBlock / 64);                      // the workgroup's first group
  const uint32_t s0 = e.n_grp > kSuperGroups ? G0 & ~63u : 0u;         // groups before s0: by their blocks
  const uint32_t own = G0 + lane < e.n_grp && lane < kBlock / 64 ? gp(e.group_pk)[(G0 + lane) * ps] : 0u;
  uint32_t part = 0u;
  for (uint32_t i = threadIdx.x; i < s0 / 64u; i += kBlock) part += gp(e.super_pk)[i * kSuperStep];
  for (uint32_t i0 = s0; i0 < G0; i0 += 8u * kBlock) {  // uniform; eight loads in flight
    uint32_t x[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const uint32_t i = i0 + k * kBlock + threadIdx.x;
      x[k] = i < G0 ? gp(e.group_pk)[i * ps] : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) part += x[k];
  }
  part = wave_sum(part);
  if (lane == 0u) s_sum[w] = part;
  lds_barrier();
  if (!live) return;
  const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane((int)own, (int)w);
  int64_t base = (int64_t)(s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]);
  for (uint32_t k = 0; k < w; ++k) base += (uint32_t)__builtin_amdgcn_readlane((int)own, (int)k);
  if (e.carry_in) base += *gp(e.carry_in);
  if (G == e.n_grp - 1u && lane == 0u) {
    *gp(e.n_found) = base + mine;
    if (e.carry_out) *gp(e.carry_out) = base + mine;
  }
  if (mine == 0u || base >= e.cap) return;  // uniform
  if (mine <= 64u) {                        // uniform
    uint32_t r = lane;
    if (!sorted) {
      r = 0u;
      for (uint32_t k = 0u; k < mine; ++k)
        r += (uint32_t)__builtin_amdgcn_readlane((int)head.x, (int)k) < head.x ? 1u : 0u;
    }
    if (lane < mine && base + r < e.cap) st_peak(e.out, base + r, head.x, head.y, a8);
    return;
  }
  if (mine <= seg_cap) {  // uniform
    if (!sorted) {
      for (uint32_t i = lane; i < mine; i += 64u) s_all[w][i] = seg[i].x;
      if (lane < 4u && mine + lane < seg_cap) s_all[w][mine + lane] = 0xffffffffu;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    }
    const u32x4* s4 = reinterpret_cast<const u32x4*>(s_all[w]);
    for (uint32_t i = lane; i < mine; i += 64u) {
      const u32x2 pk = seg[i];
      uint32_t r = i;
      if (!sorted) {
        r = 0u;
        for (uint32_t k = 0u; k < (mine + 3u) / 4u; ++k) {
          const u32x4 o = s4[k];
          r += (o.x < pk.x ? 1u : 0u) + (o.y < pk.x ? 1u : 0u) + (o.z < pk.x ? 1u : 0u) + (o.w < pk.x ? 1u : 0u);
        }
      }
      if (base + r < e.cap) st_peak(e.out, base + r, pk.x, pk.y, a8);
    }
    return;
  }
  const uint32_t gj = (uint32_t)g.j.group_jobs, nb = (uint32_t)g.n_b;
  const uint64_t first = (uint64_t)(e.grp0 + G) * gj;
  const uint32_t nj = (uint32_t)min((uint64_t)gj, (uint64_t)g.j.n_jobs - first);
  const uint64_t l0 = (uint64_t)G * gj;
  const uint32_t P = (uint32_t)g.j.sub, ch = (uint32_t)g.j.ch, strips = (uint32_t)g.j.row_jobs;
  const uint32_t sub = P > 1u ? lane / (uint32_t)g.j.units : 0u;
  const uint32_t unit0 = P > 1u ? lane - sub * (uint32_t)g.j.units : lane;
  uint32_t n = 0u;  // cells listed in s_all[w]
  auto flush = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
#pragma unroll 1
    for (uint32_t i0 = 0u; i0 < n; i0 += 64u) {  // uniform
      bool pk = i0 + lane < n;
      const uint32_t c = s_all[w][min(i0 + lane, n - 1u)];
      const uint32_t v = gp((const uint32_t*)e.acc)[c];
      if (!sorted) {  // uniform
        const TestCell x = test_cell(g, c, v);
        pk = pk && !slice_wins<NARROW, 0>(g, e.acc, x) && !slice_wins<NARROW, -1>(g, e.acc, x) &&
             !slice_wins<NARROW, 1>(g, e.acc, x);
      }
      const uint64_t b = __builtin_amdgcn_ballot_w64(pk);
      const int64_t o = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
      if (pk && o < e.cap) st_peak(e.out, o, c, v, a8);
      base += (int64_t)__builtin_popcountll(b);
    }
    n = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  };
  auto mask_of = [&](uint32_t j) -> uint32_t {  // job j of the group; 0 without survivors
    const size_t i = (size_t)(l0 + j) * 64u + lane;
    const uint32_t m = g.j.elem_bytes == 2 ? ((const GLOBAL uint16_t*)gp((const uint8_t*)e.masks))[i]
                                           : gp((const uint8_t*)e.masks)[i];
    return gp((const uint8_t*)e.job_any)[l0 + j] ? m : 0u;
  };
  auto list = [&](uint32_t j, uint32_t nib, uint32_t row) {  // a lane's columns of one row of job j
    if (__builtin_amdgcn_ballot_w64(nib != 0u) == 0ull) return;  // uniform
    const JobAt at = job_at(g, (uint32_t)(first + j));
    const uint32_t c = (at.slab * (uint32_t)g.n_a + at.a0 + row) * nb + 4u * (P > 1u ? unit0 : at.st * 64u + lane);
    const uint32_t k = (uint32_t)__builtin_popcount(nib), incl = wave_incl_scan(k);
    uint32_t i = n + incl - k;
    for (; nib; nib &= nib - 1u) s_all[w][i++] = c + (uint32_t)__builtin_ctz(nib);
    n += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    if (n > kSegMax - 128u) flush();  // uniform; a row of a job has at most 128 survivors
  };
  if (strips <= 8u) {  // uniform, as all that follow
    const uint32_t rows = 8u / strips;  // job rows at a time
    for (uint32_t j0 = 0u; j0 < nj; j0 += rows * strips) {
      const uint32_t jobs = min(rows * strips, nj - j0);
#pragma unroll
      for (uint32_t s = 0; s < 8; ++s) s_m[w][s * 64u + lane] = s < jobs ? (uint16_t)mask_of(j0 + s) : (uint16_t)0;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      for (uint32_t r = 0u; r < jobs; r += strips)
        for (uint32_t b = 0u; b < P; ++b)
          for (uint32_t q = 0u; q < ch; ++q)
            for (uint32_t s = 0u; s < strips; ++s)
              list(j0 + r + s, sub == b ? s_m[w][(r + s) * 64u + lane] >> (4u * q) & 15u : 0u, b * ch + q);
    }
  } else {  // wide rows: one band per job row
    for (uint32_t j0 = 0u; j0 < nj; j0 += strips)
      for (uint32_t q = 0u; q < ch; ++q)
        for (uint32_t s = 0u; s < strips; ++s) list(j0 + s, mask_of(j0 + s) >> (4u * q) & 15u, q);
  }
  flush();
}

constexpr int kWriteStage = 4096;  // peaks of a group staged in LDS by the dense writer

// ---------------------------------------------------------------------------------------------
// Peak search of crowded events: an LDS-halo stencil over the whole matrix (one read of it), in
// place of the survivor masks. A workgroup owns one chunk of kChunkCells B columns of every
// (theta, phi) slab and walks down a segment of S A rows. Wave p holds phi cell p of every theta
// cell, so its theta neighbours are in its own registers: lane j holds cell b = base + j - 1 of
// slab (t, p) for each t, where base = kChunkCells * chunk. Lanes 1..62 are tested; lanes 0 and
// 63 hold the cells just outside the chunk, so that every tested cell's B neighbours are in the
// wave (neighbouring chunks overlap by those two cells).
//
// The strict maximum under (votes, -index) splits the 80 neighbours of a cell c into those of
// lower index ("before": theta cell t - 1, the phi cell of lower index in theta cell t, the row
// above in its own slab, the cell left of it) and the others ("after"). A before-neighbour w
// beats c iff w >= v(c); an after-neighbour iff w > v(c). With Mb and Ma the maxima over the
// before- and after-neighbours (absent cells count 0),
//   c is a peak  iff  v(c) >= T,  v(c) >= Mb + 1  and  v(c) >= Ma.
// Per row a a wave forms, for each t, R3(a, b) = the maximum over b-1..b+1 (neighbour lanes by
// DPP wave shifts), then W9(a-1, b) = the maximum of R3 over rows a-2..a (the 3 x 3 (A, B)
// window), and puts W9 into LDS. After one barrier it reads the W9 of its two phi neighbours,
// P3 = the maximum of the three phi cells' W9, and tests row a-1: the own slab's parts come from
// registers, theta cell t - 1 gives P3(t - 1) (before), t + 1 gives P3(t + 1) (after), and the
// two phi neighbours in theta cell t join the before- or after-neighbours by their index (phi
// wraps: phi cell 0's left neighbour is the last one, an after-neighbour; the last one's right
// neighbour is phi cell 0, a before-neighbour). With phi sectors there are no phi neighbours,
// no LDS exchange and no barrier.
//
// Rows are read with buffer loads, one resource per row spanning that row of every theta cell's
// slab: a lane whose cell lies outside the row, or a row outside the segment's rows
// a_beg - 1 .. a_end (or outside the matrix), reads zero without touching memory. Each row is
// loaded kStAhead rows before its step into a ring of kStAhead + 1 register slots; the step loop
// is unrolled by kStUnroll, a multiple of the ring slots, of the three rows of R3 history and of
// the two LDS buffers, so all of them are fixed registers and offsets. The test of a row is a
// ballot; its bits 1..62 are the chunk's peak bits, one 64-bit peak word per (slab, row, chunk),
// staged in LDS and stored once per segment. The words are counted when they are stored, and each
// wave adds one count per group of tiles its words fall in (a segmented scan over its lanes): a
// count kept per row in scalar registers cost 35 scalar registers and about a tenth of the
// kernel's time.
// ---------------------------------------------------------------------------------------------
constexpr int kStAhead = 3;
constexpr int kStSlots = kStAhead + 1;
constexpr int kStUnroll = 12;
static_assert(kStUnroll % kStSlots == 0 && kStUnroll % 3 == 0, "ring slots, R3 history and LDS buffers must align");
// the fourth word of a buffer resource on gfx9-family parts: 32-bit data format, no swizzle
constexpr int kRsrcWord3 = 0x00020000;
constexpr uint64_t kTestedLanes = 0x7ffffffffffffffeull;  // lanes 1..62
constexpr uint32_t kStOutside = 0x80000000u;                // a load offset past every resource
constexpr int kStWholeRows = 48;  // segments up to this many rows keep all their peak words in LDS

// Inclusive maximum over a wave64, with the DPP steps of the inclusive sum (a lane whose source
// lies outside its row takes the maximum with 0). Every lane of the wave must be active.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v)
{
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v)
{
  v = dpp_max<0x111, 0xf>(v);
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);
  v = dpp_max<0x143, 0xc>(v);
  return v;
}

// Adds the peaks of one 64-bit peak word per lane to the peak counts of their groups of tiles.
// The words a wave holds are in (theta cell, row) order, so the lanes of one group form one run:
// a scan of the counts and a maximum-scan of the runs' starting sums give each run's total, which
// its last lane adds with one atomic. A lane with valid false (no word, or a row past the
// matrix) adds nothing and splits runs. Every lane of the wave must be active.
__device__ __forceinline__ void add_group_counts(uint32_t* group_pk, bool valid, uint32_t grp, uint64_t word)
{
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t gv = valid ? grp : 0xffffffffu;  // group numbers are below 2^31
  const uint32_t c = valid ? (uint32_t)__builtin_popcountll(word) : 0u;
  const uint32_t incl = wave_incl_scan(c);
  // the neighbours' groups are read by every lane (no short-circuit: a DPP read of a lane that
  // is switched off returns 0)
  const uint32_t gl = lane_left(gv), gr = lane_right(gv);
  const bool start = (lane == 0u) | (gl != gv);
  const bool last = (lane == 63u) | (gr != gv);
  const uint32_t run0 = wave_incl_max(start ? incl - c : 0u);
  if (valid && last && incl != run0) gatomic_add(group_pk + grp, incl - run0);
}

template <int NT, bool SECT>
__global__ __launch_bounds__(1024) void k_peak_stencil(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  // two buffers of W9, each [theta cell][16 phi slots][64 lanes]: fixed strides, so every LDS
  // address is one of three lane addresses plus a constant
  extern __shared__ uint32_t s_w9[];
  constexpr uint32_t kTBytes = 16u * 256u, kBufBytes = NT * kTBytes;
  EvDesc e = load_ev(ev0, evs);
  if (!e.dense) return;  // uniform: this event's peaks come from the fill's survivors
  const uint32_t nb = (uint32_t)g.n_b;
  const int na = g.n_a, np = g.n_phi, S = g.dense_rows;
  const uint32_t lane = threadIdx.x & 63u;
  const int p = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nch = (int)((nb + kChunkCells - 1) / kChunkCells);
  // Workgroups are dealt to the eight XCDs in turn; renumbered so that each XCD takes one
  // contiguous range (adjacent chunks of the same rows, then the next rows), the cache lines that
  // neighbouring workgroups share (chunk edges overlap by two cells, segment edges by two rows)
  // are fetched into one L2. The row bounds are uniform (read from the first lane), so the row
  // loop and its tests stay scalar.
  const uint32_t lb = xcd_contiguous(blockIdx.x, gridDim.x);
  const int chunk = __builtin_amdgcn_readfirstlane((int)lb % nch);
  const int a_beg = __builtin_amdgcn_readfirstlane(((int)lb / nch) * S);
  const int a_end = min(a_beg + S, na);
  const uint32_t base = (uint32_t)chunk * kChunkCells;
  const uint32_t row_bytes = nb * 4u;
  // The next row to load (row a_beg - 1 first), as a byte address in slab (0, p). One buffer
  // resource per row covers the NT rows of slabs (0..NT-1, p), theta cell t's row t t_bytes
  // further (a scalar offset). A lane's offset is its cell's, or kStOutside for cells outside the
  // row (the cell left of B = 0, cells past n_b), which the range check turns into zeros (with
  // or without the scalar offset counted in it: kStOutside is past the resource either way), as
  // it does every load of a row outside the segment's rows a_beg - 1 .. a_end or the matrix (an
  // empty resource). The address is never dereferenced outside the rows read.
  const uintptr_t slab_bytes = (uintptr_t)na * row_bytes;
  const uint32_t t_bytes = (uint32_t)((uintptr_t)np * slab_bytes);  // (NT-1) t_bytes + row_bytes < 2^31
  const uint32_t span = (uint32_t)(NT - 1) * t_bytes + row_bytes;
  const bool cell_in = !(base == 0u && lane == 0u) && base + lane - 1u < nb;
  const uint32_t off = cell_in ? (base + lane - 1u) * 4u : kStOutside;
  uintptr_t rp = (uintptr_t)e.acc + (uintptr_t)p * slab_bytes + (uintptr_t)a_beg * row_bytes - row_bytes;
  int ra = a_beg - 1;  // the row of the next load
  const uint32_t own_a = (uint32_t)p * 256u + 4u * lane;
  const uint32_t pm_a = (uint32_t)(p == 0 ? np - 1 : p - 1) * 256u + 4u * lane;
  const uint32_t pq_a = (uint32_t)(p + 1 == np ? 0 : p + 1) * 256u + 4u * lane;
  const bool p_mid = p > 0 && p + 1 < np;  // phi neighbours: one before, one after
  const uint32_t T = g.threshold;
  const uint32_t rows_log2 = (uint32_t)__ffs(g.rows) - 1u;
  const uint32_t gt_log2 = (uint32_t)__ffs(g.group_tiles) - 1u;
  // The peak word of (slab sl, row a = seg S + r, chunk c) is at ((sl n_seg + seg) nch + c) S + r:
  // a wave's words of one theta cell form one contiguous run of S words, and the words of a
  // group of tiles (rows of one or two slabs) lie close together for the writer. A wave's words
  // wait in its own LDS staging slots, [row][theta cell] after the W9 buffers: for the whole
  // segment when it has at most kStWholeRows rows (the default), and go out at the end; else for
  // a block of kStUnroll rows, and go out after each block. Stores of peak words are slow to
  // complete, and every one is waited for with the loads of the rows that follow it, so a wave
  // stores as few times as it can.
  // (the word's position, computed where the words are stored: kept out of the step loop's
  // scalar registers)
#define HT_ST_MW()                                                                             \
  const uint32_t n_seg_ = ((uint32_t)na + (uint32_t)S - 1u) / (uint32_t)S;                     \
  GLOBAL uint64_t* const mw = reinterpret_cast<GLOBAL uint64_t*>(gp(e.pk_mask)) +              \
      (((size_t)p * n_seg_ + (size_t)(lb / (uint32_t)nch)) * (size_t)nch + (size_t)chunk) * (size_t)S; \
  const uint32_t mt_words = (uint32_t)np * n_seg_ * (uint32_t)nch * (uint32_t)S  /* t to t + 1 */
  constexpr uint32_t kStageStep = NT * 8u;  // bytes per row in a wave's slots
  const bool whole = S <= kStWholeRows;     // uniform
  const uint32_t slot_rows = whole ? (uint32_t)S : (uint32_t)kStUnroll;
  char* const stage_w = reinterpret_cast<char*>(s_w9) + (SECT ? 0u : 2u * kBufBytes) +
                        (uint32_t)p * slot_rows * kStageStep;
  // slot (row u, t) is at stage_w + 8 (u NT + t): written by lane 0, read back by the flush
  char* stage_blk = stage_w;  // lane 0's slots of the block's first row
  // group of tiles of theta cell t's row a (a below n_a)
  auto group_of = [&](uint32_t t, uint32_t a) {
    return ((t * (uint32_t)np + (uint32_t)p) * (uint32_t)g.tiles_per_slab + (a >> rows_log2)) >> gt_log2;
  };
  uint32_t ring[kStSlots][NT], hist[3][NT];

  // The next row (rows outside [a_beg - 1, a_end] or the matrix read zeros) into ring slot
  // slot_ (a constant).
#define HT_ST_LOAD(slot_)                                                                      \
  do {                                                                                         \
    const int nr_ = (ra >= 0 && ra <= a_end && ra < na) ? (int)span : 0;                      \
    const __amdgpu_buffer_rsrc_t r_ = __builtin_amdgcn_make_buffer_rsrc((void*)rp, 0, nr_, kRsrcWord3); \
    _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_)                                          \
      ring[slot_][t_] = __builtin_amdgcn_raw_buffer_load_b32(r_, off, (uint32_t)t_ * t_bytes, 0); \
    rp += row_bytes;                                                                           \
    ++ra;                                                                                      \
  } while (0)
  // R3 of step kc_'s row (kc_ a constant congruent to the step modulo kStUnroll) into history
  // slot kc_ % 3
#define HT_ST_R3(kc_)                                                                          \
  do {                                                                                         \
    _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_) {                                        \
      const uint32_t v_ = ring[(kc_) % kStSlots][t_];                                          \
      hist[(kc_) % 3][t_] = max(max(lane_left(v_), v_), lane_right(v_));                       \
    }                                                                                          \
  } while (0)
  // The test of the row in ring slot vs_ (R3 above in h0_, below in h2_) for every theta cell.
  // Its phi neighbours in the own theta cell join the before- or after-neighbours by the wave's
  // class c_ (a constant; uniform per wave): 0 phi cells 1 .. n_phi - 2 (phi - 1 before, phi + 1
  // after; also sectors, which have none), 1 phi cell 0 (both after: phi - 1 wraps to the last),
  // 2 the last phi cell (both before: phi + 1 wraps to 0).
#define HT_ST_TEST(c_)                                                                         \
  do {                                                                                         \
    _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_) {                                        \
      const uint32_t vm_ = ring[vs_][t_];                                                      \
      uint32_t mb_ = max(lane_left(vm_), hist[h0_][t_]);                                       \
      uint32_t ma_ = max(lane_right(vm_), hist[h2_][t_]);                                      \
      const uint32_t pb_ = t_ > 0 ? p3_[t_ > 0 ? t_ - 1 : 0] : 0u;                             \
      const uint32_t pa_ = t_ + 1 < NT ? p3_[t_ + 1 < NT ? t_ + 1 : 0] : 0u;                   \
      if (SECT) {                                                                              \
        mb_ = max(mb_, pb_);                                                                   \
        ma_ = max(ma_, pa_);                                                                   \
      } else if ((c_) == 0) {                                                                  \
        mb_ = max3u(mb_, pb_, wm_[t_]);                                                        \
        ma_ = max3u(ma_, pa_, wq_[t_]);                                                        \
      } else if ((c_) == 1) {                                                                  \
        mb_ = max(mb_, pb_);                                                                   \
        ma_ = max3u(ma_, pa_, max(wm_[t_], wq_[t_]));                                          \
      } else {                                                                                 \
        mb_ = max3u(mb_, pb_, max(wm_[t_], wq_[t_]));                                          \
        ma_ = max(ma_, pa_);                                                                   \
      }                                                                                        \
      pk_[t_] = __builtin_amdgcn_ballot_w64(vm_ >= max3u(mb_ + 1u, ma_, T)) & kTestedLanes;   \
    }                                                                                          \
  } while (0)
  // Step kb_ + kc_ (kc_ >= 2 a constant, kb_ a multiple of kStUnroll): R3 of its row completes W9
  // of the row before; W9 goes to LDS buffer kc_ % 2, and after one barrier the phi neighbours'
  // are read and the row before is tested; then the row kStAhead steps on is loaded into the
  // slot of that tested row.
#define HT_ST_STEP(kc_, kb_)                                                                   \
  do {                                                                                         \
    HT_ST_R3(kc_);                                                                             \
    constexpr int h0_ = ((kc_) + 1) % 3, h1_ = ((kc_) + 2) % 3, h2_ = (kc_) % 3;               \
    constexpr int vs_ = ((kc_) + kStSlots - 1) % kStSlots;                                     \
    uint32_t w9_[NT], p3_[NT], wm_[NT], wq_[NT];                                               \
    _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_)                                          \
      w9_[t_] = max3u(hist[h0_][t_], hist[h1_][t_], hist[h2_][t_]);                            \
    if (!SECT) {                                                                               \
      char* B_ = reinterpret_cast<char*>(s_w9) + ((kc_) % 2) * kBufBytes;                      \
      _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_)                                        \
        *reinterpret_cast<uint32_t*>(B_ + t_ * kTBytes + own_a) = w9_[t_];                     \
      lds_barrier();                                                                           \
      _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_) {                                      \
        wm_[t_] = *reinterpret_cast<const uint32_t*>(B_ + t_ * kTBytes + pm_a);                \
        wq_[t_] = *reinterpret_cast<const uint32_t*>(B_ + t_ * kTBytes + pq_a);                \
        p3_[t_] = max3u(wm_[t_], w9_[t_], wq_[t_]);                                            \
      }                                                                                        \
    } else {                                                                                   \
      _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_) p3_[t_] = wm_[t_] = wq_[t_] = w9_[t_]; \
    }                                                                                          \
    uint64_t pk_[NT];                                                                          \
    if (SECT || p_mid) HT_ST_TEST(0);                                                          \
    else if (p == 0) HT_ST_TEST(1);                                                            \
    else HT_ST_TEST(2);                                                                        \
    if (lane == 0u) { /* lane 0 puts the words into the wave's staging slots */               \
      _Pragma("unroll") for (int t_ = 0; t_ < NT; ++t_)                                        \
        *reinterpret_cast<uint64_t*>(stage_blk + ((kc_) - 2) * kStageStep + 8 * t_) = pk_[t_]; \
    }                                                                                          \
    HT_ST_LOAD(vs_);                                                                           \
  } while (0)

  // steps 0 and 1 (rows a_beg - 1 and a_beg) only start the R3 history
#pragma unroll
  for (int k = 0; k < kStAhead; ++k) HT_ST_LOAD(k);
  HT_ST_R3(0);
  HT_ST_LOAD(kStAhead % kStSlots);
  HT_ST_R3(1);
  HT_ST_LOAD((1 + kStAhead) % kStSlots);
  // steps 2 .. S + 1 test rows a_beg .. a_beg + S - 1 (S is a multiple of kStUnroll)
  for (int kb = 0; kb < S; kb += kStUnroll) {  // uniform
    HT_ST_STEP(2, kb);
    HT_ST_STEP(3, kb);
    HT_ST_STEP(4, kb);
    HT_ST_STEP(5, kb);
    HT_ST_STEP(6, kb);
    HT_ST_STEP(7, kb);
    HT_ST_STEP(8, kb);
    HT_ST_STEP(9, kb);
    HT_ST_STEP(10, kb);
    HT_ST_STEP(11, kb);
    HT_ST_STEP(12, kb);
    HT_ST_STEP(13, kb);
    if (whole) {  // uniform
      stage_blk += kStUnroll * kStageStep;
    } else {
      // the block's words leave the staging slots: lane t kStUnroll + u stores theta cell t's
      // word of the block's u-th row (runs of kStUnroll words). Lane 0 wrote the slots: the
      // fence keeps these reads after its writes (with phi sectors no barrier orders them).
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      HT_ST_MW();
      const bool in = lane < (uint32_t)(kStUnroll * NT);
      const uint32_t t = in ? lane / kStUnroll : 0u, u = in ? lane - t * kStUnroll : 0u;
      const uint64_t w = *reinterpret_cast<const uint64_t*>(stage_w + 8u * (u * NT + t));
      if (in) mw[(size_t)t * mt_words + (size_t)kb + u] = w;
      const uint32_t a = (uint32_t)(a_beg + kb) + u;
      add_group_counts(e.group_pk, in && a < (uint32_t)na, group_of(t, a), w);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    }
  }
  if (whole) {  // uniform: the segment's words, a run of S per theta cell
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    HT_ST_MW();
    const uint32_t n_w = (uint32_t)S * NT;
    for (uint32_t j0 = 0; j0 < n_w; j0 += 64u) {  // uniform: every lane counts
      const uint32_t j = j0 + lane;
      const bool in = j < n_w;
      const uint32_t t = in ? j / (uint32_t)S : 0u, r = in ? j - t * (uint32_t)S : 0u;
      const uint64_t w = *reinterpret_cast<const uint64_t*>(stage_w + 8u * (r * NT + t));
      if (in) mw[(size_t)t * mt_words + r] = w;
      const uint32_t a = (uint32_t)a_beg + r;
      add_group_counts(e.group_pk, in && a < (uint32_t)na, group_of(t, a), w);
    }
  }
#undef HT_ST_STEP
#undef HT_ST_TEST
#undef HT_ST_MW
#undef HT_ST_R3
#undef HT_ST_LOAD
}

// Ordered output of a dense event: one workgroup per group of tiles (a contiguous range of rows
// of the matrix, so of peak-mask words); its output offset is the sum of the earlier groups'
// peak counts. Thread t takes the t-th of 256 equal, contiguous pieces of the group's words, all
// loaded at once; one block scan of the pieces' peak counts gives each thread where its peaks
// go, in cell order (words in row, then chunk order; bits 1..62 of a word are the chunk's cells
// in B order).
__global__ __launch_bounds__(kBlock) void k_peak_write_dense(DevGrid g, EvDesc ev0, const EvDesc* evs,
                                                               uint32_t stage_cap)
{
  __shared__ uint32_t smem[32];
  __shared__ uint32_t s_cells[kWriteStage];
  EvDesc e = load_ev(ev0, evs);
  if (!e.dense) return;
  const int G = blockIdx.x;
  const int t0 = G * g.group_tiles;
  const int nt = min(g.group_tiles, g.n_tiles - t0);
  const bool a8 = ((uintptr_t)e.out & 7u) == 0;
  uint32_t c_beg, L0, c_last, L1;
  tile_range(g, t0, &c_beg, &L0);
  tile_range(g, t0 + nt - 1, &c_last, &L1);
  const uint32_t nb = (uint32_t)g.n_b, nch = (nb + kChunkCells - 1) / kChunkCells;
  // The group's rows [c_beg / nb, (c_last + L1) / nb) of the slab-major row order, so its words
  // in cell order ("logical" words w = (slab n_a + a) nch + chunk). The stencil stored the word
  // of (slab sl, row a = seg S + r, chunk c) at ((sl n_seg + seg) nch + c) S + r; a thread walks
  // its logical words with that position kept up to date.
  const uint32_t w0 = (c_beg / nb) * nch, w1 = (uint32_t)(((uint64_t)c_last + L1) / nb) * nch;
  const uint32_t per = (w1 - w0 + kBlock - 1) / kBlock;
  const uint32_t lo = min(w1, w0 + per * threadIdx.x), hi = min(w1, lo + per);
  const GLOBAL uint64_t* mw = reinterpret_cast<const GLOBAL uint64_t*>(gp((const uint8_t*)e.pk_mask));
  const uint32_t na = (uint32_t)g.n_a, S = (uint32_t)g.dense_rows;
  const uint32_t n_seg = (na + S - 1u) / S;
  uint32_t ch = lo % nch, a = (lo / nch) % na, sl = lo / nch / na;
  uint32_t seg = a / S, r = a - seg * S;
  auto rewind = [&]() {
    ch = lo % nch;
    a = (lo / nch) % na;
    sl = lo / nch / na;
    seg = a / S;
    r = a - seg * S;
  };
  auto phys = [&]() { return ((sl * n_seg + seg) * nch + ch) * S + r; };
  auto next = [&]() {
    if (++ch == nch) {
      ch = 0;
      if (++r == S) {
        r = 0;
        ++seg;
      }
      if (++a == na) {
        a = 0;
        seg = 0;
        r = 0;
        ++sl;
      }
    }
  };
  constexpr int kMaxW = 16;  // up to 16 words per thread held in registers
  uint64_t wv[kMaxW];
  uint32_t cnt = 0;
  const int nw = (int)(hi - lo);
  if (per <= (uint32_t)kMaxW) {  // uniform
#pragma unroll
    for (int k = 0; k < kMaxW; ++k) {
      wv[k] = k < nw ? mw[phys()] : 0ull;
      next();
    }
  }
  // the earlier groups' peak counts give the output offset (loaded while the words arrive)
  uint32_t part = 0;
  for (int i0 = 0; i0 < G; i0 += 4 * kBlock) {  // uniform
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = i0 + k * kBlock + (int)threadIdx.x;
      w[k] = i < G ? gp(e.group_pk)[i] : 0u;
    }
    part += w[0] + w[1] + w[2] + w[3];
  }
  const int64_t base = (int64_t)block_sum(part, smem);
  if (G == (int)gridDim.x - 1 && threadIdx.x == 0) *gp(e.n_found) = base + gp(e.group_pk)[G];
  if (base >= e.cap) return;  // uniform
  if (per <= (uint32_t)kMaxW) {  // uniform
#pragma unroll
    for (int k = 0; k < kMaxW; ++k) cnt += (uint32_t)__builtin_popcountll(wv[k]);
  } else {
    for (uint32_t w = lo; w < hi; ++w) {
      cnt += (uint32_t)__builtin_popcountll(mw[phys()]);
      next();
    }
  }
  uint32_t tot;
  const uint32_t lo_pk = block_excl_scan(cnt, smem, &tot);  // the thread's first peak in the group
  // Cell of bit j of word w: row w / nch, chunk w % nch, B = chunk * kChunkCells + j - 1. A group
  // of at most kWriteStage peaks (the common case) first lists its cells in LDS, in order; then
  // every thread loads the votes of every 256th of them at once and stores those peaks, so the
  // group's vote loads take one round trip whichever threads own the crowded words, and the
  // stores are contiguous. A larger group emits each thread's peaks itself, loading the votes of
  // up to four at a time.
#define HT_FOR_PEAKS(w_, bits_, body_)                                                         \
  do {                                                                                         \
    uint64_t b_ = (bits_);                                                                     \
    if (b_) {                                                                                  \
      const uint32_t row_ = (w_) / nch;                                                        \
      const uint32_t c0_ = row_ * nb + ((w_) - row_ * nch) * kChunkCells - 1u;                 \
      while (b_) {                                                                             \
        const uint32_t c_ = c0_ + (uint32_t)__builtin_ctzll(b_);                               \
        b_ &= b_ - 1ull;                                                                       \
        body_;                                                                                 \
      }                                                                                        \
    }                                                                                          \
  } while (0)
  if (tot <= stage_cap) {  // uniform (stage_cap <= kWriteStage)
    uint32_t i = lo_pk;
    if (per <= (uint32_t)kMaxW) {  // uniform
#pragma unroll
      for (int k = 0; k < kMaxW; ++k) HT_FOR_PEAKS(lo + (uint32_t)k, wv[k], s_cells[i++] = c_);
    } else {
      rewind();
      for (uint32_t w = lo; w < hi; ++w) {
        HT_FOR_PEAKS(w, mw[phys()], s_cells[i++] = c_);
        next();
      }
    }
    lds_barrier();
    constexpr int kRounds = kWriteStage / kBlock;
    uint32_t c[kRounds], v[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint32_t k = (uint32_t)r * kBlock + threadIdx.x;
      c[r] = s_cells[k < tot ? k : 0u];
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
      if ((uint32_t)r * kBlock < tot) v[r] = gp(e.acc)[c[r]];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint32_t k = (uint32_t)r * kBlock + threadIdx.x;
      if (k < tot && base + (int64_t)k < e.cap) st_peak(e.out, base + (int64_t)k, c[r], v[r], a8);
    }
    return;
  }
  int64_t o = base + (int64_t)lo_pk;
  if (o >= e.cap || cnt == 0) return;
#define HT_EMIT_WORD(w_, bits_)                                                                \
  do {                                                                                         \
    uint64_t b_ = (bits_);                                                                     \
    if (b_) {                                                                                  \
      const uint32_t row_ = (w_) / nch;                                                        \
      const uint32_t c0_ = row_ * nb + ((w_) - row_ * nch) * kChunkCells - 1u;                 \
      while (b_) {                                                                             \
        uint32_t c_[4], v_[4];                                                                 \
        int n_ = 0;                                                                            \
        _Pragma("unroll") for (int q_ = 0; q_ < 4; ++q_) {                                     \
          c_[q_] = c0_ + (b_ ? (uint32_t)__builtin_ctzll(b_) : 1u);                            \
          n_ += b_ ? 1 : 0;                                                                    \
          b_ &= b_ - 1ull;                                                                     \
        }                                                                                      \
        _Pragma("unroll") for (int q_ = 0; q_ < 4; ++q_) v_[q_] = gp(e.acc)[c_[q_]];          \
        _Pragma("unroll") for (int q_ = 0; q_ < 4; ++q_) {                                     \
          if (q_ < n_ && o < e.cap) st_peak(e.out, o, c_[q_], v_[q_], a8);                     \
          o += q_ < n_ ? 1 : 0;                                                                \
        }                                                                                      \
      }                                                                                        \
    }                                                                                          \
  } while (0)
  if (per <= (uint32_t)kMaxW) {  // uniform
#pragma unroll
    for (int k = 0; k < kMaxW; ++k) HT_EMIT_WORD(lo + (uint32_t)k, wv[k]);
  } else {
    rewind();
    for (uint32_t w = lo; w < hi; ++w) {
      HT_EMIT_WORD(w, mw[phys()]);
      next();
    }
  }
#undef HT_EMIT_WORD
#undef HT_FOR_PEAKS
}

// ---------------------------------------------------------------------------------------------
// Plain fill: zero the matrix, then one global atomicAdd per vote. One block per hit, its
// threads over the A bins (the decomposition the paper describes, kept as a baseline).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_zero_acc(DevGrid g, EvDesc ev0, const EvDesc* evs,
                                                     uint64_t cells)
{
  EvDesc e = load_ev(ev0, evs);
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < cells; i += stride)
    e.acc[i] = 0u;
}

__global__ __launch_bounds__(kBlock) void k_fill_atomic(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  EvDesc e = load_ev(ev0, evs);
  const int64_t h = blockIdx.x;
  if (h >= e.n_hits) return;
  int slabs[4];
  int ns = 0;
  for (int q = 0; q < 4; ++q) {
    int s = e.hit_slab[4 * h + q];
    if (s >= 0) slabs[ns++] = s;
  }
  if (ns == 0) return;
  const float4 rec = e.hit_rec[h];
  const float x = rec.x, r2 = rec.y, k = rec.z;
  for (int i = threadIdx.x; i < g.n_a; i += kBlock) {
    float ax = g.a2[i] * x;
    float num = r2 - ax;
    float B = num * k;
    float d = B - g.b_min;
    float f = d * g.inv_db;
    if (f >= 0.0f && f < g.nb_f) {
      const uint32_t j = (uint32_t)(int)f;
      for (int q = 0; q < ns; ++q)
        atomicAdd(&e.acc[((uint64_t)slabs[q] * g.n_a + i) * g.n_b + j], 1u);
    }
  }
}

// Track parameters of each peak: bin indices, bin-centre (A, B), rho, phi, theta in double.
__global__ __launch_bounds__(kBlock) void k_readout(DevGrid g, const ht_peak* peaks, const int64_t* n_found,
                                                    int64_t cap, ht_track* tracks, double b_min,
                                                    double db)
{
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t n = min(*n_found, cap);
  if (i >= n) return;
  const ht_peak pk = peaks[i];
  uint32_t t, p, a, b;
  cell_coords(g, pk.cell, &t, &p, &a, &b);
  const double A = 0.5 * (double)g.a2[a];
  const double B = b_min + ((double)b + 0.5) * db;
  double phi = atan2(B, A);
  if (phi < 0.0) phi += 2.0 * 3.14159265358979323846;
  ht_track tr;
  tr.cell = pk.cell;
  tr.votes = pk.votes;
  tr.t = (int32_t)t;
  tr.p = (int32_t)p;
  tr.a = (int32_t)a;
  tr.b = (int32_t)b;
  tr.A = (float)A;
  tr.B = (float)B;
  tr.rho = (float)sqrt(A * A + B * B);
  tr.phi = (float)phi;
  tr.theta = (float)(((double)t + 0.5) * 3.14159265358979323846 / (double)g.n_theta);
  tracks[i] = tr;
}

__global__ __launch_bounds__(kBlock) void k_debug_hits(DevGrid g, const float* x, const float* y,
                                                       const float* z, int64_t n, int32_t* info,
                                                       float* vals, int32_t* slabs)
{
  const int64_t h = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (h >= n) return;
  HitPrep p = prep_hit(g, g.phi_cs, g.th_cs, x[h], y[h], z[h]);
  info[4 * h + 0] = p.n > 0;
  info[4 * h + 1] = p.s_theta;
  info[4 * h + 2] = p.s_phi;
  info[4 * h + 3] = p.n;
  vals[3 * h + 0] = p.r2;
  vals[3 * h + 1] = p.r;
  vals[3 * h + 2] = p.k;
  for (int q = 0; q < 4; ++q) slabs[4 * h + q] = q < p.n ? p.slab[q] : -1;
}

__global__ __launch_bounds__(kBlock) void k_debug_unary(const float* v, float* root, float* inv2,
                                                        int64_t n)
{
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
    const float a = v[i];
    root[i] = hit_root(a);
    inv2[i] = hit_inv2(a);
  }
}
hipError_t launch_fill_nt(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, bool nt,
                          bool vec, bool emit, bool long_lists, size_t lds, hipStream_t s)
{
  switch (g.rows) {
    case 1: return launch_fill_for_rows<1>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    case 2: return launch_fill_for_rows<2>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    case 4: return launch_fill_for_rows<4>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    case 8: return launch_fill_for_rows<8>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    case 16: return launch_fill_for_rows<16>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    case 32: return launch_fill_for_rows<32>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    case 64: return launch_fill_for_rows<64>(g, ev0, evs, n_ev, nt, vec, emit, long_lists, lds, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int n_groups(const DevGrid& g) { return (g.n_tiles + g.group_tiles - 1) / g.group_tiles; }

size_t fill_lds_bytes(const DevGrid& g, bool long_l)
{
  return (size_t)g.rows * ((((size_t)g.n_b + 3) & ~(size_t)3) + (long_l ? kSpill : 0)) * sizeof(uint32_t);
}

hipError_t launch_fetch(EvDesc* evs, const EvDesc* host, int n_ev, hipStream_t s)
{
  static_assert(sizeof(EvDesc) % sizeof(u32x2) == 0 && alignof(EvDesc) == alignof(u32x2), "whole 8-byte words");
  const uint32_t n = (uint32_t)n_ev * (uint32_t)(sizeof(EvDesc) / sizeof(u32x2));
  hipLaunchKernelGGL(k_fetch, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, (u32x2*)evs, (const u32x2*)host, n);
  return hipGetLastError();
}

hipError_t launch_prep(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                       int64_t max_hits, bool direct, hipStream_t s)
{
  const unsigned blocks = (unsigned)std::max<int64_t>(1, (max_hits + kBlock - 1) / kBlock);
  // the boundary tables: 4 n_phi + 2 (2 n_theta + 1) floats (about 300 B for the paper grid)
  const size_t tab = (size_t)(4 * g.n_phi + 2 * (2 * g.n_theta + 1)) * sizeof(float);
  const bool lds = tab <= kLdsTableBytes;
  if (direct) {
    if (lds) hipLaunchKernelGGL(k_prep_direct<true>, dim3(blocks, n_ev), dim3(kBlock), tab, s, g, ev0, evs);
    else hipLaunchKernelGGL(k_prep_direct<false>, dim3(blocks, n_ev), dim3(kBlock), 0, s, g, ev0, evs);
    return hipGetLastError();
  }
  if (lds) hipLaunchKernelGGL(k_prep<true>, dim3(blocks, n_ev), dim3(kBlock), tab, s, g, ev0, evs);
  else hipLaunchKernelGGL(k_prep<false>, dim3(blocks, n_ev), dim3(kBlock), 0, s, g, ev0, evs);
  hipLaunchKernelGGL(k_bucket, dim3(blocks, n_ev), dim3(kBlock), 0, s, g, ev0, evs);
  return hipGetLastError();
}

// A measure of the survivors of an event at a threshold of nine votes or so: the cube of its hits per
// (slab, B) column, times the cells.
static double survivor_measure(const DevGrid& g, int64_t hits, double* per_cell)
{
  const double ratio = 4.0 * (double)hits / ((double)g.n_slabs * g.n_b);
  *per_cell = ratio * ratio * ratio;
  return *per_cell * (double)g.n_slabs * g.n_a * g.n_b;
}

bool long_lists(const DevGrid& g, int n_ev, int64_t max_hits)
{
  // more than two records per thread of the short-list fill expected per slab (a hit has at most
  // four cells, about three on average), in tiles narrow enough for it to matter; and votes that
  // are never NaN, which the long-list fill cannot tell from bin 0
  const int64_t longest = (int64_t)2 * kBlock * g.n_slabs;
  if (g.rows > 8 || !g.finite_votes || max_hits * 3 <= longest) return false;
  if (!g.search || dense_peaks(g, max_hits)) return true;
  // Lists of up to six times that whose events leave few survivors (more at low thresholds) stay with
  // the short-list fill: it lists the survivors, and their test takes half the time of the masks'.
  // Short and long, whole calls in us: 2700 hits on 2x4x256x9000 27.8 and 34.7, 5461 (5e5) 30.9 and
  // 34.7; 2048 on 1x3x2000x5000 (5e6) 34 and 47; 2785 on sectors 4x4x1024x1024 (5e6) 29.5 and 33.8;
  // 5461 on 2x4x256x2500 (7e6) 25.4 and 26.1, 10922 (53e6, eight times as long) 31.4 and 29.0; 11141 on
  // 4x16x1024x1024 (21e6) 65 and 69, 13107 (34e6) 76 and 72; T 3, 2048 on 2x4x256x9000 (3e4) 31 and 39,
  // 5461 58 and 45; T 2, 2048 65 and 47.
  double per_cell;
  const double low = std::max(1.0, 9.0 / g.threshold);
  return max_hits * 3 > 6 * longest || survivor_measure(g, max_hits, &per_cell) * n_ev * std::pow(low, 5) > 12e6;
}

bool use_lists(const DevGrid& g, int n_ev, int64_t max_hits, int64_t hits)
{
  // The long-list fill makes none: with the code for them it spills registers (a 14142-hit event's
  // fill took 68 us, not 55, and its test 23 us, not 24).
  if (long_lists(g, n_ev, max_hits)) return false;
  // Survivors come about as the cube of the hits per (slab, B) column, times the cells: on the paper
  // grid 2.7k at 5000 hits, 46k at 14142, 661k at 40000. They must fit the lists, 65k. And where a
  // job has several, the masks' test of a cell per lane is the faster one, once the launch is more
  // than latency. Lists and masks, in us: seven events of 6585 hits on 4x16x256x256 134 and 85, two
  // of them 58 and 46, one (18e6) 34 and 31; 16 of 4000 135 and 116; 20 of 2500 on 4x16x128x128 83
  // and 64; 14 of 1139 on 4x4x130x259 (10e6) 39.5 and 43; one of 8000 on 4x16x512x512 (16e6) 39 and
  // 42; twelve of 8000 on the paper grid (0.1 per cell) 569 and 619.
  double cube;
  const double measure = survivor_measure(g, hits, &cube);
  // At a threshold of one vote most cells of a vote survive. Lists and masks, in us: 4x16x256x256, 32
  // hits (B 32768) 53 and 40, eight (8192) 25 and 28; 4x16x128x128, 32 hits (16384) 42 and 37, 250 (128000)
  // 59 and 46; 4x16x512x512, 16 hits (32768) 34 and 36, 32 hits 62 and 50.
  if (g.threshold == 1 && (double)hits * (g.phi_sectors ? 2 : 4) * g.n_a * n_ev > 30e3) return false;
  if (cube > 0.5 && measure * n_ev > 20e6) return false;
  return measure <= 48e6;
}

hipError_t launch_fill(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                       bool emit, bool long_l, hipStream_t s)
{
  // store kind 2: 4-byte stores (the dword path), otherwise 16-byte stores where rows allow
  const bool vec = (g.n_b % 4) == 0 && g.nt_store != 2;
  const size_t lds = fill_lds_bytes(g, long_l);
  return launch_fill_nt(g, ev0, evs, n_ev, g.nt_store == 1, vec, emit, long_l, lds, s);
}

// the tile and the boundary tables
static size_t tiny_lds_bytes(const DevGrid& g)
{
  return fill_lds_bytes(g, false) + (size_t)(4 * g.n_phi + 2 * (2 * g.n_theta + 1)) * sizeof(float);
}

int64_t cells_bound(const DevGrid& g, int64_t hits)
{
  // a hit votes once per A row in each of its (theta, phi) cells
  return hits * (g.phi_sectors ? 2 : 4) * g.n_a / (int64_t)g.threshold;
}

bool few_cells(const DevGrid& g, int64_t max_hits)
{
  // Of the cells that can reach the threshold far fewer do in ordinary events, unless one or two votes are enough: then most of them
  // do, more than one workgroup tests in the time of two launches. One workgroup and the general
  // search from lists, in us: T 1, 4x16x64x64, one hit (bound 256) 12 and 15, two 19 and 17, 32 (8192)
  // 59 and 18; two hits on 4x16x1024x1024 (8192) 179 and 51; T 2, 4x16x64x64, 32 hits (4096) 15 and
  // 16, 64 (8192) 28 and 17; T 3, 64 hits (5461) 15.4 and 16.6; T 4, 128 (8192) 16.5 and 17.0.
  const int64_t limit = g.threshold == 1 ? 256 : g.threshold == 2 ? kFewCells / 2 : kFewCells;
  return max_hits <= kFewHits && cells_bound(g, max_hits) <= limit;
}

bool tiny_launch(const DevGrid& g, int n_ev, int64_t max_hits)
{
  // Every workgroup prepares every hit, so the hits fit its LDS, and there are no more workgroups
  // than the chip holds at once. 250 hits on 4x16x64x64 (256 workgroups): 15.6 us a call in four
  // launches, 9.6 in two; on 256x256 planes (1024): 16.5 and 13.4; 200 on 512x512 (4096): 24.8 and
  // 33.9; batches of 16 of the first (1024) 38.0 and 36.9 us, of 32 (2048) 41.7 and 44.7, of 100
  // 60 and 84.
  if (!g.lds_fill || g.packed_lists || g.j.ch != 4 || max_hits > kTinyHits || !few_cells(g, max_hits)) return false;
  return (int64_t)g.n_tiles * n_ev <= 1024 && tiny_lds_bytes(g) + 12 * kTinyHits + 64 <= 65536;
}

hipError_t launch_tiny_fill(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, hipStream_t s)
{
  const size_t lds = tiny_lds_bytes(g);
  const dim3 grid(g.n_tiles, n_ev);
  const bool vec = g.n_b % 4 == 0 && g.nt_store != 2, nt = g.nt_store == 1;
  if (vec && nt) hipLaunchKernelGGL((k_tiny_fill<true, true>), grid, dim3(kBlock), lds, s, g, ev0, evs);
  else if (vec) hipLaunchKernelGGL((k_tiny_fill<true, false>), grid, dim3(kBlock), lds, s, g, ev0, evs);
  else if (nt) hipLaunchKernelGGL((k_tiny_fill<false, true>), grid, dim3(kBlock), lds, s, g, ev0, evs);
  else hipLaunchKernelGGL((k_tiny_fill<false, false>), grid, dim3(kBlock), lds, s, g, ev0, evs);
  return hipGetLastError();
}

hipError_t launch_few_peaks(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, hipStream_t s)
{
  if (g.n_b < 3) hipLaunchKernelGGL(k_few_peaks<true>, dim3(1, n_ev), dim3(1024), 0, s, g, ev0, evs);
  else hipLaunchKernelGGL(k_few_peaks<false>, dim3(1, n_ev), dim3(1024), 0, s, g, ev0, evs);
  return hipGetLastError();
}

hipError_t launch_scan(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, uint32_t n_grp,
                       bool counters, hipStream_t s)
{
  const uint64_t jobs = std::min<uint64_t>((uint64_t)n_grp * g.j.group_jobs, g.j.n_jobs);
  dim3 grid((unsigned)((jobs + 7) / 8), n_ev);
  const bool vec = g.n_b % 4 == 0;
  if (g.j.ch == 4 && vec) hipLaunchKernelGGL((k_scan<true, 4>), grid, dim3(kBlock), 0, s, g, ev0, evs, counters ? 1 : 0);
  else if (g.j.ch == 4) hipLaunchKernelGGL((k_scan<false, 4>), grid, dim3(kBlock), 0, s, g, ev0, evs, counters ? 1 : 0);
  else if (vec) hipLaunchKernelGGL((k_scan<true, 1>), grid, dim3(kBlock), 0, s, g, ev0, evs, counters ? 1 : 0);
  else hipLaunchKernelGGL((k_scan<false, 1>), grid, dim3(kBlock), 0, s, g, ev0, evs, counters ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_peaks(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, uint32_t n_grp,
                        hipStream_t s)
{
  // A workgroup per group, so that the hardware deals the uneven ones out as CUs come free (16384
  // groups of 8x32x2048x2048 cells, four events: 1.24 ms with 2048 workgroups each, 1.16 with all).
  // Batches of more than eight events on grids of up to 4096 groups share kTestGrid, within 5% either
  // way of a workgroup per group: thirty events of 2000 hits on the paper grid (2048 groups) 1383 us
  // and 1418 with all, nine of 10000 on 8x32x1024x1024 (4096) 1639 and 1665, 100 of 6585 on
  // 4x16x256x256 (128) 727 and 762; but 100 of 5000 on 4x16x512x512 (512) 1918 and 1837, sixteen of
  // 22000 on the paper grid 1227 and 1209. Past them all groups win where they are crowded (nine events
  // of 105600 hits on 8x32x2048x2048, 8192 groups, 9298 and 9037 us; of 20000 hits 6947 and 6991). For
  // the lists of small grids at least one per CU over all events. A multiple of the XCDs.
  const unsigned least = std::max(kTestBlocks, 256u / (unsigned)n_ev);
  const unsigned most = n_ev <= 8 || n_grp > 4096u ? 16384u : std::max(least, kTestGrid / (unsigned)n_ev);
  const dim3 tg((std::min(std::max(n_grp, least), most) + 7u) & ~7u, n_ev);
  if (g.n_b < 3) hipLaunchKernelGGL(k_peak_test<true>, tg, dim3(kBlock), 0, s, g, ev0, evs);
  else hipLaunchKernelGGL(k_peak_test<false>, tg, dim3(kBlock), 0, s, g, ev0, evs);
  const dim3 wg((n_grp + 3) / 4, n_ev);
  if (g.n_b < 3) hipLaunchKernelGGL(k_peak_write<true>, wg, dim3(kBlock), 0, s, g, ev0, evs);
  else hipLaunchKernelGGL(k_peak_write<false>, wg, dim3(kBlock), 0, s, g, ev0, evs);
  return hipGetLastError();
}

int dense_blocks(const DevGrid& g)
{
  return ((g.n_b + kChunkCells - 1) / kChunkCells) * ((g.n_a + g.dense_rows - 1) / g.dense_rows);
}

hipError_t launch_peaks_dense(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                              hipStream_t s)
{
  // one wave per phi cell; two LDS buffers of 16 phi slots of 64 window maxima per theta cell
  // (none with sectors), then every wave's staging slots for the peak words of its segment's
  // rows (or of 12 rows when the segment is longer than kStWholeRows)
  const dim3 grid(dense_blocks(g), n_ev), block(64 * g.n_phi);
  const int slot_rows = g.dense_rows <= kStWholeRows ? g.dense_rows : kStUnroll;
  const size_t lds = (g.phi_sectors ? 0 : 2 * (size_t)g.n_theta * 16 * 256) +
                     (size_t)g.n_phi * slot_rows * g.n_theta * 8;
#define HT_ST_CASE(nt_)                                                                        \
  case nt_:                                                                                    \
    if (g.phi_sectors) hipLaunchKernelGGL((k_peak_stencil<nt_, true>), grid, block, lds, s, g, ev0, evs); \
    else hipLaunchKernelGGL((k_peak_stencil<nt_, false>), grid, block, lds, s, g, ev0, evs);  \
    break
  switch (g.n_theta) {
    HT_ST_CASE(1);
    HT_ST_CASE(2);
    HT_ST_CASE(3);
    HT_ST_CASE(4);
    default: return hipErrorInvalidValue;  // the tiling offers the stencil for 1-4 theta cells only
  }
#undef HT_ST_CASE
  // HT_DENSE_STAGE (tests): stage at most that many peaks of a group in LDS, so that smaller
  // groups take the writer's other path
  uint32_t stage_cap = kWriteStage;
  if (const char* v = std::getenv("HT_DENSE_STAGE")) {
    const long c = std::strtol(v, nullptr, 10);
    if (c >= 0 && c < kWriteStage) stage_cap = (uint32_t)c;
  }
  hipLaunchKernelGGL(k_peak_write_dense, dim3(n_groups(g), n_ev), dim3(kBlock), 0, s, g, ev0, evs, stage_cap);
  return hipGetLastError();
}

hipError_t launch_fill_atomic(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                              int64_t max_hits, hipStream_t s)
{
  const uint64_t cells = (uint64_t)g.n_slabs * g.n_a * g.n_b;
  hipLaunchKernelGGL(k_zero_acc, dim3(4096, n_ev), dim3(kBlock), 0, s, g, ev0, evs, cells);
  hipLaunchKernelGGL(k_fill_atomic, dim3((unsigned)std::max<int64_t>(max_hits, 1), n_ev), dim3(kBlock), 0,
                     s, g, ev0, evs);
  return hipGetLastError();
}

hipError_t launch_readout(const DevGrid& g, const ht_peak* peaks, const int64_t* n_found, int64_t cap,
                          ht_track* tracks, double b_min, double db, hipStream_t s)
{
  if (cap > 0)
    hipLaunchKernelGGL(k_readout, dim3((unsigned)((cap + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, g,
                       peaks, n_found, cap, tracks, b_min, db);
  return hipGetLastError();
}

hipError_t launch_debug_hits(const DevGrid& g, const float* x, const float* y, const float* z,
                             int64_t n, int32_t* info, float* vals, int32_t* slabs, hipStream_t s)
{
  if (n > 0)
    hipLaunchKernelGGL(k_debug_hits, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       g, x, y, z, n, info, vals, slabs);
  return hipGetLastError();
}

hipError_t launch_debug_unary(const float* v, float* root, float* inv2, int64_t n, hipStream_t s)
{
  if (n > 0) {
    const int64_t blocks = std::min<int64_t>((n + kBlock - 1) / kBlock, 16384);
    hipLaunchKernelGGL(k_debug_unary, dim3((unsigned)blocks), dim3(kBlock), 0, s, v, root, inv2, n);
  }
  return hipGetLastError();
}

}  // namespace ht