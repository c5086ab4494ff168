// ht_device.h -- device code shared by the kernel translation units of libht.so: memory
// helpers, wave and block scans, the survivors of an LDS tile's cells, and the fill kernel
// template (its row counts are instantiated in separate translation units so that they compile
// in parallel).
//
// Every floating-point step of the bin rule is one binary32 operation, rounded to nearest even,
// in the documented order: contraction is off wherever this header is included.
#pragma once

#include "ht_internal.h"

#pragma clang fp contract(off)

namespace ht {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 256;
constexpr int kSpill = 64;  // spill words per row of a long-list fill tile

// A launch's event descriptor: the kernel argument for one event, else evs[blockIdx.y]. The
// descriptor array is read through the constant address space: both sources are then
// scalar-loaded (a generic pointer chosen between the two would make every field a vector
// memory load, one more round trip before each workgroup's first real load).
#define CONSTANT __attribute__((address_space(4)))
__device__ __forceinline__ EvDesc load_ev(const EvDesc& ev0, const EvDesc* evs)
{
#if defined(__HIP_DEVICE_COMPILE__)
  if (evs) return ((const CONSTANT EvDesc*)evs)[blockIdx.y];
#else
  if (evs) return evs[blockIdx.y];  // the host pass only parses device functions
#endif
  return ev0;
}

// ---------------------------------------------------------------------------------------------
// Memory helpers. Pointers reached through descriptors are generic to the compiler, which then
// emits FLAT instructions: those count against the LDS counter too, so every LDS wait would also
// wait for outstanding global stores, and the compiler must assume they may alias LDS. gp()
// states that a pointer is global memory (device memory or host memory mapped into the GPU's
// address space). lds_barrier() synchronises the workgroup for LDS only: no workgroup here reads
// global data written by another of its threads in the same launch, so outstanding global
// stores need not complete before a barrier.
// ---------------------------------------------------------------------------------------------
#define GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GLOBAL T* gp(T* p)
{
  return (GLOBAL T*)p;
}
template <typename T>
__device__ __forceinline__ const GLOBAL T* gp(const T* p)
{
  return (const GLOBAL T*)p;
}
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// (x, r2, k) of a record: three 4-byte loads the compiler merges into one 12-byte load (the
// unused fourth word is not loaded, so it cannot hold up a register)
__device__ __forceinline__ void ld_xyz(const float4* p, size_t i, float* x, float* r2, float* k)
{
  const GLOBAL float* q = (const GLOBAL float*)p + 4 * i;
  *x = q[0];
  *r2 = q[1];
  *k = q[2];
}
__device__ __forceinline__ void st_rec(float4* p, size_t i, float4 v)
{
  const f32x4 w = {v.x, v.y, v.z, v.w};
  ((GLOBAL f32x4*)p)[i] = w;
}
// an output peak: one 8-byte store when the caller's array is 8-byte aligned (a wave's peaks
// then go out as one contiguous run, which matters when the array is host memory mapped into
// the GPU: every store becomes a bus write), else two 4-byte stores (the array need only be
// 4-byte aligned). a8 is uniform.
__device__ __forceinline__ void st_peak(ht_peak* p, int64_t i, uint32_t cell, uint32_t votes, bool a8)
{
  if (a8) {
    const u32x2 w = {cell, votes};
    ((GLOBAL u32x2*)p)[i] = w;
    return;
  }
  GLOBAL uint32_t* q = (GLOBAL uint32_t*)p + 2 * i;
  q[0] = cell;
  q[1] = votes;
}
__device__ __forceinline__ uint32_t gatomic_add(uint32_t* p, uint32_t v)
{
  return __hip_atomic_fetch_add(gp(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void lds_barrier()
{
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------------------------
// Wave / block scans (wave64)
// ---------------------------------------------------------------------------------------------
// Inclusive scan over a wave64 with DPP moves, which stay in the VALU (no LDS round trips):
// Hillis-Steele shifts inside each row of 16 lanes, then the last lane of row 0 is added to
// row 1 and row 3, and that of row 1 (lane 31) to rows 2 and 3. A lane whose source lies
// outside its row is masked off and adds 0. Every lane of the wave must be active.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v)
{
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
  v = dpp_add<0x111, 0xf>(v);  // row_shr:1
  v = dpp_add<0x112, 0xf>(v);  // row_shr:2
  v = dpp_add<0x114, 0xf>(v);  // row_shr:4
  v = dpp_add<0x118, 0xf>(v);  // row_shr:8
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Sum over a wave64 (every lane active); the result is uniform.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v), 63);
}

// Exclusive scan over the block (blockDim a multiple of 64, at most 1024). smem: >= 17 words.
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t* smem, uint32_t* total)
{
  const int lane = __lane_id();
  const int w = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  uint32_t inc = wave_incl_scan(v);
  if (lane == 63) smem[w] = inc;
  lds_barrier();
  if (threadIdx.x < 64) {
    uint32_t s = threadIdx.x < (unsigned)nw ? smem[threadIdx.x] : 0u;
    uint32_t si = wave_incl_scan(s);
    if (threadIdx.x < (unsigned)nw) smem[threadIdx.x] = si - s;
    if (threadIdx.x == (unsigned)nw - 1) smem[16] = si;
  }
  lds_barrier();
  uint32_t res = smem[w] + inc - v;
  *total = smem[16];
  lds_barrier();
  return res;
}

__device__ uint32_t block_sum(uint32_t v, uint32_t* smem)
{
  uint32_t total;
  block_excl_scan(v, smem, &total);
  return total;
}


__device__ __forceinline__ uint32_t max3u(uint32_t a, uint32_t b, uint32_t c) { return max(a, max(b, c)); }
// lane j - 1's value (wave_shr:1; lane 0 gets 0)
__device__ __forceinline__ uint32_t lane_left(uint32_t v)
{
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);
}
// lane j + 1's value (wave_shl:1; lane 63 gets 0)
__device__ __forceinline__ uint32_t lane_right(uint32_t v)
{
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);
}

// ---------------------------------------------------------------------------------------------
// Survivors of a job (JobGeom): the cells >= T that no neighbour among the job's own cells beats
// under (votes, -index). v[q] holds the lane's four columns of row q (zeros where there is no
// cell); lmask / rmask are 0 in lanes whose left / right neighbour lane holds another row's cells.
// Neighbours outside the job are not looked at, so the test only drops cells that are no peaks:
// on a 40k-hit event it leaves 0.26 of the candidates, and the candidate test does the rest.
// Per row: R3 = the 3-maximum along B. A cell must exceed the R3 above it and its left neighbour
// (lower indices) and reach the R3 below it and its right neighbour: four VALU instructions per
// cell. A job with no cell >= T (nine in ten on an ordinary event) stops after one comparison.
// Returns the lane's mask, bit 4 q + k; every lane of the wave must be active.
// ---------------------------------------------------------------------------------------------
template <int CH>
__device__ __forceinline__ uint32_t job_survivors(const u32x4 (&v)[CH], uint32_t T, uint32_t lmask, uint32_t rmask)
{
  uint32_t mx = 0u;
#pragma unroll
  for (int q = 0; q < CH; ++q) mx = max(max3u(mx, v[q].x, v[q].y), max(v[q].z, v[q].w));
  if (__builtin_amdgcn_ballot_w64(mx >= T) == 0u) return 0u;  // uniform
  u32x4 r3[CH];
  uint32_t lf[CH], rt[CH];
#pragma unroll
  for (int q = 0; q < CH; ++q) {
    lf[q] = lane_left(v[q].w) & lmask;
    rt[q] = lane_right(v[q].x) & rmask;
    r3[q].x = max3u(lf[q], v[q].x, v[q].y);
    r3[q].y = max3u(v[q].x, v[q].y, v[q].z);
    r3[q].z = max3u(v[q].y, v[q].z, v[q].w);
    r3[q].w = max3u(v[q].z, v[q].w, rt[q]);
  }
  uint32_t m = 0u;
#pragma unroll
  for (int q = 0; q < CH; ++q) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const u32x4 up = q > 0 ? r3[q > 0 ? q - 1 : 0] : zero;
    const u32x4 dn = q + 1 < CH ? r3[q + 1 < CH ? q + 1 : 0] : zero;
    const bool k0 = (v[q].x > max(up.x, lf[q])) & (v[q].x >= max3u(dn.x, v[q].y, T));
    const bool k1 = (v[q].y > max(up.y, v[q].x)) & (v[q].y >= max3u(dn.y, v[q].z, T));
    const bool k2 = (v[q].z > max(up.z, v[q].y)) & (v[q].z >= max3u(dn.z, v[q].w, T));
    const bool k3 = (v[q].w > max(up.w, v[q].z)) & (v[q].w >= max3u(dn.w, rt[q], T));
    m |= (k0 ? 1u << (4 * q) : 0u) | (k1 ? 2u << (4 * q) : 0u) | (k2 ? 4u << (4 * q) : 0u) |
         (k3 ? 8u << (4 * q) : 0u);
  }
  return m;
}


// Stores a job's masks and its flag, if it has survivors. job: its index in the event's arrays.
template <int CH>
__device__ __forceinline__ void put_mask(const EvDesc& e, uint32_t job, uint32_t lane, uint32_t m)
{
  if (CH == 4) ((GLOBAL uint16_t*)gp(e.masks))[(size_t)job * 64u + lane] = (uint16_t)m;
  else gp(e.masks)[(size_t)job * 64u + lane] = (uint8_t)m;
  if (lane == 0u) gp(e.job_any)[job] = 1;
}

// Adds a job's survivors to one of the event's lists (cell, votes, group of jobs), one reservation
// per job. Entries past the list's end are dropped: the test then works from the masks instead.
// c0: the lane's first cell; v: its cells, as in job_survivors.
template <int CH>
__device__ __forceinline__ void list_survivors(const EvDesc& e, uint32_t job, uint32_t grp, uint32_t lane, uint32_t m,
                                               uint32_t c0, uint32_t nb, const u32x4 (&v)[CH])
{
  const uint32_t l = (job * 0x9e3779b1u) >> 29 & e.lists >> kListShift;  // neighbouring jobs' survivors cluster: spread them
  static_assert(kLists == 8, "the hash's top three bits choose the list");
  const uint32_t cap = e.lists & kListEntries;
  const uint32_t c = (uint32_t)__builtin_popcount(m), incl = wave_incl_scan(c);
  uint32_t from = 0u;
  if (lane == 63u) from = gatomic_add(e.slab_cnt + kListLens + l * kListLine, incl);
  from = (uint32_t)__builtin_amdgcn_readlane((int)from, 63);
  if (lane == 63u && from + incl > cap) gp(e.slab_cnt)[kListOver] = 1u;
  // byte offsets in vector registers, one for the next entry and one for the end: the scalar registers
  // are all taken, and spilled ones were fetched for every entry (100 paper events' fill: 4045 us with
  // a scalar end and an index, 3982 so, 4024 so with entries of 12 bytes)
  uint32_t o = (l * cap + from + incl - c) * 16u, end = (l + 1u) * cap * 16u;
  asm volatile("" : "+v"(end));
#pragma unroll
  for (int q = 0; q < CH; ++q)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (m >> (4 * q + k) & 1u) {
        const u32x4 en = {c0 + (uint32_t)q * nb + (uint32_t)k, v[q][k], grp, 0u};
        if (o < end) *(GLOBAL u32x4*)((GLOBAL char*)gp(e.surv) + o) = en;
        o += 16u;
      }
}

// floor(f) as a signed integer, saturated (v_cvt_flr_i32_f32; a NaN gives 0)
__device__ __forceinline__ int32_t floor_i32(float f)
{
#if defined(__HIP_DEVICE_COMPILE__)
  int32_t r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(f));
  return r;
#else
  return (int32_t)f;  // the host pass only parses device functions
#endif
}

typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
// A lane's unit of four columns of a row of nb cells: one 16-byte access (of 4-byte alignment
// where rows are not whole units), the row's last unit cell by cell.
template <bool NT>
__device__ __forceinline__ void st_unit(uint32_t* acc, uint32_t c, uint32_t left, u32x4 v)
{
  GLOBAL uint32_t* const d = gp(acc) + c;
  if (left >= 4u) {
    if (NT) __builtin_nontemporal_store(v, (GLOBAL u32x4_a4*)d);
    else *(GLOBAL u32x4_a4*)d = v;
    return;
  }
#pragma unroll
  for (uint32_t k = 0; k < 3; ++k)
    if (k < left) d[k] = v[k];
}

// Sweeps a filled LDS tile, each wave its jobs in turn: every job's cells are read from LDS once,
// written to the matrix, cleared, and given to on_job (job of the tile, the lane's first cell, its
// cells by row; called by every lane of the wave) to be searched for survivors in registers. No
// wave waits for another here: what bounds the fill of an ordinary event is its stores, and a
// pass that counted candidates, a barrier, a pool reservation and a second pass over the tile cost
// 9 us of 47 on the paper event.
// ldr4s: 16-byte units of an LDS row; ldr4: those of them that hold cells; sub, unit0: the lane's
// band and unit (of its strip) in a job. SPILL: words past a row's cells may hold counts.
template <int CH, bool VEC, bool NT, bool SPILL, int WAVES, typename F>
__device__ __forceinline__ void sweep_jobs(const DevGrid& g, uint32_t* acc, u32x4* s4, uint32_t ldr4s, uint32_t ldr4,
                                           uint32_t nb, uint32_t cell0, int rows, uint32_t wave, uint32_t lane,
                                           uint32_t sub, uint32_t unit0, F on_job)
{
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  uint32_t bg = 0u, st = wave;  // job = bg * strips + st
  while (st >= (uint32_t)g.j.strips) { st -= (uint32_t)g.j.strips; ++bg; }
  for (uint32_t job = wave; job < (uint32_t)g.j.tile_jobs; job += WAVES) {  // uniform
    const uint32_t u = g.j.sub > 1 ? unit0 : st * 64u + lane;
    const uint32_t r0 = (bg * (uint32_t)g.j.sub + sub) * CH;
    const bool in = u < ldr4 && sub < (uint32_t)g.j.sub;
    u32x4 v[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) v[q] = in && (int)r0 + q < rows ? s4[(r0 + q) * ldr4s + u] : zero4;
    if (SPILL && !VEC) {  // the first spill words complete a ragged row's last unit: they are no cells
      const uint32_t left = nb - 4u * u;
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        v[q].y = left > 1u ? v[q].y : 0u;
        v[q].z = left > 2u ? v[q].z : 0u;
        v[q].w = left > 3u ? v[q].w : 0u;
      }
    }
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      if (in && (int)r0 + q < rows) {
        const uint32_t c = cell0 + (r0 + q) * nb + 4u * u;
        if (VEC) {
          GLOBAL u32x4* d4 = reinterpret_cast<GLOBAL u32x4*>(gp(acc) + c);
          if (NT) __builtin_nontemporal_store(v[q], d4);
          else *d4 = v[q];
        } else {
          st_unit<NT>(acc, c, nb - 4u * u, v[q]);
        }
        s4[(r0 + q) * ldr4s + u] = zero4;
      }
    }
    on_job(job, cell0 + r0 * nb + 4u * u, v);
    st += WAVES;
    while (st >= (uint32_t)g.j.strips) { st -= (uint32_t)g.j.strips; ++bg; }
  }
}

// ---------------------------------------------------------------------------------------------
// Fill through an LDS tile of ROWS x n_b counters. The grid holds ceil(n_tiles / fill_tiles)
// workgroups; workgroup w fills tiles w, w + G, w + 2G, ... (G workgroups), so at any moment the
// workgroups write one contiguous stretch of the matrix. Per tile: the slab's record list is
// read (with direct lists the first CACHE records per thread are loaded together with the list
// length, in one memory round trip; longer lists come in further chunks of CACHE records per
// thread, each chunk's loads issued together) and the votes go to LDS. Then the waves take the
// tile's jobs in turn, with no further barrier: a wave reads its job's cells once, writes them to
// the matrix, clears them in LDS, and (EMIT) stores the survivors' masks of the peak search.
// Short lists: 256 threads, two records per thread and round trip. LONG lists: 512 threads and
// four records each, so that the 32 KiB tile, of which a CU holds four, has 32 waves to vote, not
// 16.
// ---------------------------------------------------------------------------------------------
template <int ROWS, bool VEC, bool EMIT, bool NT, bool LONG>
__global__ __launch_bounds__(LONG ? 2 * kBlock : kBlock, LONG || ROWS <= 4 ? 8 : 1) void k_fill(DevGrid g, EvDesc ev0, const EvDesc* evs)
{
  constexpr int kThreads = LONG ? 2 * kBlock : kBlock;
  constexpr int CACHE = LONG ? 4 : 2;
  extern __shared__ uint32_t smem[];
  EvDesc e = load_ev(ev0, evs);
  const uint32_t nb = (uint32_t)g.n_b;
  // row stride in LDS: whole 16-byte units where jobs read them; long lists: then kSpill words
  // that take the votes outside the row, the lane's own from word n_b + lane on
  const uint32_t ldr4 = (nb + 3u) / 4u, ldr = LONG ? 4u * ldr4 + (uint32_t)kSpill : EMIT ? 4u * ldr4 : nb;
  const uint32_t ldr4s = ldr / 4u;
  const uint32_t Lpad = ((uint32_t)ROWS * ldr + 3u) & ~3u;
  uint32_t* s_tile = smem;
  u32x4* s4 = reinterpret_cast<u32x4*>(s_tile);
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  for (uint32_t i = threadIdx.x; i < Lpad / 4; i += kThreads) s4[i] = zero4;

  const float b_min = g.b_min, inv_db = g.inv_db, nb_f = g.nb_f;
  const uint32_t spill = nb + (threadIdx.x & 63u);  // long lists
  // the wave's jobs: lane -> (band of the job, 4-column unit); wide rows: unit = 64 strip + lane
  constexpr int CH = ROWS < 4 ? ROWS : 4;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t sub = g.j.sub > 1 ? lane / ldr4 : 0u;
  const uint32_t unit0 = g.j.sub > 1 ? lane - sub * ldr4 : lane;
  const uint32_t lmask = unit0 > 0u ? ~0u : 0u;  // a strip's first lane reads 0 anyway
  const uint32_t rmask = g.j.sub > 1 && unit0 + 1u == ldr4 ? 0u : ~0u;
  // Workgroups are dealt to the eight XCDs in turn, so consecutive tiles land on different
  // XCDs and a slab's record list is fetched into every XCD's L2. Giving each XCD one
  // contiguous range of tiles instead measured 11% slower on the paper grid (eight separate
  // write streams); the plain order is kept.
  //
  // With long lists and several tiles per workgroup, a workgroup instead fills consecutive
  // tiles, the A rows of one slab in turn, and keeps the slab's records in registers from one
  // tile to the next when they all fit (no list load after the first tile).
  const bool consecutive = LONG && g.fill_tiles > 1;  // uniform
  const int t_begin = consecutive ? (int)blockIdx.x * g.fill_tiles : (int)blockIdx.x;
  const int t_end = consecutive ? min(t_begin + g.fill_tiles, g.n_tiles) : g.n_tiles;
  const int t_step = consecutive ? 1 : (int)gridDim.x;
  int held_slab = -1;  // slab whose whole record list is in registers, or -1
  size_t beg = 0;
  uint32_t n = 0;
  float cx[CACHE], cr2[CACHE], ck[CACHE];
  constexpr bool kSplit = !LONG && ROWS >= 4;  // see the votes of very short lists
  constexpr int kPart = kSplit ? ROWS / (kThreads / 64) : ROWS;
  float sx = 0.0f, sr2 = 0.0f, sk = 0.0f, sa2 = 0.0f;
  for (int tile = t_begin; tile < t_end; tile += t_step) {  // uniform
    const int slab = tile / g.tiles_per_slab;
    const int a0 = (tile - slab * g.tiles_per_slab) * ROWS;
    const int rows = min(ROWS, g.n_a - a0);
    if (!LONG || slab != held_slab) {  // the short-list variant never holds a list
      uint32_t last;  // last readable record (before n is known)
      if (e.list_cap > 0) {
        beg = (size_t)slab * (size_t)e.list_cap;
        n = gp(e.slab_cnt)[slab];
        last = (uint32_t)e.list_cap - 1u;
      } else {
        // the packed list has one record of slack past its end, so beg is always readable
        const uint32_t o = gp(e.slab_off)[slab];
        beg = o;
        n = gp(e.slab_off)[slab + 1] - o;
        last = n > 0 ? n - 1u : 0u;
      }
      // unconditional loads from clamped indices: no branch, so the values land straight in
      // the registers the votes read, and the loads overlap the list-length load
#pragma unroll
      for (int c = 0; c < CACHE; ++c)
        ld_xyz(e.list, beg + min(threadIdx.x + (uint32_t)c * (uint32_t)kThreads, last), &cx[c], &cr2[c], &ck[c]);
      if (kSplit) ld_xyz(e.list, beg + min(lane, last), &sx, &sr2, &sk);
      held_slab = (consecutive && n <= (uint32_t)(CACHE * (uint32_t)kThreads)) ? slab : -1;
    }
    // tall tiles read each row's A from the lane that holds it: 64 of them in scalar registers spill
    constexpr bool kLaneA2 = ROWS >= 16;
    if (kSplit || kLaneA2) sa2 = gp(g.a2)[min(a0 + (int)lane, g.n_a - 1)];
    constexpr int kVoteUnroll = ROWS < 8 ? ROWS : 8;
    float a2r[kLaneA2 ? 1 : ROWS];
    if (!kLaneA2) {
#pragma unroll
      for (int r = 0; r < ROWS; ++r) a2r[kLaneA2 ? 0 : r] = g.a2[min(a0 + r, g.n_a - 1)];
    }
    auto lane_a2 = [&](int row) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sa2), row)); };
    // the LDS tile is zero: set at the start, restored at the end of every tile
    lds_barrier();
    // Long lists (crowded events) vote with no branch: every row (rows past a short last tile are
    // cleared after it), and a vote outside the row goes to the spill words past it. floor(f) as a
    // signed integer, taken as unsigned and held at n_b + lane, is f's bin where 0 <= f < n_b, and
    // a spill word elsewhere: negative values floor to at least 2^31, large ones and infinities
    // saturate. (f is no NaN: launch_fill's rule and the preparation see to that. -0 floors to 0,
    // its bin.) That is eight VALU instructions per vote. Comparing bit patterns and selecting a
    // spill word past the tile took ten, and branches slowed a 40k-hit event's fill by 11%; the
    // short-list fill of the paper event is 4% faster with the branch and keeps it.
    auto vote_row = [&](int r, float a2, float x, float r2, float k) {
      if (!LONG && r >= rows) return;
      float ax = a2 * x;
      float num = r2 - ax;
      float B = num * k;
      float d = B - b_min;
      float f = d * inv_db;
      if (LONG) {
        atomicAdd(&s_tile[(uint32_t)r * ldr + min((uint32_t)floor_i32(f), spill)], 1u);
      } else if (f >= 0.0f && f < nb_f) {
        atomicAdd(&s_tile[(uint32_t)r * ldr + (uint32_t)(int)f], 1u);
      }
    };
    auto vote = [&](float x, float r2, float k) {
#pragma unroll kVoteUnroll
      for (int r = 0; r < ROWS; ++r) vote_row(r, kLaneA2 ? lane_a2(r) : a2r[kLaneA2 ? 0 : r], x, r2, k);
    };
    // Lists of at most one record per lane (small events: 13 records in a slab on average) would
    // leave all but one wave idle through ROWS dependent votes: each wave takes a quarter of the
    // rows instead, every lane the record of its lane number.
    if (kSplit && n <= 64u) {  // uniform
#pragma unroll 4
      for (int r = 0; r < kPart; ++r) {
        const int row = (int)wave * kPart + r;
        const float a2 = lane_a2(row);
        if (lane < n) vote_row(row, a2, sx, sr2, sk);
      }
    } else {
#pragma unroll
      for (int c = 0; c < CACHE; ++c)
        if (threadIdx.x + (uint32_t)c * (uint32_t)kThreads < n) vote(cx[c], cr2[c], ck[c]);
    }
    // longer lists: further chunks of CACHE records per thread, each chunk's loads issued
    // together (one round trip per chunk)
    for (uint32_t base = CACHE * (uint32_t)kThreads; base < n; base += CACHE * (uint32_t)kThreads) {  // uniform
#pragma unroll
      for (int c = 0; c < CACHE; ++c)
        ld_xyz(e.list, beg + min(base + threadIdx.x + (uint32_t)c * (uint32_t)kThreads, n - 1u), &cx[c], &cr2[c], &ck[c]);
#pragma unroll
      for (int c = 0; c < CACHE; ++c)
        if (base + threadIdx.x + (uint32_t)c * (uint32_t)kThreads < n) vote(cx[c], cr2[c], ck[c]);
    }
    lds_barrier();

    const uint32_t cell0 = ((uint32_t)slab * (uint32_t)g.n_a + (uint32_t)a0) * nb;
    if (!EMIT && !LONG) {
      // no search of the tile: one linear sweep over it
      const uint32_t L = (uint32_t)rows * nb;
      GLOBAL uint32_t* dst = gp(e.acc) + cell0;
      if (VEC) {
        GLOBAL u32x4* d4 = reinterpret_cast<GLOBAL u32x4*>(dst);
        for (uint32_t i = threadIdx.x; i < L / 4u; i += kThreads) {
          const u32x4 v = s4[i];
          if (NT) __builtin_nontemporal_store(v, d4 + i);
          else d4[i] = v;
          s4[i] = zero4;
        }
      } else {
        for (uint32_t i = threadIdx.x; i < L; i += kThreads) {
          const uint32_t v = s_tile[i];
          if (NT) __builtin_nontemporal_store(v, dst + i);
          else dst[i] = v;
          s_tile[i] = 0u;
        }
      }
      continue;
    }
    const bool emit = EMIT && !e.dense;  // uniform; a crowded event's peaks come from the stencil
    sweep_jobs<CH, VEC, NT, LONG, kThreads / 64>(g, e.acc, s4, ldr4s, ldr4, nb, cell0, rows, wave, lane, sub, unit0,
                                           [&](uint32_t job, uint32_t c0, const u32x4 (&v)[CH]) {
      if (!emit) return;
      const uint32_t m = job_survivors<CH>(v, g.threshold, lmask, rmask);
      if (__builtin_amdgcn_ballot_w64(m != 0u) == 0u) return;  // uniform
      const uint32_t id = (uint32_t)tile * (uint32_t)g.j.tile_jobs + job;
      put_mask<CH>(e, id, lane, m);
      if (!LONG && e.lists)  // uniform
        list_survivors<CH>(e, id, id / (uint32_t)g.j.group_jobs, lane, m, c0, nb, v);
    });
    if (LONG && rows < ROWS)  // uniform: the rows past a short last tile took votes
      for (uint32_t i = (uint32_t)rows * ldr4s + threadIdx.x; i < Lpad / 4u; i += kThreads) s4[i] = zero4;
    // the LDS tile is all zero again; the next tile's votes start after its first barrier
  }
}

template <int ROWS, bool NT, bool LONG>
hipError_t launch_fill_form(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                             bool vec, bool emit, size_t lds, hipStream_t s)
{
  dim3 grid((g.n_tiles + g.fill_tiles - 1) / g.fill_tiles, n_ev);  // interleaved tiles
  if (vec) {
    if (emit) hipLaunchKernelGGL((k_fill<ROWS, true, true, NT, LONG>), grid, dim3(LONG ? 2 * kBlock : kBlock), lds, s, g, ev0, evs);
    else hipLaunchKernelGGL((k_fill<ROWS, true, false, NT, LONG>), grid, dim3(LONG ? 2 * kBlock : kBlock), lds, s, g, ev0, evs);
  } else {
    if (emit) hipLaunchKernelGGL((k_fill<ROWS, false, true, NT, LONG>), grid, dim3(LONG ? 2 * kBlock : kBlock), lds, s, g, ev0, evs);
    else hipLaunchKernelGGL((k_fill<ROWS, false, false, NT, LONG>), grid, dim3(LONG ? 2 * kBlock : kBlock), lds, s, g, ev0, evs);
  }
  return hipGetLastError();
}

template <int ROWS, bool NT>
hipError_t launch_fill_rows(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                            bool vec, bool emit, bool long_lists, size_t lds, hipStream_t s)
{
  // long-list variant only where tiles are narrow enough for it to matter (rows <= 8)
  if (ROWS <= 8 && long_lists) return launch_fill_form<ROWS, NT, true>(g, ev0, evs, n_ev, vec, emit, lds, s);
  return launch_fill_form<ROWS, NT, false>(g, ev0, evs, n_ev, vec, emit, lds, s);
}
}  // namespace

// Fill launch for one A-row count per tile (ht_fill_rows.hip instantiates each).
template <int ROWS>
hipError_t launch_fill_for_rows(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, bool nt,
                                bool vec, bool emit, bool long_lists, size_t lds, hipStream_t s);

}  // namespace ht
