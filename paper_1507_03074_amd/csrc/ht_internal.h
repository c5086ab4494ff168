// ht_internal.h -- types shared by the translation units of libht.so (kernels, C ABI, server).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "ht.h"

namespace ht {

// Largest number of (theta, phi) cells (slabs); their counters live in LDS during the prep.
constexpr int kMaxSlabs = 4096;
// Per-event slab counters: a pair of arrays used alternately by successive calls. A call counts
// into the array that is zero and clears the other one for the next call, so no call needs a
// separate clearing launch. They live in memory of their own, cleared once when allocated.
// Each array holds kMaxSlabs slab counters, then the lengths of the survivor lists (from kListLens
// on) and a word that is set when a survivor did not fit its list (kListOver). An event's survivors
// (cell, votes, group of jobs) go to kLists lists of up to kListCap entries each, chosen by
// a hash of the job. One list would do but for its counter: atomic additions to one cache line take
// 10 ns each, and an event of 10k hits has 5000 jobs with survivors; the lists' lengths are a
// cache line (kListLine words) apart. An event with more survivors is tested group by group. An event
// of few cells (few_cells) has one list that holds them all.
constexpr uint32_t kLists = 8;
constexpr uint32_t kListCap = 8192;
constexpr uint32_t kListLine = 32;
constexpr uint32_t kListShift = 28;  // of EvDesc::lists
constexpr uint32_t kListEntries = (1u << kListShift) - 1u;
constexpr int kListLens = kMaxSlabs;
constexpr int kListOver = kListLens + (int)(kLists * kListLine);
constexpr int kCounterWords = kListOver + (int)kListLine;
constexpr size_t kCounterBytes = 2 * sizeof(uint32_t) * kCounterWords;
// Direct slab lists (one fixed-capacity list per slab, capacity = the event's hit count) are
// used while they need at most this many bytes per event; above it, a counting sort.
constexpr size_t kDirectListMax = (size_t)1 << 29;
// A batch uses direct lists only while the scratch of all its events stays within this.
constexpr size_t kBatchDirectMax = (size_t)8 << 30;

// Jobs of the peak search. A wave64 takes one job: `ch` consecutive A rows (a band, up to 4) of
// 4 B columns per lane, so up to 256 columns (a strip). Rows narrower than 32 units of 4 columns
// put `sub` bands one after another into one job; wider rows take `strips` jobs per band. A
// tile (tile_rows A rows of one slab) holds tile_jobs jobs, in (band, strip) order; the strips of
// one band or of `sub` bands are a job row. Each lane's survivors of a job are one mask element of
// elem_bytes bytes: bit 4 q + k is row q, column k of its cells.
struct JobGeom {
  int32_t ch, sub, strips, units;   // units: 4-column units per row
  int32_t tile_rows, tiles_per_slab, tile_jobs;
  int32_t elem_bytes;               // mask bytes per lane: 2 (ch 4) or 1
  int32_t row_jobs;                 // jobs in whose order cells are not in order: a job row, or 1
  int32_t group_jobs;               // jobs per group of the peak test (whole job rows)
  int32_t pk_step;                  // words from one group's peak count to the next
  int32_t seg;                      // peaks of a group that its segment holds (at most kSegMax)
  uint32_t n_jobs, n_groups;
};
constexpr uint32_t kSegMax = 1024;
constexpr uint32_t kSuperStep = 32;  // words: a cache line each
// Few peaks: at most this many cells can reach the threshold.
constexpr uint32_t kFewCells = 8192;
constexpr int64_t kFewHits = 65535;  // and hits
constexpr int kTinyHits = 1024;  // of an event that takes two launches (tiny_launch)

// Grid constants and tables as the kernels see them (passed by value as a kernel argument).
struct DevGrid {
  int32_t n_theta, n_phi, n_a, n_b;
  float b_min;
  float inv_db;     // (float)(n_b / (b_max - b_min))
  float nb_f;       // (float)n_b, exact because n_b <= 2^24
  uint32_t threshold;
  int32_t n_slabs;         // n_theta * n_phi: one (A, B) slab per (theta, phi) cell
  int32_t rows;            // A rows per tile; a tile is rows x n_b contiguous cells of one slab
  int32_t tiles_per_slab;  // ceil(n_a / rows)
  int32_t n_tiles;         // n_slabs * tiles_per_slab
  int32_t lds_fill;        // 1: fill through an LDS tile; 0: global atomics (very wide B rows)
  int32_t group_tiles;     // tiles per workgroup of the peak search (16, 32 or 64)
  int32_t nt_store;        // fill store kind: 0 16-byte, 1 non-temporal 16-byte, 2 4-byte
  int32_t fill_tiles;      // fill tiles per workgroup (filled in turn)
  int32_t phi_sectors;     // 1: phi cells are independent sectors (no phi widening or neighbours)
  int32_t packed_lists;    // 1: always the counting-sort (packed) slab lists, never direct ones
  int32_t search;          // 1: the launch searches the fill's survivors (0: a fill alone)
  int32_t finite_votes;    // 1: no vote of a hit with finite 1/(2y) is NaN (bounded A, finite inv_db)
  int32_t dense_w;         // 1: the stencil peak search is available on this grid (0: not)
  int32_t dense_rows;      // A rows per workgroup of the stencil peak search (a multiple of 12)
  int32_t dense_hits;      // events with at least this many hits take the stencil (0: never)
  JobGeom j;               // jobs of the survivor search (of fill tiles, or of a scanned matrix)
  const float* a2;         // device [n_a]
  const float* phi_cs;     // device [2 * 2 n_phi] (cos, sin)
  const float* th_cs;      // device [2 * (2 n_theta + 1)] (cos, sin)
};

// One event's inputs, outputs and scratch (device pointers).
struct EvDesc {
  const float* x;
  const float* y;
  const float* z;
  int64_t n_hits;
  uint32_t* acc;        // [cells]
  ht_peak* out;         // [cap]
  int64_t cap;
  int64_t* n_found;     // [1]
  // scratch
  uint32_t* slab_cnt;       // [n_slabs] counters of this call, zero on entry (kCounterBytes)
  uint32_t* slab_cnt_next;  // [n_slabs] the other counter array, cleared by this call
  int64_t list_cap;         // > 0: direct lists, list_cap records per slab; 0: counting sort
  uint32_t* slab_off;       // [n_slabs + 1] (counting sort)
  int32_t* hit_slab;    // [4 n_hits] slab of each (hit, cell) or -1
  uint32_t* hit_pos;    // [4 n_hits] position of the (hit, cell) in its slab list
  float4* hit_rec;      // [n_hits] (x, r2, k, 0)
  float4* list;         // hit records bucketed by slab: [n_slabs * list_cap] or [4 n_hits]
  // survivor search (ordinary events): the groups [grp0, grp0 + n_grp) of the event, all of them
  // except where a caller's fixed scratch holds only a slice at a time
  uint32_t grp0, n_grp;
  uint32_t* group_pk;   // peaks per group of jobs, g.j.pk_step words apart (or [groups of tiles]: stencil)
  uint32_t* super_pk;   // [n_grp / 64, rounded up] peaks per 64 groups, kSuperStep words apart
  uint8_t* job_any;     // [jobs] 1: the job has survivors (its masks are valid)
  uint8_t* masks;       // [jobs][64 lanes] mask elements; jobs without the flag are not written
  uint2* seg;           // [n_grp][g.j.seg] each group's peaks (cell, votes)
  uint4* surv;          // [lists][entries] survivors (cell, votes, group, 0) in no order
  uint32_t lists;       // their number - 1 << kListShift | entries of one; 0: none are made (crowded
                        // slabs). One word, as every scalar register counts in the fill, which
                        // stores the masks also of an event of few cells: no search reads them
  void* clear;          // what the preparation clears: super_pk, group_pk and job_any, or the
  uint32_t clear_n16;   // stencil's group_pk; in 16-byte units
  const int64_t* carry_in;  // peaks of the earlier slices, or NULL
  int64_t* carry_out;       // receives the peaks up to and with this slice, or NULL
  int32_t dense;        // 1: peaks from the stencil over the matrix (crowded events), no masks
  uint8_t* pk_mask;     // 64-bit words of peak bits of a dense event, kChunkCells cells per
                        // (slab, row, chunk) word, stored by the stencil's workgroups
};

// B columns tested per wave of the stencil peak search: a wave64 holds them and the cell on
// either side.
constexpr int kChunkCells = 62;

// Launch shape of one grid (ht_tuning resolved against the defaults).
struct Tiling {
  int32_t rows, tiles_per_slab, n_tiles, lds_fill, group_tiles, nt_store, fill_tiles;
  int32_t auto_rows, auto_nt;  // 1: not set by the caller, so each launch may take its own
  int32_t cand_cap;  // of the no-alloc call's limit only: no search keeps a candidate list
  int32_t packed_lists;
  int32_t dense_w, dense_rows;  // stencil peak search (DevGrid fields of these names)
  int32_t dense_hits;           // hits from which it is used: as reported,
  int32_t dense_from;           // and as done (DevGrid::dense_hits)
};
Tiling choose_tiling(const ht_grid& g);

// Device copies of the bin-rule tables of one grid.
struct DevTables {
  float* a2 = nullptr;
  float* phi = nullptr;
  float* th = nullptr;
  float inv_db = 0.0f;
};
// Floats of each table: a2[n_a], phi (cos, sin)[2 n_phi], theta (cos, sin)[2 n_theta + 1].
inline size_t a2_floats(const ht_grid& g) { return (size_t)g.n_a; }
inline size_t phi_floats(const ht_grid& g) { return 4 * (size_t)g.n_phi; }
inline size_t th_floats(const ht_grid& g) { return 2 * (2 * (size_t)g.n_theta + 1); }
// The tables computed on the host in double and rounded once to float, into caller arrays of
// the sizes above.
void host_tables_into(const ht_grid& g, float* a2, float* inv_db, float* phi, float* th);
// n_ev, max_hits: what the launches it is for hold; search: whether they search for peaks.
DevGrid make_devgrid(const ht_grid& g, const DevTables& t, const Tiling& tl, int n_ev, int64_t max_hits,
                     bool search = true);
// The hits from which the events of a launch of n_ev events of up to max_hits hits take the stencil
// (DevGrid::dense_hits; 0: none).
int32_t stencil_from(const Tiling& tl, int n_ev, int64_t max_hits);
// Sets g.j: the jobs of tiles of `tile_rows` rows, or with 0 those of a matrix that k_scan reads
// (bands of four rows, or of one in very wide rows). n_ev: events of the launch.
void set_jobs(DevGrid* g, int tile_rows, int n_ev);

// Whether an event of n_hits hits uses direct slab lists (see kDirectListMax).
bool direct_lists(const DevGrid& g, int64_t n_hits);
// Whether the fused fill + peaks of an event of n_hits hits searches its peaks with the stencil
// over the matrix (crowded events) instead of testing the fill's survivors.
bool dense_peaks(const DevGrid& g, int64_t n_hits);
// What an event's peak-search scratch holds: the survivors' masks, the stencil's peak words, or
// both (request-loop slots, which serve events of either kind), the one list of an event of few cells
// (and room for masks), or nothing.
enum PeakScratch { kPeakBands = 1, kPeakMask = 2, kPeakFew = 4 };
// Bytes of per-event scratch for a grid tiling and an event size (below 0: no hits, but a matrix of
// any counts), and the carving of it.
size_t event_scratch_bytes(const DevGrid& g, int64_t n_hits, bool direct, int peaks = kPeakBands);
size_t mask_bytes(const DevGrid& g);  // of the stencil's peak words
void carve_event_scratch(const DevGrid& g, int64_t n_hits, bool direct, char* base, EvDesc* ev,
                         int peaks = kPeakBands);
// The peak-search part of it alone, for n_grp groups from grp0 on.
void carve_peak_scratch(const DevGrid& g, int64_t n_hits, char* base, EvDesc* ev, int peaks, uint32_t grp0, uint32_t n_grp);
size_t surv_bytes(const DevGrid& g, int64_t n_hits, int peaks);  // of the survivor lists

// The preparation clears the stencil's peak counts (an event of a layout with both searches).
void clear_groups(const DevGrid& g, EvDesc* ev);

// Kernel launchers (ht_kernels.hip). `evs` is a device array of n_ev descriptors, or nullptr
// for a single event passed by value in `ev0`. `max_hits` bounds n_hits over the events.
// launch_fetch copies the descriptors to `evs` from pinned host memory, which has to stay as it is
// until the launch is done.
hipError_t launch_fetch(EvDesc* evs, const EvDesc* host, int n_ev, hipStream_t s);
hipError_t launch_prep(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                       int64_t max_hits, bool direct, hipStream_t s);
hipError_t launch_fill(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                       bool emit, bool long_l, hipStream_t s);
// Survivors of a written matrix (g.j set for a scan), for n_grp groups per event. counters: the
// scan uses the counter pair (no preparation of the same call does): the lists' lengths in one
// array, and it clears the other.
hipError_t launch_scan(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, uint32_t n_grp,
                       bool counters, hipStream_t s);
hipError_t launch_peaks(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, uint32_t n_grp,
                        hipStream_t s);
// Stencil peak search and ordered write of the events marked dense (others are skipped).
hipError_t launch_peaks_dense(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                              hipStream_t s);
// Peak search of filled events whose survivors are in one list (kPeakFew), as their grid and hits
// leave at most kFewCells cells at the threshold (few_cells): one launch.
int64_t cells_bound(const DevGrid& g, int64_t hits);  // cells that can reach the threshold
bool few_cells(const DevGrid& g, int64_t max_hits);
hipError_t launch_few_peaks(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, hipStream_t s);
// Launches of tiny events (g.j set for fill tiles, few cells): whether these are, and their fill with
// the preparation in it (it uses the counter pair).
bool tiny_launch(const DevGrid& g, int n_ev, int64_t max_hits);
hipError_t launch_tiny_fill(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev, hipStream_t s);
// Plain fill: zero the matrix, then one global atomicAdd per vote (reference path and the
// fallback for B rows too wide for an LDS tile).
hipError_t launch_fill_atomic(const DevGrid& g, const EvDesc& ev0, const EvDesc* evs, int n_ev,
                              int64_t max_hits, hipStream_t s);

hipError_t launch_readout(const DevGrid& g, const ht_peak* peaks, const int64_t* n_found, int64_t cap,
                          ht_track* tracks, double b_min, double db, hipStream_t s);

// Whether the fill of a launch of n_ev events of up to max_hits hits makes lists of the survivors of
// an event of `hits` hits. (If it does for one, it does for those of fewer hits.)
bool use_lists(const DevGrid& g, int n_ev, int64_t max_hits, int64_t hits);
// Whether that fill takes its long-list variant (given g.rows).
bool long_lists(const DevGrid& g, int n_ev, int64_t max_hits);
size_t fill_lds_bytes(const DevGrid& g, bool long_l);
int n_groups(const DevGrid& g);

// The layout of one no-alloc call (ht_noalloc.hip): whether its peaks come from the stencil, the
// kind of its slab lists, and whether the search runs slice by slice (the grid's jobs are then
// those of a scan, and slice_groups of them make a slice). HT_EINVAL for an event that it refuses.
struct NoallocPlan {
  bool dense, direct, sliced;
  int layout;
  size_t scratch_bytes;
  uint32_t slice_groups;
};
int plan_noalloc(const ht_grid& grid, const Tiling& tl, const DevGrid& g, int64_t n_hits, NoallocPlan* plan);

// Host helpers (ht_api.cpp).
// 0: not usable by a kernel; 1: device memory; 2: pinned host memory mapped into the device;
// 3: managed memory.
int pointer_kind(const void* ptr);
int check_accessible(const void* ptr, const char* what);
// Enqueues one event's stages on s: prep (counting into ev.slab_cnt and clearing
// ev.slab_cnt_next), then the fill, then the peak search, as do_fill / do_peaks ask; `atomic`
// takes the global-atomic fill and a scan of the matrix for survivors. *counters_used is set once
// a kernel that uses the counter pair is on the stream (the caller then flips to the other
// array for its next call). `timed` records the stage timers of ht_profile_enable.
int enqueue_event(const DevGrid& g, const EvDesc& ev, int64_t n_hits, bool direct, bool atomic,
                  bool do_fill, bool do_peaks, bool timed, hipStream_t s, bool* counters_used);
int fail(int code, const char* fmt, ...);
int fail_hip(hipError_t e, const char* what);
int validate_grid(const ht_grid* g);
uint64_t n_cells(const ht_grid& g);
// Validates the grid, uploads its tables once per device and picks the tiling.
int make_device_grid(const ht_grid& g, int dev, int n_ev, int64_t max_hits, DevGrid* out, Tiling* tl = nullptr,
                     bool search = true);
// What a batch of n_ev events of up to max_hits hits launches, besides what g says.
struct BatchShape {
  int64_t prep_hits;  // that the preparation's grid is made for: at least max_hits
  bool long_l;        // the fill's variant for long lists
  bool few;           // the search of few cells: the ordinary events have the layout kPeakFew
  bool tiny;          // and the launches of tiny events
};
BatchShape batch_shape(const DevGrid& g, int n_ev, int64_t max_hits, bool any_dense, int pieces);
// Scratch of one slot of a request loop (g made for batches of max_batch events of max_hits hits), and
// the layout of those of its batches that are not of few cells, whose slots are carved as kPeakFew.
size_t slot_scratch_bytes(const DevGrid& g, const Tiling& tl, int max_batch, int64_t max_hits, int* layout);
// The whole batched pipeline (prep, fill with survivors, peaks) for n_ev events whose
// descriptors are already in device memory.
// *prep_enqueued is set once the preparation (which counts into and clears the events' counter
// arrays) is on the stream.
// A batch split into runs of events whose peak searches run on a side stream beside the next
// run's fill (pieces <= kMaxPieces; pieces 1: no split).
constexpr int kMaxPieces = 8;
struct BatchSplit {
  int pieces;
  hipStream_t side;
  hipEvent_t filled[kMaxPieces];  // recorded on the launch stream after each run's fill
  hipEvent_t done;                // recorded on the side stream after the last peak search
};
// any_bands / any_dense: whether some event searches its peaks through the fill's survivors /
// the stencil (only the kernels needed are launched). split: NULL, or how to overlap.
int launch_batch(const DevGrid& g, const EvDesc* d_ev, int n_ev, const BatchShape& bs, bool direct,
                 bool any_bands, bool any_dense, hipStream_t s, bool* prep_enqueued,
                 const BatchSplit* split = nullptr);

}  // namespace ht
