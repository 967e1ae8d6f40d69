// Workspace layout and launch interface of the LST chain (host + device).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lst {

// Counter slots (int32) at the start of the workspace.
enum Ctr : int {
  C_STATUS = 0,  // bit 0: invalid hit data, bit 1: invalid seed data, bit 2: capacity exceeded
  C_NMD = 1, C_NLS, C_NT3, C_NT5, C_NPT3, C_NPT5, C_NTC, C_NTCHITS,   // built counts (clamped)
  C_RMD = 9, C_RLS, C_RT3, C_RT5, C_RPT3, C_RPT5,                      // required counts
  C_NT5KEEP = 15, C_NTC0 = 16, C_NTC1, C_NTC2, C_NTC3,                 // survivors, TCs per type
  C_NINC = 21, C_NBIN = 25,      // scratch totals
  C_NMDLIST = 26,                // entries of the mini-doublet search's lists
  C_NLSOVF = 27,                 // MDs with more segments than the count pass caches
  C_NEXTHITS = 28,               // hits of the extended track-candidate collection
  C_EXT = 29,                    // 1 once the track extensions of the event are written
  C_COUNT = 64
};
enum : int { ST_BAD_HIT = 1, ST_BAD_SEED = 2, ST_CAPACITY = 4 };

// Tile choices of the chain, set per geometry at run time (lst_set_tile_config,
// lst_autotune): how many passing partners a count pass remembers per parent
// (its fill copies them instead of searching again), the seed search's LDS
// list and slice table, and the candidates per wave of the extension search.
// Storage and LDS arrays are sized for the maxima (the kXxx constants below);
// results never depend on the choice.
struct Tiles {
  int md_cache;      // partners per lower hit the MD search keeps, 0..kMdCache (at most kMdKeep are kept)
  int ls_cache;      // segments per MD the segment count pass keeps, 0..kLsCache
  int t3_cache;      // triplets per segment the triplet count pass keeps, 0..kT3Cache
  int t5_cache;      // quintuplets per triplet the quintuplet count pass keeps, 0..kT5Cache
  int pt3_cache;     // pT3 per seed the seed-search count keeps with attributes, 0..kPt3Cache
  int pt5_cache;     // pT5 per seed, 0..kPt5Cache
  int pass_list;     // passing objects per seed ranked in LDS by the fill, 1..kPassList (else: ordered scan)
  int max_slices;    // marked bins per seed gathered into one flat list, 1..kMaxSlices (else: bin by bin)
  int ext_per_wave;  // track candidates per wave of the extension search: 4, 8 or 16
  int ls_group;      // inner MDs per wave of the segment count pass, 1..kLsGroup; 0: chosen per launch
};

struct DevGeom {
  int n_mod, n_edges;
  int map_asc;        // 1: every module's targets ascend
  const int *map_off, *map_tgt;
  const float4 *win;  // per module: W, A1, A2, A3
  const int *info;    // per module: bit 0 = 2S, bit 1 = endcap
  int ext;            // 1: the chain ends with the track extensions
  float d0max;        // transverse impact-parameter bound of the selections [cm]
  int stub16;         // 1: MD stubs stored as binary16 pairs (dense half2), else float2
  const float2 *t5cut;  // per quintuplet category (1024): chi2_xy and chi2_rz bounds
  Tiles tiles;
};

// One array cleared to zero at the start of the chain: n entries, `stride` ints apart.
struct FillJob {
  int *p;
  int n, stride;
};
enum FillId : int { FL_CTR, FL_TS, FL_SEED_CNT, FL_SEED_TC, FL_PLS_NEAR, FL_BIN_CNT, FL_COUNT };

// Sums a count pass keeps so that its fill pass finds its own output offsets
// (no scan launches between them): one sum per tile of 2^tile_shift(capacity)
// consecutive parents, at most kMaxSumTiles of them.  Each sum has a 128-byte
// line of its own: a count pass adds to a tile's sum from many waves, and
// atomics on one line run one after another (about 5 ns each; with 32 sums a
// line the segment count of one event went from 0.119 to 0.165 ms).
constexpr int kMaxSumTiles = 512;
constexpr int kSumStride = 32;
constexpr int kTaskShards = 16;  // lines that the seed search's tasks are counted in
__host__ __device__ inline int tile_shift(long cap) {
  int s = 8;
  while ((cap >> s) >= kMaxSumTiles) ++s;
  return s;
}
__host__ __device__ inline long n_sum_tiles(long cap) { return (cap >> tile_shift(cap)) + 1; }

// Passing partners remembered between a stage's count and fill passes: per
// module for mini-doublets, per MD for segments, per seed for pT3 / pT5 (more
// than this: the fill searches again).
constexpr int kLsCache = 32;
constexpr int kLsGroup = 16;  // most inner MDs per wave of the segment count pass
constexpr int kAzBins = 32;    // azimuth bins of a module's MDs
constexpr int kMinParents = 16;  // fewest parents per wave of the triplet and quintuplet passes
constexpr int kMdCache = 32;  // largest md_cache tile
constexpr int kMdKeep = 6;    // partners per lower hit the MD search keeps
constexpr int kT3Cache = 2;   // triplets per parent segment whose candidate the T3 count pass keeps
constexpr int kT5Cache = 2;   // quintuplets per parent triplet whose candidate the T5 count pass keeps
constexpr int kPt3Cache = 256;  // pT3 per seed (most PU200 events' largest is below, about one seed an event has more)
constexpr int kPt5Cache = 16;   // pT5 per seed
// Hit bucketing: block tiles of kHitTile to 4 kHitTile input hits; (module,
// sensor) keys in coarse buckets of kFineKeys consecutive keys (at most
// kMaxCoarse of them, so 2 n_mod <= kFineKeys * kMaxCoarse).  kScanTileHits: the
// tile that bounds an event's hits on a detector.
constexpr int kHitTile = 1024, kScanTileHits = 4096;
constexpr int kFineBits = 5, kFineKeys = 1 << kFineBits;
constexpr int kMaxCoarse = 2048;
constexpr int kMaxModules = kFineKeys * kMaxCoarse / 2;
__host__ __device__ inline int n_coarse(int n_mod) { return (2 * n_mod + kFineKeys - 1) / kFineKeys; }
__host__ __device__ inline int n_hit_tiles(long n_hits, int tile) { return (int)((n_hits + tile - 1) / tile); }
constexpr int kPassList = 1024;  // passing objects of one seed ranked in LDS by the seed-search fill
constexpr int kMaxSlices = 512;  // marked bins of one seed gathered into a flat list in LDS
constexpr int kExtPerWaveMax = 16;
constexpr Tiles kTilesDefault{kMdCache, kLsCache, kT3Cache, kT5Cache, kPt3Cache, kPt5Cache, kPassList, kMaxSlices, 8, 0};

// First-anchor bins of the seed search: 10 radius rings x 256 azimuth bins x
// 55 z bins (10 cm over |z| < 275 cm); bins of one (ring, azimuth) pair, a row,
// are contiguous, z ascending, with the row's end as a 56th offset.
constexpr int kBinRows = 10 * 256, kZBins = 55, kBinStride = kZBins + 1;
constexpr int kSeedBins = kBinRows * kBinStride;
constexpr int kDirBins = 512;             // azimuth bins of the seeds' directions at the beam line
constexpr int kSeedKeys = 4 * kDirBins;   // direction groups: each bin in four of the slope

// Device pointers of one event (all inside the workspace except the inputs).
// Kernels of a batch read descriptor blockIdx.y of a device array of these.
struct Ws {
  // inputs (device)
  int n_hits, n_seeds;
  const float *x, *y, *z, *px, *py, *pz;
  const int *module, *sensor, *q, *hits4;
  // capacities
  int cap_md, cap_ls, cap_t3, cap_t5, cap_pt3, cap_pt5, cap_tc;
  int *ctr;
  // hit buckets by (module, sensor)
  int *boff, *hidx;  // (module, sensor) buckets: offsets (2 n_mod + 1), input index per bucketed hit
  // hits per (tile, coarse bucket), then the bucket's hits in earlier tiles; hits per coarse
  // bucket; where each bucket starts
  int *tile_hist, *coarse_cnt, *coarse_off;
  // hits in coarse-bucket order (stable): x, y, z, input index | key within the bucket << 23
  // (bits); once sorted, per lower hit the partners the MD search found (6 x 16 bits, count)
  float4 *hcp;
  float4 *hpos;
  // mini-doublets
  int *md_cnt, *md_off;
  int *md_tot;      // MDs per coarse bucket (kFineKeys / 2 modules)
  int2 *md_hits;    // input indices of the lower and upper hit
  int *md_mod;
  float4 *md_pos;   // anchor (lower hit) x, y, z, r
  float2 *md_stub;  // tangential displacement, sensor separation (dense half2 with DevGeom::stub16)
  float4 *mod_disc;  // two per module with MDs: x-y disc (cx, cy, radius, |c|) around its anchors; r and z ranges
  int *md_az;        // each module's MDs grouped by bins of azimuth (azimuth_bin)
  unsigned short *mod_az;  // per module: the first place of each bin, from the module's first MD
  // segments
  int *ls_cnt, *ls_off;
  int *ls_cache;    // per MD: up to kLsCache passing partners found by the count pass (| info << 30)
  int *ls_ovf;      // the MDs with more, listed (in any order) with the tile sums
  int2 *ls_md;
  float2 *ls_beta;
  float4 *ls_opos;  // the outer MD's anchor (a copy, read by the triplet search)
  int *ls_oinf;      // and its module's info word
  // triplets
  int *t3_off;      // triplets per segment (count pass), then their offsets (written in place by the fill)
  int4 *t3_md;      // a, b, c, -
  float4 *t3_attr;  // kappa, dkappa, chi2_rz, lambda
  float2 *t3_first; // anchor x, y of the first MD
  int *t3_cache;    // per segment: up to kT3Cache passing candidate segments of the count pass
  // quintuplets
  int *t5_off;      // quintuplets per triplet, then their offsets, likewise
  int2 *t5_t3;
  int *t5_md;       // 5 per T5
  float *t5_attr;   // 8 per T5
  int *t5_keep;
  float2 *t5_first;
  int *t5_cache;    // per triplet: up to kT5Cache passing candidate triplets of the count pass
  // T5s on each MD (until the lists are placed: those it is not the first MD of), where
  // its list starts (lists in any order), and what its T5s as first MD add to their index
  int *inc_cnt, *inc_off, *inc_b0;
  int *t5_slot;     // 4 per T5: its place in the lists of its second to fifth MDs
  int2 *inc_list;   // T5s containing each MD: (T5, bits of its chi2_xy score)
  int4 *inc_mds;    // and, in step with inc_list, that T5's four other MDs
  // pixel seeds
  float *pls;       // 8 per seed: pT, cx, cy, lambda, kappa, x0, y0, z0
  int *pls_keep;
  int *seed_key, *seed_slot, *seed_cnt;  // each seed's direction group and place in it; seeds per group
  // seeds using each pixel hit: one of them (the owner), and the others as a linked list of
  // (4 seed + hit number): the hit's first entry (-1: none) and each entry's next one.  Set
  // for the seeds' hits only.
  int *ph_owner, *ph_head, *ph_next;
  // pixel triplets / quintuplets
  int *pt3_cnt, *pt3_off, *pt5_cnt, *pt5_off;
  // seeds with more than those, per kind: the tasks of the fill (2 seed + kind), and n_spill
  // lists of kPassList objects for the first of them
  int *pt_tasks, *pt_spill;
  int n_spill;
  int *pt3_cache, *pt5_cache;  // per seed: up to kPt3Cache / kPt5Cache passing objects found by the count pass
  float4 *pt3_cattr, *pt5_cattr;  // and their attributes
  int2 *pt3_so, *pt5_so;      // seed, object
  float4 *pt3_attr, *pt5_attr;
  int *pt3_keep, *pt5_keep;
  // per T3 / T5: the largest ~(score bits << 32 | seed) of the pT3 / pT5 entries on it,
  // i.e. its entry with the smallest (score, seed) (scores are >= 0, so their bits order them)
  unsigned long long *o3_best, *o5_best;
  // MDs that start a triplet, by (ring, azimuth, z) bin of their anchor: counts and offsets
  // per bin, each MD's bin (-1: none) and place in it, and per list entry the anchor x, y, z
  // with the module info bits and the MD's triplets and quintuplets (first, count, first, count)
  int *bin_cnt, *bin_off;
  int2 *md_bin;
  float4 *bin_pos;
  int4 *bin_rng;
  // track candidates
  int *t5_used;
  // the seeds sorted by group of their direction at the beam line (the seed search's order
  // too): (dx, dy, lambda, seed bits), azimuth bin offsets, each seed's place, and per place
  // the candidates the seed is in (1 pT5, 2 pT3)
  float4 *sdir;
  int *sdir_off, *sdir_pos, *sdir_tc;
  int *w_pt5, *w_pt3;           // per seed: its surviving pT5 / pT3 entry, or -1
  // track-candidate flags, one bit a seed (pT5, pT3, pLS) or quintuplet, 64 a word;
  // pls_near: the seeds near a T5 candidate
  unsigned long long *m_pt5, *m_pt3, *m_pls, *m_t5;
  unsigned *pls_near;
  // n types, n + 1 offsets, then the hit lists, end to end (n: C_NTC), so that one copy reads them
  int *tc_out;
  // host memory (pinned; may be NULL): the counters, written at the chain's end, and the
  // same candidates (with track extensions: ext_out) when they take at most h_tc_cap ints
  int *h_ctr, *h_tc;
  int h_tc_cap;
  int *tc_md;                                   // its outer-tracker MDs, inner to outer (5 per TC)
  float2 *tc_kap;                               // its curvature and curvature tolerance
  // track extensions, end to end for n candidates (ExtOut): types, MDs added (0-2), triplets
  // (-1: none), (chi2_xy, chi2_rz, kappa, -), n + 1 offsets, the extended hit lists; and the
  // hit count of each extended candidate with its exclusive scan
  int *ext_out, *ext_cnt, *ext_off;
  // the count passes' sums per tile of parents (tile_shift) and, for triplets and
  // quintuplets, per wave (parent_shift)
  int *ts_ls, *ts_t3, *ts_t5, *ts_p3, *ts_p5;
  int *ts_task;  // kTaskShards counts of tasks, likewise a line each
  int sh_ls, sh_t3, sh_t5, sh_pt;
  int *ws_t3, *ws_t5;
  // scan scratch and the table of the clears
  int *scan_tmp;
  FillJob fills[FL_COUNT];
};

// Parts of ext_out for n candidates.
struct ExtOut {
  int *type, *added, *t3, *attr, *off, *hits;
  __host__ __device__ ExtOut(int *p, long n)
      : type(p), added(p + n), t3(p + 2 * n), attr(p + 3 * n), off(p + 7 * n), hits(p + 8 * n + 1) {}
  __host__ __device__ static long ints(long n, long n_hits) { return 8 * n + 1 + n_hits; }
};

// Capacities and sizes (host-side).
struct Caps {
  int64_t md, ls, t3, t5, pt3, pt5;
};

// Carves one event's arrays from `base` (nullptr: size only) and fills the
// scan / clear job tables; counters go to `ctr` (64 ints) when given.
// Array sizes follow n_hits_alloc / n_seeds_alloc when those are >= 0 (a
// slot of a captured plan is sized for the largest event it may hold).
size_t workspace_layout(int n_mod, int n_hits, int n_seeds, const Caps &c, Ws *ws, char *base, int *ctr,
                        int n_hits_alloc = -1, int n_seeds_alloc = -1);
// Brackets launch site `site` of the chain with two recorded HIP events.
struct KernelTimer {
  int site;
  hipEvent_t beg, end;
};
constexpr int kChainSite = 1000;  // KernelTimer::site that brackets the whole chain
extern const char *const kSiteNames[];
extern const int kNumSites;
constexpr int kMaxSites = 64;
// True for the launch sites that take a block of 64, 128 or 256 threads.
bool site_tunable(int site);
bool site_shaped(int site);  // and its launch reads the shape
// Enqueues the whole chain for B events whose descriptors are d_ws[0..B) in
// device memory; `bound` holds, field by field, the largest sizes and
// capacities of the batch (it sets the launch grids).  site_block (kMaxSites
// entries or NULL): threads per block of each tunable site, 0 = the default.
// value (one event only): the descriptor, which the first launch carries and
// writes to d_ws; NULL: d_ws is there already.
void enqueue_chain(const DevGeom &g, Ws *d_ws, int B, const Ws &bound, hipStream_t st, const KernelTimer *kt,
                   const int *site_block, const Ws *value);
void launch_module_windows(const int *info, const float *pos_lo, const float *pos_up, const float *lmin,
                           const float *lmax, int n_mod, double d0, float4 *win, hipStream_t st);
// Allocation-free form: the track candidates copied to caller device buffers
// (counts: n, hits, status).
void launch_tc_export(const Ws *d_ws, int max_tc, int max_hits, int *type, int *off, int *hits, int *counts,
                      hipStream_t st);

}  // namespace lst
