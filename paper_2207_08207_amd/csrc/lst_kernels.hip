// gfx950 kernels of the Line Segment Tracking chain (arXiv:2207.08207).
//
// Every stage follows one pattern: count objects per parent (module, MD, LS,
// T3, seed), then fill each parent's objects at the prefix of the counts, which
// the fill sums for itself from the count's tile sums, in a fixed order.  No
// atomic decides an output position, so the object arrays are identical run to
// run; the atomics that remain are sums, histogram counts, list places (per-MD
// and per-hit lists, bins) and maxima, whose consumers are order-independent.
// Object counts stay on the device: later kernels read them and stride over
// them, so the whole chain is enqueued without a host round trip.  Work that no
// launch waits for (clears, seeds, bins) rides on further blocks of launches
// that are there anyway: a launch costs 4 to 5 us on one event.
#include <hip/hip_fp16.h>

#include <cstring>
#include <type_traits>

#include "lst_select.hpp"
#include "lst_ws.hpp"

namespace lst {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kScanItems = 8;                       // per thread
constexpr int kScanTile = kBlock * kScanItems;      // per block
constexpr int kMaxScanBlocks = 4096;                // tile sums a scan keeps (scan_tmp): n < 8M
static_assert((long)kMaxScanBlocks * kScanTile > 8000000L, "scan of the largest count of an event");

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
// Set bits of a ballot below this lane (its rank among the set lanes).
__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Wave-uniform values in scalar registers: the compiler cannot prove a value
// derived from threadIdx.x, or loaded through a generic pointer, uniform, and
// would otherwise keep it (and every address computed from it) in vector
// registers.  uload is for loads whose address is the same on every lane.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
__device__ __forceinline__ int uload(const int *p) { return __builtin_amdgcn_readfirstlane(*p); }
// The same pointer in the global address space: the workspace and geometry
// pointers are read from memory, so the compiler cannot infer their address
// space and would issue flat loads, which also count against the LDS wait
// counter (every LDS wait then waits for the gathers in flight too) and take a
// 64-bit address per lane.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T *gp(const T *p) {
  return (const __attribute__((address_space(1))) T *)p;
}
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gp(T *p) {
  return (__attribute__((address_space(1))) T *)p;
}
// Loads and stores of vector types through the global address space (their
// member operators take a generic `this`): by their bits, as native vectors.
template <int N> struct NativeOf;
template <> struct NativeOf<4> { typedef int type; };
template <> struct NativeOf<8> { typedef int type __attribute__((ext_vector_type(2))); };
template <> struct NativeOf<16> { typedef int type __attribute__((ext_vector_type(4))); };
template <class T>
__device__ __forceinline__ T gload(const T *p, long i) {
  typedef typename NativeOf<sizeof(T)>::type N;
  const N n = ((const __attribute__((address_space(1))) N *)p)[i];
  T v;
  __builtin_memcpy(&v, &n, sizeof(T));
  return v;
}
template <class T>
__device__ __forceinline__ void gstore(T *p, long i, const T &v) {
  typedef typename NativeOf<sizeof(T)>::type N;
  N n;
  __builtin_memcpy(&n, &v, sizeof(T));
  ((__attribute__((address_space(1))) N *)p)[i] = n;
}

// The hardware reciprocal and reciprocal square root (within 1 ulp), for pre-tests.
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float frsq(float x) { return __builtin_amdgcn_rsqf(x); }

__device__ __forceinline__ int block_sum(int v, int *s_red) {
  // wave reduction by shuffles, then across waves in LDS
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if (lane_id() == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  int t = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) t += s_red[w];
  __syncthreads();
  return t;
}

// ------------------------------------------------------------------ start
// On further blocks (q of nq) of the chain's first launch: clears what later
// launches count into, empties the lists of the pixel hits that seeds use and
// gives each such hit an owner, the seed whose store came last (the rest of
// ph_head and ph_owner is never read).  Arrays indexed by MDs or quintuplets are
// cleared where those are written, so no launch of the chain only clears.
__device__ __forceinline__ void start_blocks(const Ws &w, int q, int nq) {
  const int tid = q * blockDim.x + threadIdx.x, nt = nq * blockDim.x;
  for (int j = 0; j < FL_COUNT; ++j) {
    int *p = w.fills[j].p;
    const int n = w.fills[j].n, st = w.fills[j].stride;
    for (long i = tid; i < n; i += nt) gp(p)[i * st] = 0;
  }
  for (long i = tid; i < 4L * w.n_seeds; i += nt) {
    const int h = gp(w.hits4)[i];
    if (h >= 0 && h < w.n_hits) {
      gp(w.ph_head)[h] = -1;
      gp(w.ph_owner)[h] = (int)(i >> 2);
    }
  }
}

// ------------------------------------------------------------------ scan
// Exclusive scan of the extended candidates' hit counts, out[n] = total.  Two
// passes: tile sums, then each tile's scan offset by the sum of the tiles before
// it.
__global__ void k_scan_reduce(const Ws *__restrict__ wb) {
  __shared__ int s_red[kWaves];
  const Ws &w = wb[blockIdx.y];
  const int n = uload(w.ctr + C_NTC);
  // tiles 0 .. n / kScanTile (the last one may be empty), strided over the grid
  for (long t = blockIdx.x; t * kScanTile <= n; t += gridDim.x) {
    const long base = t * kScanTile;
    int v = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const long i = base + (long)k * kBlock + threadIdx.x;
      if (i < n) v += gp(w.ext_cnt)[i];
    }
    v = block_sum(v, s_red);
    if (threadIdx.x == 0) w.scan_tmp[t] = v;
  }
}

// Each tile adds the tile sums before it (at most a few hundred) to its own
// exclusive scan; the tile holding index n writes out[n] and the total.  (Two
// launches instead of a third, single-block pass over the tile sums.)  Both passes
// stride over the tiles, so the grid need not cover the capacity.
__global__ void k_scan_apply(const Ws *__restrict__ wb) {
  __shared__ int s_wave[kWaves], s_red[kWaves];
  const Ws &w = wb[blockIdx.y];
  const int n = uload(w.ctr + C_NTC);
  for (long t = blockIdx.x; t * kScanTile <= n; t += gridDim.x) {
    const long base = t * kScanTile;
    int pre = 0;
    for (int j = threadIdx.x; j < (int)t; j += blockDim.x) pre += w.scan_tmp[j];
    int run = block_sum(pre, s_red);
    // the tile in kScanItems rounds of kBlock consecutive items
    for (int k = 0; k < kScanItems; ++k) {
      const long i = base + (long)k * kBlock + threadIdx.x;
      const int v = (i < n) ? gp(w.ext_cnt)[i] : 0;
      // inclusive scan within the wave
      int x = v;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane_id() >= o) x += y;
      }
      if (lane_id() == 63) s_wave[threadIdx.x >> 6] = x;
      __syncthreads();
      int wbs = 0, tot = 0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) {
        const int c = s_wave[q];
        wbs += (q < (int)(threadIdx.x >> 6)) ? c : 0;
        tot += c;
      }
      if (i <= n) gp(w.ext_off)[i] = run + wbs + x - v;  // [n] = total
      __syncthreads();
      run += tot;
    }
    if (base + kScanTile > n && threadIdx.x == 0) w.ctr[C_NEXTHITS] = run;  // every item of the later tiles is past n
  }
}

// Blocks for n items, one wave per item (grid_waves) or one thread per item
// (grid_for), at `block` threads per block; kernels stride over the rest.
static inline int grid_waves(long n, int block = kBlock) {
  const int wpb = block / 64;
  long g = (n + wpb - 1) / wpb;
  if (g < 1) g = 1;
  if (g > 16384) g = 16384;
  return (int)g;
}

// Waves per launch that grid-stride kernels share among the launch's events: eight
// per wave slot of the chip (256 CUs x 32); the searches whose work is a large
// fraction of their capacity (the segment count, the quintuplets' duplicate
// removal) take four times that, since waves with more work left than the others
// hide each other's latency (measured: two per slot made the segment count 1.24x
// slower than eight; four times the blocks for the triplets and quintuplets of
// eight PU200 events cost 20 us).
constexpr long kLaunchWaves = 8L * 256 * 32;

static inline int grid_for(long n, int block = kBlock) {
  long g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 8192) g = 8192;
  return (int)g;
}

// The scan in every event of the batch; n_cap bounds the item count.
static void scan(const Ws *wb, int B, long n_cap, hipStream_t st) {
  // tiles covering n_cap + 1 outputs (capacities are checked on the host so that every scan's
  // count stays below kMaxScanBlocks tiles), at most an equal share of kLaunchWaves per event
  const long share = std::max(64L, kLaunchWaves / B / kWaves);
  const int nb = (int)std::min<long>(std::min<long>((n_cap + kScanTile) / kScanTile, kMaxScanBlocks), share);
  k_scan_reduce<<<dim3(nb, B), kBlock, 0, st>>>(wb);
  k_scan_apply<<<dim3(nb, B), kBlock, 0, st>>>(wb);
}

// ------------------------------------------------- offsets inside a fill pass
// A stage's objects are counted per parent, then written at the exclusive
// prefix of the counts.  The prefix of a wave's first parent is the sum of the
// tile sums before its tile (added by the count pass, one atomic per wave) plus
// the counts inside the tile before it, so the fill finds its own offsets and
// the chain has no scan launches there: each cost about 5 us on one event, which
// is launch and drain time and not work (the two-launch scans of the segment,
// triplet, quintuplet and pixel stages were 0.06 ms of a 1.0 ms event).

// Sum over the wave, in a scalar register.
__device__ __forceinline__ int wave_total(int v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return __builtin_amdgcn_readfirstlane(v);
}
// Inclusive prefix of v over the wave's lanes.
__device__ __forceinline__ int wave_inclusive(int v) {
  const int lane = lane_id();
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}
// Prefix of the wave's parent p0: tile sums ts (2^sh parents each) before its
// tile, then the sums `part` of 2^psh parents each (psh = 0: the counts
// themselves) from the tile's start to p0.
__device__ __forceinline__ int wave_prefix(const int *ts, int sh, const int *part, int psh, int p0) {
  const int lane = lane_id();
  const int T = p0 >> sh;
  int v = 0;
  for (int j = lane; j < T; j += 64) v += gp(ts)[j * kSumStride];
  const int w1 = p0 >> psh;
  for (int j = (T << (sh - psh)) + lane; j < w1; j += 64) v += gp(part)[j];
  return wave_total(v);
}
// The same for a block (all its threads call it; p0 the block's first parent):
// one read of the sums for its waves.  (With one per wave the fills of a launch
// of eight events took 0.11 ms longer.)
__device__ __forceinline__ int block_prefix(const int *ts, int sh, const int *part, int psh, int p0, int *s_red) {
  const int T = p0 >> sh;
  int v = 0;
  for (int j = threadIdx.x; j < T; j += blockDim.x) v += gp(ts)[j * kSumStride];
  const int w1 = p0 >> psh;
  for (int j = (T << (sh - psh)) + (int)threadIdx.x; j < w1; j += blockDim.x) v += gp(part)[j];
  v = wave_total(v);
  const int wpb = blockDim.x >> 6;
  __syncthreads();  // s_red may still be read by the previous call
  if (lane_id() == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  int t = 0;
  for (int q = 0; q < wpb; ++q) t += s_red[q];
  return __builtin_amdgcn_readfirstlane(t);
}
// The stage's total: required and built counts, the capacity flag.
__device__ __forceinline__ void put_total(const Ws &w, int tot, int cap, int req, int built) {
  w.ctr[req] = tot;
  w.ctr[built] = tot < cap ? tot : cap;
  if (tot > cap) atomicOr(w.ctr + C_STATUS, (int)ST_CAPACITY);
}

// ------------------------------------------------------------- windows
__global__ void k_module_windows(const int *info, const float *pos_lo, const float *pos_up, const float *lmin,
                                 const float *lmax, int n_mod, double d0, float4 *win) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_mod) return;
  double w[4];
  module_windows((info[m] >> 1) & 1, info[m] & 1, (double)pos_lo[m], (double)pos_up[m], (double)lmin[m],
                 (double)lmax[m], d0, w);
  win[m] = make_float4((float)w[0], (float)w[1], (float)w[2], (float)w[3]);
}

void launch_module_windows(const int *info, const float *pos_lo, const float *pos_up, const float *lmin,
                           const float *lmax, int n_mod, double d0, float4 *win, hipStream_t st) {
  k_module_windows<<<(n_mod + 127) / 128, 128, 0, st>>>(info, pos_lo, pos_up, lmin, lmax, n_mod, d0, win);
}

// ------------------------------------------------- allocation-free forms
// Copies an event's track candidates to caller device buffers: counts[0] =
// candidates, counts[1] = their hits, counts[2] = the chain's status flags;
// the arrays are written only when the chain succeeded and both fit.
__global__ void k_tc_export(const Ws *__restrict__ wb, int max_tc, int max_hits, int *type, int *off, int *hits,
                            int *counts) {
  const Ws &w = wb[0];
  const int st = w.ctr[C_STATUS], n = uload(w.ctr + C_NTC), nh = uload(w.ctr + C_NTCHITS);
  const int tid = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
  if (tid == 0) {
    counts[0] = n;
    counts[1] = nh;
    counts[2] = st;
  }
  if (st != 0 || n > max_tc || nh > max_hits) return;
  for (int i = tid; i <= n; i += stride) {
    if (i < n) type[i] = gp(w.tc_out)[i];
    off[i] = gp(w.tc_out)[n + i];
  }
  for (int i = tid; i < nh; i += stride) hits[i] = gp(w.tc_out)[2L * n + 1 + i];
}

void launch_tc_export(const Ws *d_ws, int max_tc, int max_hits, int *type, int *off, int *hits, int *counts,
                      hipStream_t st) {
  k_tc_export<<<256, 256, 0, st>>>(d_ws, max_tc, max_hits, type, off, hits, counts);
}

// ---- binned search: objects grouped by first anchor (radius ring, azimuth bin, z bin)
constexpr int kRings = 10;
constexpr float kRing0 = 20.0f, kRingW = 10.0f;      // rings [20, 30), ..., [110, 120) cm, ends clamped
constexpr int kPhiBins = 256;
constexpr int kObjBins = kRings * kPhiBins;          // (ring, azimuth) pairs: the bits of a seed's mask
constexpr float kZHalf = 275.0f, kZW = 10.0f;        // z bins [-275, -265), ..., ends clamped
static_assert(kObjBins == kBinRows && kPhiBins * 8 == kSeedKeys, "seed-search bins and direction groups");
constexpr int kMaskWords = kObjBins / 32;
constexpr float kSampleStep = 2.0f;                  // trajectory sampling step [cm]
constexpr int kMaxSamples = 112;                     // 224 cm of arc

__device__ __forceinline__ int ring_of(float r) {
  const int k = (int)floorf((r - kRing0) / kRingW);
  return k < 0 ? 0 : (k >= kRings ? kRings - 1 : k);
}
__device__ __forceinline__ int phibin_of(float ph) {
  const int b = (int)floorf((ph + (float)M_PI) * (float)(kPhiBins / (2.0 * M_PI)));
  return b < 0 ? 0 : (b >= kPhiBins ? kPhiBins - 1 : b);
}
__device__ __forceinline__ int zbin_of(float z) {
  const int b = (int)floorf((z + kZHalf) / kZW);
  return b < 0 ? 0 : (b >= kZBins ? kZBins - 1 : b);
}
// Bin of the objects whose first anchor is a.
__device__ __forceinline__ int obj_bin(const float4 &a) {
  const float ph = atan2f(a.y, a.x);
  const int rp = ph == ph ? ring_of(a.w) * kPhiBins + phibin_of(ph) : 0;
  return rp * kBinStride + zbin_of(a.z);
}
// Proximity queries (near_dir) read the seeds' directions at the beam line,
// binned by azimuth, so that a query reads only the bins that can hold a near
// entry.  The seed search takes the seeds in the table's order: each azimuth bin
// in four groups of the slope, so that waves that run together scan nearly the
// same object bins and reuse each other's lists in cache (results do not depend
// on the order).  Near entries have |dphi| < asin(D) (the test requires sin^2 dphi < D^2
// and a positive dot product), so with bins of width 2 pi / kDirBins the query
// covers ceil(asin(D) / width) + 1 bins on each side, one more than needed to
// absorb atan2f rounding.  The decision itself is near_dir, unchanged.
__device__ __forceinline__ int dir_bin(float dx, float dy) {
  const float ph = atan2f(dy, dx);
  if (!(ph == ph)) return 0;
  const int b = (int)floorf((ph + (float)M_PI) * (float)(kDirBins / (2.0 * M_PI)));
  return b < 0 ? 0 : (b >= kDirBins ? kDirBins - 1 : b);
}
constexpr int bin_reach(double D) {
  // ceil(asin(D) / (2 pi / kDirBins)) + 1 for the D values used (asin(D) < 1.0005 D for D <= 0.05)
  return (int)(D * 1.0005 / (2.0 * 3.14159265358979 / kDirBins)) + 2;
}

// ------------------------------------------------------------- a0: hits
// Hits are bucketed by key = 2 module + sensor, stably (input order within a
// key), with no global atomic: a two-level counting sort.
//  1. k_hits_count: each block counts the hits of its tile of input hits per
//     coarse bucket (key >> kFineBits) in LDS;
//  2. k_hits_rows turns each bucket's counts into the hits of earlier tiles (the
//     scatter does so itself for few tiles);
//  3. k_hits_scatter: each wave places its 64 to 512 hits of the tile in input
//     order, 64 at a time, after the waves before it; hits of one coarse bucket
//     in a round find each other with ballots and take consecutive positions
//     after the bucket's running position (stable), writing one 16-byte record
//     (x, y, z, input index and key within the bucket);
//  4. k_bucket_md: one block per coarse bucket counts its keys, writes their
//     offsets, moves every hit (input index; x, y, z, r) to its key's running
//     position, again 64 hits at a time in order, and searches the bucket's
//     modules for mini-doublets.

// The bucket key of hit i, or -1 for a pixel hit or invalid data (*bad).
__device__ __forceinline__ int hit_key(const Ws &w, int i, int n_mod, bool *bad) {
  const int m = gp(w.module)[i], sn = gp(w.sensor)[i];  // (a pixel hit's sensor is read, not used)
  const float x = gp(w.x)[i], y = gp(w.y)[i], z = gp(w.z)[i];
  bool b = !(isfinite(x) && isfinite(y) && isfinite(z)) || m < -1 || m >= n_mod;
  int key = -1;
  if (m >= 0) {
    b |= (sn != 0 && sn != 1);
    if (!b) key = 2 * m + sn;
  }
  *bad = b;
  return key;
}

// A hit's input index (below 2^23: events hold at most 8,000,000 hits) and its
// key's position in its coarse bucket, packed into the fourth word of its
// coarse-order record.
__device__ __forceinline__ int hit_tag(int i, int key) { return i | ((key & (kFineKeys - 1)) << 23); }
__device__ __forceinline__ int tag_index(float t) { return __float_as_int(t) & 0x7fffff; }
__device__ __forceinline__ int tag_fine(float t) { return (int)((unsigned)__float_as_int(t) >> 23); }
static_assert(kFineBits + 23 <= 32, "index and fine key in one word");

// Lanes (of the active ones) whose `nbits`-bit value v equals this lane's.
__device__ __forceinline__ unsigned long long match_value(int v, int nbits, bool active) {
  unsigned long long m = __ballot(active);
  for (int b = 0; b < nbits; ++b) {
    const bool bit = (v >> b) & 1;
    const unsigned long long bb = __ballot(active && bit);
    m &= bit ? bb : ~bb;
  }
  return m;
}

__device__ __forceinline__ int bits_for(int n) {  // bits of the values 0 .. n - 1
  int b = 0;
  while ((1 << b) < n) ++b;
  return b;
}

// ------------------------------------------------------------- a6: pLS
__device__ __forceinline__ Seed load_seed(const Ws &w, int s) {
  const float *p = w.pls + 8 * (long)s;
  Seed sd;
  sd.pt = p[0]; sd.cx = p[1]; sd.cy = p[2]; sd.lam = p[3]; sd.ks = p[4]; sd.x0 = p[5]; sd.y0 = p[6]; sd.z0 = p[7];
  return sd;
}

// Pixel line segment of seed s (Section 2.4): validated (returns true if its
// data are invalid), its parameters computed, entered in the lists of its pixel
// hits and counted in its direction group.
__device__ __forceinline__ bool seed_prepare(const Ws &w, int s) {
  const float px = gp(w.px)[s], py = gp(w.py)[s], pz = gp(w.pz)[s];
  const int q = gp(w.q)[s];
  bool bad = !(q == 1 || q == -1) || !(isfinite(px) && isfinite(py) && isfinite(pz));
  bad |= !(px * px + py * py > 0.0f);
  int h0 = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int h = gp(w.hits4)[4 * (long)s + k];
    const bool in = h >= 0 && h < w.n_hits;
    bad |= !in;
    if (in) {
      bad |= gp(w.module)[h] != -1;
      // a hit that another seed owns (few): join its list
      if (gp(w.ph_owner)[h] != s) gp(w.ph_next)[4 * (long)s + k] = atomicExch(w.ph_head + h, 4 * s + k);
      if (k == 0) h0 = h;
    }
  }
  const bool any = w.n_hits > 0;
  Seed sd;
  sd.pt = sqrtf(px * px + py * py);
  sd.cx = px / sd.pt;
  sd.cy = py / sd.pt;
  sd.lam = pz / sd.pt;
  sd.ks = (-(float)q * kCurv) / sd.pt;
  sd.x0 = any ? gp(w.x)[h0] : 0.f;
  sd.y0 = any ? gp(w.y)[h0] : 0.f;
  sd.z0 = any ? gp(w.z)[h0] : 0.f;
  float4 *o = reinterpret_cast<float4 *>(w.pls + 8 * (long)s);
  gstore(o, 0, make_float4(sd.pt, sd.cx, sd.cy, sd.lam));
  gstore(o, 1, make_float4(sd.ks, sd.x0, sd.y0, sd.z0));
  const Dir d = seed_dir(sd);
  const int key = 4 * dir_bin(d.dx, d.dy) + (d.lam < 0.0f ? 0 : 2) + (fabsf(d.lam) < 1.5f ? 0 : 1);
  gp(w.seed_key)[s] = key;
  gp(w.seed_slot)[s] = atomicAdd(w.seed_cnt + key, 1);
  return bad;
}

// A tile is NW waves x R rounds of 64 hits: sixteen waves where their rows of
// 16-bit counts fit LDS (n_coarse up to 1,700), else eight.  (Four waves of 16
// rounds, as one block took before, left a tile's hits to a serial chain: 28 +
// 43 us for the count and the scatter of one PU200 event.)
//
// The chain's first launch, with start_blocks on the blocks from n_tiles on (a
// launch of their own, 5 to 9 us, before).  Nothing of theirs is used here: the
// hits' validity is reported by the scatter, the seeds are prepared beside the
// bucket sort (with the count, their chain of gathers made it 20 us for a PU200
// event).  For one event (VALUE) the launch's arguments carry the descriptor,
// which the first of those blocks writes where the later launches read it,
// instead of a copy before the chain.
template <bool VALUE, int NW, int R>
__global__ __launch_bounds__(64 * NW) void k_hits_count(Ws value, Ws *wb, int n_mod, int n_tiles) {
  extern __shared__ int s_hits[];  // nc counts
  const Ws &w = VALUE ? value : wb[blockIdx.y];
  if ((int)blockIdx.x >= n_tiles) {
    if (VALUE && (int)blockIdx.x == n_tiles) {
      static_assert(sizeof(Ws) % 4 == 0 && sizeof(Ws) <= 3584, "the first launch argument, within the argument block");
      const auto *src = (const __attribute__((address_space(4))) int *)__builtin_amdgcn_kernarg_segment_ptr();
      for (int i = threadIdx.x; i < (int)(sizeof(Ws) / 4); i += blockDim.x) gp(reinterpret_cast<int *>(wb))[i] = src[i];
    }
    start_blocks(w, (int)blockIdx.x - n_tiles, (int)gridDim.x - n_tiles);
    return;
  }
  const int nc = n_coarse(n_mod), tb = blockIdx.x;
  const long i0 = (long)tb * (64 * NW * R);
  if (i0 < w.n_hits) {
    for (int c = threadIdx.x; c < nc; c += 64 * NW) s_hits[c] = 0;
    int key[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = (int)i0 + r * 64 * NW + (int)threadIdx.x;
      bool bad;
      key[r] = i < w.n_hits ? hit_key(w, i, n_mod, &bad) : -1;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (key[r] >= 0) atomicAdd(&s_hits[key[r] >> kFineBits], 1);  // LDS
    __syncthreads();
    for (int c = threadIdx.x; c < nc; c += 64 * NW) gp(w.tile_hist)[(long)tb * nc + c] = s_hits[c];
  }
}

// Each coarse bucket's counts per tile, in place, into the bucket's hits in
// earlier tiles, and its total: 32 buckets per block, the tiles in 32 segments.
__global__ __launch_bounds__(1024) void k_hits_rows(const Ws *__restrict__ wb, int n_mod, int tile) {
  __shared__ int s_seg[32][33];
  const Ws &w = wb[blockIdx.y];
  const int nc = n_coarse(n_mod), nt = n_hit_tiles(w.n_hits, tile);
  const int col = threadIdx.x & 31, seg = threadIdx.x >> 5, c = blockIdx.x * 32 + col;
  const int t0 = (int)((long)nt * seg / 32), t1 = (int)((long)nt * (seg + 1) / 32);
  int sum = 0;
  if (c < nc)
    for (int t = t0; t < t1; ++t) sum += gp(w.tile_hist)[(long)t * nc + c];
  s_seg[seg][col] = sum;
  __syncthreads();
  int run = 0;
  for (int q = 0; q < seg; ++q) run += s_seg[q][col];
  if (c >= nc) return;
  for (int t = t0; t < t1; ++t) {
    const int v = gp(w.tile_hist)[(long)t * nc + c];
    gp(w.tile_hist)[(long)t * nc + c] = run;
    run += v;
  }
  if (seg == 31) gp(w.coarse_cnt)[c] = run;
}

// Stable scatter of a tile's hits into coarse-bucket order: each wave's first
// slot in bucket c is the bucket's start (every block scans the bucket counts
// for itself; the first writes the starts), plus the hits of earlier tiles, plus
// those of the waves before it; in each round of 64 hits, a hit's rank among
// the round's hits of its bucket (match_value) places it.  The hit's
// coordinates, input index and key within its bucket travel with it (one
// 16-byte store), so the per-bucket sort reads them contiguously.
// With few tiles (direct: at most kDirectTiles in the launch's largest event) every
// block sums the tiles' counts for itself and there is no launch of k_hits_rows:
// 4 us less on a tiny event (two tiles of 1,400 hits).  With the 130 tiles of a
// PU50 event the blocks would read 80 MB for it.
constexpr int kDirectTiles = 16;
template <int NW, int R>
__global__ __launch_bounds__(64 * NW) void k_hits_scatter(const Ws *__restrict__ wb, int n_mod, int direct) {
  extern __shared__ int s_hits[];  // nc positions, then NW rows of 16-bit counts, two a word
  __shared__ int s_wave[NW];
  constexpr int T = 64 * NW;
  const Ws &w = wb[blockIdx.y];
  const int wv = wave_id(), lane = lane_id(), t = threadIdx.x;
  const int nc = n_coarse(n_mod), row = (nc + 1) / 2, tb = blockIdx.x;
  const long i0 = (long)tb * (T * R) + wv * (64 * R);
  if ((long)tb * (T * R) >= w.n_hits && tb > 0) return;  // the whole block
  int *s_base = s_hits;
  unsigned *rows = reinterpret_cast<unsigned *>(s_hits + nc);
  for (int i = t; i < NW * row; i += T) rows[i] = 0u;
  // the wave's hits, kept in registers
  int key[R];
  float x[R], y[R], z[R];
  bool any_bad = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = (int)i0 + r * 64 + lane;
    bool bad = false;
    key[r] = i < w.n_hits ? hit_key(w, i, n_mod, &bad) : -1;
    any_bad |= bad;
    x[r] = y[r] = z[r] = 0.f;
    if (key[r] >= 0) {
      x[r] = gp(w.x)[i];
      y[r] = gp(w.y)[i];
      z[r] = gp(w.z)[i];
    }
  }
  if (any_bad) atomicOr(&w.ctr[C_STATUS], (int)ST_BAD_HIT);
  // bucket starts: an exclusive scan of the bucket counts, kPer consecutive ones a thread
  constexpr int kPer = (kMaxCoarse + T - 1) / T;
  int v[kPer], own[kPer], sum = 0;  // the bucket's hits, and those in earlier tiles
  const int n_tiles = direct ? n_hit_tiles(w.n_hits, T * R) : 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int c = t * kPer + i;
    v[i] = own[i] = 0;
    if (c < nc) {
      if (!direct) v[i] = gp(w.coarse_cnt)[c];
      for (int q = 0; q < n_tiles; ++q) {
        if (q == tb) own[i] = v[i];
        v[i] += gp(w.tile_hist)[(long)q * nc + c];
      }
    }
    sum += v[i];
  }
  const int inc = wave_inclusive(sum);
  if (lane == 63) s_wave[wv] = inc;
  __syncthreads();
  int ex = inc - sum;
  for (int q = 0; q < wv; ++q) ex += s_wave[q];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int c = t * kPer + i;
    if (c < nc) {
      s_base[c] = ex + own[i];
      if (tb == 0) {
        gp(w.coarse_off)[c] = ex;
        if (c == nc - 1) gp(w.coarse_off)[nc] = ex + v[i];
      }
    }
    ex += v[i];
  }
  // each wave's hits per bucket (at most 64 R < 2^16)
  unsigned *mine = rows + wv * row;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (key[r] >= 0) {
      const int c = key[r] >> kFineBits;
      atomicAdd(&mine[c >> 1], 1u << (16 * (c & 1)));  // LDS
    }
  __syncthreads();
  // ... into the hits of the waves before it, both halves of a word at once
  for (int i = t; i < row; i += T) {
    unsigned run = 0u;
    for (int q = 0; q < NW; ++q) {
      const unsigned u = rows[q * row + i];
      rows[q * row + i] = run;
      run += u;
    }
  }
  if (!direct && (long)tb * (T * R) < w.n_hits)
    for (int c = t; c < nc; c += T) s_base[c] += gp(w.tile_hist)[(long)tb * nc + c];
  __syncthreads();
  unsigned short *s_run = reinterpret_cast<unsigned short *>(mine);
  const int nbits = bits_for(nc);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool act = key[r] >= 0;
    const int c = act ? key[r] >> kFineBits : 0;
    const unsigned long long peers = match_value(c, nbits, act);
    int base = 0;
    if (act) {
      base = s_run[c];
      const int pos = s_base[c] + base + lanes_below(peers);
      gstore(w.hcp, pos, make_float4(x[r], y[r], z[r], __int_as_float(hit_tag((int)i0 + r * 64 + lane, key[r]))));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (act && lanes_below(peers) == 0) s_run[c] = (unsigned short)(base + __popcll(peers));  // the bucket's first lane
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------- a1: MD
// MD stubs are stored as float2 or, with the geometry's 16-bit stub switch, as
// a dense array of binary16 pairs (rounded to nearest even) read back as float.
__device__ __forceinline__ void put_stub(const Ws &w, const DevGeom &g, int pos, float2 st) {
  if (g.stub16)
    gstore(reinterpret_cast<__half2 *>(w.md_stub), pos, __floats2half2_rn(st.x, st.y));
  else
    gstore(w.md_stub, pos, st);
}
__device__ __forceinline__ float2 get_stub(const Ws &w, const DevGeom &g, int i) {
  if (g.stub16) return __half22float2(gload(reinterpret_cast<const __half2 *>(w.md_stub), i));
  return gload(w.md_stub, i);
}

// Anchor disc of a module for the segment stage's module-level azimuth
// pre-test, from the lower hits' bounding box (min/max reduced by the caller).
__device__ __forceinline__ float4 anchor_disc(float x0, float x1, float y0, float y1) {
  const float cx = 0.5f * (x0 + x1), cy = 0.5f * (y0 + y1);
  const float hx = 0.5f * (x1 - x0), hy = 0.5f * (y1 - y0);
  const float rho = sqrtf(hx * hx + hy * hy) * 1.0001f + 1e-3f;
  return make_float4(cx, cy, rho, sqrtf(cx * cx + cy * cy));
}

// Bin of an azimuth in a module, from the sine of its angle from the disc's
// centre: kAzBins equal steps over the disc's own |sine| <= radius / |c| = 1 / scale, the
// values outside in the first and last.  Non-decreasing in the sine.
__device__ __forceinline__ int azimuth_bin(float scale, float s) {
  const float u = (s * scale + 1.0f) * (0.5f * kAzBins);
  return (int)fminf(fmaxf(u, 0.0f), (float)(kAzBins - 1));  // (NaN: 0)
}

// Quotient and remainder of t / n for 0 <= t < 2^22 and n >= 1 from rn, the
// float reciprocal of n: t is exact in float and the two roundings (of 1 / n
// and of the product) are 2^-24 relative each, so the float quotient is within
// (t / n) 2^-23 < 1/2 of t / n; truncated, it is the quotient or one off, and
// one correction step each way makes it exact.  (Integer division has no
// instruction: the compiler's sequence for a variable divisor costs some 30
// instructions, in 64 bits far more.)
__device__ __forceinline__ int2 divmod22(int t, int n, float rn) {
  int q = (int)((float)t * rn);
  int r = t - q * n;
  if (r < 0) {
    --q;
    r += n;
  }
  if (r >= n) {
    ++q;
    r -= n;
  }
  return make_int2(q, r);
}

// Floats as ints of the same order (for LDS atomic minima and maxima).
__device__ __forceinline__ int ordered(float f) {
  const int b = __float_as_int(f);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float unordered(int b) { return __int_as_float(b ^ ((b >> 31) & 0x7fffffff)); }

// One block of kSortWaves waves per coarse bucket: the bucket's hits (in input
// order) are split into kSortWaves consecutive runs; each wave counts its
// run's keys, the block turns the counts into each (wave, key)'s first
// position (key order, then wave order: stable), writes the keys' offsets, and
// every wave places its run's hits 64 at a time in order.
//
// Then the MD search of the bucket's kBucketMods modules.  A module's window
// admits about a hundredth of its (lower, upper) pairs, so each upper hit joins,
// as it is placed, the list in LDS of one of its module's kMdBins bins of u =
// tan(azimuth from one of the module's lower hits), and each lower hit (one a
// lane, the bucket's modules end to end) tests only the uppers of the two bins
// that its window touches.  For |u| <= 1/2 a pair that passes md_pass has
// |u_j - u_i| = |sin(azimuth change)| / (cos cos) <= 5/4 W, up to rounding (each
// u within 4e-7, W's test within 1e-6); bins are a little wider than twice that
// bound (so a window touches two, whatever u inv rounds to) and wrap round (the
// exact test decides, so sharing a bin only costs a test).
//
// A module with a hit outside that range (or nearly on the beam line, where products
// may underflow, or far out) or a wide window, or a bucket with more hits than the
// lists hold, has every pair tested, and the fill tests a lower hit's again if it has
// more than kMdKeep partners (they are kept in order).  That is too slow for
// detectors of few, wide modules, so in launches with many hits a module
// (CROWDED, kCrowdedHits):
//  - modules with a hit outside the range of u (if one with more than kMdWalk upper
//    hits is among the bucket's), and all of a bucket with more hits than the lists
//    hold, are listed again in a second pass, by direction (md_bins), with the lists of
//    such a bucket in the records of its upper hits, which are read no more; only those
//    with few hits, with one near the beam line or far out and with windows of more
//    than about a radian have every pair tested;
//  - lower hits with more than kMdKeep partners in a module of more than kMdWalk upper
//    hits have all of them written to a list in global memory (the segments' cache,
//    not yet in use).
//
// (Testing all pairs, 8.8M on a PU200 event for 138k MDs, took 25 + 27 us to
// count and 24 + 14 us to fill for one event, 318 us for eight; the kernel is
// bound by the chain of its steps in the densest bucket, hence few passes over
// the hits.  Crowded, 6 x 1,000 and 24 x 1,000 hits a sensor on modules of a whole and
// of a quarter of the azimuth take 0.23 and 0.77 ms here and 0.06 and 0.32 in the fill,
// else 2.21, 6.47, 0.06 and 3.06.  The line, 48 hits a module: with 55, PU400, the
// densest bucket has 8,500 hits, and the crowded form takes 0.14 ms instead of 0.60;
// below about 50 every bucket's hits fit the lists, and its checks only lengthen the
// densest bucket's chain, by 1 to 2 us.)
// At most 80 scalar registers (72 and the reserved ones): with 80 and those a SIMD
// held seven waves, so a CU three of these blocks instead of four, and eight PU50
// events took 78 us instead of 71.
constexpr int kSortWaves = 8, kSortThreads = 64 * kSortWaves;
constexpr int kBucketMods = kFineKeys / 2;
constexpr int kMdBins = 64;    // per module
constexpr int kMdList = 8192;  // hits of a bucket that the lists can hold
constexpr int kMdWalk = 64;    // upper hits that the fill tests again one after another
constexpr long kCrowdedHits = 48;  // hits a module, of the launch's largest event
static_assert((kMdBins & (kMdBins - 1)) == 0, "bins wrap round by a mask");

// The module of the bucket's q-th lower hit (modules' lower hits before: lpre[0..kBucketMods]).
__device__ __forceinline__ int lower_module(const int *lpre, int q) {
  int m = 0;
#pragma unroll
  for (int s = kBucketMods / 2; s > 0; s >>= 1)
    if (lpre[m + s] <= q) m += s;
  return m;
}
// Direction of (x, y) from the beam line: non-decreasing in the azimuth from -pi to
// pi, from -2 to 2, with a slope of at most 1 (a half to 1).
__device__ __forceinline__ float direction(float x, float y) {
  const float t = y * frcp(fabsf(x) + fabsf(y));
  return x >= 0.0f ? t : (y >= 0.0f ? 2.0f - t : -2.0f - t);
}
// Bins of the whole circle for pairs with |sin of the azimuth change| <= W and a
// positive cosine (up to rounding, 3e-7): (d, bins per unit of direction, bins) with d
// at least the change of direction and a bin at least 2.1 d wide, so that what a
// lower hit of direction p pairs with is in the bins of p - d and p + d.  No bins
// (0) for windows that would leave fewer than four.  Up to 65,536 bins, d's 4e-6
// is more than the rounding of their edges.
__device__ __forceinline__ float3 md_bins(float W) {
  const float c2 = 1.0f - W * W;
  if (!(W >= 0.0f && c2 > 0.1f)) return make_float3(0.f, 0.f, 0.f);
  const float d = W * frsq(c2) * 1.0001f + 4e-6f;
  const float n = fminf(floorf((4.0f / 2.1f) / d), 65536.0f);
  return n >= 4.0f ? make_float3(d, 0.25f * n, n) : make_float3(0.f, 0.f, 0.f);
}
__device__ __forceinline__ int md_bin(float p, const float3 &b) {
  const float v = floorf((p + 2.0f) * b.y);
  return (int)(v < 0.0f ? v + b.z : (v >= b.z ? v - b.z : v));
}
// The first kMdKeep partners of a lower hit, ascending, and how many there are.
struct MdKept {
  unsigned kept[kMdKeep];
  int n = 0;
  __device__ __forceinline__ MdKept() {
#pragma unroll
    for (int i = 0; i < kMdKeep; ++i) kept[i] = 0xffffu;
  }
  __device__ __forceinline__ void take(int j) {
    ++n;
    unsigned v = (unsigned)min(j, 0xffff);
#pragma unroll
    for (int i = 0; i < kMdKeep; ++i) {
      const unsigned lo = min(kept[i], v);
      v = max(kept[i], v);
      kept[i] = lo;
    }
  }
  __device__ __forceinline__ int4 packed() const {
    return make_int4((int)(kept[0] | kept[1] << 16), (int)(kept[2] | kept[3] << 16), (int)(kept[4] | kept[5] << 16), n);
  }
};
// Whether a lower hit's partners, n of nup upper hits, go to a list.
__device__ __forceinline__ bool md_listed(int n, int nup) { return n > kMdKeep && nup > kMdWalk && nup <= 0xffff; }
// lpre from key0, by the first wave.
__device__ __forceinline__ void lower_prefix(const int *key0, int *lpre) {
  const int lane = lane_id();
  const int n = lane < kBucketMods ? key0[2 * lane + 1] - key0[2 * lane] : 0;
  const int x = wave_inclusive(n);
  if (lane <= kBucketMods) lpre[lane] = x - n;
}

template <bool CROWDED>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_num_sgpr(80))) void k_bucket_md(const Ws *__restrict__ wb,
                                                                                                DevGeom g) {
  __shared__ int s_cnt[kSortWaves][kFineKeys];
  __shared__ int s_key0[kFineKeys + 1], s_lpre[kBucketMods + 1];
  __shared__ int s_head[kBucketMods * kMdBins];  // per (module, bin): its first upper (position in the bucket), -1: none
  __shared__ unsigned short s_next[kMdList];     // per hit of the bucket: the next upper of its bin
  __shared__ int s_ref[kBucketMods], s_nmd[kBucketMods];
  // how a module is searched: 0 by u; 1 (a hit outside u's range, a wide window) all pairs, or by
  // direction (CROWDED, and one of them has more than kMdWalk upper hits: s_any); 2 or 3 all pairs
  __shared__ int s_odd[kBucketMods], s_any, s_more;
  __shared__ float4 s_mod[kBucketMods];          // per module: reference direction x, y, window in u, bins per unit of u
  __shared__ int s_x0[kBucketMods], s_x1[kBucketMods], s_y0[kBucketMods], s_y1[kBucketMods];
  const Ws &w = wb[blockIdx.y];
  const int wv = wave_id(), lane = lane_id(), t = threadIdx.x;
  const int n_mod = g.n_mod, nc = n_coarse(n_mod), nkeys = 2 * n_mod;
  const int c = blockIdx.x, m0 = c * kBucketMods;
  if (c >= nc) {  // the seeds
    const int nt = ((int)gridDim.x - nc) * kSortThreads;
    for (int s = (c - nc) * kSortThreads + t; s < w.n_seeds; s += nt)
      if (seed_prepare(w, s)) atomicOr(&w.ctr[C_STATUS], (int)ST_BAD_SEED);
    return;
  }
  const int j0 = uload(w.coarse_off + c), j1 = uload(w.coarse_off + c + 1);
  const long L = j1 - j0;
  const int a = j0 + (int)(L * wv / kSortWaves), b = j0 + (int)(L * (wv + 1) / kSortWaves);
  for (int f = lane; f < kFineKeys; f += 64) s_cnt[wv][f] = 0;
  for (int i = t; i < kBucketMods * kMdBins; i += kSortThreads) s_head[i] = -1;
  if (t < kBucketMods) {
    s_ref[t] = -1;
    s_x0[t] = s_y0[t] = 0x7fffffff;
    s_x1[t] = s_y1[t] = (int)0x80000000;
    s_odd[t] = s_nmd[t] = 0;
  }
  if (CROWDED && t == 0) s_any = s_more = 0;
  __syncthreads();
  for (int j = a + lane; j < b; j += 64) {
    const int f = tag_fine(gload(w.hcp, j).w);
    atomicAdd(&s_cnt[wv][f], 1);  // LDS
    if ((f & 1) == 0) s_ref[f >> 1] = j;  // any of the module's lower hits
  }
  __syncthreads();
  // each key's total over the waves, the keys' first positions (wave 0: one key per lane)
  // and the modules' lower hits; the modules' references and windows (wave 1: one module per lane)
  if (wv == 0) {
    static_assert(kFineKeys < 64, "one key per lane");
    int tot = 0;
    if (lane < kFineKeys)
      for (int q = 0; q < kSortWaves; ++q) tot += s_cnt[q][lane];
    const int ex = j0 + wave_inclusive(tot) - tot;
    const int k = c * kFineKeys + lane;
    if (lane <= kFineKeys) s_key0[lane] = ex;  // (the last one is j1)
    if (lane < kFineKeys && k < nkeys) gp(w.boff)[k] = ex;
    if (c == nc - 1 && lane == 0) gp(w.boff)[nkeys] = j1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    lower_prefix(s_key0, s_lpre);
    // first position of each (wave, key): the key's first position plus the earlier waves' counts
    if (lane < kFineKeys) {
      int run = ex;
      for (int q = 0; q < kSortWaves; ++q) {
        const int v = s_cnt[q][lane];
        s_cnt[q][lane] = run;
        run += v;
      }
    }
  } else if (wv == 1 && lane < kBucketMods && s_ref[lane] >= 0) {
    const float4 h = gload(w.hcp, s_ref[lane]);
    const float d = gload(g.win, m0 + lane).x * 1.27f + 4e-6f;
    s_mod[lane] = make_float4(h.x, h.y, d, 0.47f / d);
    const float r = sqrtf(h.x * h.x + h.y * h.y);
    if (!CROWDED && !(r >= 1e-3f && r <= 1e6f && d < 0.25f)) s_odd[lane] = 1;
  }
  __syncthreads();
  // u of a hit of module m; false outside the range that the bins cover
  auto u_of = [&](const float4 &mod, const float4 &h, float *u) {
    const float dot = mod.x * h.x + mod.y * h.y, cr = mod.x * h.y - mod.y * h.x;
    *u = cr * frcp(dot);
    return (CROWDED || (h.w >= 1e-3f && h.w <= 1e6f)) && dot > 0.0f && fabsf(cr) <= 0.5f * dot;
  };
  auto bin_of = [](float u, float inv) { return (int)floorf(u * inv) & (kMdBins - 1); };
  for (int r0 = a; r0 < b; r0 += 64) {
    const int j = r0 + lane;
    const bool act = j < b;
    const float4 h = act ? gload(w.hcp, j) : make_float4(0.f, 0.f, 0.f, 0.f);
    const int f = act ? tag_fine(h.w) : 0;
    const unsigned long long peers = match_value(f, kFineBits, act);
    int base = 0;
    if (act) {
      base = s_cnt[wv][f];
      const int pos = base + lanes_below(peers), m = f >> 1;
      const float4 hr = make_float4(h.x, h.y, h.z, sqrtf(h.x * h.x + h.y * h.y));
      gp(w.hidx)[pos] = tag_index(h.w);
      gstore(w.hpos, pos, hr);
      if (s_ref[m] >= 0) {  // the module has lower hits
        const float4 mod = s_mod[m];
        float u;
        if (CROWDED && !(hr.w >= 1e-3f && hr.w <= 1e6f)) {
          atomicOr(&s_odd[m], 2);
        } else if (!CROWDED && !u_of(mod, hr, &u)) {
          s_odd[m] = 1;
        } else if (CROWDED && (!u_of(mod, hr, &u) || !(mod.z < 0.25f))) {
          atomicOr(&s_odd[m], 1);
          if (s_key0[2 * m + 2] - s_key0[2 * m + 1] > kMdWalk) s_any = 1;
        } else if (f & 1) {
          const int i = pos - j0;
          if (i < kMdList) s_next[i] = (unsigned short)atomicExch(&s_head[m * kMdBins + bin_of(u, mod.w)], i);
        }
        if ((f & 1) == 0) {  // the module's anchors' bounding box
          atomicMin(&s_x0[m], ordered(h.x));
          atomicMax(&s_x1[m], ordered(h.x));
          atomicMin(&s_y0[m], ordered(h.y));
          atomicMax(&s_y1[m], ordered(h.y));
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (act && lanes_below(peers) == 0) s_cnt[wv][f] = base + __popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  const bool fits = L <= kMdList;
  const bool again = CROWDED && (!fits || __builtin_amdgcn_readfirstlane(s_any));
  if (again) {  // (the whole block) modules that are listed by direction
    if (t < kBucketMods && s_ref[t] >= 0) {
      int mode = s_odd[t];
      if (mode == 0 && !fits) mode = 1;
      if (mode == 1) {
        const float3 b = md_bins(gload(g.win, m0 + t).x);
        s_mod[t] = make_float4(b.x, b.y, b.z, 0.0f);
        if (b.z == 0.0f) mode = 2;
      }
      s_odd[t] = mode;
    }
    __syncthreads();
    for (int i = t; i < kBucketMods * kMdBins; i += kSortThreads)
      if (s_odd[i / kMdBins] == 1) s_head[i] = -1;
    __syncthreads();
    for (int p = j0 + t; p < j1; p += kSortThreads) {
      int f = 0;  // its key
#pragma unroll
      for (int q = kFineKeys / 2; q > 0; q >>= 1)
        if (s_key0[f + q] <= p) f += q;
      const int m = f >> 1;
      if (!(f & 1) || s_odd[m] != 1 || s_ref[m] < 0) continue;
      const float4 h = gload(w.hpos, p);
      const int b = md_bin(direction(h.x, h.y), make_float3(s_mod[m].x, s_mod[m].y, s_mod[m].z));
      const int old = atomicExch(&s_head[m * kMdBins + (b & (kMdBins - 1))], p - j0);
      if (fits) s_next[p - j0] = (unsigned short)old;
      else gp(reinterpret_cast<int *>(w.hcp + p))[0] = old;
    }
    __syncthreads();
  }
  // ---- the MD search
  static_assert(kMdKeep == 6 && kMdList <= 0x8000, "packed in three words; list ends are negative");
  const int n_lower = s_lpre[kBucketMods];
  for (int q = t; q < n_lower && !again; q += kSortThreads) {
    const int m = lower_module(s_lpre, q);
    const int p = s_key0[2 * m] + (q - s_lpre[m]), up0 = s_key0[2 * m + 1], nup = s_key0[2 * m + 2] - up0;
    MdKept r;
    if (nup > 0) {
      const float4 hi = gload(w.hpos, p), win = gload(g.win, m0 + m);
      const ModInfo mi{gp(g.info)[m0 + m]};
      if ((CROWDED || fits) && !s_odd[m]) {
        const float4 mod = s_mod[m];
        float u;
        u_of(mod, hi, &u);
        const int b0 = bin_of(u - mod.z, mod.w), b1 = bin_of(u + mod.z, mod.w);
        const int *head = s_head + m * kMdBins;
        // the two bins' lists one after the other
        int k = head[b0], rest = b1 != b0 ? head[b1] : -1;
        if (k < 0) {
          k = rest;
          rest = -1;
        }
        while (k >= 0) {
          const float4 hj = gload(w.hpos, j0 + k);
          const int j = j0 + k - up0;
          k = (int)(short)s_next[k];  // -1 at the end
          if (k < 0) {
            k = rest;
            rest = -1;
          }
          if (md_pass(hi, hj, win, mi)) r.take(j);
        }
      } else {
        for (int j = 0; j < nup; ++j)
          if (md_pass(hi, gload(w.hpos, up0 + j), win, mi)) r.take(j);
      }
    }
    if (CROWDED && md_listed(r.n, nup)) s_more = 1;
    gstore(reinterpret_cast<int4 *>(w.hcp), p, r.packed());
    if (r.n > 0) atomicAdd(&s_nmd[m], r.n);
  }
  __syncthreads();
  // the same with modules listed by direction, and the lists of the lower hits with many partners
  if (CROWDED && (again || __builtin_amdgcn_readfirstlane(s_more))) {  // (the whole block)
    for (int q0 = 0; q0 < n_lower; q0 += kSortThreads) {
      const int q = q0 + t;
      int m = 0, p = 0, up0 = 0, nup = 0, n = 0;
      int h0 = -1, h1 = -1;  // the lists of the two bins
      bool listed = true, mine = q < n_lower;
      if (mine) {
        m = lower_module(s_lpre, q);
        p = s_key0[2 * m] + (q - s_lpre[m]);
        up0 = s_key0[2 * m + 1];
        nup = s_key0[2 * m + 2] - up0;
        if (!again) {
          n = gload(reinterpret_cast<const int4 *>(w.hcp), p).w;
          mine = md_listed(n, nup);
        }
      }
      float4 hi = make_float4(0.f, 0.f, 0.f, 0.f), win = hi;
      ModInfo mi{0};
      if (mine && nup > 0) {
        hi = gload(w.hpos, p);
        win = gload(g.win, m0 + m);
        mi.bits = gp(g.info)[m0 + m];
        const int mode = s_odd[m];
        const float4 mod = s_mod[m];
        int b0 = 0, b1 = 0;
        if (mode == 0) {
          float u;
          u_of(mod, hi, &u);
          b0 = bin_of(u - mod.z, mod.w);
          b1 = bin_of(u + mod.z, mod.w);
        } else if (mode == 1 && again) {
          const float d = direction(hi.x, hi.y);
          const float3 b = make_float3(mod.x, mod.y, mod.z);
          b0 = md_bin(d - b.x, b) & (kMdBins - 1);
          b1 = md_bin(d + b.x, b) & (kMdBins - 1);
        } else {
          listed = false;
        }
        if (listed) {
          h0 = s_head[m * kMdBins + b0];
          h1 = b1 != b0 ? s_head[m * kMdBins + b1] : -1;
        }
      }
      // the first pass counts (again: no search has), the second fills the list
      int list = -1, k = 0;
      for (int pass = again ? 0 : 1; pass < 2; ++pass) {
        if (pass == 1) {
          const int all = mine && md_listed(n, nup) ? n : 0, x = wave_inclusive(all), sum = __builtin_amdgcn_readlane(x, 63);
          if (sum == 0) break;
          int at = 0;
          if (lane == 63) at = atomicAdd(w.ctr + C_NMDLIST, sum);
          at = __builtin_amdgcn_readlane(at, 63) + x - all;
          mine = all > 0;
          if (mine && at >= 0 && at + (long)all <= (long)kLsCache * w.cap_md) list = at;
          // in any order from the bins, if the fill ranks them with fewer steps than one pass over
          // the module takes, which finds them in order
          listed = listed && (long)all * all <= 4L * nup;
          if (mine) gstore(reinterpret_cast<int4 *>(w.hcp), p, make_int4(list, listed ? 0 : 1, 0, n));  // (-1: the fill tests again)
          mine = list >= 0;
        }
        MdKept r;
        auto take = [&](int j) {
          if (pass == 0) r.take(j);
          else if (k < n) gp(w.ls_cache)[(long)list + k++] = j;
        };
        if (mine && listed) {
          int i = h0, rest = h1;
          if (i < 0) {
            i = rest;
            rest = -1;
          }
          while (i >= 0) {
            const float4 hj = gload(w.hpos, j0 + i);
            const int j = j0 + i - up0;
            i = fits ? (int)(short)s_next[i] : gp(reinterpret_cast<const int *>(w.hcp + j0 + i))[0];
            if (i < 0) {
              i = rest;
              rest = -1;
            }
            if (md_pass(hi, hj, win, mi)) take(j);
          }
        } else if (mine) {
          for (int j = 0; j < nup; ++j)
            if (md_pass(hi, gload(w.hpos, up0 + j), win, mi)) take(j);
        }
        if (pass == 0 && mine) {
          n = r.n;
          gstore(reinterpret_cast<int4 *>(w.hcp), p, r.packed());
          if (n > 0) atomicAdd(&s_nmd[m], n);
        }
      }
    }
    __syncthreads();
  }
  if (t < kBucketMods && m0 + t < n_mod) {
    gp(w.md_cnt)[m0 + t] = s_nmd[t];
    if (s_nmd[t] > 0)
      gstore(w.mod_disc, 2 * (m0 + t), anchor_disc(unordered(s_x0[t]), unordered(s_x1[t]), unordered(s_y0[t]), unordered(s_y1[t])));
  }
  if (t == 0) {
    int tot = 0;
    for (int m = 0; m < kBucketMods; ++m) tot += s_nmd[m];
    gp(w.md_tot)[c] = tot;
  }
}

// The MDs of a coarse bucket, in row-major (lower, upper) order per module: the
// offset of each of the bucket's lower hits is the MDs of the buckets before
// (summed here) plus a scan over the lower hits before it.  Partners that the
// search did not keep come from its list, or are searched again.
template <bool CROWDED>
__global__ __launch_bounds__(kSortThreads) void k_md_fill(const Ws *__restrict__ wb, DevGeom g) {
  __shared__ int s_key0[kFineKeys + 1], s_lpre[kBucketMods + 1], s_red[kSortWaves];
  __shared__ int s_at[kBucketMods + 1];  // the modules' first MDs, from the bucket's first
  __shared__ int s_r0[kBucketMods], s_r1[kBucketMods], s_z0[kBucketMods], s_z1[kBucketMods];
  __shared__ int s_az[kBucketMods * kAzBins];  // MDs per module and azimuth bin
  static_assert(kBucketMods * kAzBins == kSortThreads, "one bin a thread");
  const Ws &w = wb[blockIdx.y];
  const int wv = wave_id(), lane = lane_id(), t = threadIdx.x;
  const int n_mod = g.n_mod, nc = n_coarse(n_mod), nkeys = 2 * n_mod, c = blockIdx.x;
  if (c >= nc) return;  // the whole block
  int v = 0;
  for (int j = t; j < c; j += kSortThreads) v += gp(w.md_tot)[j];
  v = wave_total(v);
  if (lane == 0) s_red[wv] = v;
  if (t <= kFineKeys) s_key0[t] = gp(w.boff)[min(c * kFineKeys + t, nkeys)];
  s_az[t] = 0;
  if (t < kBucketMods) {
    s_r0[t] = s_z0[t] = 0x7fffffff;
    s_r1[t] = s_z1[t] = (int)0x80000000;
  }
  __syncthreads();
  int run = 0;
#pragma unroll
  for (int q = 0; q < kSortWaves; ++q) run += s_red[q];
  const int m0 = c * kBucketMods;
  if (wv == 0) {
    lower_prefix(s_key0, s_lpre);
    // the modules' offsets; after the last one, the totals
    const int n = lane < kBucketMods && m0 + lane < n_mod ? gp(w.md_cnt)[m0 + lane] : 0;
    const int at = run + wave_inclusive(n) - n;
    if (lane <= kBucketMods) s_at[lane] = at - run;  // (lanes past the modules count none)
    if (lane < kBucketMods && m0 + lane < n_mod) {
      gp(w.md_off)[m0 + lane] = at;
      if (m0 + lane == n_mod - 1) {
        gp(w.md_off)[n_mod] = at + n;
        put_total(w, at + n, w.cap_md, C_RMD, C_NMD);
      }
    }
  }
  __syncthreads();
  const int n_lower = s_lpre[kBucketMods], keep = min(g.tiles.md_cache, kMdKeep), first = run;
  for (int q0 = 0; q0 < n_lower; q0 += kSortThreads) {
    const int q = q0 + t;
    int m = 0, p = 0;
    int4 r = make_int4(0, 0, 0, 0);
    if (q < n_lower) {
      m = lower_module(s_lpre, q);
      p = s_key0[2 * m] + (q - s_lpre[m]);
      r = gload(reinterpret_cast<const int4 *>(w.hcp), p);
    }
    const int n = r.w, x = wave_inclusive(n);
    __syncthreads();  // the previous reads of s_red
    if (lane == 63) s_red[wv] = x;
    __syncthreads();
    int pos = run + x - n;
    for (int i = 0; i < kSortWaves; ++i) {
      if (i < wv) pos += s_red[i];
      run += s_red[i];
    }
    if (n == 0) continue;
    const int up0 = s_key0[2 * m + 1], nup = s_key0[2 * m + 2] - up0;
    const ModInfo mi{gp(g.info)[m0 + m]};
    const float4 hi = gload(w.hpos, p);
    const int lower = gp(w.hidx)[p];
    const float4 disc = gload(w.mod_disc, 2 * (m0 + m));
    const int bin = m * kAzBins + azimuth_bin(disc.w * frcp(disc.z), (disc.x * hi.y - disc.y * hi.x) * (frcp(disc.w) * frcp(hi.w)));
    atomicMin(&s_r0[m], ordered(hi.w));
    atomicMax(&s_r1[m], ordered(hi.w));
    atomicMin(&s_z0[m], ordered(hi.z));
    atomicMax(&s_z1[m], ordered(hi.z));
    auto put = [&](int at, int j, const float4 &hj) {
      if (at >= w.cap_md) return;
      gstore(w.md_hits, at, make_int2(lower, gp(w.hidx)[up0 + j]));
      gp(w.md_mod)[at] = m0 + m;
      gp(w.inc_cnt)[at] = 0;
      gstore(w.md_pos, at, hi);
      gp(w.inc_off)[at] = (int)((unsigned)bin | (unsigned)atomicAdd(&s_az[bin], 1) << 9);
      put_stub(w, g, at, md_stub(hi, hj, mi));
    };
    if (n <= keep && nup <= 0xffff) {
      for (int i = 0; i < n; ++i) {
        const int word = i < 2 ? r.x : (i < 4 ? r.y : r.z);
        const int j = (word >> (16 * (i & 1))) & 0xffff;
        put(pos + i, j, gload(w.hpos, up0 + j));
      }
    } else if (CROWDED && md_listed(n, nup) && r.x >= 0 && keep == kMdKeep) {
      const auto list = gp(w.ls_cache) + r.x;
      for (int i = 0; i < n; ++i) {
        const int j = list[i];
        int at = i;
        if (r.y == 0) {  // (in any order: its place is its rank)
          at = 0;
#pragma unroll 8
          for (int k = 0; k < n; ++k) at += list[k] < j ? 1 : 0;
        }
        const int jj = min(max(j, 0), nup - 1);  // (lists overlap only if their count overflowed: the event is refused)
        put(pos + at, jj, gload(w.hpos, up0 + jj));
      }
    } else {
      const float4 win = gload(g.win, m0 + m);
      for (int j = 0; j < nup; ++j) {
        const float4 hj = gload(w.hpos, up0 + j);
        if (md_pass(hi, hj, win, mi)) put(pos++, j, hj);
      }
    }
  }
  // each module's MDs grouped by azimuth, and its anchors' ranges of radius and z
  __syncthreads();
  int at = s_az[t];
  for (int o = 1; o < kAzBins; o <<= 1) {
    const int v = __shfl_up(at, o, kAzBins);
    if ((t & (kAzBins - 1)) >= o) at += v;
  }
  at -= s_az[t];
  if (m0 + t / kAzBins < n_mod) gp(w.mod_az)[(long)m0 * kAzBins + t] = (unsigned short)min(at, 0xffff);
  __syncthreads();
  s_az[t] = first + s_at[t / kAzBins] + at;
  __syncthreads();
  const int last = min(first + s_at[kBucketMods], w.cap_md);
  for (int i = first + t; i < last; i += kSortThreads) {
    const unsigned v = (unsigned)gp(w.inc_off)[i];  // bin and place in it (below 2^23, the largest capacity)
    const int p = s_az[v & 511u] + (int)(v >> 9);
    if (p < w.cap_md) gp(w.md_az)[p] = i;
  }
  if (t < kBucketMods && s_at[t + 1] > s_at[t])
    gstore(w.mod_disc, 2 * (m0 + t) + 1,
           make_float4(unordered(s_r0[t]), unordered(s_r1[t]), unordered(s_z0[t]), unordered(s_z1[t])));
}

// ------------------------------------------------------------- a2: LS
// Pre-tests of the segment azimuth window that only save work.  For inner
// anchor A and a partner module whose anchors lie in an x-y disc (centre C,
// radius rho; written by the MD fill), every term of ls_pass's window W is at
// most its value at the largest partner radius r_B <= |C| + rho: the
// threshold term (ub - ua) / sqrt(1 - ub^2) and the impact-parameter term
// D0 (1/r_A - 1/r_B) grow with r_B (the latter is below D0 / r_A) and the
// pitch terms are below (h_A + h_B) / r_A for an outgoing segment.  With the
// margins below (far above rounding) Wmax >= W, so a candidate failing
// |A x B| <= Wmax r_A r_B fails ls_pass; and since |A x B| = r_A |n.B| >= r_A
// (|n.C| - rho) for the unit normal n of A, with r_B <= |C| + rho, a module
// failing |n.C| - rho <= Wmax (|C| + rho) has no candidate that can pass.
//
// The pre-tests use the hardware reciprocal, reciprocal square root and
// square root (v_rcp_f32, v_rsq_f32, v_sqrt_f32: within 1 ulp each) instead of
// correctly rounded division and square root; their results differ from the
// exact values by a few parts in 1e7, far inside each pre-test's margin, so
// the pre-tests stay supersets of the exact selection that decides.

__device__ __forceinline__ float ls_window_bound(const float4 &A, ModInfo ma, float4 disc, ModInfo mb, float d0) {
  const float ub = kHalfKmax * ((disc.w + disc.z) + mb.er());
  if (!(ub < 0.99f)) return 3.0e38f;  // no useful bound
  const float ua = kHalfKmax * (A.w - ma.er());
  const float w = (ub - ua) * frsq(1.0f - ub * ub) + (d0 + ma.hphi() + 0.005f) * frcp(A.w);
  return (w * kMargin + kEps) * 1.01f + 1e-6f;
}

__device__ __forceinline__ bool ls_module_may_pass(const float4 &A, float4 disc, float wmax) {
  const float dn = fabsf(A.x * disc.y - A.y * disc.x) * frcp(A.w);
  return dn - disc.z <= (wmax * (disc.w + disc.z)) * 1.001f + 1e-4f;
}

// What the pair loop of the count pass needs of a linked module: its centre's
// direction, distance, radius (anchor_disc), ranges of r and z, the window
// bound's two terms (ls_window_bound) and the scale of azimuth_bin.
struct LsLink {
  float nx, ny, c, rho;
  float4 rng;
  float ub, rs, bins;
};
__device__ __forceinline__ LsLink ls_link(const float4 &disc, const float4 &rng, ModInfo mb) {
  LsLink l;
  const float ic = frcp(disc.w);
  l.nx = disc.x * ic; l.ny = disc.y * ic; l.c = disc.w; l.rho = disc.z;
  l.rng = rng;
  l.ub = kHalfKmax * ((disc.w + disc.z) + mb.er());
  l.rs = l.ub < 0.99f ? frsq(1.0f - l.ub * l.ub) : -1.0f;
  l.bins = disc.z < 0.5f * disc.w ? disc.w * frcp(disc.z) : -1.0f;
  return l;
}
// And of an inner MD: 1 / r, 1 / separation (negative: none), the window
// bound's terms and twice the pitch.
__device__ __forceinline__ float4 ls_inner(const float4 &A, float2 st, ModInfo ma, float d0) {
  const float ia = frcp(A.w);
  return make_float4(ia, st.y > 0.0f ? frcp(st.y) : -1.0f, kHalfKmax * (A.w - ma.er()), (d0 + ma.hphi() + 0.005f) * ia);
}

// The bins of the linked module's kAzBins, first and end, that hold every MD B
// past the window and the stub check of the inner MD A; false if there is none
// (ls_window_bound and ls_module_may_pass included, on the link's constants).
// With D the azimuth from A to B, |sin D| <= wmax (ls_window_may_pass; A.B > 0
// and r_B > r_A are ls_pass's own).  A barrel A's stub check bounds t, the
// tangent of the angle at B between the chord and the radial direction
// (|st.x - st.y t| <= err, largest for the shortest chord), and t = r_A sin D /
// (r_B - r_A cos D) with r_B in the module's range and cos D in
// [sqrt(1 - wmax^2), 1]; where the window allows chords near the tangent, or r_B
// cos D <= r_A, that bound is not taken.  An endcap A's check bounds st.y r_A
// sin D / |dz|, with dz in the module's range.  The margins are those of
// ls_stub_may_pass, and a further 1e-4 of the bound and 1e-5 in sine; rounding
// stays below 1e-6 of both.  All bins for wide discs and windows, for A far
// from the module in azimuth, and where the disc has no direction (its centre on
// the beam line, or so far out that its distance overflows: sd and cd are NaN).
__device__ __forceinline__ bool ls_azimuth_bins(const float4 &A, float2 st, const float4 &in, ModInfo ma, const LsLink &l,
                                                ModInfo mb, float d0, int *b0, int *b1) {
  *b0 = 0;
  *b1 = kAzBins;
  // ls_window_bound and ls_module_may_pass, with the direction's products instead of the disc's
  const float wmax = l.rs < 0.0f ? 3.0e38f : (((l.ub - in.z) * l.rs + in.w) * kMargin + kEps) * 1.01f + 1e-6f;
  const float sd = (l.nx * A.y - l.ny * A.x) * in.x, cd = (l.nx * A.x + l.ny * A.y) * in.x;
  if (l.c * fabsf(sd) - l.rho > (wmax * (l.c + l.rho)) * 1.001f + 1e-4f) return false;  // (no direction: kept)
  if (!(l.bins > 0.0f && wmax < 0.69f && cd > 0.5f)) return true;
  const float sw = wmax * 1.0001f + 1e-6f, cw = 0.9999f * __builtin_amdgcn_sqrtf(1.0f - sw * sw);
  const float e2 = (ma.endcap() ? ma.hlong() : ma.hphi()) + (mb.endcap() ? mb.hlong() : mb.hphi());
  float lo = -sw, hi = sw;
  float near, far, err;  // sin D in [(x -+ err) * near or far] / (st.y r_A)
  bool bound;
  const float x = st.x;
  if (!ma.endcap()) {
    near = l.rng.x - A.w;
    far = l.rng.y - A.w * cw;
    bound = l.rng.x * cw > A.w * 1.0001f && A.w * sw <= 0.9f * near;
    err = (2.0f * ma.hphi() + (2.0f * st.y) * (e2 * frcp(near) + d0 * in.x)) * (kMargin * 1.0005f) + kEps +
          2e-4f * fabsf(x);
  } else {
    const float z0 = l.rng.z - A.z, z1 = l.rng.w - A.z;
    near = fminf(fabsf(z0), fabsf(z1));
    far = fmaxf(fabsf(z0), fabsf(z1));
    bound = z0 > 0.0f || z1 < 0.0f;
    const float chord = fmaxf(fabsf(l.rng.x - A.w), fabsf(l.rng.y - A.w)) + 1.1f * A.w * sw;
    err = (2.0f * ma.hphi() + st.y * (e2 + chord * d0 * in.x) * frcp(near)) * (kMargin * 1.033f) + kEps +
          0.0313f * fabsf(x);
  }
  if (bound && in.y > 0.0f) {
    const float f = in.x * in.y, x0 = x - err, x1 = x + err;
    const float p = x0 * (x0 >= 0.0f ? near : far) * f, q = x1 * (x1 >= 0.0f ? far : near) * f;
    lo = fmaxf(lo, p - (1e-4f * fabsf(p) + 1e-5f));
    hi = fminf(hi, q + (1e-4f * fabsf(q) + 1e-5f));
    if (!(lo <= hi)) return false;
  }
  // sin(D + the azimuth from the disc's centre to A), within a right angle
  const float cl = __builtin_amdgcn_sqrtf(1.0f - lo * lo), ch = __builtin_amdgcn_sqrtf(1.0f - hi * hi);
  if (cl * cd - lo * sd > 0.0f) *b0 = azimuth_bin(l.bins, lo * cd + cl * sd - 1e-5f);
  if (ch * cd - hi * sd > 0.0f) *b1 = azimuth_bin(l.bins, hi * cd + ch * sd + 1e-5f) + 1;
  return true;
}

// One MD's stub check of ls_pass (ls_stub_ok) evaluated with the fast
// operations, from the chord (sx, sy) = B - A, its inverse length il, dz = zB -
// zA, the chord's sine sn against the radial direction the check uses, eang
// and the MD's radius rp: every quantity is within 2e-6 relative of the exact
// one (a chain of at most six operations of <= 2 ulp), except that 1 - s^2
// loses relative precision as s^2 -> 1: chords within asin(sqrt(0.9)) of the
// tangent skip the pre-test (the exact test decides), which bounds the error of
// the predicted displacement at 4e-5 relative.  The margins (1e-4 of the
// prediction and of the error) exceed those bounds, so whatever passes the
// exact check passes this one.
__device__ __forceinline__ bool ls_stub_may_pass(float2 st, ModInfo m, float sn, float sx, float sy, float il, float dz,
                                                 float eang, float rp, float d0) {
  float pred, err;
  if (!m.endcap()) {
    const float sn2 = sn * sn;
    if (!(sn2 < 0.9f)) return true;
    pred = (st.y * sn) * frsq(1.0f - sn2);
    err = 2.0f * m.hphi() + (2.0f * st.y) * (eang + d0 * frcp(rp));
  } else {
    const float adz = fabsf(dz);
    if (!(adz > 0.0f)) return false;  // the exact check's own rejection, on the same operands
    const float ds = st.y * (sx * sx + sy * sy) * il * frcp(adz);
    pred = ds * sn;
    err = (2.0f * m.hphi() + (float)0.03 * fabsf(pred)) + ds * (eang + d0 * frcp(rp));
  }
  return fabsf(st.x - pred) <= (err * kMargin) * 1.0001f + kEps + 1e-4f * fabsf(pred);
}

// The inner MD's stub check (its chord sine taken at the outer anchor B).
__device__ __forceinline__ bool ls_inner_stub_may_pass(const float4 &A, const float4 &B, float2 st, ModInfo ma,
                                                       ModInfo mb, float d0) {
  const float sx = B.x - A.x, sy = B.y - A.y;
  const float il = frsq(sx * sx + sy * sy);  // 1 / |AB|
  const float sn = (B.x * sy - B.y * sx) * frcp(B.w) * il;
  const float ea2 = ma.endcap() ? ma.hlong() : ma.hphi();
  const float eb2 = mb.endcap() ? mb.hlong() : mb.hphi();
  return ls_stub_may_pass(st, ma, sn, sx, sy, il, B.z - A.z, (ea2 + eb2) * il, A.w, d0);
}

__device__ __forceinline__ bool ls_window_may_pass(const float4 &A, const float4 &B, float wmax) {
  const float c = A.x * B.y - A.y * B.x;
  return fabsf(c) <= wmax * (A.w * B.w);
}

// The checks of ls_pass that a pair past the two pre-tests above still fails
// most often, on the pair itself: the signs of dr and of A.B (the same
// operations as ls_pass), the x-y window with the outer radius of this B
// instead of the module's (all terms of w are positive for dr > 0, so the fast
// operations' few-ulp errors stay far inside the 1e-4 margin; ub >= 0.99
// leaves the decision to the exact test), and the outer MD's stub check, its
// chord sine taken at the inner anchor A.
__device__ __forceinline__ bool ls_pair_may_pass(const float4 &A, const float4 &B, float2 sb, ModInfo ma, ModInfo mb,
                                                 float d0) {
  const float dr = B.w - A.w;
  if (!(dr > 0.0f)) return false;
  if (!(A.x * B.x + A.y * B.y > 0.0f)) return false;
  const float ub = kHalfKmax * (B.w + mb.er());
  if (ub < 0.99f) {
    const float ua = kHalfKmax * (A.w - ma.er());
    const float ra = frcp(A.w), rb = frcp(B.w);
    const float wv = (ub - ua) * frsq(1.0f - ub * ub) + (d0 * dr) * (ra * rb) + ma.hphi() * ra + mb.hphi() * rb;
    const float c = A.x * B.y - A.y * B.x;
    if (!(fabsf(c) <= ((wv * kMargin + kEps) * (A.w * B.w)) * 1.0001f + 1e-6f)) return false;
  }
  const float sx = B.x - A.x, sy = B.y - A.y;
  const float il = frsq(sx * sx + sy * sy);
  const float sn = (A.x * sy - A.y * sx) * frcp(A.w) * il;
  const float ea2 = ma.endcap() ? ma.hlong() : ma.hphi();
  const float eb2 = mb.endcap() ? mb.hlong() : mb.hphi();
  return ls_stub_may_pass(sb, mb, sn, sx, sy, il, B.z - A.z, (ea2 + eb2) * il, B.w, d0);
}

constexpr int kMaxEdges = 128;  // module-map targets per module (checked when the geometry is loaded)

// Drops the first 64 entries of a wave's queue (two arrays of 128): the rest (< 64)
// entries behind them move to its front.
template <class T>
__device__ __forceinline__ void queue_pop64(int *qa, T *qb, int rest) {
  const int lane = lane_id();
  int va = 0;
  T vb = 0;
  if (lane < rest) {
    va = qa[64 + lane];
    vb = qb[64 + lane];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane < rest) {
    qa[lane] = va;
    qb[lane] = vb;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void queue_pop64(int *qa, int rest) {
  const int lane = lane_id();
  const int va = lane < rest ? qa[64 + lane] : 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane < rest) qa[lane] = va;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Count pass of the segment search: one wave per group of up to kLsGroup
// consecutive inner MDs, taken in chunks of MDs of one module whose (inner MD,
// linked module) pairs are flattened over the lanes.  A pair's candidates are
// the MDs in a run of the module's azimuth bins (ls_azimuth_bins; in MD order
// and all of them if the module map does not ascend, since the fill then could
// not put the partners in order).  They go 64 per round through the pair pre-test
// (ls_pair_may_pass: a fifth of them pass on PU200 events), its survivors,
// queued, through the full selection, which thus runs on full waves of likely
// pairs.  The pairs of one inner MD are consecutive in the queue; a passing
// pair's rank among its MD's passing pairs is the MD's count from earlier flushes
// plus the passing lanes of its run below it.  Writes each MD's count and caches
// up to tiles.ls_cache partners as found.
//
// Bound by the vector units: a PU200 event's 21.7M candidates of the modules
// that the window reaches, each tested, took 72.5M wave instructions and 120 us
// (eight events 872); the bins leave 4.9M, 53M instructions before the links'
// constants were taken out of the pair loop, and 86-90 us (588), of which the
// pairs (4.3M) take the most.  The bins cost the MD fill 13 -> 20 us (68 -> 109)
// and their order the segment fill 24 -> 32 us (115 -> 136).
constexpr int kLsPairs = 2 * kMaxEdges;  // (inner MD, linked module) pairs of a chunk in LDS

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7))) void k_ls_count(
    const Ws *__restrict__ wb, DevGeom g, int group) {
  const Ws &w = wb[blockIdx.y];
  // (inner MD, linked module) pairs left with candidates, in (MD, map) order: first
  // candidate less the candidates before it, those, and the pair's inner MD (its slot in
  // the group) with the module's info
  __shared__ int s_ej[kWaves][kLsPairs], s_ep[kWaves][kLsPairs], s_ek[kWaves][kLsPairs];
  __shared__ int s_mark[kWaves][64];            // a pair's candidates start here
  // (inner MD, candidate) pairs past the pair pre-test, in order, as partner | module info
  // << 30 and the inner MD's slot in the group
  __shared__ int s_r[kWaves][128];
  __shared__ unsigned char s_rg[kWaves][128];
  __shared__ float4 s_A[kWaves][kLsGroup], s_in[kWaves][kLsGroup];  // the group's inner MDs
  __shared__ float2 s_sa[kWaves][kLsGroup];
  __shared__ int s_mia[kWaves][kLsGroup], s_cnt[kWaves][kLsGroup], s_mm[kWaves][kLsGroup];
  const int n_md = uload(w.ctr + C_NMD);
  const int wv = wave_id(), lane = lane_id();
  const int wpb = blockDim.x >> 6;
  const int waves_total = gridDim.x * wpb;
  const int n_grp = (n_md + group - 1) / group;
  const int keep = g.tiles.ls_cache;
  for (int gi = blockIdx.x * wpb + wv; gi < n_grp; gi += waves_total) {
    const int a0 = gi * group;
    const int na = min(group, n_md - a0);
    if (lane < na) {
      const int a = a0 + lane;
      const int ma = gp(w.md_mod)[a];
      const float4 A = gload(w.md_pos, a);
      const float2 sa = get_stub(w, g, a);
      const ModInfo mia{gp(g.info)[ma]};
      s_A[wv][lane] = A;
      s_sa[wv][lane] = sa;
      s_mia[wv][lane] = mia.bits;
      s_in[wv][lane] = ls_inner(A, sa, mia, g.d0max);
      s_mm[wv][lane] = ma;
      s_cnt[wv][lane] = 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int nr = 0;
    // the full selection on the first n pairs of s_r (n <= 64)
    auto select = [&](int n) {
      bool pass = false;
      int e = 0, q = -1;
      if (lane < n) {
        e = s_r[wv][lane];
        q = s_rg[wv][lane];
        const int b = e & 0x3fffffff;
        float2 beta;
        pass = ls_pass(s_A[wv][q], gload(w.md_pos, b), s_sa[wv][q], get_stub(w, g, b), ModInfo{s_mia[wv][q]},
                       ModInfo{(int)((unsigned)e >> 30)}, &beta, g.d0max);
      }
      const unsigned long long m = __ballot(pass);
      const int qp = __shfl_up(q, 1, 64), qn = __shfl_down(q, 1, 64);
      const unsigned long long starts = __ballot(lane == 0 || q != qp);
      const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
      const int first = 63 - __clzll(starts & upto);  // first lane of this lane's run
      const int below = __popcll(m & ((1ull << lane) - 1ull) & ~((1ull << first) - 1ull));
      int before = 0;
      if (lane < n) before = s_cnt[wv][q];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (pass && before + below < keep)  // the partner and its module's info word (2 bits) in one int
        gp(w.ls_cache)[(long)(a0 + q) * kLsCache + before + below] = e;
      if (lane < n && (lane == n - 1 || qn != q)) s_cnt[wv][q] = before + below + (pass ? 1 : 0);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    // the linked modules' data of the current inner module (one per lane, when it has
    // at most 64 of them): consecutive inner MDs mostly share their module
    int cur_ma = -1, e0 = 0, ne = 0;
    int r_mb = 0, r_first = 0, r_cnt = 0, r_info = 0;
    LsLink r_l{};
    auto linked = [&](int kk, int &mb, int &first, int &cnt, int &info, LsLink &l) {
      mb = gp(g.map_tgt)[e0 + kk];
      first = gp(w.md_off)[mb];
      const int last = min(gp(w.md_off)[mb + 1], n_md);
      cnt = last > first ? last - first : 0;
      info = gp(g.info)[mb];
      l = ls_link(gload(w.mod_disc, 2 * mb), gload(w.mod_disc, 2 * mb + 1), ModInfo{info});
    };
    // Chunks of consecutive inner MDs of one module, at most kLsPairs / ne of them, so
    // that every (inner MD, linked module) pair of the chunk fits the LDS list: the
    // prologue and the candidate rounds run over the chunk's pairs flattened, which
    // fills the lanes that one MD's ~27 linked modules and ~90 candidates leave idle.
    for (int k0 = 0; k0 < na;) {
      const int ma = __builtin_amdgcn_readfirstlane(s_mm[wv][k0]);
      if (ma != cur_ma) {
        cur_ma = ma;
        e0 = uload(g.map_off + ma);
        ne = uload(g.map_off + ma + 1) - e0;  // <= kMaxEdges = kLsPairs, checked when the geometry is loaded
        if (ne <= 64 && lane < ne) linked(lane, r_mb, r_first, r_cnt, r_info, r_l);
      }
      const int cap_k = ne > 0 ? kLsPairs / ne : na;
      int k1 = k0 + 1;
      while (k1 < na && k1 - k0 < cap_k && __builtin_amdgcn_readfirstlane(s_mm[wv][k1]) == ma) ++k1;
      const int npair = (k1 - k0) * ne;
      const float rne = ne > 0 ? 1.0f / (float)ne : 0.0f;
      int run = 0, n_ne = 0;
      for (int p0 = 0; p0 < npair; p0 += 64) {
        const int p = p0 + lane;
        const int2 ke = divmod22(p < npair ? p : 0, ne > 0 ? ne : 1, rne);  // (MD of the chunk, link)
        int mb = 0, first = 0, cnt = 0, info = 0;
        LsLink l = r_l;
        if (ne <= 64) {  // the links' data from the lanes that hold them
          const auto from = [&](auto v) { return __shfl(v, ke.y, 64); };
          mb = from(r_mb); first = from(r_first); cnt = from(r_cnt); info = from(r_info);
          l = LsLink{from(r_l.nx), from(r_l.ny), from(r_l.c), from(r_l.rho),
                     make_float4(from(r_l.rng.x), from(r_l.rng.y), from(r_l.rng.z), from(r_l.rng.w)),
                     from(r_l.ub), from(r_l.rs), from(r_l.bins)};
        }
        const int kk = k0 + ke.x;
        if (p < npair) {
          if (ne > 64) linked(ke.y, mb, first, cnt, info, l);
          if (cnt > 0) {
            int az0, az1;
            if (!ls_azimuth_bins(s_A[wv][kk], s_sa[wv][kk], s_in[wv][kk], ModInfo{s_mia[wv][kk]}, l, ModInfo{info}, g.d0max,
                                 &az0, &az1)) {
              cnt = 0;
            } else if (g.map_asc && cnt < 0xffff) {
              const int l0 = gp(w.mod_az)[mb * kAzBins + az0];
              const int l1 = az1 < kAzBins ? (int)gp(w.mod_az)[mb * kAzBins + az1] : cnt;
              first += l0;
              cnt = max(l1 - l0, 0);
            }
          }
        } else {
          cnt = 0;
        }
        int x = cnt;
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(x, o, 64);
          if (lane >= o) x += y;
        }
        const unsigned long long live = __ballot(cnt > 0);
        if (cnt > 0) {
          const int q = n_ne + lanes_below(live);
          s_ep[wv][q] = run + x - cnt;
          s_ej[wv][q] = first - (run + x - cnt);
          s_ek[wv][q] = kk | info << 8;
        }
        n_ne += __popcll(live);
        run += __builtin_amdgcn_readfirstlane(__shfl(x, 63, 64));
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int total = run;
      // Candidates go 64 per round.  The candidate c of lane L lies in the last pair whose
      // candidates start at or before c: the pairs starting before the round (jlo of
      // them) plus those starting at or below L in it, found by marking the round's
      // starts (distinct, as every listed pair has candidates) and a ballot.
      int jlo = 0;
      // at least one round, so that the group's last chunk flushes the queue
      for (int c0 = 0; c0 < (total > 0 ? total : 1); c0 += 64) {
        s_mark[wv][lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (jlo + lane < n_ne) {
          const int p = s_ep[wv][jlo + lane] - c0;  // >= 0: it starts at or after c0
          if (p < 64) s_mark[wv][p] = 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const unsigned long long starts = __ballot(s_mark[wv][lane] != 0);
        const int c = c0 + lane;
        bool ok = false;
        int e = 0, q = 0;
        if (c < total) {
          const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
          const int j = jlo - 1 + __popcll(starts & upto);
          const int ki = s_ek[wv][j];
          q = ki & 0xff;
          int b = s_ej[wv][j] + c;
          if (g.map_asc) b = gp(w.md_az)[b];
          const float4 A = s_A[wv][q], B = gload(w.md_pos, b);
          const ModInfo mia{s_mia[wv][q]}, mib{ki >> 8};
          e = b | (ki >> 8) << 30;
          ok = ls_pair_may_pass(A, B, get_stub(w, g, b), mia, mib, g.d0max);
        }
        jlo += __popcll(starts);
        const unsigned long long m = __ballot(ok);
        if (ok) {
          const int pos = nr + lanes_below(m);
          s_r[wv][pos] = e;
          s_rg[wv][pos] = (unsigned char)q;
        }
        nr += __popcll(m);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the queue holds < 64 entries before a round adds at most 64, and is drained 64 at
        // a time; the group's last round drains it completely
        const bool fin = k1 == na && c0 + 64 >= total;
        while (nr >= 64) {
          select(64);
          queue_pop64(s_r[wv], s_rg[wv], nr - 64);
          nr -= 64;
        }
        if (fin && nr > 0) {
          select(nr);
          nr = 0;
        }
      }
      k0 = k1;
    }
    if (lane < na) gp(w.ls_cnt)[a0 + lane] = s_cnt[wv][lane];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Segments per tile of MDs (2^sh_ls of them), for the offsets of the fill, and
// the list of the MDs with more segments than the count pass caches (428 of
// 138k on a PU200 event), which the fill searches again.  The count pass does
// not do this itself: an atomic per group of MDs there delays the wave's next
// gathers until it is done (the count 0.119 -> 0.130 ms for one event, 0.88 ->
// 0.93 ms for eight), more than this launch takes.
//
// Blocks from n_sum on do what the pixel stages need and nothing else waits for:
// the seeds' direction table (every block scans the group counts for itself)
// and the pLS duplicate removal (seeds sharing at least 3 pixel hits; the lower
// seed index wins).
__device__ __forceinline__ bool pls_survives(const Ws &w, int s) {
  int hs[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) hs[k] = gp(w.hits4)[4 * (long)s + k];
  auto loses_to = [&](int t) {
    int sh = 0;
    for (int i = 0; i < 4; ++i) {
      bool f = false;
      for (int j = 0; j < 4; ++j) f |= (gp(w.hits4)[4 * (long)t + j] == hs[i]);
      sh += f ? 1 : 0;
    }
    return sh >= 3;
  };
  for (int k = 0; k < 4; ++k) {
    const int h = hs[k];
    if (h < 0 || h >= w.n_hits) continue;
    const int o = gp(w.ph_owner)[h];
    if (o < s && loses_to(o)) return false;
    for (int q = gp(w.ph_head)[h]; q >= 0; q = gp(w.ph_next)[q])
      if ((q >> 2) < s && loses_to(q >> 2)) return false;
  }
  return true;
}

__global__ __launch_bounds__(kBlock) void k_ls_sums(const Ws *__restrict__ wb, int keep, int n_sum) {
  __shared__ int s_red[kWaves];
  __shared__ int s_off[kSeedKeys];
  const Ws &w = wb[blockIdx.y];
  if ((int)blockIdx.x >= n_sum) {
    const int S = w.n_seeds, t = threadIdx.x, lane = lane_id();
    const int q0 = ((int)blockIdx.x - n_sum) * kBlock;
    if (q0 >= S) return;  // the whole block
    // exclusive prefix of the group counts
    constexpr int kPer = kSeedKeys / kBlock;
    int c[kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum += c[i] = gp(w.seed_cnt)[t * kPer + i];
    const int x = wave_inclusive(sum);
    if (lane == 63) s_red[t >> 6] = x;
    __syncthreads();
    int ex = x - sum;
    for (int q = 0; q < (t >> 6); ++q) ex += s_red[q];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      s_off[t * kPer + i] = ex;
      ex += c[i];
    }
    __syncthreads();
    if (q0 == 0)
      for (int b = t; b <= kDirBins; b += kBlock) gp(w.sdir_off)[b] = b < kDirBins ? s_off[4 * b] : S;
    for (int s = q0 + t; s < S; s += ((int)gridDim.x - n_sum) * kBlock) {
      const Dir d = seed_dir(load_seed(w, s));
      const int pos = s_off[gp(w.seed_key)[s]] + gp(w.seed_slot)[s];
      gstore(w.sdir, pos, make_float4(d.dx, d.dy, d.lam, __int_as_float(s)));
      gp(w.sdir_pos)[s] = pos;
      gp(w.pls_keep)[s] = pls_survives(w, s) ? 1 : 0;
    }
    return;
  }
  const int n = uload(w.ctr + C_NMD), sh = w.sh_ls;
  for (int t = blockIdx.x; (t << sh) < n; t += n_sum) {
    const int j1 = min((t + 1) << sh, n);
    int v = 0;
    for (int j = (t << sh) + (int)threadIdx.x; j < j1; j += kBlock) {
      const int c = gp(w.ls_cnt)[j];
      v += c;
      if (c > keep) gp(w.ls_ovf)[atomicAdd(w.ctr + C_NLSOVF, 1)] = j;
    }
    v = block_sum(v, s_red);
    if (threadIdx.x == 0) w.ts_ls[t * kSumStride] = v;
  }
}

// ---- flattened pair search shared by T3 and T5: a wave takes 64 consecutive
// parents (one per lane), stages what their pairs need in LDS, prefix-sums
// their candidate counts and lets its 64 lanes stride over all (parent,
// candidate) pairs in order, so a parent with many candidates does not hold
// the wave.  The rank of an accepted pair among its parent's accepted pairs
// (its output position after the parent's offset in the fill) is the
// parent's count from earlier rounds plus the accepted pairs of the same
// parent on lower lanes of this round (a parent's pairs are on consecutive
// lanes).  COUNT writes the per-parent counts, FILL the objects.
__device__ __forceinline__ int pair_rank(unsigned long long m, int seg_first_lane, int before_round) {
  return before_round + lanes_below(m) - __popcll(m & ((1ull << seg_first_lane) - 1ull));
}
// Exclusive prefix of n over the wave into seg[0..64] (seg[64] = total); returns the total.
__device__ __forceinline__ int wave_segments(int n, int *seg) {
  const int lane = lane_id();
  int x = n;
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  seg[lane] = x - n;
  const int total = __shfl(x, 63, 64);
  if (lane == 0) seg[64] = total;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return total;
}

// Parent of each lane's pair in a round of 64 consecutive pairs [c0, c0 + 64)
// of a wave's flattened (parent, candidate) list, where lane k's parent owns
// pairs [start, start + n) (wave_segments' prefix): every non-empty parent
// starting in the round marks its first position (distinct positions), and a
// lane's parent is the last mark at or below it, else `carry`, the parent of
// the previous round's last pair (0 before the first round).  No per-lane walk
// over the prefix.  Called by the whole wave; updates carry.
__device__ __forceinline__ int round_parent(int start, int n, int c0, int *mark, int &carry) {
  const int lane = lane_id();
  mark[lane] = -1;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (n > 0 && start >= c0 && start < c0 + 64) mark[start - c0] = lane;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int mk = mark[lane];
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  const unsigned long long sm = __ballot(mk >= 0) & upto;
  const int from = sm ? 63 - (int)__builtin_clzll(sm) : 0;
  const int got = __shfl(mk, from, 64);
  const int e = sm ? got : carry;
  carry = __builtin_amdgcn_readfirstlane(__shfl(e, 63, 64));
  return e;
}

// Fill pass of the segment search.  Blocks [0, n_copy) write the segments of
// the inner MDs whose partners the count pass cached: a wave takes kLsCopyMds
// consecutive MDs, finds their offsets (block_prefix) and strides over their
// segments flattened, each at its rank by partner (the count finds a module's
// partners in azimuth order), with the angles ls_pass reports.
// The other blocks search again for the MDs with more segments than the cache
// holds (listed by the count pass), one wave per inner MD a.  Its candidates
// -- the MDs of every module linked to a's module, edge by edge -- are
// flattened into one list that the 64 lanes stride over, so a wave stays full
// even though each linked module holds few MDs; candidates past the pre-tests,
// then past the pair pre-test, are compacted in list order with ballot and
// mbcnt into two LDS queues, and the full selection runs on full waves of the
// second.
// Eight waves per SIMD (64 VGPRs; a few spill): the segment search is bound by
// the latency of its dependent gathers, and more resident waves hide more of
// it (measured 9% faster than the 77-VGPR, six-wave build; the same for the
// triplet and quintuplet searches made them slower).
// direct (no seeds, MD capacity of at most kDirectMds): there is no launch of
// k_ls_sums, the copying blocks sum the counts before theirs and their waves take
// their own MDs with more segments than the cache: 4 us less on a tiny event.
constexpr int kDirectMds = 8192;
constexpr int kLsCopyMds = 16;
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) void k_ls_fill(
    const Ws *__restrict__ wb, DevGeom g, int n_copy, int direct) {
  const Ws &w = wb[blockIdx.y];
  __shared__ int s_pre[kWaves][kMaxEdges + 1];  // running MD count before each edge
  __shared__ int s_first[kWaves][kMaxEdges];    // first MD of each linked module
  __shared__ int s_info[kWaves][kMaxEdges];
  __shared__ float s_wmax[kWaves][kMaxEdges];   // window bound of each linked module
  // candidates in order, as partner | module info << 30: past the candidate pre-tests
  // (s_q) and past the pair pre-test as well (s_r)
  __shared__ int s_q[kWaves][128], s_r[kWaves][128];
  __shared__ int s_val[kWaves][256];  // the copied partners of three rounds
  __shared__ int s_red[kWaves];
  const int n_md = uload(w.ctr + C_NMD);
  const int wv = wave_id(), lane = lane_id();
  const int wpb = blockDim.x >> 6;  // waves per block (a tuned launch may run fewer than kWaves)
  const int sh = direct ? 30 : w.sh_ls;  // (no tile is before the first)
  if ((int)blockIdx.x < n_copy) {
    const int keep = g.tiles.ls_cache;
    int *s_seg = s_pre[wv], *s_off = s_first[wv], *s_mark = s_q[wv];  // 65 / 64 / 64 entries
    const int per = wpb * kLsCopyMds;  // the block's MDs (in one tile)
    for (int b0 = (int)blockIdx.x * per; b0 < n_md; b0 += n_copy * per) {
      const int a0 = b0 + wv * kLsCopyMds, a = a0 + lane;
      const bool mine = lane < kLsCopyMds && a < n_md;
      const int cnt = mine ? gp(w.ls_cnt)[a] : 0;
      int before = 0;  // the block's MDs on earlier waves
      for (int j = b0 + lane; j < min(a0, n_md); j += 64) before += gp(w.ls_cnt)[j];
      const int off = block_prefix(w.ts_ls, sh, w.ls_cnt, 0, b0, s_red) + wave_total(before) +
                      wave_inclusive(cnt) - cnt;
      if (mine) {
        gp(w.ls_off)[a] = off;
        if (a == n_md - 1) {
          gp(w.ls_off)[n_md] = off + cnt;
          put_total(w, off + cnt, w.cap_ls, C_RLS, C_NLS);
        }
      }
      s_off[lane] = off;
      const int n = cnt <= keep ? cnt : 0;  // the others are searched again below
      const int total = wave_segments(n, s_seg);
      const int start = s_seg[lane];
      // A module's partners were found in azimuth order: with ascending module maps a
      // partner's place is its rank.  The partners go through a ring in LDS, a round ahead,
      // since an MD's (at most kLsCache) may lie in two rounds.
      static_assert(kLsCache <= 64, "in at most two rounds");
      int carry = 0, e_next = 0;
      auto stage = [&](int c0) __attribute__((always_inline)) {
        const int c = c0 + lane;
        e_next = round_parent(start, n, c0, s_mark, carry);
        s_val[wv][c & 255] = c < total ? gp(w.ls_cache)[(long)(a0 + e_next) * kLsCache + (c - s_seg[e_next])] : 0;
      };
      if (total > 0) stage(0);
      for (int c0 = 0; c0 < total; c0 += 64) {
        const int c = c0 + lane, e = e_next;
        if (c0 + 64 < total) stage(c0 + 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (c < total) {
          const int v = s_val[wv][c & 255], b = v & 0x3fffffff;
          int k = c - s_seg[e];
          if (g.map_asc) {
            k = 0;
            const int j1 = s_seg[e + 1];
#pragma unroll 4
            for (int j = s_seg[e]; j < j1; ++j) k += (s_val[wv][j & 255] & 0x3fffffff) < b ? 1 : 0;
          }
          const int pos = s_off[e] + k;
          if (pos < w.cap_ls) {
            const float4 B = gload(w.md_pos, b);
            gstore(w.ls_md, pos, make_int2(a0 + e, b));
            gstore(w.ls_beta, pos, ls_beta(gload(w.md_pos, a0 + e), B));
            gstore(w.ls_opos, pos, B);
            gp(w.ls_oinf)[pos] = (int)((unsigned)v >> 30);
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    if (!direct) return;
  }
  auto process = [&](const int a) {
    const int ma = gp(w.md_mod)[a];
    const float4 A = gload(w.md_pos, a);
    const float2 sa = get_stub(w, g, a);
    const ModInfo mia{gp(g.info)[ma]};
    const int e0 = gp(g.map_off)[ma];
    const int ne = gp(g.map_off)[ma + 1] - e0;  // <= kMaxEdges, checked when the geometry is loaded
    // per-edge MD ranges and their exclusive prefix over the wave
    int run = 0;
    for (int k0 = 0; k0 < ne; k0 += 64) {
      const int k = k0 + lane;
      int first = 0, cnt = 0, info = 0;
      float wm = 0.0f;
      if (k < ne) {
        const int mb = gp(g.map_tgt)[e0 + k];
        first = gp(w.md_off)[mb];
        const int last = min(w.md_off[mb + 1], n_md);
        cnt = last > first ? last - first : 0;
        info = gp(g.info)[mb];
        if (cnt > 0) {
          const float4 disc = gload(w.mod_disc, 2 * mb);
          wm = ls_window_bound(A, mia, disc, ModInfo{info}, g.d0max);
          if (!ls_module_may_pass(A, disc, wm)) cnt = 0;
        }
      }
      int x = cnt;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (k < ne) {
        s_pre[wv][k] = run + x - cnt;
        s_first[wv][k] = first;
        s_info[wv][k] = info;
        s_wmax[wv][k] = wm;
      }
      run += __shfl(x, 63, 64);
    }
    if (lane == 0) s_pre[wv][ne] = run;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int total = run;
    int out = wave_prefix(w.ts_ls, sh, w.ls_cnt, 0, a);
    // the pair pre-test on the first n candidates of s_q (n <= 64); the passing ones join s_r
    int nr = 0;
    auto sift = [&](int n) {
      bool ok = false;
      int e = 0;
      if (lane < n) {
        e = s_q[wv][lane];
        const int b = e & 0x3fffffff;
        ok = ls_pair_may_pass(A, gload(w.md_pos, b), get_stub(w, g, b), mia, ModInfo{(int)((unsigned)e >> 30)},
                              g.d0max);
      }
      const unsigned long long m = __ballot(ok);
      if (ok) s_r[wv][nr + lanes_below(m)] = e;
      nr += __popcll(m);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    // the full selection on the first n candidates of s_r (n <= 64), in candidate order
    auto select = [&](int n) {
      bool pass = false;
      int b = 0, info = 0;
      float2 beta = make_float2(0.f, 0.f);
      if (lane < n) {
        const int e = s_r[wv][lane];
        b = e & 0x3fffffff;
        info = (int)((unsigned)e >> 30);
        pass = ls_pass(A, gload(w.md_pos, b), sa, get_stub(w, g, b), mia, ModInfo{info}, &beta, g.d0max);
      }
      const unsigned long long m = __ballot(pass);
      const int pre = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      const int pos = out + pre;
      if (pass && pos < w.cap_ls) {
        gstore(w.ls_md, pos, make_int2(a, b));
        gstore(w.ls_beta, pos, beta);
        gstore(w.ls_opos, pos, gload(w.md_pos, b));
        gp(w.ls_oinf)[pos] = info;
      }
      out += __popcll(m);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    // candidates past the azimuth pre-tests and the inner MD's own stub check (both
    // necessary conditions of ls_pass) are queued in LDS, and the full selection runs
    // on full waves of them
    int nq = 0;
    int e = 0;  // edge of this lane's candidate (candidates advance monotonically)
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int c = c0 + lane;
      bool keep = false;
      int b = 0, info = 0;
      if (c < total) {
        while (s_pre[wv][e + 1] <= c) ++e;
        b = s_first[wv][e] + (c - s_pre[wv][e]);
        const float4 Bp = gload(w.md_pos, b);
        info = s_info[wv][e];
        keep = ls_window_may_pass(A, Bp, s_wmax[wv][e]) &&
               ls_inner_stub_may_pass(A, Bp, sa, mia, ModInfo{info}, g.d0max);
      }
      const unsigned long long m = __ballot(keep);
      const int pre = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      if (keep) s_q[wv][nq + pre] = b | (info << 30);
      nq += __popcll(m);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // each queue holds < 64 entries before a round adds at most 64
      if (nq >= 64) {
        sift(64);
        queue_pop64(s_q[wv], nq - 64);
        nq -= 64;
        if (nr >= 64) {
          select(64);
          queue_pop64(s_r[wv], nr - 64);
          nr -= 64;
        }
      }
    }
    if (nq > 0) sift(nq);
    while (nr > 0) {
      const int n2 = nr < 64 ? nr : 64;
      select(n2);
      queue_pop64(s_r[wv], nr - n2);
      nr -= n2;
    }
  };
  if (direct) {  // those of the wave's own MDs
    for (int a0 = ((int)blockIdx.x * wpb + wv) * kLsCopyMds; a0 < n_md; a0 += n_copy * wpb * kLsCopyMds) {
      const bool more = lane < kLsCopyMds && a0 + lane < n_md && gp(w.ls_cnt)[a0 + lane] > g.tiles.ls_cache;
      for (unsigned long long m = __ballot(more); m; m &= m - 1) process(a0 + __builtin_ctzll(m));
    }
    return;
  }
  const int n_ovf = uload(w.ctr + C_NLSOVF);
  const int stride = ((int)gridDim.x - n_copy) * wpb;
  for (int k = ((int)blockIdx.x - n_copy) * wpb + wv; k < n_ovf; k += stride) process(uload(w.ls_ovf + k));
}


// ------------------------------------------------------------- a3: T3
// Parents: segments (a, b); candidates: the segments whose inner MD is b.
// A superset of t3_pass's azimuth-z test, in the fast operations of the segment
// pre-tests: the residual is a difference of two products, so its error is
// bounded by 1e-6 of their magnitudes (margin 1e-5 of them) and the tolerance's
// by 1e-6 relative (margin 1e-5).  The terms of the parent segment (a, b) are
// computed once for its pairs.  (The curvature cut prunes 2% of what this test
// leaves; tested as well, and the parent's terms per pair, the count took 36.5 us on
// a PU200 event and 217 on eight, now 30 and 177.)
__device__ __forceinline__ float4 t3_parent(const float4 &A, const float4 &B, ModInfo mA, ModInfo mB, float d0) {
  const float iP = frcp(A.w), iQ = frcp(B.w);
  return make_float4((A.x * B.y - A.y * B.x) * (iP * iQ), B.z - A.z,
                     (mA.hphi() * iP + mB.hphi() * iQ) + d0 * fabsf(iP - iQ), iQ);
}
__device__ __forceinline__ bool t3_may_pass(const float4 &p, const float4 &B, const float4 &C, ModInfo mA, ModInfo mB,
                                            ModInfo mC, float d0) {
  const float iR = frcp(C.w);
  const float sv = (B.x * C.y - B.y * C.x) * (p.w * iR);
  const float dzqr = C.z - B.z, t1 = p.x * dzqr, t2 = sv * p.y;
  const float eQR = (mB.hphi() * p.w + mC.hphi() * iR) + d0 * fabsf(p.w - iR);
  const float au = fabsf(p.x), av = fabsf(sv), adpq = fabsf(p.y), adqr = fabsf(dzqr);
  const float nl = (au * au + av * av) * kThird;
  const float tol = ((adqr * p.z + adpq * eQR) + (au * (mB.ez() + mC.ez()) + av * (mA.ez() + mB.ez()))) +
                    nl * (au * adqr + av * adpq);
  return fabsf(t1 - t2) <= (tol * kMargin + kEps) * 1.00001f + 1e-5f * (fabsf(t1) + fabsf(t2));
}

// First lane of the run of equal values v (lanes 0..n-1 of the wave, runs of
// equal values contiguous) that holds this lane's value.
__device__ __forceinline__ int run_first_lane(int v, int n) {
  const int lane = lane_id();
  const int prev = __shfl_up(v, 1, 64);
  const unsigned long long starts = __ballot(lane < n && (lane == 0 || v != prev));
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  return 63 - __builtin_clzll(starts & upto);
}

// Parents of a wave (as a power of two) in the triplet and quintuplet passes,
// from the launch's parents, about n in each of its events: 64 fill the lanes'
// setup and share the block's prefix among most, but a few thousand waves
// leave the chip waiting for the one with the most pairs.  Measured, count +
// fill, with 64 / 32 / 16: triplets of a PU200 event (484k segments) 58 / 62 /
// 87 us, of eight 372 / 483 / 722, of a PU50 event 22 / 17 / 18; quintuplets of
// a PU200 event (123k triplets) 87 / 72 / 60, of eight 196 / 237 / 322, of a PU50
// event 40 / 23 / 21.  So 64 from 256k parents on, 32 from 160k, else 16
// (kMinParents: the wave sums' arrays hold one per 16).
__device__ __forceinline__ int parent_shift(int n) {
  const long all = (long)n * gridDim.y;
  static_assert(kMinParents == 16, "the shift returned for the smallest groups");
  return all >= 262144 ? 6 : all >= 163840 ? 5 : 4;
}

// Seven waves per SIMD for the count (at most 72 VGPRs, no spills).
template <bool FILL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(FILL ? 6 : 7))) void k_t3(const Ws *__restrict__ wb, DevGeom g) {
  const Ws &w = wb[blockIdx.y];
  __shared__ float4 s_a[kWaves][64], s_b[kWaves][64], s_k[kWaves][64];  // anchors, the pre-test's terms
  __shared__ int s_mi[kWaves][64], s_lo[kWaves][64], s_cnt[kWaves][64], s_seg[kWaves][65], s_cached[kWaves][64];
  __shared__ int s_qe[kWaves][128], s_qc[kWaves][128];  // pairs past the pre-test, in pair order
  __shared__ int s_mark[kWaves][64];
  __shared__ int s_off[FILL ? kWaves : 1][64], s_red[kWaves];  // the parents' offsets
  const int n_ls = uload(w.ctr + C_NLS);
  const int wv = wave_id(), lane = lane_id();
  const int wpb = blockDim.x >> 6;
  if (FILL && n_ls == 0 && blockIdx.x == 0 && threadIdx.x == 0) w.t3_off[0] = 0;
  const int lw = parent_shift(n_ls), nb = wpb << lw;  // log2 of a wave's parents, the block's parents
  for (long b0 = (long)blockIdx.x * nb; b0 < n_ls; b0 += (long)gridDim.x * nb) {
    const long p0 = b0 + (wv << lw);
    if (!FILL && p0 >= n_ls) break;  // (the fill's waves share their block's prefix)
    const int l1 = lane >> lw ? n_ls : (int)p0 + lane;
    int n = 0, cached = 0, n_mine = 0;
    if (FILL) {  // the parents' offsets, in place of their counts
      n_mine = l1 < n_ls ? gp(w.t3_off)[l1] : 0;
      int off = block_prefix(w.ts_t3, w.sh_t3, w.ws_t3, lw, (int)b0, s_red) + wave_inclusive(n_mine) - n_mine;
      for (long q = b0; q < p0 && q < n_ls; q += 1 << lw) off += uload(w.ws_t3 + (q >> lw));
      s_off[wv][lane] = off;
      if (l1 < n_ls) gp(w.t3_off)[l1] = off;
      if (l1 == n_ls - 1) {
        gp(w.t3_off)[n_ls] = off + n_mine;
        put_total(w, off + n_mine, w.cap_t3, C_RT3, C_NT3);
      }
    }
    // the fill reads a parent's data only if the count pass found a triplet on it
    if (l1 < n_ls && (!FILL || n_mine > 0)) {
      const int2 ab = gload(w.ls_md, l1);
      const float4 A = gload(w.md_pos, ab.x), B = gload(w.ls_opos, l1);
      const ModInfo mA{gp(g.info)[gp(w.md_mod)[ab.x]]}, mB{gp(w.ls_oinf)[l1]};
      s_a[wv][lane] = A;
      s_b[wv][lane] = B;
      s_k[wv][lane] = t3_parent(A, B, mA, mB, g.d0max);
      s_mi[wv][lane] = mA.bits | (mB.bits << 8);
      const int lo = gp(w.ls_off)[ab.y], hi = min(gp(w.ls_off)[ab.y + 1], n_ls);
      s_lo[wv][lane] = lo;
      n = hi > lo ? hi - lo : 0;
      if (FILL && n_mine <= g.tiles.t3_cache) {  // the count pass kept them all: only those are tested again
        n = n_mine;
        cached = 1;
      }
    }
    s_cnt[wv][lane] = 0;
    s_cached[wv][lane] = cached;
    const int total = wave_segments(n, s_seg[wv]);
    // the exact selection on the first nb (<= 64) queued pairs: ranks among each parent's
    // passing pairs from the parent's running count and a ballot over the batch
    auto select = [&](int nb) {
      bool pass = false;
      int e = 0, cand = 0, cmd = 0;
      float4 attr = make_float4(0.f, 0.f, 0.f, 0.f);
      if (lane < nb) {
        e = s_qe[wv][lane];
        cand = s_qc[wv][lane];
        if (FILL) cmd = gload(w.ls_md, cand).y;
        const int mi = s_mi[wv][e];
        pass = t3_pass(s_a[wv][e], s_b[wv][e], gload(w.ls_opos, cand), ModInfo{mi & 0xff}, ModInfo{mi >> 8},
                       ModInfo{gp(w.ls_oinf)[cand]}, &attr, g.d0max);
      }
      const int first = run_first_lane(e, nb);
      const unsigned long long m = __ballot(pass);
      if (pass) {
        const int r = pair_rank(m, first, s_cnt[wv][e]);
        if (!FILL) {
          if (r < g.tiles.t3_cache) gp(w.t3_cache)[(long)((int)p0 + e) * kT3Cache + r] = cand;
        } else {
          const int pos = s_off[wv][e] + r;
          if (pos < w.cap_t3) {
            const int2 ab = gload(w.ls_md, (int)p0 + e);
            gstore(w.t3_md, pos, make_int4(ab.x, ab.y, cmd, (int)p0 + e));
            gstore(w.t3_attr, pos, attr);
            gstore(w.t3_first, pos, make_float2(s_a[wv][e].x, s_a[wv][e].y));
            gstore(w.o3_best, pos, 0ull);
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (pass) atomicAdd(&s_cnt[wv][e], 1);  // LDS
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    int nq = 0;
    const int start = s_seg[wv][lane];
    int carry = 0;
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int c = c0 + lane;
      const int e = round_parent(start, n, c0, s_mark[wv], carry);  // parent of this lane's pair
      bool keep = false;
      int cand = 0;
      if (c < total) {
        const int idx = c - s_seg[wv][e];
        cand = s_cached[wv][e] ? gp(w.t3_cache)[(long)((int)p0 + e) * kT3Cache + idx] : s_lo[wv][e] + idx;
        const int mi = s_mi[wv][e];
        keep = t3_may_pass(s_k[wv][e], s_b[wv][e], gload(w.ls_opos, cand), ModInfo{mi & 0xff}, ModInfo{mi >> 8},
                           ModInfo{gp(w.ls_oinf)[cand]}, g.d0max);
      }
      const unsigned long long m = __ballot(keep);
      if (keep) {
        const int q = nq + lanes_below(m);
        s_qe[wv][q] = e;
        s_qc[wv][q] = cand;
      }
      nq += __popcll(m);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (nq >= 64) {
        select(64);
        const int rest = nq - 64;  // < 64: move the queue's tail to its front
        int ve = 0, vc = 0;
        if (lane < rest) {
          ve = s_qe[wv][64 + lane];
          vc = s_qc[wv][64 + lane];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < rest) {
          s_qe[wv][lane] = ve;
          s_qc[wv][lane] = vc;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        nq = rest;
      }
    }
    if (nq > 0) select(nq);
    if (!FILL) {
      const int c = l1 < n_ls ? s_cnt[wv][lane] : 0;
      if (l1 < n_ls) gp(w.t3_off)[l1] = c;
      const int sum = wave_total(c);
      if (lane == 0) {
        gp(w.ws_t3)[p0 >> lw] = sum;
        if (sum > 0) atomicAdd(w.ts_t3 + (p0 >> w.sh_t3) * kSumStride, sum);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------- a4: T5
// Parents: triplets (a, b, c); candidates: the triplets whose first MD is c.
// A superset of the azimuth-z test of three anchors (phiz_pass), in the fast
// operations, with the margins of t3_may_pass's azimuth-z part.
__device__ __forceinline__ bool phiz_may_pass(const float4 &P, const float4 &Q, const float4 &R, ModInfo mp,
                                              ModInfo mq, ModInfo mr, float d0) {
  const float su = (P.x * Q.y - P.y * Q.x) * frcp(P.w * Q.w);
  const float sv = (Q.x * R.y - Q.y * R.x) * frcp(Q.w * R.w);
  const float dzpq = Q.z - P.z, dzqr = R.z - Q.z;
  const float t1 = su * dzqr, t2 = sv * dzpq;
  const float iP = frcp(P.w), iQ = frcp(Q.w), iR = frcp(R.w);
  const float ePQ = (mp.hphi() * iP + mq.hphi() * iQ) + d0 * fabsf(iP - iQ);
  const float eQR = (mq.hphi() * iQ + mr.hphi() * iR) + d0 * fabsf(iQ - iR);
  const float au = fabsf(su), av = fabsf(sv), adpq = fabsf(dzpq), adqr = fabsf(dzqr);
  const float nl = (au * au + av * av) * kThird;
  const float tol = ((adqr * ePQ + adpq * eQR) + (au * (mq.ez() + mr.ez()) + av * (mp.ez() + mq.ez()))) +
                    nl * (au * adqr + av * adpq);
  return fabsf(t1 - t2) <= (tol * kMargin + kEps) * 1.00001f + 1e-5f * (fabsf(t1) + fabsf(t2));
}

// The triplets that start at MD m: (first, end), both at most n_t3: past the
// capacity the offsets run on, and t5_off has n_t3 + 1 entries.
__device__ __forceinline__ int2 md_triplets(const Ws &w, int m, int n_ls, int n_t3) {
  const int l0 = min(gp(w.ls_off)[m], n_ls), l1 = min(gp(w.ls_off)[m + 1], n_ls);
  return make_int2(min(gp(w.t3_off)[l0], n_t3), min(gp(w.t3_off)[l1], n_t3));
}
// The quintuplets among the triplets [r.x, r.y).
__device__ __forceinline__ int2 triplets_t5(const Ws &w, int2 r, int n_t5) {
  const int lo = min(gp(w.t5_off)[r.x], n_t5), hi = min(gp(w.t5_off)[r.y], n_t5);
  return make_int2(lo, hi > lo ? hi : lo);
}

// Seed-search bins: the search tests first anchors, and the triplets and
// quintuplets of one first MD are consecutive, so the bins hold MDs (50k on a
// PU200 event, where its 124k triplets and 29k quintuplets had an entry each)
// and one test serves all of an MD's objects of both kinds.  Count, placement
// of the rows and scatter ride in the quintuplet stage's launches as further
// blocks, q = 0, 1, ... of nq.
__device__ __forceinline__ void bin_count(const Ws &w, int q, int nq) {
  if (w.n_seeds == 0) return;
  if (q == 0 && threadIdx.x < kTaskShards) gp(w.ts_task)[threadIdx.x * kSumStride] = 0;  // (the seed search's tasks)
  const int n = uload(w.ctr + C_NMD), n_ls = uload(w.ctr + C_NLS), n_t3 = uload(w.ctr + C_NT3);
  for (int m = q * blockDim.x + threadIdx.x; m < n; m += nq * blockDim.x) {
    const int2 r = md_triplets(w, m, n_ls, n_t3);
    int2 b = make_int2(-1, 0);
    if (r.y > r.x) {
      b.x = obj_bin(gload(w.md_pos, m));
      b.y = atomicAdd(w.bin_cnt + b.x, 1);
    }
    gstore(w.md_bin, m, b);
  }
}
// A row's place among the others does not matter (its bins are consecutive, z
// ascending): each block takes one atomic on the total and scans its own counts.
constexpr int kRowsPerWave = 8;
__device__ __forceinline__ void bin_place(const Ws &w, int q, int *s_wave) {
  if (w.n_seeds == 0) return;
  static_assert(kBinStride <= 64, "a row's bins on one wave");
  const int lane = lane_id(), wv = wave_id(), wpb = blockDim.x >> 6;
  const int r0 = (q * wpb + wv) * kRowsPerWave;
  int c[kRowsPerWave], sum = 0;
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r)
    sum += c[r] = (lane < kZBins && r0 + r < kBinRows) ? gp(w.bin_cnt)[(r0 + r) * kBinStride + lane] : 0;
  sum = wave_total(sum);
  if (lane == 0) s_wave[wv] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int i = 0; i < wpb; ++i) tot += s_wave[i];
    s_wave[kWaves] = atomicAdd(w.ctr + C_NBIN, tot);
  }
  __syncthreads();
  int run = s_wave[kWaves];
  for (int i = 0; i < wv; ++i) run += s_wave[i];
#pragma unroll
  for (int r = 0; r < kRowsPerWave; ++r) {
    const int x = wave_inclusive(c[r]);
    if (lane < kBinStride && r0 + r < kBinRows) gp(w.bin_off)[(r0 + r) * kBinStride + lane] = run + x - c[r];
    run += __shfl(x, 63, 64);
  }
}
__device__ __forceinline__ void bin_scatter(const Ws &w, const DevGeom &g, int q, int nq) {
  if (w.n_seeds == 0) return;
  const int n = uload(w.ctr + C_NMD), n_ls = uload(w.ctr + C_NLS), n_t3 = uload(w.ctr + C_NT3);
  const int n_t5 = uload(w.ctr + C_NT5);
  for (int m = q * blockDim.x + threadIdx.x; m < n; m += nq * blockDim.x) {
    const int2 b = gload(w.md_bin, m);
    if (b.x < 0) continue;
    const int j = gp(w.bin_off)[b.x] + b.y;
    const int2 r = md_triplets(w, m, n_ls, n_t3), v = triplets_t5(w, r, n_t5);
    const float4 a = gload(w.md_pos, m);
    gstore(w.bin_pos, j, make_float4(a.x, a.y, a.z, __int_as_float(gp(g.info)[gp(w.md_mod)[m]])));
    gstore(w.bin_rng, j, make_int4(r.x, r.y - r.x, v.x, v.y - v.x));
  }
}

template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_t5(const Ws *__restrict__ wb, DevGeom g, int n_main) {
  const Ws &w = wb[blockIdx.y];
  if ((int)blockIdx.x >= n_main) {  // the seed search's bins
    __shared__ int s_wave[kWaves + 1];
    const int q = (int)blockIdx.x - n_main, nq = (int)gridDim.x - n_main;
    if constexpr (FILL) bin_place(w, q, s_wave);
    else bin_count(w, q, nq);
    return;
  }
  __shared__ float4 s_p[kWaves][3][64], s_tin[kWaves][64];
  __shared__ int s_mi[kWaves][64], s_lo[kWaves][64], s_cnt[kWaves][64], s_seg[kWaves][65], s_cached[kWaves][64];
  __shared__ int s_qe[kWaves][128], s_qc[kWaves][128];  // pairs past the pre-test, in pair order
  __shared__ int s_off[FILL ? kWaves : 1][64], s_red[kWaves];  // the parents' offsets
  const int n_t3 = uload(w.ctr + C_NT3);
  const int n_ls = uload(w.ctr + C_NLS);
  const int wv = wave_id(), lane = lane_id();
  const int wpb = blockDim.x >> 6;
  if (FILL && n_t3 == 0 && blockIdx.x == 0 && threadIdx.x == 0) w.t5_off[0] = 0;
  const int lw = parent_shift(n_t3), nb = wpb << lw;
  for (long b0 = (long)blockIdx.x * nb; b0 < n_t3; b0 += (long)n_main * nb) {
    const long p0 = b0 + (wv << lw);
    if (!FILL && p0 >= n_t3) break;
    const int t1 = lane >> lw ? n_t3 : (int)p0 + lane;
    int n = 0, cached = 0, n_mine = 0;
    if (FILL) {  // the parents' offsets, in place of their counts
      n_mine = t1 < n_t3 ? gp(w.t5_off)[t1] : 0;
      int off = block_prefix(w.ts_t5, w.sh_t5, w.ws_t5, lw, (int)b0, s_red) + wave_inclusive(n_mine) - n_mine;
      for (long q = b0; q < p0 && q < n_t3; q += 1 << lw) off += uload(w.ws_t5 + (q >> lw));
      s_off[wv][lane] = off;
      if (t1 < n_t3) gp(w.t5_off)[t1] = off;
      if (t1 == n_t3 - 1) {
        gp(w.t5_off)[n_t3] = off + n_mine;
        put_total(w, off + n_mine, w.cap_t5, C_RT5, C_NT5);
      }
    }
    // the fill reads a parent's data only if the count pass found a quintuplet on it
    if (t1 < n_t3 && (!FILL || n_mine > 0)) {
      const int4 abc = gload(w.t3_md, t1);
      s_p[wv][0][lane] = gload(w.md_pos, abc.x);
      s_p[wv][1][lane] = gload(w.md_pos, abc.y);
      s_p[wv][2][lane] = gload(w.md_pos, abc.z);
      s_mi[wv][lane] = gp(g.info)[gp(w.md_mod)[abc.x]] | (g.info[gp(w.md_mod)[abc.y]] << 8) | (g.info[gp(w.md_mod)[abc.z]] << 16);
      s_tin[wv][lane] = gload(w.t3_attr, t1);
      // triplets with first MD c: those built from segments with inner MD c
      const int lsb = min(w.ls_off[abc.z], n_ls), lse = min(w.ls_off[abc.z + 1], n_ls);
      const int lo = gp(w.t3_off)[lsb], hi = min(w.t3_off[lse], n_t3);
      s_lo[wv][lane] = lo;
      n = hi > lo ? hi - lo : 0;
      if (FILL && n_mine <= g.tiles.t5_cache) {  // the count pass kept them all: only those are tested again
        n = n_mine;
        cached = 1;
      }
    }
    s_cnt[wv][lane] = 0;
    s_cached[wv][lane] = cached;
    const int total = wave_segments(n, s_seg[wv]);
    // the exact selection on the first nb (<= 64) queued pairs (as in k_t3)
    auto select = [&](int nb) {
      bool pass = false;
      int e = 0, t2 = 0;
      int4 cde = make_int4(0, 0, 0, 0);
      float at[8];
      if (lane < nb) {
        e = s_qe[wv][lane];
        t2 = s_qc[wv][lane];
        cde = gload(w.t3_md, t2);
        float4 P[5];
        ModInfo M[5];
        const int mi = s_mi[wv][e];
        P[0] = s_p[wv][0][e]; P[1] = s_p[wv][1][e]; P[2] = s_p[wv][2][e];
        M[0].bits = mi & 0xff; M[1].bits = (mi >> 8) & 0xff; M[2].bits = mi >> 16;
        P[3] = gload(w.md_pos, cde.y);
        P[4] = gload(w.md_pos, cde.z);
        M[3].bits = gp(g.info)[gp(w.md_mod)[cde.y]];
        M[4].bits = gp(g.info)[gp(w.md_mod)[cde.z]];
        pass = t5_pass(P, M, s_tin[wv][e], gload(w.t3_attr, t2), at, g.d0max, g.t5cut);
      }
      const int first = run_first_lane(e, nb);
      const unsigned long long m = __ballot(pass);
      if (pass) {
        const int r = pair_rank(m, first, s_cnt[wv][e]);
        if (!FILL) {
          if (r < g.tiles.t5_cache) gp(w.t5_cache)[(long)((int)p0 + e) * kT5Cache + r] = t2;
        } else {
          const int t1e = (int)p0 + e;
          const int pos = s_off[wv][e] + r;
          if (pos < w.cap_t5) {
            const int4 abc = gload(w.t3_md, t1e);
            gstore(w.t5_t3, pos, make_int2(t1e, t2));
            int *md = w.t5_md + 5 * (long)pos;
            md[0] = abc.x; md[1] = abc.y; md[2] = abc.z; md[3] = cde.y; md[4] = cde.z;
            float *dst = w.t5_attr + 8 * (long)pos;
#pragma unroll
            for (int k = 0; k < 8; ++k) dst[k] = at[k];
            gp(w.t5_keep)[pos] = 1;  // until a better duplicate is found
            gp(w.t5_used)[pos] = 0;
            gstore(w.t5_first, pos, make_float2(s_p[wv][0][e].x, s_p[wv][0][e].y));
            gstore(w.o5_best, pos, 0ull);
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (pass) atomicAdd(&s_cnt[wv][e], 1);  // LDS
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    int nq = 0;
    int e = 0;  // parent of this lane's pair (pairs advance monotonically; the walk takes fewer
                // registers than round_parent)
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int c = c0 + lane;
      bool keep = false;
      int t2 = 0;
      if (c < total) {
        while (s_seg[wv][e + 1] <= c) ++e;
        const int idx = c - s_seg[wv][e];
        t2 = s_cached[wv][e] ? gp(w.t5_cache)[(long)((int)p0 + e) * kT5Cache + idx] : s_lo[wv][e] + idx;
        // the radius compatibility cut exactly (no division), then the fast azimuth-z test
        const float4 tin = s_tin[wv][e], tout = gload(w.t3_attr, t2);
        if (fabsf(tin.x - tout.x) <= tin.y + tout.y) {
          const int4 cde = gload(w.t3_md, t2);
          const int mi = s_mi[wv][e];
          keep = phiz_may_pass(s_p[wv][0][e], s_p[wv][2][e], gload(w.md_pos, cde.z), ModInfo{mi & 0xff},
                               ModInfo{mi >> 16}, ModInfo{gp(g.info)[gp(w.md_mod)[cde.z]]}, g.d0max);
        }
      }
      const unsigned long long m = __ballot(keep);
      if (keep) {
        const int q = nq + lanes_below(m);
        s_qe[wv][q] = e;
        s_qc[wv][q] = t2;
      }
      nq += __popcll(m);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (nq >= 64) {
        select(64);
        const int rest = nq - 64;
        int ve = 0, vc = 0;
        if (lane < rest) {
          ve = s_qe[wv][64 + lane];
          vc = s_qc[wv][64 + lane];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < rest) {
          s_qe[wv][lane] = ve;
          s_qc[wv][lane] = vc;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        nq = rest;
      }
    }
    if (nq > 0) select(nq);
    if (!FILL) {
      const int c = t1 < n_t3 ? s_cnt[wv][lane] : 0;
      if (t1 < n_t3) gp(w.t5_off)[t1] = c;
      const int sum = wave_total(c);
      if (lane == 0) {
        gp(w.ws_t5)[p0 >> lw] = sum;
        if (sum > 0) atomicAdd(w.ts_t5 + (p0 >> w.sh_t5) * kSumStride, sum);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------- a5: T5 dedup
// Lists of the T5s on each MD.  The T5s that start at an MD are consecutive, so
// only the other four of a T5's MDs count it: one thread per (T5, MD) takes the
// T5's place in the MD's list (blocks [0, n5); the others scatter the seed
// search's bins).  Device atomics run at about 8 per ns whatever waits for them;
// taken inside the quintuplet fill, with its fewer and longer waves, they cost it
// 46 us against 17 here.
__global__ __launch_bounds__(kBlock) void k_t5_inc(const Ws *__restrict__ wb, DevGeom g, int n5) {
  const Ws &w = wb[blockIdx.y];
  if ((int)blockIdx.x >= n5) {
    bin_scatter(w, g, (int)blockIdx.x - n5, (int)gridDim.x - n5);
    return;
  }
  const long n = 4L * uload(w.ctr + C_NT5);
  for (long i = blockIdx.x * (long)kBlock + threadIdx.x; i < n; i += (long)n5 * kBlock) {
    const int md = gp(w.t5_md)[5 * (i >> 2) + 1 + (i & 3)];
    gp(w.t5_slot)[i] = atomicAdd(w.inc_cnt + md, 1);
  }
}
// Places of the lists: a list's place among the others does not matter, so each
// block takes one atomic on the total and scans its own counts.
__global__ __launch_bounds__(kBlock) void k_list_place(const Ws *__restrict__ wb) {
  __shared__ int s_wave[kWaves], s_base;
  const Ws &w = wb[blockIdx.y];
  const int t = threadIdx.x, lane = lane_id(), wv = wave_id();
  const int n = uload(w.ctr + C_NMD), n_ls = uload(w.ctr + C_NLS), n_t3 = uload(w.ctr + C_NT3);
  const int n_t5 = uload(w.ctr + C_NT5);
  constexpr int kItems = 2;
  for (long b0 = (long)blockIdx.x * kItems * kBlock; b0 < n; b0 += (long)gridDim.x * kItems * kBlock) {
    int c[kItems], sum = 0;
    int2 own[kItems];  // the T5s it is the first MD of
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const long m = b0 + k * kBlock + t;
      own[k] = make_int2(0, 0);
      c[k] = 0;
      if (m < n) {
        own[k] = triplets_t5(w, md_triplets(w, (int)m, n_ls, n_t3), n_t5);
        c[k] = gp(w.inc_cnt)[m];
      }
      sum += c[k] + own[k].y - own[k].x;
    }
    const int x = wave_inclusive(sum);
    __syncthreads();  // the previous round's reads
    if (lane == 63) s_wave[wv] = x;
    __syncthreads();
    if (t == 0) {
      int tot = 0;
      for (int q = 0; q < kWaves; ++q) tot += s_wave[q];
      s_base = tot > 0 ? atomicAdd(w.ctr + C_NINC, tot) : 0;
    }
    __syncthreads();
    int at = s_base + x - sum;
    for (int q = 0; q < wv; ++q) at += s_wave[q];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const long m = b0 + k * kBlock + t;
      if (m < n) {
        const int n0 = own[k].y - own[k].x;
        gp(w.inc_off)[m] = at;
        gp(w.inc_cnt)[m] = c[k] + n0;
        gp(w.inc_b0)[m] = at + c[k] - own[k].x;
        at += c[k] + n0;
      }
    }
  }
}
// The T5s into their MDs' lists, one thread per (T5, MD): every place is known.
// An entry holds the T5, its score and its four other MDs, so that the
// duplicate removal reads lists and nothing else.
__global__ __launch_bounds__(kBlock) void k_t5_inc_scatter(const Ws *__restrict__ wb) {
  const Ws &w = wb[blockIdx.y];
  const long n = 5L * uload(w.ctr + C_NT5);
  for (long i = blockIdx.x * (long)kBlock + threadIdx.x; i < n; i += (long)gridDim.x * kBlock) {
    const long t = i / 5;
    const int k = (int)(i - 5 * t);
    int m[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) m[j] = gp(w.t5_md)[5 * t + j];
    const int md = gp(w.t5_md)[i];
    const int pos = k == 0 ? gp(w.inc_b0)[md] + (int)t : gp(w.inc_off)[md] + gp(w.t5_slot)[4 * t + k - 1];
    gstore(w.inc_list, pos, make_int2((int)t, __float_as_int(gp(w.t5_attr)[8 * t + 1])));
    gstore(w.inc_mds, pos, make_int4(k > 0 ? m[0] : m[1], k > 1 ? m[1] : m[2], k > 2 ? m[2] : m[3], k > 3 ? m[3] : m[4]));
  }
}

__device__ __forceinline__ void t5_hits(const Ws &w, int t, int *h) {
  const int *md = w.t5_md + 5 * (long)t;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const int2 hh = w.md_hits[md[k]];
    h[2 * k] = hh.x;
    h[2 * k + 1] = hh.y;
  }
}
// (score, tuple) of u strictly smaller than (score, tuple) of t
template <int N>
__device__ __forceinline__ bool better(float su, const int *hu, float st, const int *ht) {
  if (su < st) return true;
  if (st < su) return false;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (hu[k] < ht[k]) return true;
    if (ht[k] < hu[k]) return false;
  }
  return false;
}

// A T5 is dropped when another T5 sharing at least two MDs has a smaller (chi2_xy, hit tuple).
// Items (T5 t, k < 4); an item's candidates are the T5s u listed at t's k-th
// MD, and u is judged there only if it shares at least two MDs with t and its
// first MD in common with t's first four is that k-th one (so each pair is
// judged once; a duplicate shares two of the five MDs, hence one of the first
// four).  A block takes 16 T5s, spread over the event, stages their MDs in LDS
// and strides all (item, candidate) pairs, flattened, with all its waves.  The
// lists are uneven (hundreds of T5s at an MD of a dense core, few elsewhere)
// and consecutive T5s have the same ones, so the longest chain bounds the
// launch: with 16 consecutive items a wave a PU200 event took 58 us and with
// 64 211 us; 64 consecutive items a block, 55 us; 64 of T5s n / 16 apart, 19 us
// (eight events: 241, 104 and 110 us).  Candidates' MDs come with the list: eight
// events took 256 us when they were gathered from t5_md.
// t5_keep starts at 1 (written by the fill); a strictly better duplicate
// clears it (every writer writes 0).
__global__ __launch_bounds__(kBlock) void k_t5_dedup(const Ws *__restrict__ wb) {
  __shared__ int s_mt[5][64], s_lo[64], s_cnt[64], s_seg[kWaves][65], s_mark[kWaves][64];
  __shared__ float s_st[64];
  const Ws &w = wb[blockIdx.y];
  const int n = uload(w.ctr + C_NT5);
  const int wv = wave_id(), lane = lane_id();
  const int stride = blockDim.x;
  const int n_grp = (n + 15) / 16;
  for (int q = blockIdx.x; q < n_grp; q += gridDim.x) {
    __syncthreads();  // the previous items' data is no longer read
    if (wv == 0) {
      const int t = q + (lane >> 2) * n_grp, k = lane & 3;
      int cnt = 0;
      if (t < n) {
        int mt[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) {
          mt[j] = gp(w.t5_md)[5 * (long)t + j];
          s_mt[j][lane] = mt[j];
        }
        s_lo[lane] = gp(w.inc_off)[mt[k]];
        cnt = gp(w.inc_cnt)[mt[k]];
        s_st[lane] = gp(w.t5_attr)[8 * (long)t + 1];
      }
      s_cnt[lane] = cnt;
    }
    __syncthreads();
    const int cnt = s_cnt[lane];
    const int total = wave_segments(cnt, s_seg[wv]);
    const int start = s_seg[wv][lane];
    for (int c0 = wv * 64; c0 < total; c0 += stride) {
      const int c = c0 + lane;
      // the item whose pairs run into this round, then that of each lane's pair
      const unsigned long long before = __ballot(cnt > 0 && start < c0);
      int carry = before ? 63 - (int)__builtin_clzll(before) : 0;
      const int e = round_parent(start, cnt, c0, s_mark[wv], carry);
      if (c >= total) continue;
      const int t = q + (e >> 2) * n_grp, k = e & 3;
      const int pos = s_lo[e] + (c - s_seg[wv][e]);
      const int2 ue = gload(w.inc_list, pos);
      const int u = ue.x;
      if (u == t) continue;
      // only a u that is not worse can drop t: the score first (kept in the list entry),
      // then sharing, then on a tie of scores the hit tuples (the decision of better<10>)
      const float su = __int_as_float(ue.y), st = s_st[e];
      if (st < su) continue;
      // u has t's k-th MD; its others are in the list (the MDs of a T5 are distinct)
      const int4 mu = gload(w.inc_mds, pos);
      unsigned in = 0u;
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const int v = s_mt[j][e];
        in |= (v == mu.x || v == mu.y || v == mu.z || v == mu.w) ? 1u << j : 0u;
      }
      if (in >> k == 0u || (in & ((1u << k) - 1u)) != 0u) continue;
      bool drop = su < st;
      if (!drop) {
        int ht[10], hu[10];
        t5_hits(w, t, ht);
        t5_hits(w, u, hu);
        drop = better<10>(su, hu, st, ht);
      }
      if (drop) gp(w.t5_keep)[t] = 0;
    }
  }
}

// The same decision with every pair of T5s, one wave per T5 t and its lanes over
// the others (at most 32 rounds), for capacities up to kPairsT5: no lists, so
// three launches less (with the removal itself 16 -> 5 us on a tiny event of 179
// T5s; the lists of a PU50 event, with ten times as many, take 21 us, and pairs
// grow with the square).  The seed search's bins are scattered on further blocks.
constexpr int kPairsT5 = 2048;
__global__ __launch_bounds__(kBlock) void k_t5_pairs(const Ws *__restrict__ wb, DevGeom g, int n_main) {
  const Ws &w = wb[blockIdx.y];
  if ((int)blockIdx.x >= n_main) {
    bin_scatter(w, g, (int)blockIdx.x - n_main, (int)gridDim.x - n_main);
    return;
  }
  const int n = uload(w.ctr + C_NT5);
  const int lane = lane_id(), wpb = blockDim.x >> 6;
  for (int t = blockIdx.x * wpb + wave_id(); t < n; t += n_main * wpb) {
    int mt[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) mt[j] = uload(w.t5_md + 5L * t + j);
    const float st = __int_as_float(uload(reinterpret_cast<const int *>(w.t5_attr) + 8L * t + 1));
    bool drop = false;
    for (int u = lane; u < n; u += 64) {
      const float su = gp(w.t5_attr)[8L * u + 1];
      if (u == t || st < su) continue;
      int shared = 0;
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const int m = gp(w.t5_md)[5L * u + j];
        shared += m == mt[0] || m == mt[1] || m == mt[2] || m == mt[3] || m == mt[4] ? 1 : 0;
      }
      if (shared < 2) continue;
      bool better_u = su < st;
      if (!better_u) {
        int ht[10], hu[10];
        t5_hits(w, t, ht);
        t5_hits(w, u, hu);
        better_u = better<10>(su, hu, st, ht);
      }
      drop |= better_u;
    }
    if (__ballot(drop) && lane == 0) gp(w.t5_keep)[t] = 0;
  }
}

// ------------------------------------------------------------- a7: pT3 / pT5
template <int K>
__device__ __forceinline__ void load_object(const Ws &w, const DevGeom &g, int t, float4 *P, ModInfo *M, float *kT,
                                            float *dkT) {
  if constexpr (K == 3) {
    const int4 abc = gload(w.t3_md, t);
    const int md[3] = {abc.x, abc.y, abc.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) { P[k] = w.md_pos[md[k]]; M[k].bits = gp(g.info)[gp(w.md_mod)[md[k]]]; }
    const float4 a3 = gload(w.t3_attr, t);
    *kT = a3.x; *dkT = a3.y;
  } else {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const int md = gp(w.t5_md)[5 * (long)t + k];
      P[k] = gload(w.md_pos, md);
      M[k].bits = gp(g.info)[gp(w.md_mod)[md]];
    }
    const float4 a3 = w.t3_attr[gload(w.t5_t3, t).y];
    *kT = a3.x; *dkT = a3.y;
  }
}

// Marks, in the wave's bin mask, every (ring, azimuth) bin that can hold the
// first anchor of an object inside the seed's window: the anchor lies within
// 1.01 cm of the seed circle on its forward half-turn (algebraic distance
// <= 1 cm with |kappa| <= 0.02/cm), hence within d = 1.01 + step/2 + 0.05 cm
// of a trajectory sample taken every `kSampleStep` of arc.
static_assert(kPhiBins % 32 == 0, "a ring's row of the bin mask is whole words");

// Sets bits id0 .. id0 + n - 1 of the mask, one atomic per word.
__device__ __forceinline__ void mark_run(unsigned *mask, int id0, int n) {
  const int end = id0 + n;
  for (int id = id0; id < end;) {
    const int bit = id & 31;
    const int take = min(32 - bit, end - id);
    const unsigned m = take == 32 ? 0xffffffffu : ((1u << take) - 1u) << bit;
    atomicOr(&mask[id >> 5], m);
    id += take;
  }
}

__device__ void mark_seed_bins(const Seed &sd, unsigned *mask, int *s_lo, int *s_hi) {
  const int lane = lane_id();
  const float d = 1.01f * kBoxXY + 0.5f * kSampleStep + 0.05f;
  const float bw = (float)(2.0 * M_PI / kPhiBins);
  const float k = sd.ks;
  const float ak = fabsf(k) > 1e-9f ? fabsf(k) : 1e-9f;
  const float s_max = (float)M_PI / ak;
  const float px = -sd.cy, py = sd.cx;  // perpendicular of the direction
  for (int i = lane; i < kMaxSamples; i += 64) {
    const float sarc = i * kSampleStep;
    if (sarc > s_max + kSampleStep) continue;
    const float a = k * sarc;
    const float s1 = fabsf(k) > 1e-9f ? sinf(a) / k : sarc;
    const float sh = sinf(0.5f * a);
    const float s2 = fabsf(k) > 1e-9f ? 2.0f * sh * sh / k : 0.0f;
    const float x = sd.x0 + sd.cx * s1 + px * s2;
    const float y = sd.y0 + sd.cy * s1 + py * s2;
    const float r = sqrtf(x * x + y * y);
    if (r + d < kRing0 - 5.0f || r - d > kRing0 + kRings * kRingW + 5.0f) continue;
    const int r0 = ring_of(r - d), r1 = ring_of(r + d);
    const float rin = r - d;
    int b0, b1;
    if (rin <= 1e-3f || d / rin >= 1.0f) {
      b0 = 0;
      b1 = kPhiBins - 1;
    } else {
      // an anchor within d of the sample, at radius >= rin, is within asin(d / rin) of
      // its azimuth; 2e-4 rad (1% of a bin) covers the rounding of these bin edges
      // against phibin_of's
      const float hw = asinf(d / rin);
      const float ph = atan2f(y, x);
      b0 = (int)floorf((ph - hw - 2e-4f + (float)M_PI) / bw);
      b1 = (int)floorf((ph + hw + 2e-4f + (float)M_PI) / bw);
      if (b1 - b0 >= kPhiBins) { b0 = 0; b1 = kPhiBins - 1; }
    }
    // bins b0..b1 (fewer than kPhiBins, may wrap round) as at most two runs of
    // one ring's row; a ring's row is whole mask words, so each word a run
    // touches takes one atomic
    const int lo = ((b0 % kPhiBins) + kPhiBins) % kPhiBins;
    const int len = b1 - b0 + 1;
    const int n1 = min(len, kPhiBins - lo);
    for (int rr = r0; rr <= r1; ++rr) {
      // arc lengths are >= 0, so their float bits order like ints
      atomicMin(&s_lo[rr], __float_as_int(sarc));
      atomicMax(&s_hi[rr], __float_as_int(sarc));
      mark_run(mask, rr * kPhiBins + lo, n1);
      if (len > n1) mark_run(mask, rr * kPhiBins, len - n1);
    }
  }
}

// z bins of ring rr that can hold the first anchor of an object inside the
// seed's window, from the arc-length range [lo, hi] of the samples that marked
// the ring: the anchor's arc length from the seed hit (the chord series of
// pt_pass) is within d + step + 1.5 cm of such a sample's, and its z within
// the first-anchor z window (3 cm + 2 sigma_z, sigma_z at most
// max(2.5, 2.5 |lambda| + 0.01) cm) of z0 + lambda s; margins on top.
__device__ __forceinline__ int2 seed_zbins(const Seed &sd, float lo, float hi) {
  const float ds = 1.01f * kBoxXY + 1.5f * kSampleStep + 1.6f;
  const float al = fabsf(sd.lam);
  const float zw = (kBoxZ0 + 2.0f * fmaxf(2.5f, 2.5f * al + 0.01f)) * 1.01f + 0.1f;
  const float za = sd.z0 + sd.lam * (lo - ds), zb = sd.z0 + sd.lam * (hi + ds);
  return make_int2(zbin_of(fminf(za, zb) - zw), zbin_of(fmaxf(za, zb) + zw));
}

// The key that orders a pT entry for the same-object rule: smaller (score,
// seed) is better, and since scores are >= 0 their bits order them as
// integers; complemented so that the best is the largest, found with an
// atomic maximum per outer object (a value, not a position: order-independent).
__device__ __forceinline__ unsigned long long pt_obj_key(float score, int seed) {
  return ~(((unsigned long long)__float_as_uint(score) << 32) | (unsigned long long)(unsigned)seed);
}

// One entry of the output, which also offers its key to its outer object.
template <int KO>
__device__ __forceinline__ void put_pt(const Ws &w, int pos, int s, int t, const float4 &attr) {
  if (pos >= (KO == 3 ? w.cap_pt3 : w.cap_pt5)) return;
  gstore(KO == 3 ? w.pt3_so : w.pt5_so, pos, make_int2(s, t));
  gstore(KO == 3 ? w.pt3_attr : w.pt5_attr, pos, attr);
  atomicMax((KO == 3 ? w.o3_best : w.o5_best) + t, pt_obj_key(attr.z, s));
}

// Entries of the seeds whose passing objects the count pass kept (block q of nq):
// a wave takes kPtSeeds seeds, finds their offsets and strides their entries,
// flattened, through LDS, where an entry's place is its rank by object index
// (indices are distinct): the order of the full scan.  A wave's time is its chain
// of gathers (sums, counts, entries, attributes), which more seeds share, and the
// ranks of its longest lists: with 1 / 4 / 16 seeds 22 / 21 / 28 us on a PU200
// event (93k triplet entries), 140 / 83 / 75 on eight.
constexpr int kPtSeeds = 4;
constexpr int kPtStage = 512;  // entries of a wave in LDS at a time
struct PtCopyLds {
  int seg[65], off[64], mark[64], val[kPtStage];
  unsigned char par[kPtStage];
};
template <int KO>
__device__ __forceinline__ void pt_copy(const Ws &w, const DevGeom &g, int q, int nq, PtCopyLds &L, int *s_red) {
  constexpr int kCache = KO == 3 ? kPt3Cache : kPt5Cache;
  static_assert(kCache <= kPtStage && kPtSeeds <= 64, "a seed's entries fit the stage");
  const int wv = wave_id(), lane = lane_id(), wpb = blockDim.x >> 6, S = w.n_seeds;
  const int keep = KO == 3 ? g.tiles.pt3_cache : g.tiles.pt5_cache;  // <= kCache
  const int *cnts = KO == 3 ? w.pt3_cnt : w.pt5_cnt;
  int *offs = KO == 3 ? w.pt3_off : w.pt5_off;
  if (S == 0 && q == 0 && threadIdx.x == 0) offs[0] = 0;
  const int per = wpb * kPtSeeds;
  for (int b0 = q * per; b0 < S; b0 += nq * per) {
    const int s0 = b0 + wv * kPtSeeds, s = s0 + lane;
    const bool mine = lane < kPtSeeds && s < S;
    const int cnt = mine ? gp(cnts)[s] : 0;
    int before = 0;  // the block's seeds on earlier waves
    for (int j = b0 + lane; j < min(s0, S); j += 64) before += gp(cnts)[j];
    const int off = block_prefix(KO == 3 ? w.ts_p3 : w.ts_p5, w.sh_pt, cnts, 0, b0, s_red) + wave_total(before) +
                    wave_inclusive(cnt) - cnt;
    if (mine) {
      gp(offs)[s] = off;
      if (s == S - 1) {
        gp(offs)[S] = off + cnt;
        put_total(w, off + cnt, KO == 3 ? w.cap_pt3 : w.cap_pt5, KO == 3 ? C_RPT3 : C_RPT5, KO == 3 ? C_NPT3 : C_NPT5);
      }
    }
    L.off[lane] = off;
    const int n = cnt <= keep ? cnt : 0;  // the others are searched again
    wave_segments(n, L.seg);
    const int start = L.seg[lane];
    for (int e0 = 0; e0 < kPtSeeds;) {
      // as many whole seeds as the stage holds
      const int c0 = L.seg[e0];
      const int e1 = e0 + __popcll(__ballot(lane >= e0 && lane < kPtSeeds && L.seg[lane + 1] - c0 <= kPtStage));
      const int c1 = L.seg[e1];
      int carry = e0;
      for (int r = c0; r < c1; r += 64) {
        const int c = r + lane, e = round_parent(start, n, r, L.mark, carry);
        if (c < c1) {
          L.val[c - c0] = gp(KO == 3 ? w.pt3_cache : w.pt5_cache)[(long)(s0 + e) * kCache + (c - L.seg[e])];
          L.par[c - c0] = (unsigned char)e;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (int c = c0 + lane; c < c1; c += 64) {
        const int e = L.par[c - c0], t = L.val[c - c0], a = L.seg[e] - c0, b = L.seg[e + 1] - c0;
        const float4 attr = gload(KO == 3 ? w.pt3_cattr : w.pt5_cattr, (long)(s0 + e) * kCache + (c - c0 - a));
        int rank = 0;
#pragma unroll 8
        for (int j = a; j < b; ++j) rank += L.val[j] < t ? 1 : 0;
        put_pt<KO>(w, L.off[e] + rank, s0 + e, t, attr);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      e0 = e1;
    }
  }
}

// The seed search over the objects of the bins a seed's trajectory can reach.
// The count: one wave per seed, both kinds on one mask; it counts the passing
// objects and keeps up to pt3_cache / pt5_cache of them with their attributes.
// A seed with more of a kind (seven of eight PU200 events') is a task of the fill,
// listed where its place among them says (pt_task); the first n_spill places have a
// list in global memory for the others' indices.
// The fill copies the kept ones (blocks [0, nc) the triplets, [nc, 2 nc) the
// quintuplets); the first waves of the other blocks share the tasks: a task's
// objects, from cache and list, or from a second search without a list, are ranked
// by object index in LDS and written at the seed's offset; with more of them than
// the LDS list holds (tile pass_list <= kPassList) an ordered scan over all objects
// is taken instead.  (Searching again for the seven made the fill 193 us.  With one
// wave to each 64 consecutive seeds' tasks the fill of a PU200 event with nothing
// cached took 1.53 ms, now 0.29, and with 16 triplets cached 117 us, now 50; that
// of a PU400 event 8.7, now 8.1, which is one seed's scan.)  More than max_slices marked bins are searched bin by bin.
// Tasks are counted in 16 lines by seed, since additions to one run one after
// another (a PU200 event's count took 197 us with 17,800 tasks on one counter, 72
// without); few seeds have one, so that the places stay below 4 n_seeds.
__device__ __forceinline__ int pt_shards(const Ws &w) { return w.n_seeds >= 256 ? kTaskShards : 1; }
__device__ __forceinline__ int pt_task(const Ws &w, int s) {  // called by one lane
  const int n = pt_shards(w), q = s & (n - 1);
  return atomicAdd(w.ts_task + q * kSumStride, 1) * n + q;
}

template <bool FILL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void k_pt_binned(const Ws *__restrict__ wb,
                                                                                              DevGeom g, int nc) {
  constexpr int kSets = FILL ? 1 : kWaves;  // waves that search
  __shared__ unsigned s_mask[kSets][kMaskWords];
  __shared__ int s_slo[kSets][kRings], s_shi[kSets][kRings];
  __shared__ int2 s_zb[kSets][kRings];
  __shared__ int s_sl_j0[kSets][kMaxSlices];       // bin id of each slice, then first list entry of each slice with candidates
  __shared__ int s_sl_pre[kSets][kMaxSlices];      // candidates before each slice with candidates
  __shared__ int s_list[FILL ? kPassList : 1];
  __shared__ int s_pq[kSets][128];  // MDs past the first-anchor test, their objects awaiting the full one
  __shared__ int s_mark[kSets][64];  // a slice's candidates start here (this round)
  __shared__ int s_seg[kSets][65], s_first[kSets][64];  // the queued MDs' objects
  const Ws &w = wb[blockIdx.y];
  const int wv = wave_id(), lane = lane_id();
  int s = 0;
  if constexpr (FILL) {
    __shared__ PtCopyLds s_copy[kWaves];
    __shared__ int s_red[kWaves];
    if ((int)blockIdx.x < nc) return pt_copy<3>(w, g, blockIdx.x, nc, s_copy[wv], s_red);
    if ((int)blockIdx.x < 2 * nc) return pt_copy<5>(w, g, (int)blockIdx.x - nc, nc, s_copy[wv], s_red);
    if (wv > 0) return;
  } else {
    const int si = (int)blockIdx.x * (int)(blockDim.x >> 6) + wv;
    if (si >= w.n_seeds) return;
    s = __float_as_int(gload(w.sdir, si).w);  // seeds of one direction on neighbouring waves
  }
  Seed sd{};
  if (!FILL) sd = load_seed(w, s);
  const int pass_list = g.tiles.pass_list;                            // <= kPassList
  const int max_slices = g.tiles.max_slices;                          // <= kMaxSlices
  unsigned *mask = s_mask[FILL ? 0 : wv];
  auto mark_bins = [&]() __attribute__((always_inline)) {  // the seed's (ring, azimuth) mask and z ranges
    for (int i = lane; i < kMaskWords; i += 64) mask[i] = 0u;
    if (lane < kRings) {
      s_slo[FILL ? 0 : wv][lane] = 0x7f7fffff;  // largest finite float
      s_shi[FILL ? 0 : wv][lane] = 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    mark_seed_bins(sd, mask, s_slo[FILL ? 0 : wv], s_shi[FILL ? 0 : wv]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane < kRings)
      s_zb[FILL ? 0 : wv][lane] = seed_zbins(sd, __int_as_float(s_slo[FILL ? 0 : wv][lane]), __int_as_float(s_shi[FILL ? 0 : wv][lane]));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // entries of one kind (KO = 3: triplets, 5: quintuplets) that passed so far
  int n_pass3 = 0, n_pass5 = 0;
  // the seed's tasks (-1: none), whose lists take its entries past the cache
  int spill3 = -1, spill5 = -1;
  const int n_spill = w.n_spill;
  // the full selection on one object per active lane; passing ones are counted in ballot
  // order and remembered (count: the cache with their attributes; fill: the LDS list)
  auto full = [&](auto kind, bool active, int t, int n_pass) __attribute__((always_inline)) {
    constexpr int KO = decltype(kind)::value;
    bool pass = false;
    float4 attr = make_float4(0.f, 0.f, 0.f, 0.f);
    // (quintuplets: those that survive the duplicate removal)
    if (active && (KO == 3 || gp(w.t5_keep)[t] != 0)) {
      float4 P[KO];
      ModInfo M[KO];
      float kT, dkT;
      load_object<KO>(w, g, t, P, M, &kT, &dkT);
      pass = pt_pass<KO>(sd, P, M, kT, dkT, &attr);
    }
    const unsigned long long m = __ballot(pass);
    const int keep = KO == 3 ? g.tiles.pt3_cache : g.tiles.pt5_cache;
    int &spill = KO == 3 ? spill3 : spill5;
    if (!FILL && n_pass + __popcll(m) > keep && spill == -1) {
      int v = 0;
      if (lane == 0) v = pt_task(w, s);
      spill = __builtin_amdgcn_readfirstlane(v);
    }
    if (pass) {
      const int r = n_pass + lanes_below(m);
      if (FILL) {
        if (r < kPassList) s_list[r] = t;
      } else if (r < keep) {
        constexpr int kCache = KO == 3 ? kPt3Cache : kPt5Cache;
        gp(KO == 3 ? w.pt3_cache : w.pt5_cache)[(long)s * kCache + r] = t;
        gstore(KO == 3 ? w.pt3_cattr : w.pt5_cattr, (long)s * kCache + r, attr);
      } else if (spill < n_spill && r < kPassList) {
        gp(w.pt_spill)[(long)spill * kPassList + r] = t;
      }
    }
    return n_pass + __popcll(m);
  };
  // the objects of the first n (<= 64) queued MDs, flattened over the lanes, one kind after the other
  auto expand = [&](auto kind, int n, int n_pass) __attribute__((always_inline)) {
    constexpr int KO = decltype(kind)::value;
    int first = 0, cnt = 0;
    if (lane < n) {
      const int4 r = gload(w.bin_rng, s_pq[FILL ? 0 : wv][lane]);
      first = KO == 3 ? r.x : r.z;
      cnt = KO == 3 ? r.y : r.w;
    }
    s_first[FILL ? 0 : wv][lane] = first;
    const int total = wave_segments(cnt, s_seg[FILL ? 0 : wv]);
    const int start = s_seg[FILL ? 0 : wv][lane];
    int carry = 0;
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int c = c0 + lane;
      const int e = round_parent(start, cnt, c0, s_mark[FILL ? 0 : wv], carry);
      n_pass = full(kind, c < total, c < total ? s_first[FILL ? 0 : wv][e] + (c - s_seg[FILL ? 0 : wv][e]) : 0, n_pass);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return n_pass;
  };
  // every marked bin's MDs through the exact first-anchor part of the selection (from the
  // packed anchor); MDs passing it are queued, and their objects of the wanted kinds get the
  // full selection
  auto search = [&](auto want3, auto want5) __attribute__((always_inline)) {
    // every marked (ring, azimuth) bin becomes a slice of the MD list (its reachable
    // z bins, possibly empty); bit ids first, ranked over the wave by a prefix of the
    // mask words' popcounts, then converted in place, 64 at a time, to (first entry,
    // candidates before it)
    int n_bits = 0;
    for (int w0 = 0; w0 < kMaskWords; w0 += 64) {
      const unsigned bits = w0 + lane < kMaskWords ? s_mask[FILL ? 0 : wv][w0 + lane] : 0u;
      const int pc = __popc(bits);
      const int x = wave_inclusive(pc);
      const int tot = __shfl(x, 63, 64);
      if (n_bits + tot <= max_slices) {
        int k = n_bits + x - pc;
        for (unsigned bb = bits; bb; bb &= bb - 1u) s_sl_j0[FILL ? 0 : wv][k++] = (w0 + lane) * 32 + __builtin_ctz(bb);
      }
      n_bits += tot;
    }
    const bool flat = n_bits <= max_slices;
    int run = 0, n_live = 0;
    if (flat) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // slices with candidates only, compacted in place (an entry is read before any
      // write of its round, and compacted positions never pass the round's own)
      for (int c0 = 0; c0 < n_bits; c0 += 64) {
        const int k = c0 + lane;
        int j0 = 0, len = 0;
        if (k < n_bits) {
          const int bin = s_sl_j0[FILL ? 0 : wv][k];
          const int2 zb = s_zb[FILL ? 0 : wv][bin / kPhiBins];
          j0 = gp(w.bin_off)[bin * kBinStride + zb.x];
          len = gp(w.bin_off)[bin * kBinStride + zb.y + 1] - j0;
        }
        const int x = wave_inclusive(len);
        const unsigned long long live = __ballot(len > 0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (len > 0) {
          const int q = n_live + lanes_below(live);
          s_sl_j0[FILL ? 0 : wv][q] = j0;
          s_sl_pre[FILL ? 0 : wv][q] = run + x - len;
        }
        n_live += __popcll(live);
        run += __builtin_amdgcn_readfirstlane(__shfl(x, 63, 64));
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    // Rounds of 64 MDs, from the slices laid end to end (flat), or, with more marked bins
    // than the slice table holds, bin by bin; one place that drains the queue.
    int c0 = 0, jlo = 0;                       // flat: round start, slices that start before it
    int wd = -1, j_at = 0, j_end = 0;          // bin by bin: mask word, list entries left of a bin
    unsigned bits = 0u;
    int nq = 0;
    for (bool last = false;;) {
      bool active = false;
      int j = 0;
      if (flat) {
        last = c0 >= run;
        if (!last) {
          // the slice of each lane's candidate: the slices starting before the round (jlo)
          // plus those starting at or below the lane in it (distinct starts, marked)
          const int c = c0 + lane;
          s_mark[FILL ? 0 : wv][lane] = 0;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          if (jlo + lane < n_live) {
            const int p = s_sl_pre[FILL ? 0 : wv][jlo + lane] - c0;  // >= 0
            if (p < 64) s_mark[FILL ? 0 : wv][p] = 1;
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          const unsigned long long starts = __ballot(s_mark[FILL ? 0 : wv][lane] != 0);
          active = c < run;
          if (active) {
            const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
            const int e = jlo - 1 + __popcll(starts & upto);
            j = s_sl_j0[FILL ? 0 : wv][e] + (c - s_sl_pre[FILL ? 0 : wv][e]);
          }
          jlo += __popcll(starts);
          c0 += 64;
        }
      } else {
        while (j_at >= j_end && !last) {  // the next marked bin with MDs
          while (bits == 0u && ++wd < kMaskWords) bits = mask[wd];
          last = wd >= kMaskWords;
          if (!last) {
            const int bin = wd * 32 + __builtin_ctz(bits);
            bits &= bits - 1u;
            const int2 zb = s_zb[FILL ? 0 : wv][bin / kPhiBins];
            j_at = uload(w.bin_off + bin * kBinStride + zb.x);
            j_end = uload(w.bin_off + bin * kBinStride + zb.y + 1);
          }
        }
        j = j_at + lane;
        active = !last && j < j_end;
        j_at += 64;
      }
      bool keep = false;
      if (active) {
        const float4 f = gload(w.bin_pos, j);
        keep = pt_first_anchor(sd, f, ModInfo{__float_as_int(f.w)});
      }
      const unsigned long long m = __ballot(keep);
      if (keep) s_pq[FILL ? 0 : wv][nq + lanes_below(m)] = j;
      nq += __popcll(m);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (nq >= 64 || (last && nq > 0)) {
        const int n = nq < 64 ? nq : 64;
        if constexpr (decltype(want3)::value) n_pass3 = expand(std::integral_constant<int, 3>{}, n, n_pass3);
        if constexpr (decltype(want5)::value) n_pass5 = expand(std::integral_constant<int, 5>{}, n, n_pass5);
        queue_pop64(s_pq[FILL ? 0 : wv], nq - n);
        nq -= n;
      }
      if (last && nq == 0) break;
    }
  };
  if constexpr (!FILL) {  // both kinds in one search
    mark_bins();
    search(std::true_type{}, std::true_type{});
    if (lane == 0) {
      gp(w.pt3_cnt)[s] = n_pass3;
      gp(w.pt5_cnt)[s] = n_pass5;
      if (n_pass3 > 0) atomicAdd(w.ts_p3 + (s >> w.sh_pt) * kSumStride, n_pass3);
      if (n_pass5 > 0) atomicAdd(w.ts_p5 + (s >> w.sh_pt) * kSumStride, n_pass5);
      if (spill3 >= 0) gp(w.pt_tasks)[spill3] = 2 * s;
      if (spill5 >= 0) gp(w.pt_tasks)[spill5] = 2 * s + 1;
    }
    return;
  }
  auto again = [&](auto kind, int spill) __attribute__((always_inline)) {
    constexpr int KO = decltype(kind)::value;
    const int keep = KO == 3 ? g.tiles.pt3_cache : g.tiles.pt5_cache;
    const int *cnts = KO == 3 ? w.pt3_cnt : w.pt5_cnt;
    const int expect = uload(cnts + s);
    sd = load_seed(w, s);
    int base = wave_prefix(KO == 3 ? w.ts_p3 : w.ts_p5, w.sh_pt, cnts, 0, s);
    if (expect > pass_list) {
      const float2 *first = KO == 3 ? w.t3_first : w.t5_first;
      const int n_obj = KO == 3 ? w.ctr[C_NT3] : w.ctr[C_NT5];
      for (int t0 = 0; t0 < n_obj; t0 += 64) {
        const int t = t0 + lane;
        bool pass = false;
        float4 attr = make_float4(0.f, 0.f, 0.f, 0.f);
        if (t < n_obj && (KO == 3 || gp(w.t5_keep)[t])) {
          const float2 f = first[t];
          if (seed_box(sd, f.x, f.y)) {
            float4 P[KO];
            ModInfo M[KO];
            float kT, dkT;
            load_object<KO>(w, g, t, P, M, &kT, &dkT);
            pass = pt_pass<KO>(sd, P, M, kT, dkT, &attr);
          }
        }
        const unsigned long long mp = __ballot(pass);
        if (pass) put_pt<KO>(w, base + lanes_below(mp), s, t, attr);
        base += __popcll(mp);
      }
      return;
    }
    int n = expect;
    if (spill < n_spill) {
      constexpr int kCache = KO == 3 ? kPt3Cache : kPt5Cache;
      for (int i = lane; i < n; i += 64)
        s_list[i] = i < keep ? gp(KO == 3 ? w.pt3_cache : w.pt5_cache)[(long)s * kCache + i]
                             : gp(w.pt_spill)[(long)spill * kPassList + i];
    } else {
      n_pass3 = n_pass5 = 0;
      mark_bins();
      search(std::integral_constant<bool, KO == 3>{}, std::integral_constant<bool, KO == 5>{});
      n = KO == 3 ? n_pass3 : n_pass5;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < n; i += 64) {
      const int t = s_list[i];
      int rank = 0;
#pragma unroll 8
      for (int r = 0; r < n; ++r) rank += s_list[r] < t ? 1 : 0;
      float4 attr;
      float4 P[KO];
      ModInfo M[KO];
      float kT, dkT;
      load_object<KO>(w, g, t, P, M, &kT, &dkT);
      pt_pass<KO>(sd, P, M, kT, dkT, &attr);
      put_pt<KO>(w, base + rank, s, t, attr);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (w.n_seeds == 0) return;  // (an event without seeds beside others: its counts are not cleared)
  const int shards = pt_shards(w), b = (int)blockIdx.x - 2 * nc, q = b & (shards - 1);
  const int n_task = uload(w.ts_task + q * kSumStride), step = ((int)gridDim.x - 2 * nc) / shards;
  for (int i = b / shards; i < n_task; i += step) {
    const int spill = i * shards + q, task = uload(w.pt_tasks + spill);
    s = task >> 1;
    if (task & 1) again(std::integral_constant<int, 5>{}, spill);
    else again(std::integral_constant<int, 3>{}, spill);
  }
}

template <int K>
__device__ __forceinline__ void obj_hits(const Ws &w, int t, int *h) {
  if constexpr (K == 3) {
    const int4 abc = gload(w.t3_md, t);
    const int md[3] = {abc.x, abc.y, abc.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int2 hh = w.md_hits[md[k]];
      h[2 * k] = hh.x;
      h[2 * k + 1] = hh.y;
    }
  } else {
    t5_hits(w, t, h);
  }
}

// pT duplicate removal: dropped when another entry with the same seed or the
// same outer object has a smaller (score, seed, hit tuple).  Entries of one
// seed differ in their outer object, so of a seed's entries only the one
// with the smallest (score, hit tuple) can survive; G lanes per seed find
// it (a minimum over the seed's entries, the hit tuples compared only on an
// exact tie of scores) and check it alone against the entries sharing its
// outer object, whose tuples differ from it in the seed only: it survives if
// it has the object's smallest (score, seed) (offered to it by the fill).
// G = 32 for pT3 (11 entries a seed on a PU200 event, up to 190), 8 for pT5 (0.8): a
// wave per seed left most lanes idle (89 us for eight events).
template <int K, int G>
__device__ __forceinline__ void pt_dedup(const Ws &w, int q, int nq) {
  const int n = uload(w.ctr + (K == 3 ? C_NPT3 : C_NPT5));
  const int2 *so = K == 3 ? w.pt3_so : w.pt5_so;
  const float4 *at = K == 3 ? w.pt3_attr : w.pt5_attr;
  const int *soff = K == 3 ? w.pt3_off : w.pt5_off;
  const unsigned long long *obest = K == 3 ? w.o3_best : w.o5_best;
  int *keep = K == 3 ? w.pt3_keep : w.pt5_keep;
  int *won = K == 3 ? w.w_pt3 : w.w_pt5;
  constexpr int H = 2 * K + 1;
  const int per = (int)blockDim.x / G, sub = threadIdx.x & (G - 1);
  // (whole groups: every lane of a group follows the same path)
  for (int s = q * per + (int)threadIdx.x / G; s < w.n_seeds; s += nq * per) {
    const int j0 = min(gp(soff)[s], n), j1 = min(gp(soff)[s + 1], n);
    // the smallest score of the seed's entries (scores of accepted entries are finite), an
    // entry that has it and how many do
    float best = 3.0e38f;
    int ties = 0, win = -1;
    for (int j = j0 + sub; j < j1; j += G) {
      const float z = gload(at, j).z;
      ties = z < best ? 1 : ties + (z == best ? 1 : 0);
      win = z <= best ? j : win;
      best = fminf(best, z);
    }
    for (int o = G / 2; o > 0; o >>= 1) {
      const float ob = __shfl_xor(best, o, G);
      const int ot = __shfl_xor(ties, o, G), ow = __shfl_xor(win, o, G);
      ties = ob < best ? ot : ties + (ob == best ? ot : 0);
      win = ob < best ? ow : (ob == best ? max(win, ow) : win);
      best = fminf(best, ob);
    }
    if (ties > 1) {  // (a tenth of a PU200 event's seeds)
      win = -1;
      int tw[H];
      const int g0 = lane_id() & ~(G - 1);  // the group's first lane in its wave
      for (int c0 = j0; c0 < j1; c0 += G) {
        const int j = c0 + sub;
        const unsigned long long m = __ballot(j < j1 && gload(at, min(j, j1 - 1)).z == best);
        for (unsigned mine = (unsigned)((m >> g0) & ((1ull << G) - 1)); mine; mine &= mine - 1u) {
          const int jt = c0 + __builtin_ctz(mine);
          int tj[H];
          tj[0] = s;
          obj_hits<K>(w, gload(so, jt).y, tj + 1);
          if (win < 0 || better<H>(best, tj, best, tw)) {
            win = jt;
#pragma unroll
            for (int i = 0; i < H; ++i) tw[i] = tj[i];
          }
        }
      }
    }
    // the winner survives the same-object rule if it is its object's best (score, seed)
    int obj = 0;
    bool kp = false;
    if (win >= 0) {
      obj = gload(so, win).y;
      kp = gload(obest, obj) == pt_obj_key(gload(at, win).z, s);
    }
    for (int j = j0 + sub; j < j1; j += G) gp(keep)[j] = (j == win && kp) ? 1 : 0;
    if (sub == 0) {
      gp(won)[s] = kp ? win : -1;
      if (K == 5 && kp) {  // every surviving pT5 is a candidate; its seed and T5 are used
        gp(w.sdir_tc)[gp(w.sdir_pos)[s]] = 1;
        gp(w.t5_used)[obj] = 1;
      }
    }
  }
}
// Quintuplet entries on blocks [0, n5), triplet entries on the others.
__global__ __launch_bounds__(kBlock) void k_pt_dedup(const Ws *__restrict__ wb, int n5) {
  const Ws &w = wb[blockIdx.y];
  if ((int)blockIdx.x < n5) pt_dedup<5, 8>(w, blockIdx.x, n5);
  else pt_dedup<3, 32>(w, (int)blockIdx.x - n5, (int)gridDim.x - n5);
}

// ------------------------------------------------------------- a8: TC
__device__ __forceinline__ Dir dir_of_t5(const Ws &w, int t) {
  const float *a = w.t5_attr + 8 * (long)t;
  Dir d;
  d.dx = gp(a)[6]; d.dy = gp(a)[7]; d.lam = gp(a)[3];
  return d;
}
__device__ __forceinline__ Dir dir_of(const float4 &e) {
  Dir d;
  d.dx = e.x; d.dy = e.y; d.lam = e.z;
  return d;
}

// The candidates' cleaning keeps one flag per seed or quintuplet, as bits of
// 64-bit words, so no launch counts or compacts between the steps and the
// writer ranks the candidates from the words' popcounts (1,000 words on a PU200
// event).  A wave takes the kCleanItems items of one byte: most have no
// candidate left to query, and the queries of one wave follow each other (with
// 16 items a wave the T5 step of a PU200 event took 28 us).
constexpr int kCleanItems = 8;
__device__ __forceinline__ int clean_waves(long n) { return (int)((n + 63) / 64) * 8; }  // bytes of whole words

// Calls f(place, entry) for the entries of the seeds' direction table within
// `reach` bins of direction d, 64 a round on the wave's lanes (on all lanes:
// active or not), until a call of a round returns true on some lane; returns
// whether one did.
template <class F>
__device__ __forceinline__ bool near_seeds(const Ws &w, const Dir &d, int reach, F &&f) {
  const int lane = lane_id();
  const int b = dir_bin(d.dx, d.dy), lo = b - reach, hi = b + reach + 1;  // bins [lo, hi), wrapping round
  const int a0 = uload(w.sdir_off + max(lo, 0)), a1 = uload(w.sdir_off + min(hi, kDirBins));
  int c0 = 0, c1 = 0;
  if (lo < 0) {
    c0 = uload(w.sdir_off + lo + kDirBins);
    c1 = w.n_seeds;
  } else if (hi > kDirBins) {
    c1 = uload(w.sdir_off + hi - kDirBins);
  }
  const int n1 = a1 - a0, n = n1 + c1 - c0;
  for (int r = 0; r < n; r += 64) {
    const int i = r + lane;
    const bool hit = i < n && f(i < n1 ? a0 + i : c0 + (i - n1));
    if (__ballot(hit)) return true;
  }
  return false;
}
// Whether a seed that is in a candidate (of the kinds in `kinds`) is near d.
__device__ __forceinline__ bool near_candidate(const Ws &w, const Dir &d, int kinds, float D, int reach) {
  return near_seeds(w, d, reach, [&](int j) {
    return (gp(w.sdir_tc)[j] & kinds) != 0 && near_dir(d, dir_of(gload(w.sdir, j)), D);
  });
}
__device__ __forceinline__ void put_flags(unsigned long long m, unsigned long long *words, int byte) {
  if (lane_id() == 0) reinterpret_cast<unsigned char *>(words)[byte] = (unsigned char)m;
}

// pT3 candidates: surviving pT3 whose seed no pT5 candidate uses and that is not
// near any pT5 candidate.
__global__ __launch_bounds__(kBlock) void k_tc_pt3(const Ws *__restrict__ wb) {
  const Ws &w = wb[blockIdx.y];
  const int lane = lane_id(), wpb = blockDim.x >> 6, n = clean_waves(w.n_seeds);
  for (int i = blockIdx.x * wpb + wave_id(); i < n; i += gridDim.x * wpb) {
    const int s = i * kCleanItems + lane;
    const bool mine = lane < kCleanItems && s < w.n_seeds;
    const bool five = mine && gp(w.w_pt5)[s] >= 0;
    const bool three = mine && !five && gp(w.w_pt3)[s] >= 0;
    const int pos = three ? gp(w.sdir_pos)[s] : 0;
    unsigned long long acc = 0;
    for (unsigned long long m = __ballot(three); m; m &= m - 1) {
      const int q = __builtin_ctzll(m);
      const Dir d = dir_of(gload(w.sdir, __builtin_amdgcn_readlane(pos, q)));
      if (!near_candidate(w, d, 1, kDpT3, bin_reach(0.02))) acc |= 1ull << q;
    }
    // (the other waves' queries ask for the pT5 bit alone)
    if (three && (acc >> lane & 1)) gp(w.sdir_tc)[pos] = 2;
    put_flags(__ballot(five), w.m_pt5, i);
    put_flags(acc, w.m_pt3, i);
  }
}

// T5 candidates (blocks [0, n5)): surviving T5 not used by a pT5 candidate and
// not near any pT5 or pT3 candidate; each marks the unused seeds near it.  pLS
// candidates (the others): surviving pLS used by no candidate and not near any
// pT5 or pT3 candidate; those marked by a T5 are left out when they are written.
__global__ __launch_bounds__(kBlock) void k_tc_t5(const Ws *__restrict__ wb, int n5) {
  const Ws &w = wb[blockIdx.y];
  const int lane = lane_id(), wpb = blockDim.x >> 6;
  if ((int)blockIdx.x < n5) {
    const int n_t5 = uload(w.ctr + C_NT5), n = clean_waves(n_t5);
    for (int i = blockIdx.x * wpb + wave_id(); i < n; i += n5 * wpb) {
      const int t = i * kCleanItems + lane;
      const bool cand = lane < kCleanItems && t < n_t5 && gp(w.t5_keep)[t] && !gp(w.t5_used)[t];
      unsigned long long acc = __ballot(cand);
      if (w.n_seeds > 0)
        for (unsigned long long m = acc; m; m &= m - 1) {
          const int q = __builtin_ctzll(m);
          const Dir d = dir_of_t5(w, __builtin_amdgcn_readlane(t, q));
          if (near_candidate(w, d, 3, kDT5, bin_reach(0.02))) {
            acc &= ~(1ull << q);
            continue;
          }
          near_seeds(w, d, bin_reach(0.05), [&](int j) {
            if (gp(w.sdir_tc)[j] == 0) {
              const float4 e = gload(w.sdir, j);
              const int s = __float_as_int(e.w);
              if (near_dir(dir_of(e), d, kDpLS)) atomicOr(w.pls_near + (s >> 5), 1u << (s & 31));
            }
            return false;
          });
        }
      put_flags(acc, w.m_t5, i);
    }
    return;
  }
  const int n = clean_waves(w.n_seeds), nw = ((int)gridDim.x - n5) * wpb;
  for (int i = ((int)blockIdx.x - n5) * wpb + wave_id(); i < n; i += nw) {
    const int s = i * kCleanItems + lane;
    const bool mine = lane < kCleanItems && s < w.n_seeds;
    const int pos = mine ? gp(w.sdir_pos)[s] : 0;
    unsigned long long acc = __ballot(mine && gp(w.pls_keep)[s] && gp(w.sdir_tc)[pos] == 0);
    for (unsigned long long m = acc; m; m &= m - 1) {
      const int q = __builtin_ctzll(m);
      const Dir d = dir_of(gload(w.sdir, __builtin_amdgcn_readlane(pos, q)));
      if (near_candidate(w, d, 3, kDpLS, bin_reach(0.05))) acc &= ~(1ull << q);
    }
    put_flags(acc, w.m_pls, i);
  }
}

// What the track-extension step reads of a candidate: its MDs and its
// curvature with tolerance (the seed's, three resolutions, for pT5 / pT3;
// the five-anchor fit's and the outer triplet's resolution for a T5).
__device__ __forceinline__ float2 seed_kappa(const Ws &w, int seed) {
  const float ks = gp(w.pls)[8 * (long)seed + 4];
  return make_float2(ks, 3.0f * (kSeedDpt * fabsf(ks)));
}
__device__ __forceinline__ void ext_record(const Ws &w, int k, const int *md, int K, float2 kap) {
  for (int i = 0; i < K; ++i) w.tc_md[5 * (long)k + i] = md[i];
  gstore(w.tc_kap, k, kap);
}

// Output: type, offsets, hit lists (pixel hits first, then MD hits inner to
// outer), in the order pT5, pT3, T5, pLS.  A wave takes one word of flags of one
// kind; its candidates' ranks come from the popcounts of the words before it and
// of the kinds before its own, which every block sums for itself; its hit lists
// are consecutive, so they are put together in LDS and written as one run, to
// host memory as well if all candidates fit there.  last_launch: this launch ends the
// chain (no track extensions), so its results go to the host.
__global__ __launch_bounds__(kBlock) void k_tc_write(const Ws *__restrict__ wb, int n_seed_blocks, int last_launch) {
  __shared__ int s_sum[kWaves][5];
  __shared__ int s_hits[kWaves][64 * 14];
  const Ws &w = wb[blockIdx.y];
  const int S = w.n_seeds, n_t5 = uload(w.ctr + C_NT5);
  const int sw = (S + 63) >> 6, tw = (n_t5 + 63) >> 6;
  // kind 0 pT5, 1 pT3, 2 pLS: n_seed_blocks each; 3 T5: the rest
  const int kind = min((int)blockIdx.x / n_seed_blocks, 3);
  const int q = (int)blockIdx.x - kind * n_seed_blocks, nq = kind < 3 ? n_seed_blocks : (int)gridDim.x - 3 * n_seed_blocks;
  const int words = kind < 3 ? sw : tw;
  const int lane = lane_id(), wv = wave_id();
  // the block's words: a consecutive share of the kind's
  const int share = ((words + nq - 1) / nq + kWaves - 1) / kWaves * kWaves;
  const long first = (long)q * share, last = min(first + share, (long)words);
  const bool totals = blockIdx.x == 0;
  if (first >= last && !totals) return;
  auto pls_word = [&](int j) {
    return gp(w.m_pls)[j] & ~gp(reinterpret_cast<const unsigned long long *>(w.pls_near))[j];
  };
  auto word = [&](int k, int j) {
    return k == 0 ? gp(w.m_pt5)[j] : k == 1 ? gp(w.m_pt3)[j] : k == 2 ? pls_word(j) : gp(w.m_t5)[j];
  };
  int v[5] = {0, 0, 0, 0, 0};  // candidates of each kind, and of this kind before `first`
  for (int j = threadIdx.x; j < sw; j += kBlock) {
    v[0] += __popcll(word(0, j));
    v[1] += __popcll(word(1, j));
    v[2] += __popcll(word(2, j));
  }
  for (int j = threadIdx.x; j < tw; j += kBlock) v[3] += __popcll(word(3, j));
  for (int j = threadIdx.x; j < first; j += kBlock) v[4] += __popcll(word(kind, j));
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int x = wave_total(v[i]);
    if (lane == 0) s_sum[wv][i] = x;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    int x = 0;
    for (int p = 0; p < kWaves; ++p) x += s_sum[p][i];
    v[i] = x;
  }
  const int n0 = v[0], n1 = v[1], n2 = v[3], n3 = v[2], n = n0 + n1 + n2 + n3;
  const long h1 = 14L * n0, h2 = h1 + 10L * n1, h3 = h2 + 10L * n2, nh = h3 + 4L * n3;
  int *host = (last_launch && w.h_tc && 2L * n + 1 + nh <= w.h_tc_cap) ? w.h_tc : nullptr;
  auto put = [&](long i, int x) {
    gp(w.tc_out)[i] = x;
    if (host) gp(host)[i] = x;
  };
  if (totals && wv == 0) {
    const int mine[6] = {C_NTC0, C_NTC1, C_NTC2, C_NTC3, C_NTC, C_NTCHITS};
    const int val[6] = {n0, n1, n2, n3, n, (int)nh};
    int x = gp(w.ctr)[lane];
    static_assert(C_COUNT == 64, "a counter per lane");
#pragma unroll
    for (int i = 0; i < 6; ++i)
      if (lane == mine[i]) {
        x = val[i];
        gp(w.ctr)[lane] = x;
      }
    if (last_launch && w.h_ctr) gp(w.h_ctr)[lane] = x;
    if (lane == 0) put(2L * n, (int)nh);  // the offsets' end
  }
  const int width = kind == 0 ? 14 : (kind == 2 ? 4 : 10);
  const int at = kind == 0 ? 0 : (kind == 1 ? n0 : (kind == 3 ? n0 + n1 : n0 + n1 + n2));  // the kind's first candidate
  const long hat = kind == 0 ? 0 : (kind == 1 ? h1 : (kind == 3 ? h2 : h3));               // and its first hit
  int run = v[4];  // this kind's candidates before the round
  for (long r = first; r < last; r += kWaves) {
    int k0 = run;
    unsigned long long m = 0;
    for (int p = 0; p < kWaves; ++p) {
      const unsigned long long mp = r + p < last ? word(kind, (int)r + p) : 0ull;
      if (p < wv) k0 += __popcll(mp);
      if (p == wv) m = mp;
      run += __popcll(mp);
    }
    if (m >> lane & 1) {
      const int row = lanes_below(m), k = at + k0 + row;
      const int i = (int)(r + wv) * 64 + lane;  // the seed or the quintuplet
      int *h = &s_hits[wv][row * width];
      if (kind != 3)
        for (int p = 0; p < 4; ++p) h[p] = gp(w.hits4)[4 * (long)i + p];
      if (kind == 0) {
        const int2 so = gload(w.pt5_so, gp(w.w_pt5)[i]);
        t5_hits(w, so.y, h + 4);
        ext_record(w, k, w.t5_md + 5 * (long)so.y, 5, seed_kappa(w, i));
      } else if (kind == 1) {
        const int2 so = gload(w.pt3_so, gp(w.w_pt3)[i]);
        obj_hits<3>(w, so.y, h + 4);
        const int4 abc = gload(w.t3_md, so.y);
        const int md[3] = {abc.x, abc.y, abc.z};
        ext_record(w, k, md, 3, seed_kappa(w, i));
      } else if (kind == 3) {
        t5_hits(w, i, h);
        ext_record(w, k, w.t5_md + 5 * (long)i, 5,
                   make_float2(w.t5_attr[8 * (long)i], w.t3_attr[gload(w.t5_t3, i).y].y));
      }
      put(k, kind == 2 ? 3 : (kind == 3 ? 2 : kind));
      put((long)n + k, (int)(hat + (long)width * (k0 + row)));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int cnt = __popcll(m) * width;
    for (int i = lane; i < cnt; i += 64) put(2L * n + 1 + hat + (long)width * k0 + i, s_hits[wv][i]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------- track extensions (S2.5)
// A candidate with outer MDs (pT5, pT3, T5) is tested against the triplets
// whose first two MDs are its last two (one MD added) and those whose first
// MD is its last (two added): curvatures within their resolutions (the
// seed's for pT5 / pT3, three resolutions; the outer triplet's for a T5),
// azimuth linear in z over the first, the candidate's last and the last
// added anchor, and the widened quintuplet fits (ext_fit).  The passing
// triplet adding more MDs wins, then the smaller chi2_xy + chi2_rz, then the
// smaller hit tuple of the added MDs.
//
// A wave takes kExtPerWave candidates; their (candidate, triplet) pairs are
// laid out flat (wave_segments) so the lanes test one pair each, and every
// candidate's lane then merges the passing pairs of its segment from LDS.  (A thread per
// candidate walking its own triplets is bound by the longest such walk.)
// (add, score, hits) of a strictly better than those of b
__device__ __forceinline__ bool ext_better(int add_a, float sc_a, int4 h_a, int add_b, float sc_b, int4 h_b) {
  if (add_a != add_b) return add_a > add_b;
  if (sc_a < sc_b) return true;
  if (sc_b < sc_a) return false;
  const int ha[4] = {h_a.x, h_a.y, h_a.z, h_a.w}, hb[4] = {h_b.x, h_b.y, h_b.z, h_b.w};
  for (int i = 0; i < 2 * add_a; ++i)
    if (ha[i] != hb[i]) return ha[i] < hb[i];
  return false;
}

// The K anchors of a candidate (K = 3 or 5; sP / sM [0..K)[e], staged in
// LDS) followed by the ADD MDs of triplet abc in the kExtMax slots of ext_fit
// (the slots past the chain repeat its last anchor), tested with the
// lever-arm azimuth-z check and ext_fit; the added MDs' hits come back in h.
template <int C>
__device__ __forceinline__ bool ext_eval(const Ws &w, const DevGeom &g, const float4 (*sP)[C], const int (*sM)[C],
                                         int e, int K, int add, int4 abc, float3 *a, int4 *h) {
  const int nm0 = add == 1 ? abc.z : abc.y;
  const float4 A0 = gload(w.md_pos, nm0);
  const int mod0 = gp(w.md_mod)[nm0];
  const int2 h0 = gload(w.md_hits, nm0);
  float4 A1 = A0;
  int mod1 = mod0;
  int2 h1 = make_int2(0, 0);
  if (add == 2) {
    A1 = gload(w.md_pos, abc.z);
    mod1 = gp(w.md_mod)[abc.z];
    h1 = gload(w.md_hits, abc.z);
  }
  ModInfo I0, I1;
  I0.bits = gp(g.info)[mod0];
  I1.bits = gp(g.info)[mod1];
  float4 P[kExtMax];
  ModInfo M[kExtMax];
#pragma unroll
  for (int i = 0; i < kExtMax; ++i) {
    if (i < 5 && i < K) {
      P[i] = sP[i][e];
      M[i].bits = sM[i][e];
    } else {
      P[i] = i == K ? A0 : A1;
      M[i] = i == K ? I0 : I1;
    }
  }
  *h = make_int4(h0.x, h0.y, h1.x, h1.y);
  const float4 PK = K == 5 ? P[4] : P[2];
  const ModInfo MK = K == 5 ? M[4] : M[2];
  return phiz_pass(P[0], PK, A1, M[0], MK, I1, g.d0max) && ext_fit(P, M, K + add, a);
}

// Candidates per wave, C (tile ext_per_wave: 4, 8 or 16): few enough that
// their (candidate, triplet) pairs (about 1.3 per candidate) spread over many
// waves.
template <int C>
__global__ __launch_bounds__(kBlock) void k_tc_ext(const Ws *__restrict__ wb, DevGeom g) {
  const Ws &w = wb[blockIdx.y];
  constexpr int kExtPerWave = C;
  __shared__ float4 s_P[kWaves][5][C];  // the candidates' anchors
  __shared__ int s_M[kWaves][5][C], s_md[kWaves][C], s_k[kWaves][C], s_lo2[kWaves][C], s_n2[kWaves][C],
      s_lo1[kWaves][C];  // module info bits, last MD, MD count, triplet ranges
  __shared__ int s_seg[kWaves][65];
  __shared__ float s_kt[kWaves][C], s_dkt[kWaves][C];
  __shared__ int s_rt[kWaves][64], s_radd[kWaves][64];  // per pair of the round: triplet (-1: fails), MDs added
  __shared__ float s_rsc[kWaves][64];
  __shared__ int4 s_rh[kWaves][64];
  __shared__ float4 s_ra[kWaves][64];
  const int n = uload(w.ctr + C_NTC);
  const int n_ls = uload(w.ctr + C_NLS), n_t3 = uload(w.ctr + C_NT3);
  const int wv = wave_id(), lane = lane_id();
  const int wpb = blockDim.x >> 6;
  for (long p0 = ((long)blockIdx.x * wpb + wv) * kExtPerWave; p0 < n; p0 += (long)gridDim.x * wpb * kExtPerWave) {
    const int k = (int)p0 + lane;
    const bool mine = lane < kExtPerWave && k < n;
    int cnt = 0;
    if (mine) {
      const int type = gp(w.tc_out)[k];
      const int K = type == 3 ? 0 : (type == 1 ? 3 : 5);
      s_k[wv][lane] = K;
      if (K > 0) {
        int md[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) md[i] = i < K ? w.tc_md[5 * (long)k + i] : 0;
        const float2 kap = gload(w.tc_kap, k);
        s_kt[wv][lane] = kap.x;
        s_dkt[wv][lane] = kap.y;
#pragma unroll
        for (int i = 0; i < 5; ++i)
          if (i < K) {
            s_P[wv][i][lane] = w.md_pos[md[i]];
            s_M[wv][i][lane] = gp(g.info)[gp(w.md_mod)[md[i]]];
          }
        // triplets with first MD m: those built from segments with inner MD m
        const int m2 = K == 5 ? md[3] : md[1], m1 = K == 5 ? md[4] : md[2];
        s_md[wv][lane] = m1;
        const int l2b = min(w.ls_off[m2], n_ls), l2e = min(w.ls_off[m2 + 1], n_ls);
        const int l1b = min(w.ls_off[m1], n_ls), l1e = min(w.ls_off[m1 + 1], n_ls);
        const int lo2 = gp(w.t3_off)[l2b], hi2 = min(w.t3_off[l2e], n_t3);
        const int lo1 = gp(w.t3_off)[l1b], hi1 = min(w.t3_off[l1e], n_t3);
        const int n2 = hi2 > lo2 ? hi2 - lo2 : 0, n1 = hi1 > lo1 ? hi1 - lo1 : 0;
        s_lo2[wv][lane] = lo2;
        s_n2[wv][lane] = n2;
        s_lo1[wv][lane] = lo1;
        cnt = n2 + n1;
      }
    }
    const int total = wave_segments(cnt, s_seg[wv]);
    int best_n = 0, best_t = -1;
    float best_s = 0.0f;
    int4 best_h = make_int4(0, 0, 0, 0);
    float4 best_a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    int e = 0;  // candidate of this lane's pair (pairs advance monotonically)
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int c = c0 + lane;
      int rt = -1, radd = 0;
      float rsc = 0.0f;
      int4 rh = make_int4(0, 0, 0, 0);
      float4 ra = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (c < total) {
        while (s_seg[wv][e + 1] <= c) ++e;
        const int idx = c - s_seg[wv][e];
        const int K = s_k[wv][e], n2 = s_n2[wv][e];
        const int ov = idx < n2 ? 2 : 1;
        const int t = ov == 2 ? s_lo2[wv][e] + idx : s_lo1[wv][e] + (idx - n2);
        const int4 abc = gload(w.t3_md, t);
        const float4 ta = gload(w.t3_attr, t);
        const int add = 3 - ov;
        const float dk = ta.x - s_kt[wv][e];
        bool ok = ov == 1 || abc.y == s_md[wv][e];
        ok = ok && fabsf(dk) <= ta.y + s_dkt[wv][e];
        if (ok) {
          // the anchors fill ext_fit's fixed slots (static indices: they stay in registers)
          float3 a;
          int4 h;
          if (ext_eval(w, g, s_P[wv], s_M[wv], e, K, add, abc, &a, &h)) {
            rt = t;
            radd = add;
            rsc = a.x + a.y;
            rh = h;
            ra = make_float4(a.x, a.y, a.z, 0.0f);
          }
        }
      }
      s_rt[wv][lane] = rt;
      s_radd[wv][lane] = radd;
      s_rsc[wv][lane] = rsc;
      s_rh[wv][lane] = rh;
      s_ra[wv][lane] = ra;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // every candidate merges the pairs of its segment that fell in this round
      const int q0 = max(s_seg[wv][lane], c0) - c0, q1 = min(s_seg[wv][lane + 1], c0 + 64) - c0;
      for (int q = q0; q < q1; ++q) {
        const int t = s_rt[wv][q];
        if (t < 0) continue;
        const int add = s_radd[wv][q];
        const float sc = s_rsc[wv][q];
        const int4 h = s_rh[wv][q];
        if (best_t < 0 || ext_better(add, sc, h, best_n, best_s, best_h)) {
          best_n = add; best_t = t; best_s = sc; best_h = h; best_a = s_ra[wv][q];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    if (mine) {
      const ExtOut x(w.ext_out, n);
      gp(x.added)[k] = best_n;
      gp(x.t3)[k] = best_t;
      const float at[4] = {best_a.x, best_a.y, best_a.z, best_a.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) gp(x.attr)[4L * k + i] = __float_as_int(at[i]);
      w.ext_cnt[k] = (gp(w.tc_out)[n + k + 1] - gp(w.tc_out)[n + k]) + 2 * best_n;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// The extended collection: each candidate's hits, then those of its added MDs,
// and the types and offsets beside what the search wrote.  A wave takes 64
// candidates, whose hit lists are consecutive: put together in LDS and written
// as one run, to host memory as well (with the rest of ext_out) if it fits there.
__global__ __launch_bounds__(kBlock) void k_tc_ext_write(const Ws *__restrict__ wb) {
  __shared__ int s_hits[kWaves][64 * 18];
  const Ws &w = wb[blockIdx.y];
  const int n = uload(w.ctr + C_NTC), nh = uload(w.ctr + C_NEXTHITS);
  const int lane = lane_id(), wv = wave_id();
  if (blockIdx.x == 0 && wv == 0) {  // the chain's end: the counters to the host
    static_assert(C_COUNT == 64, "a counter per lane");
    int x = gp(w.ctr)[lane];
    if (lane == C_EXT) {
      x = 1;
      gp(w.ctr)[lane] = x;
    }
    if (w.h_ctr) gp(w.h_ctr)[lane] = x;
  }
  int *host = (w.h_tc && ExtOut::ints(n, nh) <= w.h_tc_cap) ? w.h_tc : nullptr;
  const ExtOut x(w.ext_out, n), y(host, n);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    x.off[n] = nh;
    if (host) y.off[n] = nh;
  }
  for (long c0 = ((long)blockIdx.x * kWaves + wv) * 64; c0 < n; c0 += (long)gridDim.x * kWaves * 64) {
    const int k = (int)c0 + lane;
    const int first = uload(w.ext_off + c0);
    const int end = uload(w.ext_off + min(c0 + 64, (long)n));
    if (k < n) {
      const int type = gp(w.tc_out)[k], b0 = gp(w.tc_out)[n + k], b1 = gp(w.tc_out)[n + k + 1];
      const int off = gp(w.ext_off)[k], na = gp(x.added)[k], t3 = gp(x.t3)[k];
      int *dst = &s_hits[wv][off - first];
      for (int h = b0; h < b1; ++h) *dst++ = gp(w.tc_out)[2L * n + 1 + h];
      if (na > 0) {
        const int4 abc = gload(w.t3_md, t3);
        int2 hh = gload(w.md_hits, na == 1 ? abc.z : abc.y);
        dst[0] = hh.x;
        dst[1] = hh.y;
        if (na == 2) {
          hh = gload(w.md_hits, abc.z);
          dst[2] = hh.x;
          dst[3] = hh.y;
        }
      }
      gp(x.type)[k] = type;
      gp(x.off)[k] = off;
      if (host) {
        gp(y.type)[k] = type;
        gp(y.off)[k] = off;
        gp(y.added)[k] = na;
        gp(y.t3)[k] = t3;
        for (int i = 0; i < 4; ++i) gp(y.attr)[4L * k + i] = gp(x.attr)[4L * k + i];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < end - first; i += 64) {
      const int v = s_hits[wv][i];
      gp(x.hits)[(long)first + i] = v;
      if (host) gp(y.hits)[(long)first + i] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------- chain
// Launch sites of the chain, in order; each runs once per event, those whose
// work rides in another site's launch without one of their own.  One of them can
// be bracketed by HIP events (KernelTimer) to time it live.
const char *const kSiteNames[] = {
    "fill_counters", "hits_count", "hits_scan", "hits_scatter", "bucket_sort",
    "md_count", "md_scan", "md_fill", "ls_count", "ls_scan", "ls_fill",
    "t3_count", "t3_scan", "t3_fill", "t5_count", "t5_scan", "t5_fill",
    "t5_inc_count", "t5_inc_scan", "t5_inc_scatter", "t5_dedup",
    "pls", "pls_hit_scan", "pls_hit_scatter", "pls_dedup",
    "pt3_bin", "pt5_bin", "pt_count", "pt3_scan", "pt3_fill", "pt5_scan", "pt5_fill",
    "pt_obj_best", "pt3_dedup", "pt5_dedup",
    "tc_pt5", "tc_pt5_scan", "tc_pt5_dirs", "tc_pt3", "tc_pt3_scan", "tc_pt3_dirs",
    "tc_t5", "tc_t5_scan", "tc_t5_dirs", "tc_pls", "tc_pls_scan", "tc_write",
    "tc_ext", "tc_ext_scan", "tc_ext_write"};
const int kNumSites = (int)(sizeof(kSiteNames) / sizeof(kSiteNames[0]));
static_assert(sizeof(kSiteNames) / sizeof(kSiteNames[0]) <= kMaxSites, "launch-site table");

// Sites whose kernels take any block of 64, 128 or 256 threads (grid-stride
// loops over threads or waves, LDS sized for the largest block): the launch
// shape the autotuner may choose.  (md_count, md_fill, pt5_fill and tc_pls, whose
// work is in other launches or a block of fixed size, take a shape, as in files
// that were saved when they read it, and have none to choose.)
static const char *const kTunableSites[] = {"md_count", "md_fill",  "ls_count", "ls_fill",  "t3_count",
                                            "t3_fill",  "t5_count", "t5_fill",  "t5_dedup", "pt_count",
                                            "pt3_fill", "pt5_fill", "tc_pt3",   "tc_t5",    "tc_pls",
                                            "tc_ext"};

bool site_tunable(int site) {
  if (site < 0 || site >= kNumSites) return false;
  for (const char *n : kTunableSites)
    if (std::strcmp(n, kSiteNames[site]) == 0) return true;
  return false;
}

bool site_shaped(int site) {
  if (!site_tunable(site)) return false;
  for (const char *n : {"md_count", "md_fill", "pt5_fill", "tc_pls"})
    if (std::strcmp(n, kSiteNames[site]) == 0) return false;
  return true;
}

// Inner MDs per wave of the segment count pass: the tile when set, else the
// square root of the launch's expected MDs (a quarter of the MD capacity, which
// defaults to the hit count) / 2048.  Large groups fill the lanes of the pair,
// candidate and selection rounds; a launch with few MDs needs the waves more.
// Measured with 1 / 2 / 4 / 6 / 8 MDs: tiny event (1.4k MDs) 9 / 14 / 21 / 27 / 33 us,
// PU50 (37k) 40 / 32 / 28 / 34 / 40, PU140 (75k) - / 76 / 64 / 57 / 58, PU200 (138k)
// - / 115 / 90 / 90 / 85; eight PU200 events with 4 / 8 / 12 708 / 631 / 622.
int ls_group_for(const Tiles &t, int B, long cap_md) {
  if (t.ls_group > 0) return t.ls_group < kLsGroup ? t.ls_group : kLsGroup;
  const long n = (long)B * (cap_md / 4);
  int q = 1;
  while (q < kLsGroup && (q + 1) * (q + 1) * 2048L <= n) ++q;
  return q;
}

void enqueue_chain(const DevGeom &g, Ws *wb, int B, const Ws &b, hipStream_t st, const KernelTimer *kt,
                   const int *site_block, const Ws *value) {
  int site = 0;
  int tb = kBlock;  // block size of the current site (tunable sites only)
  // Runs one launch site; the timed site is bracketed by the timer's events.
  auto run = [&](auto &&launch) {
    const bool timed = kt && kt->site == site;
    tb = (site_block && site_block[site] > 0) ? site_block[site] : kBlock;
    if (timed) (void)hipEventRecord(kt->beg, st);
    launch();
    if (timed) (void)hipEventRecord(kt->end, st);
    ++site;
  };
  const int M = g.n_mod;
  const long N = b.n_hits, S = b.n_seeds;  // largest of the batch
  const bool seeds = S > 0;
  // Blocks per event: what the capacity would ask for, but at most an equal share of
  // kLaunchWaves.  The kernels launched through these stride over their device-side
  // counts, and the counts are far below the capacities: a launch over many events
  // would otherwise spend most of its time dispatching blocks that find no work.
  const long ev_waves = std::max(256L, kLaunchWaves / B);
  auto share = [&](int blocks, int threads) {
    return (unsigned)std::max(1L, std::min((long)blocks, ev_waves / (threads / 64)));
  };
  auto share_big = [&](int blocks, int threads) {
    return (unsigned)std::max(1L, std::min((long)blocks, 4 * ev_waves / (threads / 64)));
  };
  auto grid = [&](long n) { return dim3(share(grid_for(n), kBlock), B); };
  auto gridwt = [&](long n) { return dim3(share(grid_waves(n, tb), tb), B); }; // tuned wave-per-item sites
  auto gridwb = [&](long n) { return dim3(share_big(grid_waves(n, tb), tb), B); }; // the heavy searches
  // one wave per seed, every seed its own wave (the seed search does not stride)
  auto seedwaves = [&] { return dim3((unsigned)((S + tb / 64 - 1) / (tb / 64) > 0 ? (S + tb / 64 - 1) / (tb / 64) : 1), B); };
  const dim3 one(1, B);
  const bool whole = kt && kt->site == kChainSite;  // the timer brackets the whole chain
  if (whole) (void)hipEventRecord(kt->beg, st);
  // a0: buckets
  run([&] {});  // fill_counters: with hits_count
  // hits: the tile (rounds of 64 hits a wave) grows with the launch's hits, so that a
  // small event still fills blocks and a large launch amortises a block's tables
  const long n_co = n_coarse(M);
  const int rounds = N * B <= 262144 ? 1 : (N * B <= 1048576 ? 2 : 4);
  const int tile = kHitTile * rounds;
  const long n_tiles = n_hit_tiles(N, tile);
  const bool wide = n_co <= 1700;  // sixteen waves' rows fit 64 KiB of LDS
  const unsigned hit_blocks = (unsigned)std::max(1L, n_tiles);
  const size_t lds_scatter = n_co * sizeof(int) + (wide ? 16 : 8) * ((n_co + 1) / 2) * sizeof(int);
  auto by_tile = [&](auto &&f) {
    using std::integral_constant;
    if (wide) {
      if (rounds == 1) f(integral_constant<int, 16>{}, integral_constant<int, 1>{});
      else if (rounds == 2) f(integral_constant<int, 16>{}, integral_constant<int, 2>{});
      else f(integral_constant<int, 16>{}, integral_constant<int, 4>{});
    } else {
      if (rounds == 1) f(integral_constant<int, 8>{}, integral_constant<int, 2>{});
      else if (rounds == 2) f(integral_constant<int, 8>{}, integral_constant<int, 4>{});
      else f(integral_constant<int, 8>{}, integral_constant<int, 8>{});
    }
  };
  run([&] {  // one block per hit tile, the clears on further blocks
    by_tile([&](auto nw, auto r) {
      constexpr int T = 64 * nw();
      const dim3 d(hit_blocks + std::max(1u, grid(seeds ? kSeedBins : 4096).x * kBlock / T), B);
      if (value) k_hits_count<true, nw(), r()><<<d, T, n_co * sizeof(int), st>>>(*value, wb, M, (int)hit_blocks);
      else k_hits_count<false, nw(), r()><<<d, T, n_co * sizeof(int), st>>>(Ws{}, wb, M, (int)hit_blocks);
    });
  });
  const int direct = n_tiles <= kDirectTiles ? 1 : 0;
  run([&] { if (!direct) k_hits_rows<<<dim3((unsigned)((n_co + 31) / 32), B), 1024, 0, st>>>(wb, M, tile); });
  run([&] {
    by_tile([&](auto nw, auto r) {
      k_hits_scatter<nw(), r()><<<dim3(hit_blocks, B), 64 * nw(), lds_scatter, st>>>(wb, M, direct);
    });
  });
  // the bucket sort and a1: MD
  const bool crowded = N > kCrowdedHits * M;
  // (with the seeds in further blocks)
  run([&] {
    const unsigned n_seed = (unsigned)std::min((S + kSortThreads - 1) / kSortThreads, 4096L);
    const dim3 d((unsigned)n_co + n_seed, B);
    if (crowded) k_bucket_md<true><<<d, kSortThreads, 0, st>>>(wb, g);
    else k_bucket_md<false><<<d, kSortThreads, 0, st>>>(wb, g);
  });
  for (int q = 0; q < 2; ++q) run([&] {});  // md_count, md_scan: with bucket_sort, md_fill
  run([&] {
    if (crowded) k_md_fill<true><<<dim3((unsigned)n_co, B), kSortThreads, 0, st>>>(wb, g);
    else k_md_fill<false><<<dim3((unsigned)n_co, B), kSortThreads, 0, st>>>(wb, g);
  });
  // a2: LS
  run([&] {
    const int lg = ls_group_for(g.tiles, B, b.cap_md);
    k_ls_count<<<gridwb((b.cap_md + lg - 1) / lg), tb, 0, st>>>(wb, g, lg);
  });
  const bool ls_direct = !seeds && b.cap_md <= kDirectMds;
  run([&] {
    if (ls_direct) return;
    const unsigned n_sum = (unsigned)std::min<long>(n_sum_tiles(b.cap_md), 256);
    const unsigned n_seed = seeds ? grid(S).x : 0;
    k_ls_sums<<<dim3(n_sum + n_seed, B), kBlock, 0, st>>>(wb, g.tiles.ls_cache, (int)n_sum);
  });
  run([&] {
    const unsigned n_copy = gridwt((b.cap_md + kLsCopyMds - 1) / kLsCopyMds).x;
    const unsigned n_ovf = ls_direct ? 0 : gridwt(std::min(b.cap_md, 4096)).x;  // the overflow MDs (428 on a PU200 event)
    k_ls_fill<<<dim3(n_copy + n_ovf, B), tb, 0, st>>>(wb, g, (int)n_copy, ls_direct ? 1 : 0);
  });
  // a3: T3
  run([&] { k_t3<false><<<gridwt(b.cap_ls / kMinParents + 1), tb, 0, st>>>(wb, g); });
  run([&] {});  // t3_scan
  run([&] { k_t3<true><<<gridwt(b.cap_ls / kMinParents + 1), tb, 0, st>>>(wb, g); });
  // a4: T5
  // (with the seed search's bins in further blocks)
  run([&] {
    const dim3 d = gridwt(b.cap_t3 / kMinParents + 1);
    const unsigned nq = seeds ? share(grid_for(b.cap_md, tb), tb) : 0;
    k_t5<false><<<dim3(d.x + nq, B), tb, 0, st>>>(wb, g, (int)d.x);
  });
  run([&] {});  // t5_scan
  run([&] {
    const dim3 d = gridwt(b.cap_t3 / kMinParents + 1);
    const int rows = (tb / 64) * kRowsPerWave;
    const unsigned nq = seeds ? (kBinRows + rows - 1) / rows : 0;
    k_t5<true><<<dim3(d.x + nq, B), tb, 0, st>>>(wb, g, (int)d.x);
  });
  // a5: T5 duplicate removal through per-MD incidence lists, or over all pairs of few
  const bool pairs = b.cap_t5 <= kPairsT5;
  run([&] {
    if (pairs) return;
    const unsigned n5 = grid(4L * b.cap_t5).x, nq = seeds ? grid(b.cap_md).x : 0;
    k_t5_inc<<<dim3(n5 + nq, B), kBlock, 0, st>>>(wb, g, (int)n5);
  });
  run([&] { if (!pairs) k_list_place<<<grid((b.cap_md + 1) / 2), kBlock, 0, st>>>(wb); });
  run([&] { if (!pairs) k_t5_inc_scatter<<<grid(5L * b.cap_t5), kBlock, 0, st>>>(wb); });
  run([&] {
    if (pairs) {
      const unsigned n5 = gridwt(b.cap_t5).x, nq = seeds ? grid(b.cap_md).x : 0;
      k_t5_pairs<<<dim3(n5 + nq, B), tb, 0, st>>>(wb, g, (int)n5);
      return;
    }
    const long blocks = (4L * b.cap_t5 + 63) / 64;  // 64 items a block
    k_t5_dedup<<<dim3(share_big((int)std::min(blocks, 1L << 24), tb), B), tb, 0, st>>>(wb);
  });
  // a6: pLS (with the hit count and the segment sums); a7's bins (with the quintuplets)
  for (int q = 0; q < 6; ++q) run([&] {});  // pls, its hit lists and duplicate removal, pt3_bin, pt5_bin
  // a7: pT3, pT5: one wave per seed over its bins;
  // both counts on one trajectory mask per seed, both fills in one launch
  run([&] { if (seeds) k_pt_binned<false><<<seedwaves(), tb, 0, st>>>(wb, g, 0); });
  run([&] {});  // pt3_scan
  run([&] {
    if (!seeds) return;
    // the tasks' blocks: whole rounds of the shards, three a CU for the launch (with eight a
    // PU200 event with nothing cached takes 0.21 ms, but eight PU10 events, without a task,
    // 0.5 us longer)
    const unsigned nc = gridwt((S + kPtSeeds - 1) / kPtSeeds).x;
    const unsigned n_again = (unsigned)((std::min(2 * S, std::max(768L / B, 64L)) + kTaskShards - 1) / kTaskShards) * kTaskShards;
    k_pt_binned<true><<<dim3(2 * nc + n_again, B), tb, 0, st>>>(wb, g, (int)nc);
  });
  run([&] {});  // pt5_scan
  run([&] {});  // pt5_fill: with pt3_fill
  run([&] {});  // pt_obj_best: offered by the fill
  run([&] {
    if (!seeds) return;
    const unsigned n5 = grid(8 * S).x, n3 = grid(32 * S).x;
    k_pt_dedup<<<dim3(n5 + n3, B), kBlock, 0, st>>>(wb, (int)n5);
  });
  run([&] {});  // pt5_dedup: with pt3_dedup
  // a8: cleaning and track candidates
  for (int q = 0; q < 3; ++q) run([&] {});  // tc_pt5, its scan and directions: with the duplicate removal
  auto clean = [&](long n) { return gridwt((n + kCleanItems - 1) / kCleanItems).x; };
  run([&] { if (seeds) k_tc_pt3<<<dim3(clean(S), B), tb, 0, st>>>(wb); });
  for (int q = 0; q < 2; ++q) run([&] {});  // tc_pt3_scan, tc_pt3_dirs
  run([&] {
    const unsigned n5 = clean(b.cap_t5), ns = seeds ? clean(S) : 0;
    k_tc_t5<<<dim3(n5 + ns, B), tb, 0, st>>>(wb, (int)n5);
  });
  for (int q = 0; q < 4; ++q) run([&] {});  // tc_t5_scan, tc_t5_dirs, tc_pls (with tc_t5), tc_pls_scan
  run([&] {
    const unsigned ns = share((int)std::min(1024L, (S + 255) / 256), kBlock);
    const unsigned n5 = share((int)std::min(1024L, ((long)b.cap_t5 + 255) / 256), kBlock);
    k_tc_write<<<dim3(3 * ns + n5, B), kBlock, 0, st>>>(wb, (int)ns, g.ext ? 0 : 1);
  });
  // track extensions (when the geometry enables them)
  run([&] {
    if (!g.ext) return;
    const int c = g.tiles.ext_per_wave;
    if (c == 4) k_tc_ext<4><<<gridwt((b.cap_tc + 3) / 4), tb, 0, st>>>(wb, g);
    else if (c == 16) k_tc_ext<16><<<gridwt((b.cap_tc + 15) / 16), tb, 0, st>>>(wb, g);
    else k_tc_ext<8><<<gridwt((b.cap_tc + 7) / 8), tb, 0, st>>>(wb, g);
  });
  run([&] { if (g.ext) scan(wb, B, b.cap_tc, st); });
  run([&] { if (g.ext) k_tc_ext_write<<<grid(b.cap_tc), kBlock, 0, st>>>(wb); });
  if (whole) (void)hipEventRecord(kt->end, st);
}

}  // namespace lst
