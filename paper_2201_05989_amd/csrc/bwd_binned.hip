// Binned backward pass of the hash encoding (Fig. 3 caption of the paper: the
// gradient of the loss is accumulated in the looked-up feature vectors).
//
// Why not atomics: on this chip a device-scope fp32 atomic add costs one L2
// request per 64-byte block per wave instruction and all XCDs together retire
// about 21 G requests/s, whatever the table size; a fine hashed level needs at
// least 2^(d-1) requests per point, which bounds an atomic backward pass far
// below what the memory system can stream.  LDS fp32 atomics are slow as well
// (about 0.3 lane-ops per clock per CU) while LDS *integer* atomics run at about
// 3.6 64-bit adds per clock per CU.  So the scatter-add is done as a bucket
// sort followed by an owner-computes accumulation:
//
//   count      every (point, level) emits 2^(d-1) records, one per pair of
//              corners that differ only along dimension 0 (they are neighbours
//              in memory: index+1 on 1:1 levels, same small aligned block on
//              hashed levels because pi_1 = 1 in Eq. 4).  A record belongs to
//              the bin (chunk of the level's gradient slice, at most 2^chunk_log2
//              entries) that holds both corners.  This kernel only counts.
//   scan       per-bin totals and per-(workgroup, bin) write offsets.
//   scatter    recomputes the records, sorts them by bin in LDS one level at a
//              time and writes each to its slot.  A record names the two
//              chunk-local entries and carries the fractional position along
//              dimension 0, the weight of the other dimensions and dL/dy of the
//              level: 16 bytes when dL/dy is fp32, 12 bytes when it is fp16
//              (see Record below).  The passes that write and re-read the
//              records are bound by memory bandwidth, so the record size is
//              what sets their time.
//   accumulate one workgroup per bin (several for the few bins of coarse 1:1
//              levels, which receive very many records): sums its records into
//              LDS in 64-bit fixed point with integer atomics, then adds the
//              chunk to the fp32 gradient (plain read-modify-write when the bin
//              has a single owner).  The fixed-point scale comes from the
//              largest |dL/dy| of the call, with headroom for 8*B summands, so
//              the sum is exact and independent of the order of the records;
//              each summand is rounded once to 2^-min(62-H, 51) of the power of
//              two above that largest value (H = ceil(log2(8B))).
//
// Variants of the same plan: the forward pass can do the counting (hashgrid.hip,
// HG_BWD_COUNTED); in two dimensions large levels are sorted in tiles of 1024 points
// (tile_mult_for); plans with more than kMaxStagedBins chunks use tiles of
// kBigTileMult * 512 points and write their records unstaged (bin_scatter_direct);
// pairs whose corners lie in two chunks (hashed levels of resolution 2^chunk_log2
// or more) bypass the sort and are added with device atomics; with
// HG_BWD_OVERWRITE the owners store their sums instead of adding them, the scan
// kernel clears the levels that several workgroups share, and the atomics for the
// straddling pairs run as a last pass (bin_crossing).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "hashgrid.h"
#include "hashgrid_common.hpp"
#include "hashgrid_internal.hpp"
#include "adam_device.hpp"
#include "bwd_bins.hpp"
#include "bwd_record.hpp"

namespace hg {

// Launch shapes, each the best of a sweep on the headline configuration.
constexpr int kScanThreads = 1024;
constexpr int kAccThreads = 1024;                // accumulate workgroup (512 x 2 per CU is slower)
constexpr uint32_t kFewBins = 32;                 // bins of a level up to which the scatter pass spreads a tile's records (bin_scatter)
// Queues of work items: a counter each, 64 bytes apart.  One counter hands out an item every 13 ns, whoever asks, which is
// all of the pass where the items are short (table of 2^22 entries in two dimensions: 7600 items of 500 records, 103 us with one
// queue, 91 with four or eight); with few items one queue shares them out better.
constexpr uint32_t kQueues = 4, kQueueStride = 16, kManyItems = 1024;
constexpr uint32_t kAccWgsPerCu = 1;             // its LDS lets one accumulate workgroup run per CU
constexpr uint32_t kTargetRecordsPerAccWg = 16384;
// Eight features an entry, half-precision gradients: a record is 16 additions in LDS, so 16384 records keep a compute unit busy
// for 30 us, however little the others have to do.  Items of more than kGroupedHalfShares / 2 times a compute unit's share of the
// batch are then shared out by features, kGroupFeatures to a work item: every sum is formed from the same records in one
// place as before, where a finer cut of the records would add partial sums that are rounded to half.  The price is in each part
// reading the records again and in its sums leaving in requests that a whole item fills, so not from twice the share on (uniform
// points on equal chunks: 73 -> 81 us for both passes), and not where there are chip-filling numbers of such items already (8
// levels in one chunk each, 89981 points: 76 -> 90).  Over 180 random configurations, both passes: 0.93 of the time without on
// average, 0.72 to 1.06; 30011 points, 8 levels on 2^17 entries: 85 -> 72.5 us.  Not for single-precision gradients, whose sums
// leave one to a lane (a table of 2^14 entries, 91757 points in two dimensions: 86 -> 155 us), nor for four features (1.01 to 1.25 of
// the time without); and the code is an instance of its own, since merely having it costs the others 5 to 20 %.
constexpr int kGroupedF = 8, kGroupFeatures = 2;
constexpr uint32_t kGroupedHalfShares = 5, kShares = 256;  // shares: compute units of the chip
constexpr uint32_t kMinGroupedAdds = 1u << 15;        // records * F below which an item is short anyway (4 us)
constexpr uint32_t kMaxParts = 4;                // level parts of the scatter grid (1, 2, 8: slower)
constexpr uint32_t kCountParts = 2;              // ... of the count grid (its workgroups are lighter)
// Level parts are doubled (up to one level per part) until one part's bins fit these bounds: a count
// workgroup keeps one LDS word per bin of its part, a scatter workgroup three, next to its staging area.
constexpr uint32_t kMaxCountPartBins = 4096, kMaxScatterPartBins = 4096;
// Beyond this many chunks in all, a tile is kBigTileMult * 512 points and the scatter pass does not
// stage (bin_scatter_direct, one LDS word per bin of its part).  One level of 4096 chunks per part: the grid runs
// part after part, so the records in flight then belong to two levels (200 MB at T = 2^24), not four (-3%).
constexpr uint32_t kMaxStagedBins = 16384, kBigTileMult = 8, kMaxDirectPartBins = 4096;
// A level may have this many chunks (one level is the smallest part): T up to 2^24 at 4096 entries per chunk.
constexpr uint32_t kMaxLevelBins = 4096;

static_assert(kChunkLog2 <= 12, "a record holds a 12-bit local index");

struct Workspace {
  uint32_t* counts;     // [n_tiles + 1][n_bins] counts, then exclusive prefix over tiles (last row: totals)
  uint32_t* bin_total;  // [n_bins] records in the bin
  float* tile_max;      // [n_tiles * parts of the scatter grid (at most L)] largest |dL/dy| seen by each scatter workgroup
  uint32_t* item_counters;  // [kQueues * kQueueStride] next work item of each queue of the accumulate pass
  uint32_t* chunk_open;    // [n_bins] workgroups that have yet to add their share of a chunk (accumulate pass with the optimiser)
  uint32_t* records;    // room for [B * L * rec_per_point] records (Record::kWords words each)
  uint4* items;         // [accumulate work items] what a workgroup of that pass needs to know of each (write_items)
  uint32_t n_tiles;
  uint32_t n_bins;
};

static inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// Chunks of the largest of `parts` level parts
static uint32_t max_part_bins(const BinPlan& bp, uint32_t L, uint32_t parts) {
  uint32_t m = 0;
  for (uint32_t p = 0; p < parts; ++p) {
    const uint32_t nbp = bp.bin_base[(p + 1) * L / parts] - bp.bin_base[p * L / parts];
    m = nbp > m ? nbp : m;
  }
  return m;
}

// 32-bit words of a record (Record::kWords)
static uint32_t record_words(const hashgrid* h) { return 2u + (h->cfg.F * (h->cfg.io_dtype == HG_F16 ? 2u : 4u) + 3u) / 4u; }

// one count / scatter workgroup per tile and level part
static uint32_t tiles_for(uint32_t tile_mult, uint32_t B) {
  const uint32_t points = kBinThreads * tile_mult;
  return (uint32_t)(((uint64_t)B + points - 1) / points);
}

// Records to expect of a point and level: nearly every pair is one record, also where each corner may need its own
// (rec_per_point then leaves room for that).
static uint32_t pairs_per_point(const BinPlan& bp) { return bp.corner_records ? bp.rec_per_point / 2 : bp.rec_per_point; }

// Slices per bin of each level for a batch of B points: coarse 1:1 levels have
// few bins and receive B * 2^(d-1) records, so their bins are shared by several
// accumulate-workgroups.  Levels in group_mask: every share once for each kGroupFeatures features.
// records: of a point and level, to be shared out.
static void plan_slices_for(BinPlan& bp, const LevelTable& lv, uint32_t B, uint32_t F, bool half_grad, uint64_t records) {
  bp.group_mask = 0;
  const uint64_t share = (uint64_t)B * lv.L * records / kShares;
  uint64_t grouped_items = 0;
  for (uint32_t l = 0; l < lv.L; ++l) {
    const uint32_t nb = bp.bin_base[l + 1] - bp.bin_base[l];
    const uint64_t per_bin = ((uint64_t)B * records + nb - 1) / nb;
    uint64_t s = (per_bin + kTargetRecordsPerAccWg - 1) / kTargetRecordsPerAccWg;
    if (!((lv.dense_mask >> l) & 1u) && s < 4) s = 1;  // hashed bins are evenly filled
    if (s > 256) s = 256;
    bp.slices[l] = (uint32_t)(s < 1 ? 1 : s);
    if (F == kGroupedF && half_grad && 2 * per_bin > kGroupedHalfShares * share * bp.slices[l] &&
        per_bin * F >= (uint64_t)kMinGroupedAdds * bp.slices[l]) {
      bp.group_mask |= 1u << l;
      grouped_items += (uint64_t)nb * bp.slices[l] * (F / kGroupFeatures);
    }
  }
  if (grouped_items > kShares) bp.group_mask = 0;
  uint32_t wgs = 0;
  for (uint32_t l = 0; l < lv.L; ++l) {
    bp.wg_base[l] = wgs;
    wgs += (bp.bin_base[l + 1] - bp.bin_base[l]) * bp.slices[l] * ((bp.group_mask >> l) & 1u ? F / kGroupFeatures : 1u);
  }
  bp.wg_base[lv.L] = wgs;
}

// Plans with BinPlan::corner_records: the items that the pairs ask for, or as many as a record for every corner would (twice as many,
// half as long) where those leave the chip waiting for a few: in one dimension (neighbours in the batch are on one
// entry often, and lanes that add to one address wait for each other), for wide entries (2 F additions a record) and where
// there are fewer items than compute units.  Both passes, us, pairs' items against corners': d = 1, F = 2, points in order 116 -> 94;
// d = 3, F = 8, T = 524287, uniform 143 -> 127; d = 2, F = 2, N 2 to 3, 64075 points in order 63 -> 46.  Elsewhere the shares' partial sums
// cost more than that gains (F = 2, T = 1000003, d = 3 129 -> 132, d = 2 106 -> 109).
static void plan_slices(BinPlan& bp, const LevelTable& lv, uint32_t B, uint32_t F, bool half_grad) {
  plan_slices_for(bp, lv, B, F, half_grad, pairs_per_point(bp));
  const bool one_dimension = bp.rec_per_point == 2;
  if (bp.corner_records && (one_dimension || F >= 4 || bp.wg_base[lv.L] < kShares))
    plan_slices_for(bp, lv, B, F, half_grad, bp.rec_per_point);
}

static uint64_t max_items(const hashgrid* h, uint32_t B) {
  BinPlan bp = h->bp;
  plan_slices(bp, h->lv, B, h->cfg.F, h->cfg.grad_dtype == HG_F16);
  return bp.wg_base[h->lv.L];
}

// Bytes of the workspace; before_items: those in front of the item list, which is last.
static uint64_t carve(const hashgrid* h, uint32_t B, uint8_t* base, Workspace* ws, uint64_t* before_items = nullptr) {
  const uint32_t nb = h->bp.bin_base[h->lv.L];
  const uint32_t nt = tiles_for(h->bp.tile_mult, B);  // room for the plan's tiles, where the batch's are twice as large, too
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    uint64_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  const uint64_t o_counts = take((uint64_t)(nt + 1) * nb * 4), o_total = take((uint64_t)nb * 4),
                 o_max = take((uint64_t)nt * h->lv.L * 4), o_queues = take(kQueues * kQueueStride * 4), o_open = take((uint64_t)nb * 4),
                 o_rec = take((uint64_t)B * h->lv.L * h->bp.rec_per_point * record_words(h) * 4),
                 o_items = take(max_items(h, B) * sizeof(uint4));
  if (before_items) *before_items = o_items;
  if (ws) {
    ws->counts = reinterpret_cast<uint32_t*>(base + o_counts);
    ws->bin_total = reinterpret_cast<uint32_t*>(base + o_total);
    ws->tile_max = reinterpret_cast<float*>(base + o_max);
    ws->item_counters = reinterpret_cast<uint32_t*>(base + o_queues);
    ws->chunk_open = reinterpret_cast<uint32_t*>(base + o_open);
    ws->records = reinterpret_cast<uint32_t*>(base + o_rec);
    ws->items = reinterpret_cast<uint4*>(base + o_items);
    ws->n_tiles = tiles_for(tile_mult_for(h, B), B);
    ws->n_bins = nb;
  }
  return off;
}

// Chunking of every level's gradient slice.  1:1 levels are cut at grid-row
// boundaries (a row = all vertices that share the coordinates of dimensions
// 1..d-1, contiguous in memory), a power-of-two number of rows per chunk; hashed
// levels are cut into aligned blocks of 2^chunk_log2 entries, which the XOR with
// the low chunk_log2 bits of v_0 cannot leave.
void build_bin_plan(hashgrid* h) {
  BinPlan& bp = h->bp;
  bp = BinPlan{};
  const hashgrid_config& c = h->cfg;
  const LevelTable& lv = h->lv;
  bp.chunk_log2 = chunk_log2_of(c.F);
  // A pair record gives one corner along dimension 0 and the kernel derives the other, which takes a power-of-two T (with
  // another T Eq. 4's mod T comes after the XOR, and the upper corner's entry does not follow from the lower one's, though
  // the two are near: 99.9 % of the pairs of a hashed level in one chunk, T = 1000003) and a second dimension to cut 1:1
  // levels by grid rows; otherwise the record carries both indices, where it can (NearPair), and the corners get a record
  // each where it cannot.  100003 points, T = 1000003, fp32 records of 16 bytes, both passes, a record for every corner
  // against this: 273 against 207 us (a record for every corner writes and reads 205 MB, this 104).
  bp.corner_records = (c.d < 2 || !lv.T_is_pow2) ? 1u : 0u;
  bp.rec_per_point = bp.corner_records ? 1u << c.d : 1u << (c.d - 1);
  if (c.d < 1 || c.d > 3) return;  // F is 1, 2, 4 or 8 (hashgrid_create)
  const uint32_t cap = 1u << bp.chunk_log2;
  uint32_t bins = 0;
  for (uint32_t l = 0; l < lv.L; ++l) {
    const uint32_t verts = lv.verts[l];
    uint32_t nb;
    if (bp.corner_records) {
      nb = (lv.size[l] + cap - 1u) >> bp.chunk_log2;  // aligned blocks of the level's slice, the last one ragged
    } else if ((lv.dense_mask >> l) & 1u) {
      if (verts > cap) return;
      uint32_t s = 0;
      while (((uint64_t)verts << (s + 1)) <= cap) ++s;
      const uint64_t rows = c.d == 3 ? (uint64_t)verts * verts : verts;
      bp.row_shift[l] = s;
      nb = (uint32_t)((rows + (1ull << s) - 1) >> s);
    } else {
      // The two corners of a pair share the bits above the chunk unless stepping v_0 carries out of
      // its low chunk_log2 bits, which needs a resolution of 2^chunk_log2 or more and then happens
      // for one voxel in 2^chunk_log2: those pairs bypass the sort (see bin_scatter).
      nb = lv.T > cap ? lv.T >> bp.chunk_log2 : 1u;
    }
    if (nb > kMaxLevelBins) return;
    bp.bin_base[l] = bins;
    bins += nb;
  }
  bp.bin_base[lv.L] = bins;
  auto parts_for = [&](uint32_t start, uint32_t limit) {
    uint32_t np = lv.L < start ? lv.L : start;
    while (max_part_bins(bp, lv.L, np) > limit && np < lv.L) np = np * 2 < lv.L ? np * 2 : lv.L;
    return max_part_bins(bp, lv.L, np) <= limit ? np : 0u;
  };
  bp.count_parts = parts_for(kCountParts, kMaxCountPartBins);
  // With very many chunks a tile of 512 points leaves less than a record per chunk and level: the
  // per-chunk work of every count / scatter workgroup (and the count table) then outweighs the
  // records, and staging them for whole-line writes gains nothing.  Larger tiles, no staging.
  bp.tile_mult = bins > kMaxStagedBins ? kBigTileMult : 1u;
  bp.scatter_parts = bp.tile_mult > 1 ? parts_for(kMaxParts, kMaxDirectPartBins) : parts_for(kMaxParts, kMaxScatterPartBins);
  if (!bp.count_parts || !bp.scatter_parts) return;
  bp.supported = 1;
}

// ------------------------------------------------------------------ device

// The pairs of a hashed level whose two corners lie in different chunks (Rows::cross; one voxel
// in 2^chunk_log2 along dimension 0, and only at resolutions of 2^chunk_log2 or more) get no
// record: their 2^d products go to the gradient with device-scope atomics.  T is a power of two.
template <int D, int F>
__device__ __forceinline__ void add_crossing_pairs(const LevelTable& lv, uint32_t l, bool smooth, const float (&xp)[D],
                                                   const float (&g)[F], void* __restrict__ grad, const bool g16) {
  const float Nf = (float)lv.N[l];
  const float shift = smooth ? 0.5f : 0.0f;
  const float cmaxf = smooth ? Nf : Nf - 1.0f;
  uint32_t c0[D];
  float w[D], u[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    float wf;
    split(xp[i], Nf, shift, cmaxf, c0[i], wf);
    w[i] = smooth ? smoothstep(wf) : wf;
    u[i] = smooth ? smoothstep(1.0f - wf) : 1.0f - wf;
  }
  const uint32_t tmask = lv.T - 1u;
  float* gl = static_cast<float*>(grad) + lv.offset[l] * F;          // (g16: the same entries, as halves)
  _Float16* gl16 = static_cast<_Float16*>(grad) + lv.offset[l] * F;
#pragma unroll
  for (uint32_t r = 0; r < (1u << (D - 1)); ++r) {
    float wr = 1.0f;
    uint32_t rt = 0;
#pragma unroll
    for (int i = 1; i < D; ++i) {
      const uint32_t up = (r >> (i - 1)) & 1u;
      wr *= up ? w[i] : u[i];
      rt ^= (c0[i] + up) * prime(i);
    }
    const uint32_t ia = (c0[0] ^ rt) & tmask, ib = ((c0[0] + 1u) ^ rt) & tmask;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      if (g16) {  // uniform
        grad_atomic_add(gl16, F * (uint64_t)ia + f, u[0] * (wr * g[f]));
        grad_atomic_add(gl16, F * (uint64_t)ib + f, w[0] * (wr * g[f]));
      } else {
        grad_atomic_add(gl, F * (uint64_t)ia + f, u[0] * (wr * g[f]));
        grad_atomic_add(gl, F * (uint64_t)ib + f, w[0] * (wr * g[f]));
      }
    }
  }
}

template <int D>
__device__ __forceinline__ void load_x(const float* __restrict__ x, uint32_t b, float (&xp)[D]) {
#pragma unroll
  for (int i = 0; i < D; ++i) xp[i] = x[(uint64_t)b * D + i];
}

// Workgroup -> tile of points.  Workgroup i runs on XCD i mod 8 (each XCD has its
// own L2), so consecutive tiles are given to consecutive workgroups of one XCD:
// the runs two neighbouring tiles write into a bin are adjacent in memory, and
// the cache line they share is completed inside one L2 instead of being written
// back half-filled twice.  Returns n_tiles or more for surplus workgroups.
__device__ __forceinline__ uint32_t tile_of_workgroup(uint32_t wg, uint32_t n_tiles) {
  const uint32_t per_xcd = (n_tiles + 7u) / 8u;
  const uint32_t j = wg >> 3;
  return j < per_xcd ? (wg & 7u) * per_xcd + j : n_tiles;
}

// Levels are split into gridDim.y parts; a count / scatter workgroup serves one
// tile of points and one part.  More, lighter workgroups per CU hide the latency
// of the LDS atomics and of the per-level barriers.
__device__ __forceinline__ void part_levels(uint32_t L, uint32_t& l0, uint32_t& l1) {
  l0 = blockIdx.y * L / gridDim.y;
  l1 = (blockIdx.y + 1) * L / gridDim.y;
}

// count: records per (tile, bin).
template <int D, bool CORNERS>
__global__ __launch_bounds__(kBinThreads) void bin_count(const LevelTable lv, const BinPlan bp, const bool smooth,
                                                         const uint32_t B, const float* __restrict__ x,
                                                         uint32_t* __restrict__ counts, const uint32_t n_bins,
                                                         const uint32_t n_tiles) {
  extern __shared__ uint32_t hist[];  // bins of this part's levels
  const uint32_t tile = tile_of_workgroup(blockIdx.x, n_tiles);
  if (tile >= n_tiles) return;  // uniform: a surplus workgroup of the rounded-up grid
  uint32_t l0, l1;
  part_levels(lv.L, l0, l1);
  const uint32_t gb_a = bp.bin_base[l0], nbp = bp.bin_base[l1] - gb_a;
  for (uint32_t i = threadIdx.x; i < nbp; i += kBinThreads) hist[i] = 0;
  __syncthreads();
  for (uint32_t sub = 0; sub < bp.tile_mult; ++sub) {
    const uint64_t b64 = ((uint64_t)tile * bp.tile_mult + sub) * kBinThreads + threadIdx.x;
    if (b64 >= B) break;
    const uint32_t b = (uint32_t)b64;
    float xp[D];
    load_x<D>(x, b, xp);
    for (uint32_t l = l0; l < l1; ++l) {
      if constexpr (CORNERS) {
        CornerRows<D> cr;
        corner_rows_of<D, true>(lv, bp, l, smooth, xp, cr);
#pragma unroll
        for (uint32_t r = 0; r < (1u << (D - 1)); ++r) {
          count_one(hist, cr.bin[2 * r] - gb_a);
          if (cr.pair[r].step == NearPair::kNone) count_one(hist, cr.bin[2 * r + 1] - gb_a);
        }
      } else {
        Rows<D> rw;
        rows_of<D, true>(lv, bp, l, smooth, xp, rw);
        if (rw.cross) continue;
#pragma unroll
        for (uint32_t r = 0; r < (1u << (D - 1)); ++r)
          count_one(hist, rw.bin[r] - gb_a);
      }
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < nbp; i += kBinThreads) counts[(uint64_t)tile * n_bins + gb_a + i] = hist[i];
}

// m = max(m, v) where a NaN on either side wins, so that one NaN in dL/dy is seen at the end
__device__ __forceinline__ float nan_max(float m, float v) { return (v > m || v != v) ? v : m; }

// Exclusive prefix sum of a[0..n) in LDS, in place, by all T threads of the
// workgroup (every thread must call it).  `tmp` holds T/64 words.
template <int T>
__device__ __forceinline__ void block_exclusive_scan(uint32_t* a, uint32_t n, uint32_t* tmp) {
  const uint32_t per = (n + T - 1) / T;
  const uint32_t begin = threadIdx.x * per < n ? threadIdx.x * per : n;
  const uint32_t end = begin + per < n ? begin + per : n;
  uint32_t sum = 0;
  for (uint32_t i = begin; i < end; ++i) sum += a[i];
  uint32_t inc = sum;  // inclusive scan across the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = __shfl_up(inc, o);
    if ((threadIdx.x & 63) >= (uint32_t)o) inc += up;
  }
  if ((threadIdx.x & 63) == 63) tmp[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint32_t wave_base = 0;
  for (uint32_t w = 0; w < (threadIdx.x >> 6); ++w) wave_base += tmp[w];
  uint32_t run = wave_base + inc - sum;
  for (uint32_t i = begin; i < end; ++i) {
    const uint32_t v = a[i];
    a[i] = run;
    run += v;
  }
  __syncthreads();
}

// scan: each workgroup takes BINS bins and turns their column of
// counts[tile][bin] into the exclusive prefix over tiles; it also writes the
// bin's record count.  Workgroup 0 clears the counters of the accumulate pass's queues.
// Bound by the latency of its loads and stores, and by what the stores make of lines: rows start anywhere, so that neighbouring columns
// share a line in nearly every row, and written from two XCDs it goes out in parts.  Columns dealt out by XCD, and every row of
// a thread in registers instead of eight at a time and twice: d = 2, T = 2^22, 512 tiles of 7600 bins 18.0 -> 9.6 us (17.3 by the
// registers alone); T = 2^24, 512 tiles of 49 K bins 90 -> 46; 2048 tiles of 1508 bins 23.1 -> 14.7; 512 of them 7.9 -> 6.1.
// With HG_BWD_OVERWRITE it also clears the gradient of the levels in zero_mask (those that the
// later passes add into, see launch_binned): it is the first kernel of the call to run.
// ROWS: the rows of the table a thread has at most, all of them in registers: every load is in flight at once, and none is made
// twice.  0: any number, eight at a time and each read again for its prefix.
template <int ROWS, int BINS>
__global__ __launch_bounds__(kScanThreads) void bin_scan(const uint32_t n_tiles, const uint32_t n_bins,
                                                         uint32_t* __restrict__ counts,
                                                         uint32_t* __restrict__ bin_total,
                                                         uint32_t* __restrict__ item_counters,
                                                         const LevelTable lv,
                                                         const uint32_t zero_mask, const uint32_t F,
                                                         void* __restrict__ grad, const bool g16, const SideJob job) {
  __shared__ uint32_t seg_sum[kScanThreads];
  const uint32_t scan_wgs = gridDim.x - job.blocks;
  if (blockIdx.x >= scan_wgs) {  // uniform
    __shared__ float4 part[kScanThreads];
    run_side_job<kScanThreads>(job, blockIdx.x - scan_wgs, part);
    return;
  }
  // the accumulate pass draws its work items from these
  if (blockIdx.x == 0 && threadIdx.x < kQueues) item_counters[threadIdx.x * kQueueStride] = 0;
  for (uint32_t l = 0; l < lv.L; ++l) {  // uniform; bounded by L, not by the mask: with level 31 in it the shifts would go on to 32
    if (!((zero_mask >> l) & 1u)) continue;
    const uint64_t first = lv.offset[l] * F, n = (uint64_t)lv.size[l] * F;
    for (uint64_t i = (uint64_t)blockIdx.x * kScanThreads + threadIdx.x; i < n; i += (uint64_t)scan_wgs * kScanThreads) {
      if (g16) static_cast<_Float16*>(grad)[first + i] = (_Float16)0.0f;
      else static_cast<float*>(grad)[first + i] = 0.0f;
    }
  }
  constexpr uint32_t segs = kScanThreads / BINS;
  const uint32_t bin_in = threadIdx.x % BINS, seg = threadIdx.x / BINS;
  // Rows do not start on a line: neighbouring columns share one in nearly every row, and go to workgroups of one XCD (as in
  // tile_of_workgroup) so that it is completed inside one L2
  const uint32_t gb = tile_of_workgroup(blockIdx.x, (n_bins + BINS - 1) / BINS) * BINS + bin_in;
  const bool active = gb < n_bins;
  const uint32_t tps = (n_tiles + segs - 1) / segs;
  const uint32_t t0 = seg * tps < n_tiles ? seg * tps : n_tiles;
  const uint32_t t1 = t0 + tps < n_tiles ? t0 + tps : n_tiles;
  uint32_t* col = counts + (active ? gb : 0u);
  uint32_t sum = 0;
  uint32_t c[ROWS > 0 ? ROWS : 8];
  if constexpr (ROWS > 0) {
#pragma unroll
    for (int k = 0; k < ROWS; ++k) c[k] = col[(uint64_t)(t0 + k < n_tiles ? t0 + k : n_tiles - 1u) * n_bins];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      c[k] = t0 + k < t1 ? c[k] : 0u;
      sum += c[k];
    }
  } else if (active) {
    uint32_t t = t0;
    for (; t + 8 <= t1; t += 8) {
#pragma unroll
      for (int k = 0; k < 8; ++k) c[k] = col[(uint64_t)(t + k) * n_bins];
#pragma unroll
      for (int k = 0; k < 8; ++k) sum += c[k];
    }
    for (; t < t1; ++t) sum += col[(uint64_t)t * n_bins];
  }
  seg_sum[threadIdx.x] = sum;
  __syncthreads();
  if (active) {
    uint32_t run = 0, total = 0;
#pragma unroll 32
    for (uint32_t q = 0; q < segs; ++q) {
      const uint32_t v = seg_sum[q * BINS + bin_in];
      run += q < seg ? v : 0u;
      total += v;
    }
    if (seg == 0) {
      bin_total[gb] = total;
      col[(uint64_t)n_tiles * n_bins] = total;  // closes the prefix: count of tile t = row t+1 - row t
    }
    if constexpr (ROWS > 0) {
#pragma unroll
      for (int k = 0; k < ROWS; ++k) {
        if (t0 + k < t1) col[(uint64_t)(t0 + k) * n_bins] = run;
        run += c[k];
      }
    } else {
      uint32_t t = t0;
      for (; t + 8 <= t1; t += 8) {
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = col[(uint64_t)(t + k) * n_bins];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          col[(uint64_t)(t + k) * n_bins] = run;
          run += c[k];
        }
      }
      for (; t < t1; ++t) {
        const uint32_t v = col[(uint64_t)t * n_bins];
        col[(uint64_t)t * n_bins] = run;
        run += v;
      }
    }
  }
}

// A work item of the accumulate pass, written by the scatter workgroups of the first tile (they know where the bins
// start) so that the accumulate pass reads 16 bytes an item instead of searching the plan's level table and chasing the
// bin's start and count: with a table of 2^22 entries a level an item is 1100 records, and that chain was most of its 5 us.
//   .x, .y  first record, one past the last;  .z  first entry of the chunk in the tables (below 2^30), bits 30-31 group of features
//   .w      bits 0-11 entries of the chunk minus 1, 12-16 level, 17 1:1 index map (lb = la + 1), 18 the chunk is
//           shared by several workgroups (not set for the first share of an empty one), 19 it has records, 20-31 chunk of the level
constexpr uint32_t kItemDense = 1u << 17, kItemShared = 1u << 18, kItemLive = 1u << 19;
static_assert(kMaxLevelBins <= 1u << 12 && HG_MAX_LEVELS <= 32, "an item's last word");
template <int F>
__device__ __forceinline__ void write_items(const LevelTable& lv, const BinPlan& bp, const uint32_t l0, const uint32_t l1,
                                            const uint32_t gb, const uint32_t start, const uint32_t total,
                                            uint4* __restrict__ items, uint32_t* __restrict__ chunk_open) {
  uint32_t l = l0;
  while (l + 1 < l1 && gb >= bp.bin_base[l + 1]) ++l;
  const uint32_t bin = gb - bp.bin_base[l], n_sl = bp.slices[l], per = (total + n_sl - 1) / n_sl;
  const bool dense = ((lv.dense_mask >> l) & 1u) && !bp.corner_records;  // (BinPlan::corner_records: every level in aligned blocks)
  uint32_t e0, e1;
  if (dense) {
    e0 = (bin << bp.row_shift[l]) * lv.verts[l];
    e1 = e0 + (lv.verts[l] << bp.row_shift[l]);
  } else {
    e0 = bin << bp.chunk_log2;
    e1 = e0 + (1u << bp.chunk_log2);
  }
  if (e1 > lv.size[l]) e1 = lv.size[l];
  uint32_t groups = 1;
  if constexpr (F == kGroupedF) groups = (bp.group_mask >> l) & 1u ? F / kGroupFeatures : 1u;
  chunk_open[gb] = per ? (total + per - 1) / per : 1u;  // (ADAM: never in groups)
  const uint32_t w = (e1 - e0 - 1u) | (l << 12) | (dense ? kItemDense : 0u) | (bin << 20);
  for (uint32_t k = 0; k < n_sl; ++k) {
    const uint32_t r0 = k * per < total ? k * per : total, r1 = r0 + per < total ? r0 + per : total;
    for (uint32_t q = 0; q < groups; ++q)
      items[bp.wg_base[l] + (bin * n_sl + k) * groups + q] =
          make_uint4(start + r0, start + r1, ((uint32_t)lv.offset[l] + e0) | (q << 30),
                     w | (r0 < r1 ? kItemLive : 0u) | (n_sl > 1 && (k || total) ? kItemShared : 0u));
  }
}

// Records of a tile and level that the scatter pass sorts in LDS.  With BinPlan::corner_records some pairs take two records (up to 4 %
// on a level of resolution 16, 0.5 % on hashed levels): room for an eighth more, what is beyond goes to memory unsorted.  With room for
// two each (74 instead of 41 KB at 16 bytes, and 12 KB for the bins of a part at T = 1000003) one workgroup would be left on a compute unit
// instead of three; in one and two dimensions, where it would fit better, random configurations took 1 to 2 % longer.  Most beyond it: points in
// the first voxel of every level, d = 3, N = 256, F = 2, 100003 of them, both passes 88 us, as with a record for every corner.
__host__ __device__ constexpr uint32_t staged_records(uint32_t pairs, bool corners) {
  return pairs * kBinThreads + (corners ? pairs * kBinThreads / 8 : 0u);
}

// Dynamic LDS of a scatter workgroup: staging area, 16-bit bin of every staged record, three words per bin of its part and one more
constexpr size_t scatter_lds(uint32_t staged, uint32_t words, uint32_t part_bins) {
  return (size_t)staged * (words * 4 + 2) + (3 * (size_t)part_bins + 1) * 4;
}

// scatter: writes every record to its slot.  A bin's first record is the sum of
// the record counts of all bins before it (so the records are level-major); inside a bin the
// tiles of 512 or 1024 points (tile_mult_for) follow each other.  Level by level the workgroup sorts the
// records of its points by bin in LDS and copies them out bin after bin, so that
// what reaches memory is runs of whole records that mostly fill whole cache
// lines; 16-byte stores scattered over a thousand open runs leave the L2 as
// partial lines and cost several times the bytes.
// Per-bin arrays in LDS, indexed by bin relative to the first bin of this part's levels:
// local[nbp + 1] exclusive prefix of this tile's counts (where a bin's records
// sit in the tile's sorted order), cur[nbp] the same, advanced as records are
// placed, delta[nbp] = global slot minus tile-local position.
// CROSS: this pass adds the pairs that straddle two chunks.  CORNERS: BinPlan::corner_records.  PT: points a thread has (BinPlan::tile_mult).
template <int D, typename IT, int F, bool CROSS, bool CORNERS = false, int PT = 1>
__global__ __launch_bounds__(kBinThreads) void bin_scatter(const LevelTable lv, const BinPlan bp, const bool smooth,
                                                           const uint32_t B, const float* __restrict__ x,
                                                           const IT* __restrict__ dy,
                                                           const uint32_t* __restrict__ counts,
                                                           const uint32_t* __restrict__ bin_total,
                                                           uint4* __restrict__ items, uint32_t* __restrict__ chunk_open,
                                                           uint32_t* __restrict__ records, const uint32_t n_bins,
                                                           const uint32_t n_records, const uint32_t n_tiles,
                                                           float* __restrict__ tile_max, void* __restrict__ grad, const bool g16) {
  constexpr uint32_t R = 1u << (D - 1);
  using Rec = Record<IT, F>;
  using Stored = typename Rec::Stored;
  Stored* out = reinterpret_cast<Stored*>(records);
  __shared__ uint32_t scan_tmp[kBinThreads / 64];
  constexpr uint32_t kStage = staged_records(R * PT, CORNERS);
  // dynamic LDS: staging[kStage] records, binv[kStage] (part-relative bin of each
  // staged record, 16 bits), then the three per-bin arrays
  extern __shared__ uint32_t lds_u32[];
  Stored* staging = reinterpret_cast<Stored*>(lds_u32);
  uint16_t* binv = reinterpret_cast<uint16_t*>(lds_u32 + kStage * Rec::kWords);
  uint32_t* bins_lds = lds_u32 + kStage * Rec::kWords + kStage / 2;

  const uint32_t tile = tile_of_workgroup(blockIdx.x, n_tiles);
  if (tile >= n_tiles) return;  // uniform: a surplus workgroup of the rounded-up grid
  uint32_t l0, l1;
  part_levels(lv.L, l0, l1);
  const uint32_t gb_a = bp.bin_base[l0], nbp = bp.bin_base[l1] - gb_a;
  uint32_t* delta = bins_lds;
  uint32_t* local = bins_lds + nbp;
  uint32_t* cur = bins_lds + 2 * nbp + 1;

  bool valid[PT];
  float xp[PT][D];
  const IT* row[PT];
#pragma unroll
  for (int p = 0; p < PT; ++p) {
    const uint64_t b64 = ((uint64_t)tile * PT + p) * kBinThreads + threadIdx.x;
    valid[p] = b64 < B;
    const uint32_t b = valid[p] ? (uint32_t)b64 : 0u;
    load_x<D>(x, b, xp[p]);
    row[p] = dy + (uint64_t)b * lv.L * F;
  }

  // records of all bins before this part
  uint32_t before = 0;
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < gb_a; i += kBinThreads) before += bin_total[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if ((threadIdx.x & 63) == 0) scan_tmp[threadIdx.x >> 6] = before;
  const uint32_t* row0 = counts + (uint64_t)tile * n_bins + gb_a;  // prefix over tiles before this one
  const uint32_t* row1 = row0 + n_bins;                             // ... including this one
  for (uint32_t i = threadIdx.x; i < nbp; i += kBinThreads) {
    delta[i] = bin_total[gb_a + i];
    local[i] = row1[i] - row0[i];
  }
  if (threadIdx.x == 0) local[nbp] = 0;
  __syncthreads();
  before = 0;
  for (int i = 0; i < kBinThreads / 64; ++i) before += scan_tmp[i];
  __syncthreads();
  block_exclusive_scan<kBinThreads>(delta, nbp, scan_tmp);
  block_exclusive_scan<kBinThreads>(local, nbp + 1, scan_tmp);
  for (uint32_t i = threadIdx.x; i < nbp; i += kBinThreads) {
    const uint32_t f = before + delta[i];  // first record of the bin
    if (tile == 0) write_items<F>(lv, bp, l0, l1, gb_a + i, f, bin_total[gb_a + i], items, chunk_open);
    cur[i] = local[i];
    delta[i] = f + row0[i] - local[i];  // wrap-around arithmetic; undone when a position is added
  }
  __syncthreads();

  // dL/dy comes in as 16-byte pieces, K levels each when a level is narrower than that: a narrow
  // read per level with the stride of a row would cost the L1 a line per two lanes, L times over
  constexpr uint32_t kLevelBytes = F * sizeof(IT);
  constexpr uint32_t K = kLevelBytes >= 16 ? 1 : 16 / kLevelBytes;  // levels per piece
  constexpr uint32_t E = 16 / sizeof(IT);                           // scalars per piece
  constexpr uint32_t P = kLevelBytes >= 16 ? kLevelBytes / 16 : 1;  // pieces per level
  const bool vec_ok = (lv.L % K == 0) && (l0 % K == 0) && ((reinterpret_cast<uintptr_t>(dy) & 15) == 0);
  Vec<IT, E> gv[PT];
  float gmax = 0.0f;  // largest |dL/dy| this workgroup sees (idle lanes shadow point 0)
  for (uint32_t l = l0; l < l1; ++l) {
    const uint32_t rb0 = bp.bin_base[l] - gb_a, rb1 = bp.bin_base[l + 1] - gb_a;
    const uint32_t level_first = local[rb0], emitted = local[rb1] - level_first;
    // Position of a new record of bin rb in the tile's sorted order.  On a level of few bins a wave's
    // lanes crowd into the same counters and a tile's run for a bin is long: there the wave draws
    // its slots with one add per bin (wave_add_one) and the run is filled with a stride
    // (spread_in_run), for the accumulate pass.  Levels of many bins take the plain atomic.
    const bool few_bins = rb1 - rb0 <= kFewBins;  // uniform
    auto take_slot = [&](const uint32_t rb) {
      if (!few_bins) return __hip_atomic_fetch_add(&cur[rb], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const uint32_t first = local[rb];
      return first + spread_in_run(wave_add_one<true>(cur, rb) - first, local[rb + 1] - first);
    };
#pragma unroll
    for (int p = 0; p < PT; ++p) {
      IT g[F];
      if (vec_ok && K > 1) {  // uniform
        if ((l - l0) % K == 0) gv[p] = *reinterpret_cast<const Vec<IT, E>*>(row[p] + (uint64_t)l * F);
        const uint32_t k = (l - l0) % K;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          g[f] = gv[p].v[f];
#pragma unroll
          for (uint32_t q = 1; q < K; ++q) g[f] = k == q ? gv[p].v[F * q + f] : g[f];
        }
      } else if (vec_ok) {
#pragma unroll
        for (uint32_t q = 0; q < P; ++q) {
          const Vec<IT, E> piece = *reinterpret_cast<const Vec<IT, E>*>(row[p] + (uint64_t)l * F + q * E);
#pragma unroll
          for (uint32_t e = 0; e < E; ++e)
            if (q * E + e < (uint32_t)F) g[q * E + e] = piece.v[e];
        }
      } else {
#pragma unroll
        for (int f = 0; f < F; ++f) g[f] = row[p][(uint64_t)l * F + f];
      }
      float gf[F];
#pragma unroll
      for (int f = 0; f < F; ++f) {
        gf[f] = (float)g[f];
        gmax = nan_max(gmax, fabsf(gf[f]));
      }
      if (valid[p]) {
        if constexpr (CORNERS) {
          CornerRows<D> cr;
          corner_rows_of<D, false>(lv, bp, l, smooth, xp[p], cr);
          auto put = [&](const uint32_t rb, const Stored& rec) {
            const uint32_t pos = take_slot(rb) - level_first;
            if (pos < kStage) {
              staging[pos] = rec;
              binv[pos] = (uint16_t)rb;
            } else {  // more corners with a record of their own than the staging area has room for
              const uint32_t d = delta[rb] + level_first + pos;
              if (d < n_records) out[d] = rec;
            }
          };
#pragma unroll
          for (uint32_t r = 0; r < R; ++r) {
            const NearPair np = cr.pair[r];
            const bool near = np.step != NearPair::kNone;
            put(cr.bin[2 * r] - gb_a, Rec::make_near(cr.la[2 * r], near ? np.step : NearPair::kSingle, near ? np.fraction : 0u,
                                                     near ? cr.wrow[r] : cr.weight[2 * r], g));
            if (!near) put(cr.bin[2 * r + 1] - gb_a, Rec::make_near(cr.la[2 * r + 1], NearPair::kSingle, 0u, cr.weight[2 * r + 1], g));
          }
        } else {
          Rows<D> rw;
          rows_of<D, false>(lv, bp, l, smooth, xp[p], rw);
          if (CROSS && rw.cross) add_crossing_pairs<D, F>(lv, l, smooth, xp[p], gf, grad, g16);
#pragma unroll
          for (uint32_t r = 0; r < R && !rw.cross; ++r) {
            const uint32_t rb = rw.bin[r] - gb_a;
            const uint32_t pos = take_slot(rb) - level_first;
            if (pos < kStage) {  // holds when the count pass saw the same x
              staging[pos] = Rec::make(rw.la[r], record_k<D>(rw, r, (lv.dense_mask >> l) & 1u), rw.wf0, rw.wrow[r], g, smooth);
              binv[pos] = (uint16_t)rb;
            }
          }
        }
      }
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < emitted && j < kStage; j += kBinThreads) {
      const uint32_t d = delta[binv[j]] + level_first + j;
      // the count pass saw the same inputs, so d < n_records; the check only keeps a
      // caller who changed x in between from writing out of bounds
      if (d < n_records) out[d] = staging[j];
    }
    __syncthreads();
  }
  // the accumulate pass scales its fixed point by the largest |dL/dy| of the call: one value per workgroup
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) gmax = nan_max(gmax, __shfl_xor(gmax, o));
  float* wave_max = reinterpret_cast<float*>(scan_tmp);  // free since the prologue
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = gmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = wave_max[0];
    for (int i = 1; i < kBinThreads / 64; ++i) t = nan_max(t, wave_max[i]);
    tile_max[tile * gridDim.y + blockIdx.y] = t;
  }
}

// scatter without staging, for plans of very many bins (BinPlan::tile_mult > 2): a tile is
// tile_mult * 512 points, which the workgroup walks 512 at a time, and every record goes
// straight to its slot.  The runs a tile writes are a few records long at best, so sorting them
// in LDS first would not make whole lines of them; what merges partial lines here is the L2,
// which keeps the tile's open runs (a few bytes per bin of the part) while the workgroup lasts.
// LDS: slot[nbp], the next free record slot of each bin of this part for this tile.
template <int D, typename IT, int F, bool CROSS, bool CORNERS = false>
__global__ __launch_bounds__(kBinThreads) void bin_scatter_direct(
    const LevelTable lv, const BinPlan bp, const bool smooth, const uint32_t B, const float* __restrict__ x,
    const IT* __restrict__ dy, const uint32_t* __restrict__ counts, const uint32_t* __restrict__ bin_total,
    uint4* __restrict__ items, uint32_t* __restrict__ chunk_open, uint32_t* __restrict__ records, const uint32_t n_bins, const uint32_t n_records,
    const uint32_t n_tiles, float* __restrict__ tile_max, void* __restrict__ grad, const bool g16) {
  constexpr uint32_t R = 1u << (D - 1);
  using Rec = Record<IT, F>;
  using Stored = typename Rec::Stored;
  Stored* out = reinterpret_cast<Stored*>(records);
  __shared__ uint32_t scan_tmp[kBinThreads / 64];
  extern __shared__ uint32_t slot[];

  const uint32_t tile = tile_of_workgroup(blockIdx.x, n_tiles);
  if (tile >= n_tiles) return;  // uniform: a surplus workgroup of the rounded-up grid
  uint32_t l0, l1;
  part_levels(lv.L, l0, l1);
  const uint32_t gb_a = bp.bin_base[l0], nbp = bp.bin_base[l1] - gb_a;

  // first record of each bin = records of all bins before it; then the records of the tiles before this one
  uint32_t before = 0;
  for (uint32_t i = threadIdx.x; i < gb_a; i += kBinThreads) before += bin_total[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if ((threadIdx.x & 63) == 0) scan_tmp[threadIdx.x >> 6] = before;
  for (uint32_t i = threadIdx.x; i < nbp; i += kBinThreads) slot[i] = bin_total[gb_a + i];
  __syncthreads();
  before = 0;
  for (int i = 0; i < kBinThreads / 64; ++i) before += scan_tmp[i];
  __syncthreads();
  block_exclusive_scan<kBinThreads>(slot, nbp, scan_tmp);
  const uint32_t* row0 = counts + (uint64_t)tile * n_bins + gb_a;  // prefix over the tiles before this one
  for (uint32_t i = threadIdx.x; i < nbp; i += kBinThreads) {
    const uint32_t f = before + slot[i];
    if (tile == 0) write_items<F>(lv, bp, l0, l1, gb_a + i, f, bin_total[gb_a + i], items, chunk_open);
    slot[i] = f + row0[i];
  }
  __syncthreads();

  float gmax = 0.0f;  // largest |dL/dy| this workgroup sees
  for (uint32_t sub = 0; sub < bp.tile_mult; ++sub) {
    const uint64_t b64 = ((uint64_t)tile * bp.tile_mult + sub) * kBinThreads + threadIdx.x;
    if (b64 >= B) break;  // no barrier inside this loop
    const uint32_t b = (uint32_t)b64;
    float xp[D];
    load_x<D>(x, b, xp);
    const IT* row = dy + (uint64_t)b * lv.L * F;
    for (uint32_t l = l0; l < l1; ++l) {
      IT g[F];
      float gf[F];
#pragma unroll
      for (int f = 0; f < F; ++f) {
        g[f] = row[(uint64_t)l * F + f];
        gf[f] = (float)g[f];
        gmax = nan_max(gmax, fabsf(gf[f]));
      }
      if constexpr (CORNERS) {
        CornerRows<D> cr;
        corner_rows_of<D, false>(lv, bp, l, smooth, xp, cr);
        auto put = [&](const uint32_t bin, const Stored& rec) {
          const uint32_t d = __hip_atomic_fetch_add(&slot[bin - gb_a], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (d < n_records) out[d] = rec;
        };
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) {
          const NearPair np = cr.pair[r];
          const bool near = np.step != NearPair::kNone;
          put(cr.bin[2 * r], Rec::make_near(cr.la[2 * r], near ? np.step : NearPair::kSingle, near ? np.fraction : 0u,
                                            near ? cr.wrow[r] : cr.weight[2 * r], g));
          if (!near) put(cr.bin[2 * r + 1], Rec::make_near(cr.la[2 * r + 1], NearPair::kSingle, 0u, cr.weight[2 * r + 1], g));
        }
      } else {
        Rows<D> rw;
        rows_of<D, false>(lv, bp, l, smooth, xp, rw);
        if (rw.cross) {
          if (CROSS) add_crossing_pairs<D, F>(lv, l, smooth, xp, gf, grad, g16);
          continue;
        }
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) {
          const uint32_t d =
              __hip_atomic_fetch_add(&slot[rw.bin[r] - gb_a], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          // the count pass saw the same inputs, so d < n_records; the check only keeps a caller
          // who changed x in between from writing out of bounds
          if (d < n_records) out[d] = Rec::make(rw.la[r], record_k<D>(rw, r, (lv.dense_mask >> l) & 1u), rw.wf0, rw.wrow[r], g, smooth);
        }
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) gmax = nan_max(gmax, __shfl_xor(gmax, o));
  __syncthreads();  // scan_tmp is free again
  float* wave_max = reinterpret_cast<float*>(scan_tmp);
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = gmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = wave_max[0];
    for (int i = 1; i < kBinThreads / 64; ++i) t = nan_max(t, wave_max[i]);
    tile_max[tile * gridDim.y + blockIdx.y] = t;
  }
}

// The pairs that straddle two chunks (add_crossing_pairs), as a pass of its own after the accumulate
// pass: with HG_BWD_OVERWRITE the owners of the chunks store their sums, so these atomic adds
// must come after them.  Only the levels in level_mask can have such pairs; one thread per point.
template <int D, typename IT, int F>
__global__ __launch_bounds__(kBinThreads) void bin_crossing(const LevelTable lv, const BinPlan bp, const bool smooth,
                                                            const uint32_t B, const float* __restrict__ x,
                                                            const IT* __restrict__ dy, const uint32_t level_mask,
                                                            void* __restrict__ grad, const bool g16) {
  const uint64_t b64 = (uint64_t)blockIdx.x * kBinThreads + threadIdx.x;
  if (b64 >= B) return;
  const uint32_t b = (uint32_t)b64;
  float xp[D];
  load_x<D>(x, b, xp);
  for (uint32_t l = 0; l < lv.L; ++l) {  // uniform; bounded by L, as in bin_scan
    if (!((level_mask >> l) & 1u)) continue;
    Rows<D> rw;
    rows_of<D, true>(lv, bp, l, smooth, xp, rw);
    if (!rw.cross) continue;
    float gf[F];
#pragma unroll
    for (int f = 0; f < F; ++f) gf[f] = (float)dy[((uint64_t)b * lv.L + l) * F + f];
    add_crossing_pairs<D, F>(lv, l, smooth, xp, gf, grad, g16);
  }
}

// accumulate: work item = (bin, slice).  The grid is persistent: workgroup w
// starts with item w and then draws items from its queue's counter, two items
// ahead, so that the first records of the next item are fetched while the current
// one is streamed (the chain "offsets -> records" is paid once per workgroup, not
// once per bin) and workgroups that drew short items simply draw more of them:
// items differ in size by a factor of ten on 1:1 levels when the points crowd
// around a surface.  The LDS accumulators are re-zeroed by the lanes that have
// just read them.
//
// What bounds it: the records read and the gradient's old and new values, 293 MB in 58 us at 2^18 points and T = 2^19 (d = 3,
// F = 2), 57 us without the additions in LDS; in ray order the additions too, where lanes meet in one entry (2^20 points:
// 267 us with the optimiser, 214 without them).  Times against conditional loads that were waited for all at once, one set of sums,
// one queue: 72.8 -> 58.3 us; 2^20 points on rays with the optimiser 293 -> 267; d = 2, T = 2^22 107 -> 77; T = 2^24, 2^21 points
// 847 -> 582.
// GT: type of the gradient scalars (float, or _Float16: the sums are still exact fixed point and are
// rounded to half precision once, where they are added to the gradient).
// NEAR: records of a plan with BinPlan::corner_records (NearPair).
// GROUPS: levels in bp.group_mask have work items for some of an entry's features (half-precision gradients).
//
// ADAM: a training step has no use for the gradient itself, only for what the optimiser makes of it.  The owner of a
// chunk then takes its sums straight to Adam on the chunk's entries, instead of writing them for a pass of
// their own to read back with everything else (the step's largest streams are the two moments and the master copy:
// 26 bytes a scalar, against 8 for the gradient's round trip), and those streams run beside the
// LDS work of this kernel.  `grad` is then an array that is zero before and after: the workgroups that share a chunk add their
// sums into it, and the last one to arrive (chunk_open) takes them out again and applies them, as does the owner of
// a chunk with what the straddling pairs left there.
// Sets of sums in LDS.  With two, an item's records are added to one while other waves still empty the other, and one barrier an
// item is enough: whoever passes it has emptied his part of the other set before.  (2 x 64 KB at F = 2; one for wider entries.)
__host__ __device__ constexpr uint32_t acc_buffers(uint32_t F) { return F <= 2 ? 2u : 1u; }
struct NoAdam {};
struct AdamOut {
  AdamArgs a;
  AdamState st;
  uint32_t* chunk_open;
  uint32_t cross_mask;  // levels whose straddling pairs were added to grad by the scatter pass
};
template <typename IT, int F, bool SMOOTH, typename GT = float, bool ADAM = false, bool GROUPS = false, bool NEAR = false>
__global__ __launch_bounds__(kAccThreads) void bin_accumulate(const LevelTable lv, const BinPlan bp,
                                                              const uint32_t B, const uint32_t n_items,
                                                              const uint4* __restrict__ items,
                                                              const float* __restrict__ tile_max,
                                                              const uint32_t n_max,
                                                              const uint32_t* __restrict__ records,
                                                              uint32_t* __restrict__ item_counters, const uint32_t n_queues,
                                                              GT* __restrict__ grad, const uint32_t overwrite_mask,
                                                              const typename std::conditional<ADAM, AdamOut, NoAdam>::type ad) {
  // bit l of overwrite_mask: the owner of a chunk of level l stores its sums (HG_BWD_OVERWRITE, one
  // slice per chunk, no pairs that straddle chunks) instead of adding them to what is there
  constexpr uint32_t kBuffers = acc_buffers(F);
  __shared__ uint32_t s_ticket[2];
  extern __shared__ unsigned long long acc_lds[];  // [kBuffers][F][2^chunk_log2] fixed point: feature 0 of every entry, then
                                                   // feature 1 ..., so that consecutive entries map to consecutive banks
  bool finite = true;  // the call's dL/dy (known further down)
  constexpr uint32_t cl = chunk_log2_of(F), cap = 1u << cl, cmask = cap - 1u;
  const uint32_t n_records = B * lv.L * bp.rec_per_point;  // < 2^32 (hashgrid_bwd_workspace_bytes)
  constexpr int kPer = (int)cap / kAccThreads;  // entries per lane
  static_assert(kPer * kAccThreads == (int)cap, "every lane has as many entries of a chunk");
  struct alignas(F * sizeof(GT) > 16 ? 16 : F * sizeof(GT)) Entry {
    GT v[F];
  };
  // ADAM: one entry of the chunk that starts at entry `first` of the tables, gradient g (not all zero)
  [[maybe_unused]] auto update_entry = [&](const uint64_t at, const Entry& g, Entry p, Entry m1, Entry m2) {
    if constexpr (ADAM) {
      Vec<_Float16, F> h;
#pragma unroll
      for (int f = 0; f < F; ++f) {
        if (g.v[f] != 0.0f) adam_scalar(ad.a, g.v[f], m1.v[f], m2.v[f], p.v[f]);
        h.v[f] = (_Float16)p.v[f];
      }
      reinterpret_cast<Entry*>(ad.st.m)[at] = m1;
      reinterpret_cast<Entry*>(ad.st.v)[at] = m2;
      reinterpret_cast<Entry*>(ad.st.p32)[at] = p;
      reinterpret_cast<Vec<_Float16, F>*>(ad.st.p16)[at] = h;
    }
  };

  // The counters start at 0 (bin_scan clears them).  Item gridDim.x + n_queues t + q is number t of queue q
  const uint32_t queue = blockIdx.x % n_queues;
  uint32_t* item_counter = item_counters + queue * kQueueStride;
  auto item_of = [&](const uint32_t ticket) { return gridDim.x + ticket * n_queues + queue; };
  // (the empty asm: where the compiler knows that all lanes add to one word it adds up the lanes first and broadcasts the
  // result at once, which waits for the addition and for every load before it)
  auto draw = [&]() {
    uint32_t at = 0;
    asm volatile("" : "+v"(at));
    return __hip_atomic_fetch_add(item_counter + at, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // What the workgroup starts with is asked for all at once: its second item's number, its first item's records, the largest |dL/dy|
  uint32_t ticket;
  if (threadIdx.x == 0) ticket = draw();

  // An item as the workgroup needs it, all of it uniform (scalar registers)
  struct Item {
    uint32_t l, r0, r1, n_e, bin;
    GT* gl;
    int f0;  // grouped: this item's features are f0 .. f0 + kGroupFeatures - 1
    bool live, dense, shared, grouped;
    bool orphan;  // ADAM: no records, but straddling pairs may have added to the chunk in grad
  };
  using Rec = Record<IT, F>;
  using Stored = typename Rec::Stored;
  // Records on their way, a ring of kRing rows (a row: a record for every lane).  As soon as a lane has taken one out it requests the
  // row kRing further on, of the item itself or, in its last round, of the next item: so many loads are in flight at any time,
  // also while a chunk is flushed.  The loads carry no condition (a buffer's bound makes those beyond the item's end none): behind one
  // the compiler counts loads in flight as if they were not there, and waits for all of them before it uses the oldest.  Rows of
  // a short item's ring that hold nothing still take their instructions: 2, 4 and 8 rows are 64, 58 and 59 us at 11 rows an item,
  // 79, 77 and 88 us at half a row, 612, 582 and 674 us at two.
  constexpr int kFlushUnroll = F <= 4 ? 8 : 1;
  constexpr int kRing = F <= 4 ? 4 : 2;
  // wide entries: the registers do not hold the chunk's old gradient and the ring, so it is read when the chunk is flushed
  constexpr bool kChunkAhead = F <= 2;
  // is feature f the item's business
  auto takes = [&](const Item& c, const int f) {
    return !GROUPS || !c.grouped || (f >= c.f0 && f < c.f0 + kGroupFeatures);
  };
  auto describe = [&](const uint4 d, const bool exists) {
    Item it;
    it.l = (d.w >> 12) & 31u;
    it.bin = d.w >> 20;
    it.live = exists && (d.w & kItemLive);
    it.dense = d.w & kItemDense;
    it.shared = d.w & kItemShared;
    const ItemRecords recs = item_records(d.x, d.y, n_records);
    it.r0 = recs.r0;
    it.r1 = recs.r1;
    it.n_e = (d.w & 0xfffu) + 1u;
    it.gl = grad + (uint64_t)(d.z & 0x3fffffffu) * F;
    it.grouped = GROUPS && ((bp.group_mask >> it.l) & 1u);
    it.f0 = it.grouped ? (int)(d.z >> 30) * kGroupFeatures : 0;
    it.orphan = false;
    if constexpr (ADAM) it.orphan = exists && !(d.w & (kItemLive | kItemShared)) && ((ad.cross_mask >> it.l) & 1u);
    return it;
  };
  // the ring's loads: row j of those that start at record `first` of the item, nothing beyond its last
  const uint32_t my_byte = threadIdx.x * (Rec::kWords * 4u);
  auto window = [&](const Item& it, const uint32_t first) {
    const bool any = it.live && finite && first < it.r1;
    const uint32_t at = any ? first : 0u, left = any ? it.r1 - first : 0u;
    const uint32_t most = (uint32_t)kRing * kAccThreads;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(records) + (uint64_t)at * Rec::kWords, 0,
                                             (left < most ? left : most) * (Rec::kWords * 4u), kBufferWord3);
  };
  auto overwrites = [&](const Item& it) { return ((overwrite_mask >> it.l) & 1u) != 0; };  // uniform
  auto request_chunk = [&](const Item& it, Entry (&cur)[kPer]) {
    if (ADAM || !kChunkAhead || !it.live || !finite || it.shared || overwrites(it)) return;  // uniform
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t e = threadIdx.x + j * kAccThreads;
      if (e < it.n_e) cur[j] = reinterpret_cast<const Entry*>(it.gl)[e];
    }
  };

  auto unpack = [&](const Stored& rec, const Item& c, const double by, uint32_t& la, uint32_t& lb, float& w_lo, float& w_up,
                    bool& first, double (&G)[F]) {
    if constexpr (NEAR) {
      Rec::unpack_near(rec, cmask, by, la, lb, w_lo, w_up, first, G);  // (one corner's weights, 1 and 0, need no smoothstep)
    } else {
      Rec::unpack_scaled(rec, c.dense, cmask, c.n_e - 1u, by, la, lb, w_lo, w_up, first, G);
    }
  };
  uint32_t item = blockIdx.x;
  auto item_at = [&](const uint32_t i) { return i < n_items ? items[i] : make_uint4(0u, 0u, 0u, 0u); };  // uniform
  Item it = describe(item_at(item), item < n_items);
  Stored ring[kRing];
  {
    const auto first = window(it, it.r0);
#pragma unroll
    for (int j = 0; j < kRing; ++j) ring[j] = Rec::load_from(first, my_byte + j * kAccThreads * (Rec::kWords * 4u));
  }
  // largest |dL/dy| of the call (NaN if any is NaN) from the scatter workgroups' maxima
  __shared__ float red[kAccThreads / 64];
  float m = 0.0f;
  for (uint32_t i = threadIdx.x; i < n_max; i += 4 * kAccThreads) {
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = tile_max[i + q * kAccThreads < n_max ? i + q * kAccThreads : n_max - 1u];
#pragma unroll
    for (int q = 0; q < 4; ++q) m = nan_max(m, v[q]);
  }
  for (uint32_t i = threadIdx.x; i < kBuffers * F * cap; i += kAccThreads) acc_lds[i] = 0ull;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = nan_max(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  if (threadIdx.x == 0) s_ticket[1] = item_of(ticket);
  __syncthreads();
  uint32_t next = __builtin_amdgcn_readfirstlane(s_ticket[1]);  // every item number of n_items or more ends the loop, and tickets only grow
  m = red[0];
#pragma unroll
  for (int i = 1; i < kAccThreads / 64; ++i) m = nan_max(m, red[i]);
  m = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, m)));
  if (m == 0.0f && overwrite_mask == 0) return;  // every summand is zero
  finite = m < INFINITY;
  // fixed-point scale: |summand| <= m < 2^E, at most 8B summands per entry
  int E = 0;
  if (finite) (void)frexpf(m, &E);
  const int H = 3 + (32 - __builtin_clz(B > 1 ? B - 1 : 1));
  const int S = (62 - H < kFixedBits ? 62 - H : kFixedBits) - E;  // |summand| * 2^S < 2^min(62-H, 51)
  const double inv_scale = ldexp(1.0, -S);
  uint4 desc_n = item_at(next);
  uint32_t turn = 0;  // 0, 1, 0, ... item after item
  while (item < n_items) {
    unsigned long long* acc = acc_lds + (kBuffers == 2 ? turn * (F * cap) : 0u);
    // the item after the next one: on its way while this one is processed
    if (threadIdx.x == 0) ticket = draw();
    const Item it_n = describe(desc_n, next < n_items);
    Entry cur[kPer];
    request_chunk(it, cur);
    // HG_BWD_OVERWRITE: a chunk that gets no sums stored below is cleared by its owner
    auto clear_chunk = [&](const Item& c) {
      for (uint32_t q = threadIdx.x; q < c.n_e * F; q += kAccThreads)
        if (takes(c, (int)(q % F))) c.gl[q] = (GT)0.0f;
    };
    if (it.live && !finite) {
      if (overwrites(it)) {  // uniform
        clear_chunk(it);
        __threadfence();  // the zeros reach the L2 before any lane's atomics below
        __syncthreads();
      }
      // inf or NaN upstream: keep IEEE semantics with direct fp32 atomics (slow, rare)
      for (uint32_t i = it.r0 + threadIdx.x; i < it.r1; i += kAccThreads) {
        uint32_t la, lb;
        float w_lo, w_up;
        double G[F];
        bool first;
        unpack(Rec::load(records, i), it, 1.0, la, lb, w_lo, w_up, first, G);
        const float wu = SMOOTH && !first ? smoothstep(w_up) : w_up, wl = SMOOTH && !first ? smoothstep(w_lo) : w_lo;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          if (!takes(it, f)) continue;  // uniform
          if (la < it.n_e) grad_atomic_add(it.gl, F * la + f, wl * (float)G[f]);
          // (a corner's own record has no upper corner: 0 * inf is not to reach another entry)
          if (lb < it.n_e && !(NEAR && first)) grad_atomic_add(it.gl, F * lb + f, wu * (float)G[f]);
        }
      }
    } else if (!it.live) {
      if (overwrites(it)) clear_chunk(it);  // no records for this chunk (item < n_items inside the loop)
    }
    {
      auto add_record = [&](const Stored& rec) {
        uint32_t la8, lb8;
        double w_lo, w_up, G[F];
        Rec::template unpack_products<SMOOTH, NEAR>(rec, it.dense, cmask, it.dense ? cmask : it.n_e - 1u, SMOOTH ? S : S - 23, la8,
                                                    lb8, w_lo, w_up, G);
#pragma unroll
        for (int f = 0; f < F; ++f) {
          if (!takes(it, f)) continue;  // uniform
          char* at = reinterpret_cast<char*>(acc + f * cap);
          __hip_atomic_fetch_add(reinterpret_cast<unsigned long long*>(at + la8), fixed_product(w_lo, G[f]), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_fetch_add(reinterpret_cast<unsigned long long*>(at + lb8), fixed_product(w_up, G[f]), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      };
      uint32_t row0 = it.live && finite ? it.r0 : it.r1;  // first record of the ring's oldest row
      bool last;
      do {
        const uint32_t left = it.r1 - row0;
        last = left <= (uint32_t)kRing * kAccThreads;
        const auto ahead = last ? window(it_n, it_n.r0) : window(it, row0 + kRing * kAccThreads);
#pragma unroll
        for (int j = 0; j < kRing; ++j) {
          if (threadIdx.x + j * kAccThreads < left) add_record(ring[j]);
          ring[j] = Rec::load_from(ahead, my_byte + j * kAccThreads * (Rec::kWords * 4u));
        }
        row0 += kRing * kAccThreads;
      } while (!last);
    }
    // ADAM: the chunk's master values and moments, requested before the barrier that ends the summation.  Where the
    // chunk's records are few most entries get none, and only those that do are read (and below, written).
    const uint64_t at0 = ADAM ? (uint64_t)(it.gl - grad) / F : 0;
    const bool whole = ADAM && kChunkAhead && it.live && finite && !it.shared && (it.r1 - it.r0) * 4 >= it.n_e;  // uniform
    [[maybe_unused]] Entry pp[kPer], m1[kPer], m2[kPer];
    if constexpr (ADAM) {
      if (whole) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          const uint32_t e = threadIdx.x + j * kAccThreads;
          if (e >= it.n_e) continue;
          pp[j] = reinterpret_cast<const Entry*>(ad.st.p32)[at0 + e];
          m1[j] = reinterpret_cast<const Entry*>(ad.st.m)[at0 + e];
          m2[j] = reinterpret_cast<const Entry*>(ad.st.v)[at0 + e];
        }
      }
    }
    if (threadIdx.x == 0) s_ticket[turn] = item_of(ticket);
    __syncthreads();
    const uint32_t after_next = __builtin_amdgcn_readfirstlane(s_ticket[turn]);  // rewritten two items on, behind the next item's barrier
    desc_n = item_at(after_next);
    if (it.live && finite) {
      uint32_t tid = threadIdx.x;
      if constexpr (F >= 4) asm volatile("" : "+v"(tid));  // (addresses worked out once, ahead of the loop, would not fit the registers)
      if (GROUPS && it.grouped && !it.shared) {
        // the owner of some features of a chunk, each sum put where it belongs as below
#pragma unroll 1
        for (int j = 0; j < kPer * kGroupFeatures; ++j) {
          const uint32_t q = tid + j * kAccThreads, e = q / kGroupFeatures, f = it.f0 + q % kGroupFeatures;
          const long long a = (long long)acc[f * cap + e];
          acc[f * cap + e] = 0ull;
          if (e >= it.n_e) continue;
          GT* at = it.gl + (uint64_t)e * F + f;
          if (overwrites(it)) *at = (GT)(0.0f + (a ? (float)((double)a * inv_scale) : 0.0f));
          else *at = (GT)((float)*at + (a ? (float)((double)a * inv_scale) : -0.0f));
        }
      } else if (!it.shared) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          const uint32_t e = tid + j * kAccThreads;
          long long a[F];
#pragma unroll
          for (int f = 0; f < F; ++f) {
            a[f] = (long long)acc[f * cap + e];
            acc[f * cap + e] = 0ull;  // ready for the next item
          }
          if (e >= it.n_e) continue;
          if constexpr (ADAM) {
            Entry g;
            bool any = false;
            Entry extra;  // what the straddling pairs of this level added for this entry
            const bool cross = (ad.cross_mask >> it.l) & 1u;  // uniform
            if (cross) extra = reinterpret_cast<const Entry*>(it.gl)[e];
#pragma unroll
            for (int f = 0; f < F; ++f) {
              g.v[f] = a[f] ? (float)((double)a[f] * inv_scale) : 0.0f;
              if (cross) g.v[f] += extra.v[f];
              any = any || g.v[f] != 0.0f;
            }
            if (cross) {
              bool put = false;
#pragma unroll
              for (int f = 0; f < F; ++f) put = put || extra.v[f] != 0.0f;
              if (put) reinterpret_cast<Entry*>(it.gl)[e] = Entry{};
            }
            if (!any) continue;
            const uint64_t at = at0 + e;
            if (whole) update_entry(at, g, pp[j], m1[j], m2[j]);
            else
              update_entry(at, g, reinterpret_cast<const Entry*>(ad.st.p32)[at], reinterpret_cast<const Entry*>(ad.st.m)[at],
                           reinterpret_cast<const Entry*>(ad.st.v)[at]);
            continue;
          }
          if (overwrites(it)) {
            // what adding to a cleared entry would leave
#pragma unroll
            for (int f = 0; f < F; ++f) cur[j].v[f] = (GT)(0.0f + (a[f] ? (float)((double)a[f] * inv_scale) : 0.0f));
          } else {
            if (!kChunkAhead) cur[j] = reinterpret_cast<const Entry*>(it.gl)[e];
            // an entry no record reached gets -0.0f added, which leaves every float (either zero,
            // NaNs included) exactly as it was; storing it anyway keeps the stores of a wave contiguous
#pragma unroll
            for (int f = 0; f < F; ++f)
              cur[j].v[f] = (GT)((float)cur[j].v[f] + (a[f] ? (float)((double)a[f] * inv_scale) : -0.0f));
          }
          reinterpret_cast<Entry*>(it.gl)[e] = cur[j];
        }
      } else if constexpr (sizeof(GT) == 2) {
        // several workgroups share this chunk, half-precision gradient: packed two-half atomics, one
        // lane per aligned pair of halves (two lanes that add to the halves of one word would be
        // served one after the other); the chunk may start on the odd half of a word
        const uint32_t par = (uint32_t)(reinterpret_cast<uintptr_t>(it.gl) >> 1) & 1u;
        const int n_h = (int)(it.n_e * F);
#pragma unroll kFlushUnroll
        for (int j = 0; j < (F * kPer) / 2 + 1; ++j) {
          const int p = (int)tid + j * kAccThreads;
          const int q0 = 2 * p - (int)par;
          float v[2] = {0.0f, 0.0f};
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const int q = q0 + t;
            if (q < 0 || q >= F * (int)cap || !takes(it, q % F)) continue;
            unsigned long long* slot = &acc[(q % F) * cap + q / F];
            const long long a = (long long)*slot;
            *slot = 0ull;
            if (q < n_h && a != 0) v[t] = (float)((double)a * inv_scale);
          }
          if (v[0] != 0.0f || v[1] != 0.0f) grad_atomic_add2(it.gl + q0, 0, v[0], v[1]);
        }
      } else {
        // several workgroups share this chunk: fp32 atomics, one lane per float so that the
        // features of an entry and its neighbours travel in the same 64-byte requests
#pragma unroll kFlushUnroll
        for (int j = 0; j < F * kPer; ++j) {
          const uint32_t q = tid + j * kAccThreads;  // float index in the chunk
          const uint32_t e = q / F;
          unsigned long long* slot = &acc[(q % F) * cap + e];
          const long long a = (long long)*slot;
          *slot = 0ull;
          if (e < it.n_e && a != 0) grad_atomic_add(it.gl, q, (float)((double)a * inv_scale));
        }
      }
    }
    if constexpr (ADAM) {
      if ((it.live && (it.shared || !finite)) || it.orphan) {  // uniform: the sums of this chunk meet in grad
        __shared__ uint32_t s_last;
        // This workgroup's additions are performed before it is counted: every wave waits for its own.  They, the
        // counter and the exchanges below are all device-scope atomics, which meet behind the caches, so
        // nothing else has to be ordered; a device-scope fence would write this XCD's L2 back once per item (the
        // pass took 502 us with it, 2^18 points at Table 1's sizes).
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0)
          s_last = __hip_atomic_fetch_sub(&ad.chunk_open[bp.bin_base[it.l] + it.bin], 1u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) == 1u;
        __syncthreads();
        if (s_last) {  // every other workgroup with records of this chunk has been counted
          for (uint32_t e = threadIdx.x; e < it.n_e; e += kAccThreads) {
            Entry g;
            bool any = false;
#pragma unroll
            for (int f = 0; f < F; ++f) {  // taken out where the additions were performed, not from a cache
              g.v[f] = __hip_atomic_exchange(it.gl + (uint64_t)e * F + f, 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              any = any || g.v[f] != 0.0f;
            }
            const uint64_t at = at0 + e;
            if (any)
              update_entry(at, g, reinterpret_cast<const Entry*>(ad.st.p32)[at], reinterpret_cast<const Entry*>(ad.st.m)[at],
                           reinterpret_cast<const Entry*>(ad.st.v)[at]);
          }
        }
      }
    }
    if constexpr (kBuffers == 1) __syncthreads();
    turn ^= 1u;
    item = next;
    next = after_next;
    it = it_n;
  }
}

// Level parts of a count or scatter grid for a batch of n_tiles tiles: the plan's, doubled (up to one level per
// part) while the grid would leave most compute units without a workgroup.  A small batch is a few tiles, and a
// workgroup walks the levels of its part one after the other: 2^14 points at Table 1's sizes are 32 tiles, whose
// 128 scatter workgroups took 19 us for four levels each.
static uint32_t parts_for_batch(uint32_t plan_parts, uint32_t L, uint32_t n_tiles) {
  static const uint32_t cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    return (uint32_t)n;
  }();
  uint32_t parts = plan_parts;
  while (parts < L && (uint64_t)n_tiles * parts < 2ull * cus) parts = parts * 2 < L ? parts * 2 : L;
  return parts;
}

// In two dimensions a tile of 512 points has 1024 records a level, which on a level of 1024 chunks is one to a run: every store a part
// of a line.  Tiles of 1024 points there, two points a thread, in batches of 2^16 points and more, for records of up to 16 bytes and as
// long as a compute unit's LDS holds two scatter workgroups with them: the staging area is twice as large, and where that leaves one
// workgroup it costs what the longer runs save, or more.  Forward and backward, uniform points, us, tiles of 512 / 1024 points, T = 2^22:
//   two workgroups  F = 2 half 2^16 133 / 125, 100003 162 / 155, 2^18 242 / 228, 2^20 756 / 681; F = 1 single 116 / 107, 140 / 130,
//                   224 / 209, 738 / 657; F = 4 half on 8 levels 74 / 73, 93 / 91, 138 / 134, 422 / 396; F = 2 single in the batches that still
//                   take 8 parts 2^16 152 / 141, 100003 195 / 187
//   one workgroup   F = 2 single 2^17 215 / 218, 2^18 310 / 320, 2^20 1015 / 1010; F = 4 half 275 / 277, 382 / 394, 1098 / 1092;
//                   F = 8 single, T = 2^21, 2^16 157 / 168, 2^18 340 / 350, 2^20 1001 / 1011
//   24 bytes, two   F = 4 single on 8 levels 2^16 92 / 91, 80001 97 / 101, 2^17 133 / 127, 200001 172 / 174, 2^18 198 / 197, 2^20 642 / 631;
//   workgroups      F = 8 half, T = 2^21, 80001 117 / 120, 2^17 140 / 133, 2^18 203 / 201 (three fit with tiles of 512: left at those)
// Levels of 512 chunks lose at some sizes what they gain at others (F = 1, T = 2^21: 100003 points 88 / 92, 2^20 444 / 418;
// F = 8 on chunks of 2048, T = 2^20: 113 / 118, 624 / 621), of 32 chunks everywhere (T = 2^17: 100003 points 69 / 73); smaller
// batches take the same time (94 both).
constexpr uint32_t kWideTilesFrom = 1u << 16, kWideTilesBins = 1024, kWideTilesWords = 4;
constexpr size_t kLdsOfUnit = 160 * 1024;
uint32_t tile_mult_for(const hashgrid* h, uint32_t B) {
  const BinPlan& bp = h->bp;
  const uint32_t L = h->lv.L, widest = bp.bin_base[L] - bp.bin_base[L - 1];  // the finest level has the most entries
  if (bp.tile_mult != 1 || h->cfg.d != 2 || bp.corner_records || widest < kWideTilesBins || B < kWideTilesFrom ||
      record_words(h) > kWideTilesWords)
    return bp.tile_mult;
  const uint32_t parts = parts_for_batch(bp.scatter_parts, L, tiles_for(2, B));
  const size_t lds = scatter_lds(staged_records(2 * 2, false), record_words(h), max_part_bins(bp, L, parts)) +
                     kBinThreads / 64 * sizeof(uint32_t);  // (bin_scatter's scan_tmp)
  return 2 * lds <= kLdsOfUnit ? 2u : 1u;
}

// The count pass by itself: counts[tile][bin] for the B points (x only).
static hg_status launch_count(const hashgrid* h, uint32_t B, const float* x, const Workspace& ws, hipStream_t s) {
  BinPlan bp = h->bp;
  bp.tile_mult = tile_mult_for(h, B);
  const uint32_t L = h->lv.L, cparts = parts_for_batch(bp.count_parts, L, ws.n_tiles);
  const bool smooth = h->cfg.interp == HG_INTERP_SMOOTHSTEP;
  const dim3 grid((ws.n_tiles + 7u) / 8u * 8u, cparts);  // see tile_of_workgroup
#define HG_COUNT(D, C)                                                                                              \
  hipLaunchKernelGGL((bin_count<D, C>), grid, dim3(kBinThreads), (size_t)max_part_bins(bp, L, cparts) * 4, s, h->lv, bp, smooth, \
                     B, x, ws.counts, ws.n_bins, ws.n_tiles)
  if (bp.corner_records) {
    if (h->cfg.d == 3) HG_COUNT(3, true);
    else if (h->cfg.d == 2) HG_COUNT(2, true);
    else HG_COUNT(1, true);
  } else {
    if (h->cfg.d == 3) HG_COUNT(3, false);
    else HG_COUNT(2, false);
  }
#undef HG_COUNT
  return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
}

static void launch_scan(const hashgrid* h, const Workspace& ws, uint32_t zero_mask, void* grad, const SideJob& job, hipStream_t s) {
  auto launch = [&](auto rows, auto bins) {
    constexpr int kBins = decltype(bins)::value;
    const dim3 grid((ws.n_bins + kBins * 8 - 1) / (kBins * 8) * 8 + job.blocks);  // see tile_of_workgroup
    hipLaunchKernelGGL((bin_scan<decltype(rows)::value, kBins>), grid, dim3(kScanThreads), 0, s, ws.n_tiles, ws.n_bins, ws.counts,
                       ws.bin_total, ws.item_counters, h->lv, zero_mask, h->cfg.F, grad, h->cfg.grad_dtype == HG_F16, job);
  };
  auto rows_at = [&](uint32_t bins) { return (ws.n_tiles * bins + kScanThreads - 1) / kScanThreads; };
  // As wide as the rows a thread then has fit its registers; wider batches than 16 rows of 8 bins (2^20 points) read them twice
  constexpr std::integral_constant<int, 32> b32{};
  if (rows_at(32) <= 2) launch(std::integral_constant<int, 2>{}, b32);
  else if (rows_at(32) <= 8) launch(std::integral_constant<int, 8>{}, b32);
  else if (rows_at(32) <= 16) launch(std::integral_constant<int, 16>{}, b32);
  else if (rows_at(16) <= 16) launch(std::integral_constant<int, 16>{}, std::integral_constant<int, 16>{});
  else if (rows_at(8) <= 16) launch(std::integral_constant<int, 16>{}, std::integral_constant<int, 8>{});
  else launch(std::integral_constant<int, 0>{}, b32);
}

// The optimiser's part of a sorted backward pass (launch_binned_adam)
struct BinnedAdam {
  AdamArgs a;
  AdamState st;
  SideJob job;
};

template <int D, typename IT, int F, bool CORNERS>
static hg_status launch_binned(const hashgrid* h, uint32_t B, const float* x, const void* dy, void* grad,
                               const Workspace& ws, const bool counted, const bool overwrite, hipStream_t s,
                               const BinnedAdam* ba = nullptr) {
  const bool g16 = h->cfg.grad_dtype == HG_F16;
  using Rec = Record<IT, F>;
  constexpr uint32_t R = 1u << (D - 1);
  constexpr int DP = CORNERS ? 2 : D;  // (dimension of the kernels that only the pair records use: never D = 1)
  BinPlan bp = h->bp;
  bp.tile_mult = tile_mult_for(h, B);
  plan_slices(bp, h->lv, B, F, g16);
  const bool smooth = h->cfg.interp == HG_INTERP_SMOOTHSTEP;
  const uint32_t n_records = B * h->lv.L * bp.rec_per_point;
  const uint32_t L = h->lv.L, parts = parts_for_batch(bp.scatter_parts, L, ws.n_tiles);
  constexpr bool kWide = D == 2 && !CORNERS && Rec::kWords <= kWideTilesWords;  // (what tile_mult_for may give a tile_mult of 2)
  constexpr size_t kScatterLdsMax = scatter_lds(staged_records(R, CORNERS), Rec::kWords, kMaxScatterPartBins);
  constexpr size_t kWideLdsMax = scatter_lds(staged_records(2 * R, CORNERS), Rec::kWords, kMaxScatterPartBins);
  // The largest (146 KB: d = 3, F = 8, single precision, any table size) leaves one workgroup on a compute unit.  Unstaged such plans
  // are 3 to 12 % faster on points in no order and up to 1.8 times slower on rays (30000 points, T = 524287, both passes: 98
  // against 93 us, 108 against 196).
  static_assert(kScatterLdsMax <= kLdsOfUnit && (!kWide || kWideLdsMax <= kLdsOfUnit), "a workgroup's LDS");
  constexpr size_t kAccLds = (size_t)acc_buffers(F) * F * 8 << chunk_log2_of(F);
  constexpr bool kAdam = !CORNERS && std::is_same<IT, _Float16>::value;  // what launch_binned_adam serves
  // more dynamic LDS than the default limit of 64 KiB: opt in once per kernel
  static const hipError_t lds_ok = [] {
    hipError_t e = hipSuccess;
    if (!CORNERS && kScatterLdsMax > 64 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_scatter<DP, IT, F, true, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kScatterLdsMax);
    if (e == hipSuccess && kScatterLdsMax > 64 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_scatter<D, IT, F, false, CORNERS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kScatterLdsMax);
    if constexpr (kWide) {
      if (e == hipSuccess && kWideLdsMax > 64 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_scatter<D, IT, F, true, false, 2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideLdsMax);
      if (e == hipSuccess && kWideLdsMax > 64 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_scatter<D, IT, F, false, false, 2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideLdsMax);
    }
    if (e == hipSuccess && kAccLds > 48 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, false, float, false, false, CORNERS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
    if (e == hipSuccess && kAccLds > 48 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, true, float, false, false, CORNERS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
    if (e == hipSuccess && kAccLds > 48 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, false, _Float16, false, false, CORNERS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
    if (e == hipSuccess && kAccLds > 48 * 1024)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, true, _Float16, false, false, CORNERS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
    if constexpr (F == kGroupedF) {
      if (e == hipSuccess && kAccLds > 48 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, false, _Float16, false, true, CORNERS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
      if (e == hipSuccess && kAccLds > 48 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, true, _Float16, false, true, CORNERS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
    }
    if constexpr (kAdam) {
      if (e == hipSuccess && kAccLds > 48 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, false, float, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
      if (e == hipSuccess && kAccLds > 48 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bin_accumulate<IT, F, true, float, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAccLds);
    }
    return e;
  }();
  if (lds_ok != hipSuccess) return HG_ERR_DEVICE;
  const uint32_t part_bins = max_part_bins(bp, L, parts);
  const size_t lds_scatter = scatter_lds(staged_records(bp.tile_mult == 2 ? 2 * R : R, CORNERS), Rec::kWords, part_bins);
  const uint32_t tile_wgs = (ws.n_tiles + 7u) / 8u * 8u;  // see tile_of_workgroup
  if (!counted && launch_count(h, B, x, ws, s) != HG_OK) return HG_ERR_DEVICE;
  // HG_BWD_OVERWRITE: the owner of a chunk stores its sums, except on levels whose chunks are summed
  // by several workgroups; those levels are cleared first and added into as usual.  Pairs that
  // straddle two chunks (hashed levels of resolution 2^chunk_log2 or more) get their atomic adds
  // from a pass after the owners have stored.
  uint32_t add_mask = 0, cross_mask = 0;
  for (uint32_t l = 0; l < L; ++l) {
    const bool hashed = !((h->lv.dense_mask >> l) & 1u);
    if (bp.slices[l] > 1) add_mask |= 1u << l;
    if (!CORNERS && hashed && h->lv.N[l] + 1u >= (1u << bp.chunk_log2)) cross_mask |= 1u << l;
  }
  const uint32_t all_levels = L == 32 ? 0xffffffffu : (1u << L) - 1u;
  const uint32_t zero_mask = overwrite ? add_mask : 0u, overwrite_mask = overwrite ? all_levels & ~add_mask : 0u;
  const bool defer_cross = overwrite && cross_mask != 0;  // those atomic adds then follow the accumulate pass
  const SideJob job = ba ? ba->job : SideJob{};
  launch_scan(h, ws, zero_mask, grad, job, s);
  auto scatter = [&](auto cross) {
    constexpr bool kCross = decltype(cross)::value;
    constexpr int DS = kCross ? DP : D;  // (the straddling pairs exist with pair records only)
    if (bp.tile_mult > 2) {
      hipLaunchKernelGGL((bin_scatter_direct<DS, IT, F, kCross, CORNERS && !kCross>), dim3(tile_wgs, parts),
                         dim3(kBinThreads), (size_t)part_bins * 4, s, h->lv, bp, smooth, B, x,
                         static_cast<const IT*>(dy), ws.counts, ws.bin_total, ws.items, ws.chunk_open, ws.records, ws.n_bins,
                         n_records, ws.n_tiles, ws.tile_max, grad, g16);
    } else {
      auto staged = [&](auto points) {
        hipLaunchKernelGGL((bin_scatter<DS, IT, F, kCross, CORNERS && !kCross, decltype(points)::value>), dim3(tile_wgs, parts),
                           dim3(kBinThreads), lds_scatter, s, h->lv, bp, smooth, B, x, static_cast<const IT*>(dy),
                           ws.counts, ws.bin_total, ws.items, ws.chunk_open, ws.records, ws.n_bins, n_records, ws.n_tiles,
                           ws.tile_max, grad, g16);
      };
      if constexpr (kWide) {
        if (bp.tile_mult == 2) {
          staged(std::integral_constant<int, 2>{});
          return;
        }
      }
      staged(std::integral_constant<int, 1>{});
    }
  };
  if (CORNERS || defer_cross || cross_mask == 0)  // no such pairs at these resolutions, or bin_crossing takes them
    scatter(std::false_type{});
  else
    scatter(std::true_type{});
  const uint32_t n_items = bp.wg_base[h->lv.L];
  static const uint32_t acc_slots = [] {  // its LDS lets one workgroup run per CU; more would queue
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      cus = 256;
    return (uint32_t)cus * kAccWgsPerCu;
  }();
  const dim3 acc_grid(n_items < acc_slots ? n_items : acc_slots);
  const uint32_t n_queues = n_items >= kManyItems ? kQueues : 1u;
  auto accumulate = [&](auto smooth_t, auto* g, auto groups_t) {
    using GT = typename std::remove_pointer<decltype(g)>::type;
    hipLaunchKernelGGL((bin_accumulate<IT, F, decltype(smooth_t)::value, GT, false, decltype(groups_t)::value, CORNERS>), acc_grid,
                       dim3(kAccThreads), kAccLds, s, h->lv, bp, B, n_items, ws.items, ws.tile_max, ws.n_tiles * parts,
                       ws.records, ws.item_counters, n_queues, g, overwrite_mask, NoAdam{});
  };
  if constexpr (kAdam) {
    if (ba) {
      AdamOut out;
      out.a = ba->a;
      out.st = ba->st;
      out.chunk_open = ws.chunk_open;
      out.cross_mask = cross_mask;
      auto accumulate_adam = [&](auto smooth_t) {
        hipLaunchKernelGGL((bin_accumulate<IT, F, decltype(smooth_t)::value, float, true>), acc_grid, dim3(kAccThreads),
                           kAccLds, s, h->lv, bp, B, n_items, ws.items, ws.tile_max, ws.n_tiles * parts, ws.records, ws.item_counters, n_queues, static_cast<float*>(grad), 0u, out);
      };
      if (smooth) accumulate_adam(std::true_type{});
      else accumulate_adam(std::false_type{});
      return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
    }
  }
  if (g16 && bp.group_mask != 0) {
    if constexpr (F == kGroupedF) {
      if (smooth) accumulate(std::true_type{}, static_cast<_Float16*>(grad), std::true_type{});
      else accumulate(std::false_type{}, static_cast<_Float16*>(grad), std::true_type{});
    }
  } else if (g16) {
    if (smooth) accumulate(std::true_type{}, static_cast<_Float16*>(grad), std::false_type{});
    else accumulate(std::false_type{}, static_cast<_Float16*>(grad), std::false_type{});
  } else {
    if (smooth) accumulate(std::true_type{}, static_cast<float*>(grad), std::false_type{});
    else accumulate(std::false_type{}, static_cast<float*>(grad), std::false_type{});
  }
  if (defer_cross)
    hipLaunchKernelGGL((bin_crossing<DP, IT, F>), dim3((B + kBinThreads - 1) / kBinThreads), dim3(kBinThreads), 0, s,
                       h->lv, bp, smooth, B, x, static_cast<const IT*>(dy), cross_mask, grad, g16);
  return hipGetLastError() == hipSuccess ? HG_OK : HG_ERR_DEVICE;
}

template <int D, typename IT, bool CORNERS>
static hg_status launch_binned_f(const hashgrid* h, uint32_t B, const float* x, const void* dy, void* grad,
                                 const Workspace& ws, const bool counted, const bool overwrite, hipStream_t s) {
  switch (h->cfg.F) {
    case 1: return launch_binned<D, IT, 1, CORNERS>(h, B, x, dy, grad, ws, counted, overwrite, s);
    case 2: return launch_binned<D, IT, 2, CORNERS>(h, B, x, dy, grad, ws, counted, overwrite, s);
    case 4: return launch_binned<D, IT, 4, CORNERS>(h, B, x, dy, grad, ws, counted, overwrite, s);
    case 8: return launch_binned<D, IT, 8, CORNERS>(h, B, x, dy, grad, ws, counted, overwrite, s);
    default: return HG_ERR_UNSUPPORTED;
  }
}

hg_status launch_binned_adam(const hashgrid* h, uint32_t B, const float* x, const void* dy, float* zeros, void* workspace,
                             bool counted, const AdamArgs& a, const AdamState& st, const SideJob& job, hipStream_t s) {
  if (h->bp.corner_records || h->cfg.io_dtype != HG_F16 || h->cfg.grad_dtype != HG_F32) return HG_ERR_UNSUPPORTED;
  Workspace ws;
  carve(h, B, static_cast<uint8_t*>(workspace), &ws);
  BinnedAdam ba;
  ba.a = a;
  ba.st = st;
  ba.job = job;
#define HG_BA(D, F) launch_binned<D, _Float16, F, false>(h, B, x, dy, zeros, ws, counted, false, s, &ba)
  switch (h->cfg.d * 16 + h->cfg.F) {
    case 2 * 16 + 1: return HG_BA(2, 1);
    case 2 * 16 + 2: return HG_BA(2, 2);
    case 2 * 16 + 4: return HG_BA(2, 4);
    case 2 * 16 + 8: return HG_BA(2, 8);
    case 3 * 16 + 1: return HG_BA(3, 1);
    case 3 * 16 + 2: return HG_BA(3, 2);
    case 3 * 16 + 4: return HG_BA(3, 4);
    case 3 * 16 + 8: return HG_BA(3, 8);
    default: return HG_ERR_UNSUPPORTED;
  }
#undef HG_BA
}

template <typename IT>
static hg_status launch_binned_d(const hashgrid* h, uint32_t B, const float* x, const void* dy, void* grad,
                                 const Workspace& ws, const bool counted, const bool overwrite, hipStream_t s) {
  if (h->bp.corner_records) {
    switch (h->cfg.d) {
      case 1: return launch_binned_f<1, IT, true>(h, B, x, dy, grad, ws, counted, overwrite, s);
      case 2: return launch_binned_f<2, IT, true>(h, B, x, dy, grad, ws, counted, overwrite, s);
      default: return launch_binned_f<3, IT, true>(h, B, x, dy, grad, ws, counted, overwrite, s);
    }
  }
  return h->cfg.d == 3 ? launch_binned_f<3, IT, false>(h, B, x, dy, grad, ws, counted, overwrite, s)
                       : launch_binned_f<2, IT, false>(h, B, x, dy, grad, ws, counted, overwrite, s);
}

}  // namespace hg

extern "C" {

uint64_t hashgrid_bwd_workspace_bytes(const hashgrid_t* hg, uint32_t B) {
  if (!hg || !hg->bp.supported || B == 0 || B > HG_MAX_BATCH) return 0;
  if ((uint64_t)B * hg->lv.L * hg->bp.rec_per_point >= (1ull << 32)) return 0;
  return hg::carve(hg, B, nullptr, nullptr);
}

int hashgrid_bwd_ws_pays(const hashgrid_t* hg, uint32_t B) {
  if (hashgrid_bwd_workspace_bytes(hg, B) == 0) return 0;
  // Both passes in microseconds, from measurements on an MI355X.  Sorted pass: about 16 us of
  // launches, 0.017 us per chunk (every chunk of the gradient is visited and rewritten), then the
  // records, written once and read once: ~300 K records of 12 bytes per us, in proportion for
  // larger ones (wider entries, fp32 dL/dy).  (Any table size: priced at a record a pair.)
  // Atomic pass: ~6 us, then ~14.5 K pairs of corners per us (11 K at F = 4, 9 K at F = 8: their
  // requests are fatter), unless one 64-byte block of the gradient draws so many requests that
  // they queue up behind each other (~0.02 us each): the smallest level decides that, taking the
  // points as spread evenly over its entries.
  // Measured, sorted / atomic, d = 3, at the last size that takes the atomic pass and the first that takes the sorted one here: F = 2,
  // T = 2^19 8192 points 40 / 40, 11000 43 / 53; T = 1000003, single precision, 12288 59 / 54, 16384 60 / 69; F = 4, T = 2^17 2048 32 / 20,
  // 4096 35 / 24 (8192 41 / 41).  The price knows nothing of the longest work item, so that wide entries, whose items are 2 F additions in
  // LDS a record, change over too early: F = 8 half, T = 2^17, 8 levels 6000 points 35 / 22, 12288 43 / 34, 24576 51 / 59.
  const uint32_t F = hg->cfg.F, d = hg->cfg.d;
  const double pairs = (double)B * hg->lv.L * (1u << (d - 1));
  const double records = (double)B * hg->lv.L * hg::pairs_per_point(hg->bp);
  const double rec_bytes = 8.0 + (F * (hg->cfg.io_dtype == HG_F16 ? 2u : 4u) + 3u) / 4u * 4u;
  double per_block = 0.0;
  for (uint32_t l = 0; l < hg->lv.L; ++l) {
    const double blocks = ceil((double)hg->lv.size[l] * F * sizeof(float) / 64.0);
    per_block = fmax(per_block, (double)B * (1u << (d - 1)) / blocks);
  }
  const double pairs_per_us = F <= 2 ? 14.5e3 : F == 4 ? 11e3 : 9e3;
  const double sorted_us = 16.0 + 0.017 * hg->bp.bin_base[hg->lv.L] + records * (rec_bytes / 12.0) / 300e3;
  const double atomic_us = 6.0 + fmax(pairs / pairs_per_us, 0.02 * per_block);
  return atomic_us > sorted_us ? 1 : 0;
}

// shared argument checks of the two entry points that take the scratch buffer
static hg_status check_workspace(const hashgrid_t* hg, uint32_t B, const void* workspace, uint64_t workspace_bytes) {
  const uint64_t need = hashgrid_bwd_workspace_bytes(hg, B);
  if (need == 0) return HG_ERR_UNSUPPORTED;
  if (!workspace || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255)) return HG_ERR_INVALID_ARG;
  return HG_OK;
}

hg_status hashgrid_encode_fwd_ws(const hashgrid_t* hg, uint32_t B, const float* x, const void* params, void* y,
                                 void* workspace, uint64_t workspace_bytes, void* stream) {
  if (!hg) return HG_ERR_INVALID_ARG;
  if (B == 0) return HG_OK;
  const hg_status ok = check_workspace(hg, B, workspace, workspace_bytes);
  if (ok != HG_OK) return ok;
  if (!x || !params || !y || (reinterpret_cast<uintptr_t>(x) & 3)) return HG_ERR_INVALID_ARG;
  hg::Workspace ws;
  hg::carve(hg, B, static_cast<uint8_t*>(workspace), &ws);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // The counting kernel runs full workgroups (they cover whole tiles), which is slow for a batch that
  // cannot give every CU one: there the plain forward in small workgroups plus the count pass is
  // faster and leaves the workspace in the same state.
  // (So it is for plans with BinPlan::corner_records, which the counting kernel does not serve.)
  if (hg->bp.corner_records || hg::point_major_block(B) < 1024u) {
    const hg_status st = hashgrid_encode_fwd(hg, B, x, params, y, stream);
    return st != HG_OK ? st : hg::launch_count(hg, B, x, ws, s);
  }
  return hg::launch_fwd_counting(hg, B, x, params, y, ws.counts, ws.n_bins, ws.n_tiles, s);
}

hg_status hashgrid_encode_bwd_ws(const hashgrid_t* hg, uint32_t B, const float* x, const void* dLdy,
                                 void* grad_params, void* workspace, uint64_t workspace_bytes, uint32_t flags,
                                 void* stream) {
  if (!hg || (flags & ~(uint32_t)(HG_BWD_COUNTED | HG_BWD_OVERWRITE))) return HG_ERR_INVALID_ARG;
  if (B == 0) return HG_OK;
  const hg_status ok = check_workspace(hg, B, workspace, workspace_bytes);
  if (ok != HG_OK) return ok;
  if (!x || !dLdy || !grad_params) return HG_ERR_INVALID_ARG;
  const size_t io = hg->cfg.io_dtype == HG_F16 ? 2 : 4, F = hg->cfg.F;
  const size_t gs = hg->cfg.grad_dtype == HG_F16 ? 2 : 4;
  // one entry's gradient, up to 16 bytes (and the 4 bytes of a packed atomic at least)
  const size_t grad_align = F * gs > 16 ? 16 : (F * gs < 4 ? 4 : F * gs);
  if ((reinterpret_cast<uintptr_t>(x) & 3) || (reinterpret_cast<uintptr_t>(dLdy) & (F * io - 1) & 15) ||
      (reinterpret_cast<uintptr_t>(grad_params) & (grad_align - 1)))
    return HG_ERR_INVALID_ARG;
  hg::Workspace ws;
  hg::carve(hg, B, static_cast<uint8_t*>(workspace), &ws);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool i16 = hg->cfg.io_dtype == HG_F16, counted = flags & HG_BWD_COUNTED, ow = flags & HG_BWD_OVERWRITE;
  return i16 ? hg::launch_binned_d<_Float16>(hg, B, x, dLdy, grad_params, ws, counted, ow, s)
             : hg::launch_binned_d<float>(hg, B, x, dLdy, grad_params, ws, counted, ow, s);
}

// ---------------------------------------------------------------- entry point that allocates nothing
//
// For callers that cannot allocate (code under HIP graph capture, tight serving loops, harnesses that
// forbid hipMalloc) and have no workspace to hand over: the scratch of the sorted pass lives in a
// fixed device array that every GPU holds from the moment the library is loaded.
//
// HG_STATIC_SCRATCH_BYTES is what counts and records may take; the item list has room of its own behind them.  A level
// of n chunks has n * ceil(ceil(B R / n) / kTargetRecordsPerAccWg) items at most (plan_slices), which is below
// n + n / target + B R / target; 32 levels of 4096 chunks and records of 12 bytes and more make that the bound below.
// Levels whose items are shared out by features have kShares of them at most.
constexpr uint64_t kMostBins = (uint64_t)HG_MAX_LEVELS * hg::kMaxLevelBins;
constexpr uint64_t kMostItems = kMostBins + kMostBins / hg::kTargetRecordsPerAccWg + 1 +
                                HG_STATIC_SCRATCH_BYTES / 12 / hg::kTargetRecordsPerAccWg + 1 +
                                hg::kShares;
constexpr uint64_t kStaticBytes = HG_STATIC_SCRATCH_BYTES + (kMostItems * sizeof(uint4) + 255) / 256 * 256;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

namespace hg {
constexpr int kMaxDevices = 64;
// Device address of `scratch` on each GPU (every GPU has its own copy of the array at its own
// address); looked up once per device, with that device current.  In host code the array's name is
// only a handle for this lookup, never an address a kernel could use.
static void* static_scratch_of_current_device() {
  static std::atomic<void*> ptr_of[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void* p = ptr_of[dev].load(std::memory_order_acquire);
  if (!p) {
    void* q = nullptr;
    if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) {
      (void)hipGetLastError();
      return nullptr;
    }
    ptr_of[dev].store(q, std::memory_order_release);  // (two threads racing here store the same address)
    p = q;
  }
  return p;
}
}  // namespace hg

hg_status hashgrid_encode_bwd_static(const hashgrid_t* hg, uint32_t B, const float* x, const void* dLdy,
                                     void* grad_params, uint32_t flags, void* stream) {
  if (!hg || (flags & ~(uint32_t)HG_BWD_OVERWRITE)) return HG_ERR_INVALID_ARG;
  if (B == 0) return HG_OK;
  const uint64_t need = hashgrid_bwd_workspace_bytes(hg, B);
  if (need == 0) return HG_ERR_UNSUPPORTED;
  uint64_t before_items = 0;
  (void)hg::carve(hg, B, nullptr, nullptr, &before_items);
  if (before_items > HG_STATIC_SCRATCH_BYTES || need > kStaticBytes) return HG_ERR_UNSUPPORTED;  // batch too large for the fixed array
  void* ws = hg::static_scratch_of_current_device();
  if (!ws) return HG_ERR_DEVICE;
  // every word of the scratch that a kernel reads is written earlier in the same call (counts by
  // bin_count, totals and the queues' counters by bin_scan, items, records and maxima by bin_scatter),
  // so what the previous call left behind needs no clearing
  return hashgrid_encode_bwd_ws(hg, B, x, dLdy, grad_params, ws, kStaticBytes, flags, stream);
}

}  // extern "C"
