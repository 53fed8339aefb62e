// EmbeddingBag sum-pooling forward and the coalesced sparse-SGD backward over
// the hot cache (HBM) and the staging buffer of gathered cold rows.
//
// Lane layout: a row is covered by G lanes holding VEC consecutive elements
// each (fp32: 16-byte loads for VEC = 4; bf16: 16-byte loads for VEC = 8,
// widened to fp32),
// G = min(dim/VEC, 64); a wave holds NG = 64/G row groups; rows wider than 64
// vectors are split into column chunks over blockIdx.y.
//
// Backward: the lookups of the mini-batch are sorted by compressed row key
// (hot slot, or n_hot + staging row) with their bag as payload; then tiles of
// the sorted list are reduced by groups of E consecutive entries: a run of
// equal keys entirely inside a group is a complete segment and its row is
// updated at once; pieces of runs that cross group boundaries are combined in
// LDS in group order, and pieces that cross tile boundaries are combined by a
// second kernel in tile order.  Every row is read and written once and the
// summation order depends only on the sorted order, so results are
// deterministic.
#include <algorithm>

#include "hl_embbag_fwd.h"
#include "hl_group_sort.h"
#include "hl_internal.h"

// sorted entries per row group of the reduction: 6 for rows of 4 or more
// elements per lane (the register budget of 7 waves per SIMD), else 8
#define RB_EN(V) ((V) >= 4 ? 6 : 8)
#ifndef RB_WAVES
#define RB_WAVES 2  // waves per reduction block (2 measured fastest: a block waits for its slowest wave)
#endif
#define RB_BLOCK (RB_WAVES * 64)
static_assert(RB_WAVES >= 2, "bw_r2_longs");

template <int VEC, bool BF, int PART>
__global__ void __launch_bounds__(256)
eb_fwd(const void* w_hot, const void* stg, int32_t stg_rows, uint32_t n_hot, uint32_t k_cap,
       const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr, int32_t bps,
       const int32_t* __restrict__ sample_ids, const int32_t* n_sel_dev, int32_t n_sel_max,
       float* __restrict__ out, eb_geom g, int64_t n_lookups, int64_t n_bags_total, int32_t n_samples,
       int32_t nbg, uint32_t* err, hl_hook hk) {
  hl_hook_head(hk);
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && bag_ptr[n_bags_total] != n_lookups)
    hl_flag(err, HL_DEVERR_SHAPE);
  // (thread 0, which carries the handover, is in the first row group of every block)
  eb_fwd_body<VEC, BF, PART>(blockIdx.x, gridDim.x, w_hot, stg, stg_rows, n_hot, k_cap, codes, bag_ptr, bps,
                             sample_ids, n_sel_dev, n_sel_max, out, g, n_samples, nbg, err);
  hl_hook_tail(hk);
}

template <int VEC, bool BF, int PART>
__global__ void __launch_bounds__(256)
eb_fwd_oh(const void* w_hot, const void* stg, int32_t stg_rows, uint32_t n_hot, uint32_t k_cap,
          const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr, float* __restrict__ out, eb_geom g,
          int64_t n_lookups, int64_t n_bags, uint32_t* err, hl_hook hk) {
  hl_hook_head(hk);
  __shared__ uint32_t s_code[4][OH_UNIT];
  // (thread 0, which carries the handover, is in the first row group of every block)
  eb_fwd_oh_body<VEC, BF, PART>(blockIdx.x, gridDim.x, w_hot, stg, stg_rows, n_hot, k_cap, codes, bag_ptr, out, g,
                                n_lookups, n_bags, err, s_code);
  hl_hook_tail(hk);
}

// The forward over every bag of a one-hot mini-batch and the backward's
// grouping in one launch: T blocks each sort a table (gt_sort_body), the others
// pool the bags and check that every bag is one-hot.  Nothing one side
// writes is read by the other, so they run side by side (the sorts on a few
// compute units at LDS and latency speed, the HBM-bound forward on the rest).
// CODES: the sorts read the slot codes themselves, T apart, which spares the
// launch of gt_prep (GT_CODES_E); otherwise gt_prep's keys.  The first T blocks
// sort; with CODES the first T + GT_CHECKS take tickets, of which the first
// GT_CHECKS check the bags and then pool.
template <int VEC, bool BF, int ITEMS, bool CODES>
__global__ void __launch_bounds__(GT_THREADS)
eb_fwd_gt(const void* w_hot, const void* stg, int32_t stg_rows, uint32_t n_hot, uint32_t k_cap,
          const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr, float* __restrict__ out, eb_geom g,
          int64_t n_lookups, int64_t n_bags, gt_src src, uint32_t E, int32_t T, const uint32_t* __restrict__ tb,
          uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint32_t* err, int ballot_only, hl_hook hk) {
  __shared__ uint32_t s_code[GT_WAVES][OH_UNIT];
  __shared__ uint32_t s_ticket[2];
  hl_hook_head(hk);
  const uint32_t first = CODES ? (uint32_t)T + GT_CHECKS : (uint32_t)T, nblk = gridDim.x - (uint32_t)T;
  uint32_t t = blockIdx.x, epoch = 0, bid = blockIdx.x - first;
  if (CODES && blockIdx.x < first) {
    if (threadIdx.x == 0) s_ticket[0] = hl_ticket(src.ticket, first, &s_ticket[1]);
    __syncthreads();
    if (s_ticket[0] >= first) {  // (hl_ticket)
      if (threadIdx.x == 0) hl_flag(err, HL_DEVERR_INTERNAL);
      return;
    }
    t = s_ticket[0] - GT_CHECKS;  // (a check: past every table)
    epoch = s_ticket[1];
    if (s_ticket[0] < GT_CHECKS) {
      gt_check_bags(s_ticket[0], src, (uint32_t)n_bags, epoch);
      bid = nblk - GT_CHECKS + s_ticket[0];  // (the last to pool: a small mini-batch takes few blocks)
    }
  }
  if (t < (uint32_t)T)
    gt_sort_body<ITEMS, CODES>(t, epoch, src, E, T, (uint32_t)n_bags, tb, n_hot, kout, vout, err, ballot_only);
  else
    eb_fwd_oh_body<VEC, BF, 0>(bid, nblk, w_hot, stg, stg_rows, n_hot, k_cap, codes, bag_ptr, out, g,
                               n_lookups, n_bags, err, s_code, 0, INT64_MAX, true);
}

// ----------------------------------------------------------------------------- backward
struct bw_ws {
  hl_sort_ws sort;
  uint8_t* mask;     // [max_bags]
  float* tfirst;     // [tiles][D]
  float* tlast;      // [tiles][D]
  uint32_t* tflag;   // [tiles]
  uint32_t* tkey;    // [tiles]
  float* gc;         // [n_max][D] gradient sums of staging rows, kept between the two halves of the apply
  uint32_t* bnd;     // [1] first sorted position whose key is not a hot slot (set by the first half)
  uint32_t tiles, gc_rows;
};

static uint32_t bw_tile_entries(int32_t D, int vec) {
  eb_geom g = eb_make_geom(D, vec);
  return (uint32_t)(RB_WAVES * g.NG * RB_EN(vec));
}

// compact: no staging-row sums (gc), for plans whose apply is whole (part 0), and
// the tiles' sums where the sort's counts were (the sort clears or writes all that
// it reads there, and is done with it when the apply starts)
static void bw_carve(hl_carver& c, bw_ws& ws, uint32_t n_max, int64_t max_bags, int32_t D, bool compact = false) {
  hl_sort_ws_carve_pairs(c, ws.sort, n_max);
  if (!compact) hl_sort_ws_carve_counts(c, ws.sort);
  ws.mask = c.take<uint8_t>((size_t)max_bags + 1);
  const size_t shared = c.off;
  if (compact) hl_sort_ws_carve_counts(c, ws.sort);
  const size_t counts_end = c.off;
  if (compact) c.off = shared;
  // the smallest tile (largest count) over the vector widths the call may pick
  uint32_t te = bw_tile_entries(D, 1);
  uint32_t te2 = bw_tile_entries(D, D % 2 == 0 ? 2 : 1), te4 = bw_tile_entries(D, D % 4 == 0 ? 4 : 1);
  te = te < te2 ? te : te2;
  te = te < te4 ? te : te4;
  ws.tiles = n_max ? hl_div_up(n_max, te) : 1;
  ws.tfirst = c.take<float>((size_t)ws.tiles * D);
  ws.tlast = c.take<float>((size_t)ws.tiles * D);
  ws.tflag = c.take<uint32_t>(ws.tiles);
  ws.tkey = c.take<uint32_t>(ws.tiles);
  ws.gc_rows = compact ? 0 : n_max;
  ws.gc = c.take<float>((size_t)ws.gc_rows * D);
  ws.bnd = c.take<uint32_t>(1);
  c.off = std::max(c.off, counts_end);
}

size_t hl_bwd_ws_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags) {
  hl_carver c = hl_carver::after_header(nullptr, 0);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)max_lookups, max_bags, h->dim);
  return c.off;
}

size_t hl_bwd_ws_bytes_compact(const hl_handle* h, int64_t max_lookups, int64_t max_bags) {
  hl_carver c = hl_carver::after_header(nullptr, 0);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)max_lookups, max_bags, h->dim, true);
  return c.off;
}

static size_t bw_bytes(const hl_handle* h, int64_t n, int64_t bags, bool compact) {
  return compact ? hl_bwd_ws_bytes_compact(h, n, bags) : hl_bwd_ws_bytes(h, n, bags);
}

__global__ void bw_mask(uint8_t* mask, int32_t n_samples, const int32_t* __restrict__ ids, const int32_t* n_dev,
                        int32_t n_max, int phase) {
  if (phase == 0) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_samples; i += gridDim.x * blockDim.x) mask[i] = 0;
  } else {
    const int32_t n = eb_nsel(ids, n_dev, n_max);
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
      const int32_t s = ids[i];
      if (s >= 0 && s < n_samples) mask[s] = 1;
    }
  }
}

// (compressed key, bag) for every lookup of the mini-batch; lookups of
// unselected samples and invalid codes get the sentinel key (sorted last,
// ignored), and so do positions outside [bag_ptr[0], bag_ptr[n_bags]) (only if
// bag_ptr disagrees with n_lookups; bag_ptr is non-decreasing).

// the lookup positions no bag covers: [0, bag_ptr[0]) and [bag_ptr[n_bags], n)
__device__ __forceinline__ void bw_uncovered(const int32_t* bag_ptr, int64_t n_bags, int64_t n_lookups,
                                             int64_t* first, int64_t* covered) {
  *first = min((int64_t)max(bag_ptr[0], 0), n_lookups);
  *covered = max(min((int64_t)max(bag_ptr[n_bags], 0), n_lookups), *first);
}


#define BP_BAGS 256
__global__ void __launch_bounds__(256)
bw_prep(const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr, int64_t n_bags, int32_t bps,
        const uint8_t* __restrict__ mask, uint32_t n_hot, uint32_t k_cap, int32_t stg_rows,
        uint32_t* __restrict__ keys, uint32_t* __restrict__ vals, int64_t n_lookups, uint32_t* sflag, uint32_t sv,
        uint32_t* err) {
  __shared__ int32_t off[BP_BAGS + 1];
  bw_start_signal(sflag, sv);
  const int64_t b0 = (int64_t)blockIdx.x * BP_BAGS;
  const int nb = (int)min((int64_t)BP_BAGS, n_bags - b0);
  for (int j = threadIdx.x; j <= nb; j += blockDim.x) off[j] = bag_ptr[b0 + j];
  if (blockIdx.x == 0 && threadIdx.x == 0 && bag_ptr[n_bags] != n_lookups) hl_flag(err, HL_DEVERR_SHAPE);
  __syncthreads();
  int64_t first, covered;
  bw_uncovered(bag_ptr, n_bags, n_lookups, &first, &covered);
  const int64_t gs = (int64_t)gridDim.x * blockDim.x, t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = t0; i < first; i += gs) keys[i] = EB_SENT;
  for (int64_t i = covered + t0; i < n_lookups; i += gs) keys[i] = EB_SENT;
  const int32_t lo = off[0], hi = min((int64_t)off[nb], n_lookups);
  for (int32_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
    int a = 0, b = nb;
    while (b - a > 1) {
      int m = (a + b) >> 1;
      if (off[m] <= i) a = m; else b = m;
    }
    const int64_t bag = b0 + a;
    uint32_t key = EB_SENT;
    if (mask[bag / bps]) {
      key = bw_key((uint32_t)codes[i], n_hot, k_cap, stg_rows);
      if (key == EB_SENT) hl_flag(err, HL_DEVERR_BAD_CODE);
    }
    keys[i] = key;
    vals[i] = (uint32_t)bag;
  }
}

template <int VEC, bool BF>
__device__ __forceinline__ typename RowIO<VEC, BF>::T* bw_row(void* w_hot, void* stg, uint32_t n_hot, int32_t D,
                                                             uint32_t key) {
  typedef typename RowIO<VEC, BF>::T T;
  return key < n_hot ? (T*)w_hot + (int64_t)key * D : (T*)stg + (int64_t)(key - n_hot) * D;
}

#define GF_F 1u
#define GF_W 2u
#define GF_L 4u

// SPLIT: the run of a staging row (key n_hot + u, u < gc_rows) stores its sum
// G in gc[u] instead of updating the row, and the row is not read; bw_cold
// applies it later (the staging rows may still be in flight then).
__device__ __forceinline__ bool bw_deferred(uint32_t key, uint32_t n_hot, uint32_t gc_rows) {
  return key >= n_hot && key != EB_SENT && key - n_hot < gc_rows;
}

template <int VEC, bool BF, bool SPLIT>
__global__ void __launch_bounds__(RB_BLOCK)
bw_reduce1(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint32_t n,
           const float* __restrict__ dY, eb_geom g, void* w_hot, void* stg, uint32_t n_hot, float lr,
           float* __restrict__ tfirst, float* __restrict__ tlast, uint32_t* __restrict__ tflag,
           uint32_t* __restrict__ tkey, float* __restrict__ gc, uint32_t gc_rows, uint32_t* __restrict__ bnd,
           hl_hook hk) {
  typedef typename RowIO<VEC, BF>::T T;
  constexpr int RB_E = RB_EN(VEC);
  __shared__ float pf[RB_WAVES * 64 * VEC], pl[RB_WAVES * 64 * VEC];
  hl_hook_head(hk);
  __shared__ uint32_t gflag[RB_WAVES * 64], gkey[RB_WAVES * 64];
  __shared__ uint32_t s_tflag;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  const bool gact = gi < g.NG;
  const int grp = w * g.NG + gi;           // group index inside the block
  const int ngb = RB_WAVES * g.NG;         // groups per block
  const uint32_t te = (uint32_t)ngb * RB_E;
  const uint32_t tile = blockIdx.x;
  const uint64_t tb = (uint64_t)tile * te;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = gact && colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  const int lds_off = (grp * g.G + gl) * VEC;
  if (threadIdx.x == 0) s_tflag = 0;
  if (gact) {
    const uint64_t e0 = tb + (uint64_t)grp * RB_E;
    uint32_t kk[RB_E], bb[RB_E];
#pragma unroll
    for (int j = 0; j < RB_E; ++j) {
      const uint64_t idx = e0 + j;
      kk[j] = idx < n ? keys[idx] : EB_SENT;
      bb[j] = idx < n ? vals[idx] : 0u;
    }
    const uint32_t prevk = (e0 > 0 && e0 - 1 < n) ? keys[e0 - 1] : EB_SENT;
    const uint32_t nextk = (e0 + RB_E < n) ? keys[e0 + RB_E] : EB_SENT;
    if (SPLIT && blockIdx.y == 0 && gl == 0) {
      // the one position where the hot slots end (keys are sorted; n if they never do)
#pragma unroll
      for (int j = 0; j < RB_E; ++j) {
        const uint64_t idx = e0 + j;
        const uint32_t kp = j == 0 ? (e0 > 0 ? prevk : 0u) : kk[j - 1];
        if (idx < n && kk[j] >= n_hot && (idx == 0 || kp < n_hot)) *bnd = (uint32_t)idx;
        if (idx + 1 == n && kk[j] < n_hot) *bnd = (uint32_t)n;
      }
    }
    const bool cprev = kk[0] != EB_SENT && prevk == kk[0];
    const bool cnext = kk[RB_E - 1] != EB_SENT && nextk == kk[RB_E - 1];
    // gradient rows
    float dv[RB_E][VEC];
#pragma unroll
    for (int j = 0; j < RB_E; ++j) {
      if (kk[j] != EB_SENT && cact) ld_f32<VEC>(dY + (int64_t)bb[j] * g.D + col, dv[j]);
      else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) dv[j][e] = 0.f;
      }
    }
    // rows of complete runs (issued before the sums are formed)
    typename RowIO<VEC, BF>::Raw wr[RB_E];
    bool cpl[RB_E];
    bool from0 = true;
#pragma unroll
    for (int j = 0; j < RB_E; ++j) {
      const bool valid = kk[j] != EB_SENT;
      if (j > 0 && valid && kk[j - 1] != kk[j]) from0 = false;
      const bool end = valid && (j == RB_E - 1 || kk[j + 1] != kk[j]);
      cpl[j] = end && !(from0 && cprev) && !(j == RB_E - 1 && cnext);
      if (cpl[j] && cact && !(SPLIT && bw_deferred(kk[j], n_hot, gc_rows)))
        wr[j] = RowIO<VEC, BF>::load_raw(bw_row<VEC, BF>(w_hot, stg, n_hot, g.D, kk[j]) + col);
    }
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    uint32_t gf = 0;
    from0 = true;
#pragma unroll
    for (int j = 0; j < RB_E; ++j) {
      const bool valid = kk[j] != EB_SENT;
      if (j > 0 && valid && kk[j - 1] != kk[j]) from0 = false;
      if (valid) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += dv[j][e];
      }
      const bool end = valid && (j == RB_E - 1 || kk[j + 1] != kk[j]);
      if (end) {
        if (cpl[j]) {
          if (cact) {
            if (SPLIT && bw_deferred(kk[j], n_hot, gc_rows)) {
              st_f32<VEC>(gc + (int64_t)(kk[j] - n_hot) * g.D + col, acc);
            } else {
              float wv[VEC], nw[VEC];
              RowIO<VEC, BF>::unpack(wr[j], wv);
#pragma unroll
              for (int e = 0; e < VEC; ++e) nw[e] = wv[e] - lr * acc[e];
              RowIO<VEC, BF>::store(bw_row<VEC, BF>(w_hot, stg, n_hot, g.D, kk[j]) + col, nw);
            }
          }
        } else {
          const bool first = from0 && cprev, lastp = (j == RB_E - 1) && cnext;
          if (first) {
            gf |= GF_F | (lastp ? GF_W | GF_L : 0u);
#pragma unroll
            for (int e = 0; e < VEC; ++e) pf[lds_off + e] = acc[e];
          } else if (lastp) {
            gf |= GF_L;
#pragma unroll
            for (int e = 0; e < VEC; ++e) pl[lds_off + e] = acc[e];
          }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
      }
    }
    if (gl == 0) {
      gflag[grp] = gf;
      gkey[grp] = kk[RB_E - 1];
    }
  }
  __syncthreads();
  if (gact) {
    const uint32_t gf = gflag[grp];
    // a segment that starts in this group and continues into the next ones
    if ((gf & GF_L) && !(gf & GF_W)) {
      float acc[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] = pl[lds_off + e];
      bool done = false;
      for (int g2 = grp + 1; g2 < ngb; ++g2) {
        const int o2 = (g2 * g.G + gl) * VEC;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += pf[o2 + e];
        if (!(gflag[g2] & GF_W)) { done = true; break; }
      }
      const uint32_t key = gkey[grp];
      if (done) {
        if (cact && SPLIT && bw_deferred(key, n_hot, gc_rows)) {
          st_f32<VEC>(gc + (int64_t)(key - n_hot) * g.D + col, acc);
        } else if (cact) {
          T* p = bw_row<VEC, BF>(w_hot, stg, n_hot, g.D, key) + col;
          float wv[VEC];
          RowIO<VEC, BF>::load(p, wv);
#pragma unroll
          for (int e = 0; e < VEC; ++e) wv[e] -= lr * acc[e];
          RowIO<VEC, BF>::store(p, wv);
        }
      } else {
        if (cact) st_f32<VEC>(tlast + (int64_t)tile * g.D + col, acc);
        if (gl == 0) {
          atomicOr(&s_tflag, GF_L);
          if (blockIdx.y == 0) tkey[tile] = key;
        }
      }
    }
    // the piece of a segment that began in an earlier tile
    if (grp == 0 && (gf & GF_F)) {
      float acc[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] = pf[lds_off + e];
      bool whole = (gf & GF_W) != 0;
      if (whole) {
        for (int g2 = 1; g2 < ngb; ++g2) {
          const int o2 = (g2 * g.G + gl) * VEC;
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[e] += pf[o2 + e];
          if (!(gflag[g2] & GF_W)) { whole = false; break; }
        }
      }
      if (cact) st_f32<VEC>(tfirst + (int64_t)tile * g.D + col, acc);
      if (gl == 0) atomicOr(&s_tflag, GF_F | (whole ? GF_W : 0u));
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && blockIdx.y == 0) tflag[tile] = s_tflag;
  hl_hook_tail(hk);
}

// Segments spanning tiles: the tile where a segment starts (flag L) sums its
// own piece and the next tiles' first pieces up to the first tile that is not
// wholly inside the segment.  Piece p is summed by group p % groups in
// ascending p, then groups are added in order (so a segment of at most `groups`
// pieces in plain ascending order).
//
// A segment by the whole block: its loads that need nothing but the tile index
// (its key and piece) are issued together, and the row with the pieces of the
// later tiles.  a: a tile inside the segment up to which all after t are; f2: the
// flag of tile a + 1 + this thread; s_end: n_tiles, in LDS, seen by every thread.
// Nothing is done for one of at most `most` pieces.  Every thread of the block
// calls it.
template <int VEC, bool BF, bool SPLIT>
__device__ __forceinline__ void bw_reduce2_long(uint32_t t, uint32_t a, uint32_t f2, uint32_t* s_end, uint32_t most,
                                                uint32_t n_tiles, eb_geom g, void* w_hot, void* stg,
                                                uint32_t n_hot, float lr, const float* __restrict__ tfirst,
                                                const float* __restrict__ tlast, const uint32_t* __restrict__ tflag,
                                                const uint32_t* __restrict__ tkey, float* __restrict__ gc,
                                                uint32_t gc_rows) {
  typedef typename RowIO<VEC, BF>::T T;
  __shared__ float part[RB_WAVES * 64 * VEC];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  const bool gact = gi < g.NG;
  const int grp = w * g.NG + gi, ngb = RB_WAVES * g.NG;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = gact && colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  const uint32_t key = tkey[t];
  float v0[VEC];  // piece 0 (this tile's), summed by group 0
#pragma unroll
  for (int e = 0; e < VEC; ++e) v0[e] = 0.f;
  if (grp == 0 && cact) ld_f32<VEC>(tlast + (int64_t)t * g.D + col, v0);
  // the first tile after t that is not wholly inside the segment holds its
  // last piece (a window of RB_BLOCK tiles, then of four times as many; one lane
  // of a wave lowers s_end, since an LDS atomic goes lane by lane)
  const uint32_t w64 = (uint32_t)w * 64;
  const uint64_t m2 = __ballot(!(f2 & GF_W));
  if (m2 && lane == 0) atomicMin(s_end, a + w64 + (uint32_t)__ffsll((unsigned long long)m2));
  __syncthreads();
  uint32_t tend = *s_end;
  // the row, for group 0 (its address needs only the key)
  const bool defer = SPLIT && bw_deferred(key, n_hot, gc_rows);
  typename RowIO<VEC, BF>::Raw wr;  // (unpacked when it is used)
  T* rp = bw_row<VEC, BF>(w_hot, stg, n_hot, g.D, key) + col;
  if (grp == 0 && cact && !defer) wr = RowIO<VEC, BF>::load_raw(rp);
  for (uint32_t base = a + 1 + RB_BLOCK; tend == n_tiles && base < n_tiles; base += 4 * RB_BLOCK) {
    __syncthreads();  // (every thread has read s_end before any lowers it)
    uint32_t f3[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t t3 = base + i * RB_BLOCK + threadIdx.x;  // (clamped, not skipped: loads in flight together)
      f3[i] = tflag[min(t3, n_tiles - 1)] | (t3 < n_tiles ? 0u : GF_W);
    }
    uint32_t end = n_tiles;
#pragma unroll
    for (int i = 3; i >= 0; --i) {
      const uint64_t m3 = __ballot(!(f3[i] & GF_W));
      if (m3) end = base + i * RB_BLOCK + w64 + (uint32_t)__ffsll((unsigned long long)m3) - 1;
    }
    if (end < n_tiles && lane == 0) atomicMin(s_end, end);
    __syncthreads();
    tend = *s_end;
  }
  const uint32_t npieces = (tend < n_tiles ? tend : n_tiles - 1) - t + 1;
  if (npieces <= most) return;  // (the same for every thread of the block)
  if (gact) {
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    if (grp == 0)
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += v0[e];
    if (cact) {
      // (four pieces in flight, added in ascending order)
      for (uint32_t p = grp == 0 ? ngb : grp; p < npieces; p += 4 * ngb) {
        float v[4][VEC];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (p + i * ngb < npieces) ld_f32<VEC>(tfirst + (int64_t)(t + p + i * ngb) * g.D + col, v[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (p + i * ngb < npieces)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] += v[i][e];
      }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) part[(grp * g.G + gl) * VEC + e] = acc[e];
  }
  __syncthreads();
  if (gact && grp == 0 && cact) {
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    for (int q = 0; q < ngb; ++q)
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += part[(q * g.G + gl) * VEC + e];
    if (defer) {
      st_f32<VEC>(gc + (int64_t)(key - n_hot) * g.D + col, acc);
      return;
    }
    float wv[VEC];
    RowIO<VEC, BF>::unpack(wr, wv);
#pragma unroll
    for (int e = 0; e < VEC; ++e) wv[e] -= lr * acc[e];
    RowIO<VEC, BF>::store(rp, wv);
  }
}

// Nearly every tile ends inside a segment, and nearly every segment ends in the
// next tile or soon after.  So a row group finishes a segment of up to R2_SHORT
// pieces by itself: its tile's flag, key and piece, the next tiles' flags and the
// next piece in one round of loads, the row and any further pieces in a second.
// A longer segment lies wholly over more than R2_SHORT - 2 tiles, so one of every
// R2_SHORT - 1 tiles is inside it: the launch's first blocks look at those tiles,
// and the one at the first such tile of a segment finds its start among the tiles
// before and takes it with the whole block.  Bound by latency: a block per tile,
// with three barriers before its store, took 7.5 us for 4,438 tiles and 13.4 for
// 17,750 (f32 rows of 64), 9.2 for 6,828 with a run over 150 of them (bf16 rows
// of 128); 5.4, 7.5 and 8.7 like this (the long ones one after another in the
// blocks that met them: 5.8, 8.2 and 10.4).  One row over 5,200 tiles (f32 rows of
// 64) 80.4 us with a block per tile, 83.5 with the search and one window of flags
// after another, 74.4 with the next flags loaded beside the search and four windows
// at a time after that; 328,000 lookups of Zipf 1.2 (bf16 rows of 128, one row over
// 1,200 tiles) 25.7, 26.8 and 24.6, and the 5.4 and 8.7 above 4.7 and 7.0.
#define R2_SHORT 8
// blocks that look for long segments, and all blocks, for n_tiles tiles (at
// least two row groups to a block: RB_WAVES)
__host__ __device__ __forceinline__ uint32_t bw_r2_longs(uint32_t n_tiles, const eb_geom& g) {
  const uint32_t ngb = RB_WAVES * (uint32_t)g.NG, most = ngb < R2_SHORT ? ngb : R2_SHORT;
  return n_tiles ? (n_tiles - 1) / (most - 1) : 0;
}
__host__ __device__ __forceinline__ uint32_t bw_r2_blocks(uint32_t n_tiles, const eb_geom& g) {
  const uint32_t ngb = RB_WAVES * (uint32_t)g.NG;
  return bw_r2_longs(n_tiles, g) + (n_tiles + ngb - 1) / ngb;
}
template <int VEC, bool BF, bool SPLIT>
__device__ __forceinline__ void bw_reduce2_body(uint32_t bid, uint32_t n_tiles, eb_geom g, void* w_hot, void* stg,
                                                uint32_t n_hot, float lr, const float* __restrict__ tfirst,
                                                const float* __restrict__ tlast, const uint32_t* __restrict__ tflag,
                                                const uint32_t* __restrict__ tkey, float* __restrict__ gc,
                                                uint32_t gc_rows) {
  typedef typename RowIO<VEC, BF>::T T;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  const int grp = w * g.NG + gi, ngb = RB_WAVES * g.NG;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = gi < g.NG && colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  const uint32_t most = ngb < R2_SHORT ? ngb : R2_SHORT;
  const uint32_t longs = bw_r2_longs(n_tiles, g);
  if (bid < longs) {
    const uint32_t step = most - 1, a = (bid + 1) * step;
    uint32_t fb[R2_SHORT];  // flags of tiles a, a - 1, ..., a - step
#pragma unroll
    for (int i = 0; i < R2_SHORT; ++i) fb[i] = tflag[a - min((uint32_t)i, step)];
    // (the next tiles' flags in the same round, for a segment that goes on)
    const uint32_t t2 = a + 1 + threadIdx.x;
    const uint32_t f2 = tflag[min(t2, n_tiles - 1)] | (t2 < n_tiles ? 0u : GF_W);
    __shared__ uint32_t s_end;
    if (threadIdx.x == 0) s_end = n_tiles;
    __syncthreads();
    if (!(fb[0] & GF_W)) return;
    uint32_t back = 0;  // the segment's start, if no earlier looked-at tile is inside it
#pragma unroll
    for (int i = R2_SHORT - 1; i > 0; --i)
      if (i <= (int)step && !(fb[i] & GF_W)) back = i;
    if (back != 0)
      bw_reduce2_long<VEC, BF, SPLIT>(a - back, a, f2, &s_end, most, n_tiles, g, w_hot, stg, n_hot, lr, tfirst, tlast, tflag, tkey, gc,
                                      gc_rows);
    return;
  }
  const uint32_t t = (bid - longs) * (uint32_t)ngb + grp;
  const bool in = gi < g.NG && t + 1 < n_tiles;  // (no segment starts in the last tile and goes on)
  uint32_t f = 0, key = 0, nf[R2_SHORT - 1];
  float acc[VEC], v1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    acc[e] = 0.f;
    v1[e] = 0.f;
  }
  if (in) {
    f = tflag[t];
    key = tkey[t];
#pragma unroll
    for (int i = 0; i < R2_SHORT - 1; ++i) nf[i] = tflag[min(t + 1 + i, n_tiles - 1)];
    if (cact) {
      ld_f32<VEC>(tlast + (int64_t)t * g.D + col, acc);
      ld_f32<VEC>(tfirst + (int64_t)(t + 1) * g.D + col, v1);
    }
  }
  if (in && (f & GF_L)) {
    // pieces: this tile's and those up to the first tile not wholly inside
    uint32_t np = 0;
#pragma unroll
    for (int i = R2_SHORT - 2; i >= 0; --i)
      if (!(nf[i] & GF_W) || t + 1 + i == n_tiles - 1) np = i + 2;
    if (np != 0 && np <= most && cact) {
      const bool defer = SPLIT && bw_deferred(key, n_hot, gc_rows);
      T* rp = bw_row<VEC, BF>(w_hot, stg, n_hot, g.D, key) + col;
      float wv[VEC];
      if (!defer) RowIO<VEC, BF>::load(rp, wv);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] = 0.f + acc[e];
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += v1[e];
      for (uint32_t p = 2; p < np; ++p) {
        float v[VEC];
        ld_f32<VEC>(tfirst + (int64_t)(t + p) * g.D + col, v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += v[e];
      }
      if (defer) {
        st_f32<VEC>(gc + (int64_t)(key - n_hot) * g.D + col, acc);
      } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) wv[e] -= lr * acc[e];
        RowIO<VEC, BF>::store(rp, wv);
      }
    }
  }
}

template <int VEC, bool BF, bool SPLIT>
__global__ void __launch_bounds__(RB_BLOCK)
bw_reduce2(uint32_t n_tiles, eb_geom g, void* w_hot, void* stg, uint32_t n_hot, float lr,
           const float* __restrict__ tfirst, const float* __restrict__ tlast, const uint32_t* __restrict__ tflag,
           const uint32_t* __restrict__ tkey, float* __restrict__ gc, uint32_t gc_rows) {
  bw_reduce2_body<VEC, BF, SPLIT>(blockIdx.x, n_tiles, g, w_hot, stg, n_hot, lr, tfirst, tlast, tflag, tkey, gc,
                                  gc_rows);
}

// The deferred staging-row updates: every run end in the sorted keys whose key
// is a staging row below gc_rows applies row <- round(row - lr * gc[u]), the
// same arithmetic as the one-pass update.  Only the sorted tail from *bnd (the
// end of the hot slots, found by the first half) is scanned.  A wave tests
// CW_POS positions at a time (one per lane), then its row groups take the run
// ends found, each group its share at once (at most CW_POS / NG rows per
// group, all loads in flight together), so a wave's positions cost one round
// of row loads.
#define CW_POS 16
template <int VEC, bool BF>
__global__ void __launch_bounds__(256)
bw_cold(const uint32_t* __restrict__ keys, uint32_t n, eb_geom g, void* stg, uint32_t n_hot, float lr,
        const float* __restrict__ gc, uint32_t gc_rows, const uint32_t* __restrict__ bnd, hl_hook hk) {
  typedef typename RowIO<VEC, BF>::T T;
  hl_hook_head(hk);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = gi < g.NG && colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  const uint32_t b0 = min(*bnd, n);
  constexpr int RPG = CW_POS / 4 > 0 ? CW_POS / 4 : 1;  // rows per group for groups of 16 lanes or wider
  for (uint64_t base = b0 + ((uint64_t)blockIdx.x * 4 + w) * CW_POS; base < n;
       base += (uint64_t)gridDim.x * 4 * CW_POS) {
    const uint64_t p = base + lane;
    const bool in = lane < CW_POS && p < n;
    const uint32_t k = in ? keys[p] : EB_SENT;
    const uint32_t kn = in && p + 1 < n ? keys[p + 1] : EB_SENT;
    uint64_t m = __ballot(in && k != kn && bw_deferred(k, n_hot, gc_rows));
    while (m) {
      // run end gi + NG j of the remaining ones goes to group gi
      uint64_t mm = m;
      for (int q = 0; q < gi; ++q) mm &= mm - 1;
      int src[RPG];
      bool has[RPG];
#pragma unroll
      for (int j = 0; j < RPG; ++j) {
        has[j] = mm != 0;
        src[j] = has[j] ? __ffsll((unsigned long long)mm) - 1 : 0;
        for (int q = 0; q < g.NG && mm; ++q) mm &= mm - 1;
      }
      int64_t u[RPG];
      float wv[RPG][VEC], gv[RPG][VEC];
#pragma unroll
      for (int j = 0; j < RPG; ++j) {
        u[j] = (int64_t)__shfl(k, src[j]) - n_hot;
        if (has[j] && cact) {
          RowIO<VEC, BF>::load((T*)stg + u[j] * g.D + col, wv[j]);
          ld_f32<VEC>(gc + u[j] * g.D + col, gv[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < RPG; ++j)
        if (has[j] && cact) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) wv[j][e] = wv[j][e] - lr * gv[j][e];
          RowIO<VEC, BF>::store((T*)stg + u[j] * g.D + col, wv[j]);
        }
      for (int q = 0; q < RPG * g.NG && m; ++q) m &= m - 1;
    }
  }
  hl_hook_tail(hk);
}

// The cold half of the forward from the backward's grouping: the sorted tail
// from *bnd holds a (staging key, bag) pair for every cold lookup.  A bag is
// completed by the pair of its first cold lookup in CSR order (the first copy
// of that pair): out[bag] += its staging rows in CSR order, the same sums as
// the forward's cold half over the non-popular mu-batch.  A group of lanes
// takes FT pairs at once.
#define FT 4
// (block bid of nblk, WAVES waves per block)
template <int VEC, bool BF, int WAVES>
__device__ __forceinline__ void eb_tail_body(uint32_t bid, uint32_t nblk, const uint32_t* __restrict__ keys,
                                             const uint32_t* __restrict__ vals, uint32_t n,
                                             const uint32_t* __restrict__ bnd, eb_geom g, const void* stg_,
                                             int32_t stg_rows, uint32_t n_hot, uint32_t k_cap,
                                             const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr,
                                             float* __restrict__ out, uint32_t* err) {
  typedef typename RowIO<VEC, BF>::T T;
  const T* stg = (const T*)stg_;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  if (gi >= g.NG) return;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  const uint32_t b0 = min(*bnd, n);
  const uint64_t stride = (uint64_t)nblk * WAVES * g.NG * FT;
  for (uint64_t p0 = b0 + ((uint64_t)(bid * WAVES + w) * g.NG + gi) * FT; p0 < n; p0 += stride) {
    uint32_t key[FT], bag[FT];
    bool take[FT];
#pragma unroll
    for (int j = 0; j < FT; ++j) {
      const uint64_t p = p0 + j;
      key[j] = p < n ? keys[p] : EB_SENT;
      bag[j] = p < n ? vals[p] : 0u;
      const uint32_t kp = p > b0 && p < n ? keys[p - 1] : EB_SENT;
      const uint32_t bp = p > b0 && p < n ? vals[p - 1] : 0u;
      take[j] = key[j] != EB_SENT && key[j] >= n_hot && key[j] - n_hot < (uint32_t)stg_rows &&
                !(kp == key[j] && bp == bag[j]);
    }
    int32_t lo[FT], hi[FT];
#pragma unroll
    for (int j = 0; j < FT; ++j) {
      lo[j] = take[j] ? bag_ptr[bag[j]] : 0;
      hi[j] = take[j] ? bag_ptr[bag[j] + 1] : 0;
    }
#pragma unroll
    for (int j = 0; j < FT; ++j) {
      if (!take[j]) continue;
      const uint32_t u = key[j] - n_hot;
      if (hi[j] - lo[j] != 1) {
        // the bag's first cold lookup in CSR order names the pair that completes
        // it (row groups of 8 lanes or more search G codes at a time: a code
        // per lane, the first cold one by a ballot)
        bool mine = false;
        if (g.G >= EB_SEG_ROWS) {
          const int g0 = lane - gl;
          const uint64_t gm = g.G == 64 ? ~0ull : ((1ull << g.G) - 1ull);
          for (int32_t b0 = lo[j]; b0 < hi[j]; b0 += g.G) {
            const int32_t i = b0 + gl;
            const uint32_t c = i < hi[j] ? (uint32_t)codes[i] : ~0u;
            const bool cold = i < hi[j] && c >= k_cap && c - k_cap < (uint32_t)stg_rows;
            const uint64_t m = (__ballot(cold) >> g0) & gm;
            if (m) {
              const uint32_t cf = (uint32_t)__shfl((int)c, g0 + __ffsll((unsigned long long)m) - 1);
              mine = cf - k_cap == u;
              break;
            }
          }
        } else {
          for (int32_t i = lo[j]; i < hi[j]; ++i) {
            const uint32_t c = (uint32_t)codes[i];
            if (c >= k_cap && c - k_cap < (uint32_t)stg_rows) {
              mine = c - k_cap == u;
              break;
            }
          }
        }
        if (!mine) take[j] = false;
      }
    }
    float o[FT][VEC], v[FT][VEC];
#pragma unroll
    for (int j = 0; j < FT; ++j)
      if (take[j] && cact) {
        ld_f32<VEC>(out + (int64_t)bag[j] * g.D + col, o[j]);
        if (hi[j] - lo[j] == 1) RowIO<VEC, BF>::load(stg + (int64_t)(key[j] - n_hot) * g.D + col, v[j]);
      }
#pragma unroll
    for (int j = 0; j < FT; ++j) {
      if (!take[j]) continue;
      if (hi[j] - lo[j] == 1) {
        if (cact) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[j][e] += v[j][e];
        }
      } else {
        // the staging rows' sum, onto the stored hot sum (as PART 2 of the forward adds it)
        float c[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) c[e] = 0.f;
        bool anyc = false;
        eb_pass<VEC, BF, true>(c, nullptr, stg, stg_rows, n_hot, k_cap, codes, lo[j], hi[j], g, col, cact, gl, err,
                               &anyc);
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[j][e] += c[e];
      }
      if (cact) st_f32<VEC>(out + (int64_t)bag[j] * g.D + col, o[j]);
    }
  }
}

template <int VEC, bool BF>
__global__ void __launch_bounds__(256)
eb_fwd_tail(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint32_t n,
            const uint32_t* __restrict__ bnd, eb_geom g, const void* stg_, int32_t stg_rows, uint32_t n_hot,
            uint32_t k_cap, const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr,
            float* __restrict__ out, uint32_t* err) {
  eb_tail_body<VEC, BF, 4>(blockIdx.x, gridDim.x, keys, vals, n, bnd, g, stg_, stg_rows, n_hot, k_cap, codes, bag_ptr,
                           out, err);
}

// The cold half of the forward and the backward's segments that span tiles
// (bw_reduce2, split form) in one launch: the first blocks take the
// segments, the others the sorted tail.  They share no data (the segments
// write hot rows and staging-row sums, the tail reads staging rows and
// writes pooled outputs).
template <int VEC, bool BF>
__global__ void __launch_bounds__(RB_BLOCK)
eb_tail_r2(uint32_t n_tiles, void* w_hot, uint32_t n_hot, float lr, const float* __restrict__ tfirst,
           const float* __restrict__ tlast, const uint32_t* __restrict__ tflag, const uint32_t* __restrict__ tkey,
           float* __restrict__ gc, uint32_t gc_rows, const uint32_t* __restrict__ keys,
           const uint32_t* __restrict__ vals, uint32_t n, const uint32_t* __restrict__ bnd, eb_geom g, void* stg,
           int32_t stg_rows, uint32_t k_cap, const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr,
           float* __restrict__ out, uint32_t* err) {
  const uint32_t r2 = bw_r2_blocks(n_tiles, g);
  if (blockIdx.x < r2) {
    bw_reduce2_body<VEC, BF, true>(blockIdx.x, n_tiles, g, w_hot, stg, n_hot, lr, tfirst, tlast, tflag, tkey, gc,
                                   gc_rows);
    return;
  }
  eb_tail_body<VEC, BF, RB_WAVES>(blockIdx.x - r2, gridDim.x - r2, keys, vals, n, bnd, g, stg, stg_rows,
                                  n_hot, k_cap, codes, bag_ptr, out, err);
}

// The same launch for bags of several lookups (multi-hot), where nearly every
// bag holds a staging row: the cold half of the forward bag by bag (part 2 of
// the forward over every bag, one bag per row group) in place of the sorted
// tail.
template <int VEC, bool BF>
__global__ void __launch_bounds__(RB_BLOCK)
eb_bags_r2(uint32_t n_tiles, void* w_hot, uint32_t n_hot, float lr, const float* __restrict__ tfirst,
           const float* __restrict__ tlast, const uint32_t* __restrict__ tflag, const uint32_t* __restrict__ tkey,
           float* __restrict__ gc, uint32_t gc_rows, eb_geom g, void* stg, int32_t stg_rows, uint32_t k_cap,
           const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr, int32_t bps, int32_t n_samples,
           float* __restrict__ out, uint32_t* err) {
  const uint32_t r2 = bw_r2_blocks(n_tiles, g);
  if (blockIdx.x < r2) {
    bw_reduce2_body<VEC, BF, true>(blockIdx.x, n_tiles, g, w_hot, stg, n_hot, lr, tfirst, tlast, tflag, tkey, gc,
                                   gc_rows);
    return;
  }
  eb_fwd_body<VEC, BF, 2>(blockIdx.x - r2, gridDim.x - r2, w_hot, stg, stg_rows, n_hot, k_cap, codes,
                          bag_ptr, bps, nullptr, nullptr, n_samples, out, g, n_samples, 1, err);
}

// ----------------------------------------------------------------------------- host side
static hl_status check_common(const hl_handle* h, const int32_t* codes, const int32_t* bag_ptr, int32_t n_samples,
                              int32_t bps, int64_t n_lookups, const int32_t* sample_ids, int32_t n_sel_max,
                              int32_t stg_rows) {
  if (!h || n_samples < 0 || bps < 1 || n_lookups < 0 || n_sel_max < 0 || stg_rows < 0) return HL_ERR_INVALID_ARG;
  if (!bag_ptr || (n_lookups > 0 && !codes)) return HL_ERR_INVALID_ARG;
  if (!sample_ids && n_sel_max > n_samples) return HL_ERR_INVALID_ARG;
  if ((int64_t)n_samples * bps >= (1ll << 31) || n_lookups >= (1ll << 30)) return HL_ERR_UNSUPPORTED;
  if ((uint64_t)h->k_cap + (uint64_t)stg_rows >= (1ull << 31)) return HL_ERR_UNSUPPORTED;
  return HL_OK;
}

template <int VEC, bool BF>
static void launch_fwd(const hl_handle* h, dim3 grid, hipStream_t s, const void* w_hot, const void* stg,
                       int32_t stg_rows, const int32_t* codes, const int32_t* bag_ptr, int32_t bps,
                       const int32_t* ids, const int32_t* n_dev, int32_t n_max, float* out, eb_geom g,
                       int64_t n_lookups, int64_t n_bags, int part, int32_t nbg) {
  const hl_hook hk = hl_hook_take(h);
#define EBF(P)                                                                                                   \
  HL_KERNEL(h, s, P == 0 ? "eb_fwd" : (P == 1 ? "eb_fwd_hot" : "eb_fwd_cold"), (eb_fwd<VEC, BF, P>), grid,       \
            dim3(256), 0, s, w_hot, stg, stg_rows, h->n_hot, h->k_cap, codes, bag_ptr, bps, ids, n_dev, n_max, out, \
            g, n_lookups, n_bags, (int32_t)(n_bags / bps), nbg, h->d_err, hk);
  if (part == 0) { EBF(0) }
  else if (part == 1) { EBF(1) }
  else { EBF(2) }
#undef EBF
}

// grid of the one-hot forward: about 8 resident blocks per compute unit, each
// row group taking several chunks in turn
#define EB_OH_BLOCKS 1024
template <int VEC, bool BF>
static void launch_fwd_oh(const hl_handle* h, hipStream_t s, const void* w_hot, const void* stg, int32_t stg_rows,
                          const int32_t* codes, const int32_t* bag_ptr, float* out, eb_geom g, int64_t n_lookups,
                          int64_t n_bags, int part) {
  const hl_hook hk = hl_hook_take(h);
  const int64_t chunks = (n_bags + FC - 1) / FC;
  int64_t blocks = (chunks + 4 * g.NG - 1) / (4 * g.NG);
  if (blocks > EB_OH_BLOCKS) blocks = EB_OH_BLOCKS;
  const dim3 grid((uint32_t)blocks, g.cchunks);
  if (part == 0)
    HL_KERNEL(h, s, "eb_fwd", (eb_fwd_oh<VEC, BF, 0>), grid, dim3(256), 0, s, w_hot, stg, stg_rows, h->n_hot,
              h->k_cap, codes, bag_ptr, out, g, n_lookups, n_bags, h->d_err, hk);
  else
    HL_KERNEL(h, s, "eb_fwd_hot", (eb_fwd_oh<VEC, BF, 1>), grid, dim3(256), 0, s, w_hot, stg, stg_rows, h->n_hot,
              h->k_cap, codes, bag_ptr, out, g, n_lookups, n_bags, h->d_err, hk);
}

extern "C" hl_status hl_embbag_fwd_part(const hl_handle* h, const void* w_hot, const void* staging, int32_t stg_rows,
                                        const int32_t* codes, const int32_t* bag_ptr, int32_t n_samples, int32_t bps,
                                        int64_t n_lookups, const int32_t* sample_ids, const int32_t* n_sel_dev,
                                        int32_t n_sel_max, float* out, int32_t part, hl_stream stream) {
  hl_status st = check_common(h, codes, bag_ptr, n_samples, bps, n_lookups, sample_ids, n_sel_max, stg_rows);
  if (st != HL_OK) return st;
  if (part < 0 || part > 2) return HL_ERR_INVALID_ARG;
  if (n_sel_max == 0) return HL_OK;
  if (!out || (h->n_hot && !w_hot) || (stg_rows && !staging)) return HL_ERR_INVALID_ARG;
  const size_t es = h->dtype == HL_F32 ? 4 : 2;
  const int vec = eb_pick_vec(h->dim, es, {w_hot, staging, out});
  eb_geom g = eb_make_geom(h->dim, vec);
  const int64_t nb = (int64_t)n_samples * bps;
  const int32_t nbg = eb_bags_per_group(n_lookups, nb);
  const int64_t chunks = ((int64_t)n_sel_max * bps + nbg - 1) / nbg;
  int64_t blocks = (chunks + 4 * g.NG - 1) / (4 * g.NG);
  if (blocks > (1 << 20)) blocks = 1 << 20;
  dim3 grid((uint32_t)blocks, g.cchunks);
  hipStream_t s = (hipStream_t)stream;
  const bool bf = h->dtype == HL_BF16;
  if (part != 2 && !sample_ids && n_sel_max == n_samples && n_lookups == nb) {
    // every sample of a one-hot mini-batch
#define FOH(V, B) launch_fwd_oh<V, B>(h, s, w_hot, staging, stg_rows, codes, bag_ptr, out, g, n_lookups, nb, part)
    if (vec == 8) FOH(8, true);  // (bf16 only)
    else if (vec == 4) { if (bf) FOH(4, true); else FOH(4, false); }
    else if (vec == 2) { if (bf) FOH(2, true); else FOH(2, false); }
    else { if (bf) FOH(1, true); else FOH(1, false); }
#undef FOH
    HL_LAUNCHED();
    return HL_OK;
  }
#define FWD(V, B) launch_fwd<V, B>(h, grid, s, w_hot, staging, stg_rows, codes, bag_ptr, bps, sample_ids, n_sel_dev, \
                                   n_sel_max, out, g, n_lookups, nb, part, nbg)
  if (vec == 8) FWD(8, true);  // (bf16 only)
  else if (vec == 4) { if (bf) FWD(4, true); else FWD(4, false); }
  else if (vec == 2) { if (bf) FWD(2, true); else FWD(2, false); }
  else { if (bf) FWD(1, true); else FWD(1, false); }
#undef FWD
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_embbag_fwd(const hl_handle* h, const void* w_hot, const void* staging, int32_t stg_rows,
                                   const int32_t* codes, const int32_t* bag_ptr, int32_t n_samples, int32_t bps,
                                   int64_t n_lookups, const int32_t* sample_ids, const int32_t* n_sel_dev,
                                   int32_t n_sel_max, float* out, hl_stream stream) {
  return hl_embbag_fwd_part(h, w_hot, staging, stg_rows, codes, bag_ptr, n_samples, bps, n_lookups, sample_ids,
                            n_sel_dev, n_sel_max, out, 0, stream);
}

// Keys are compressed codes: hot slot, or n_hot + staging row.
static int bw_key_bits(const hl_handle* h, int32_t stg_rows) {
  return hl_bit_width((uint64_t)h->n_hot + (uint64_t)stg_rows);
}

// the general sort's source: the mini-batch's slot codes
static hl_sort_src bw_sort_src(const hl_handle* h, int32_t stg_rows, int32_t* codes, const int32_t* bag_ptr,
                               int64_t n_bags) {
  hl_sort_src src{};
  src.codes = codes;
  src.bag_ptr = bag_ptr;
  src.n_bags = n_bags;
  src.n_hot = h->n_hot;
  src.k_cap = h->k_cap;
  src.stg_rows = stg_rows;
  return src;
}

template <int VEC, bool BF>
static void launch_bwd(const hl_handle* h, uint32_t tiles, hipStream_t s, const uint32_t* sk, const uint32_t* sv,
                       uint32_t n, const float* dY, eb_geom g, void* w_hot, void* stg, uint32_t n_hot, float lr,
                       bw_ws& ws, int part) {
  const dim3 grid(tiles, g.cchunks), grid2(bw_r2_blocks(tiles, g), g.cchunks);
  if (part == 0) {
    HL_KERNEL(h, s, "bw_reduce1", (bw_reduce1<VEC, BF, false>), grid, dim3(RB_BLOCK), 0, s, sk, sv, n, dY, g,
              w_hot, stg, n_hot, lr, ws.tfirst, ws.tlast, ws.tflag, ws.tkey, ws.gc, ws.gc_rows, ws.bnd, hl_hook{});
    HL_KERNEL(h, s, "bw_reduce2", (bw_reduce2<VEC, BF, false>), grid2, dim3(RB_BLOCK), 0, s, tiles, g, w_hot, stg,
              n_hot, lr, ws.tfirst, ws.tlast, ws.tflag, ws.tkey, ws.gc, ws.gc_rows);
  } else if (part == 1 || part == 3) {
    HL_KERNEL(h, s, "bw_reduce1", (bw_reduce1<VEC, BF, true>), grid, dim3(RB_BLOCK), 0, s, sk, sv, n, dY, g,
              w_hot, stg, n_hot, lr, ws.tfirst, ws.tlast, ws.tflag, ws.tkey, ws.gc, ws.gc_rows, ws.bnd,
              part == 3 ? hl_hook_take(h) : hl_hook{});
    if (part == 1)
      HL_KERNEL(h, s, "bw_reduce2", (bw_reduce2<VEC, BF, true>), grid2, dim3(RB_BLOCK), 0, s, tiles, g, w_hot, stg,
                n_hot, lr, ws.tfirst, ws.tlast, ws.tflag, ws.tkey, ws.gc, ws.gc_rows);
  } else {
    // the tail (cold lookups: about a tenth of a mini-batch here) is a part of
    // n the device knows; a grid of a few thousand waves strides over it
    uint32_t b = hl_div_up(n, 4 * CW_POS);
    if (b > 1024) b = 1024;
    HL_KERNEL(h, s, "bw_cold", (bw_cold<VEC, BF>), dim3(b, g.cchunks), dim3(256), 0, s, sk, n, g, stg, n_hot, lr,
              ws.gc, ws.gc_rows, ws.bnd, hl_hook{});
  }
}

extern "C" hl_status hl_embbag_bwd_plan(hl_handle* h, int32_t stg_rows, const int32_t* codes, const int32_t* bag_ptr,
                                        int32_t n_samples, int32_t bps, int64_t n_lookups, const int32_t* sample_ids,
                                        const int32_t* n_sel_dev, int32_t n_sel_max, void* workspace, size_t ws_bytes,
                                        hl_stream stream) {
  bool sent = false;
  return hl_embbag_bwd_plan_signal(h, stg_rows, const_cast<int32_t*>(codes), bag_ptr, n_samples, bps, n_lookups,
                                   sample_ids, n_sel_dev, n_sel_max, workspace, ws_bytes, stream, nullptr, 0, &sent,
                                   nullptr);
}

hl_status hl_embbag_bwd_plan_signal(hl_handle* h, int32_t stg_rows, int32_t* codes, const int32_t* bag_ptr,
                                    int32_t n_samples, int32_t bps, int64_t n_lookups, const int32_t* sample_ids,
                                    const int32_t* n_sel_dev, int32_t n_sel_max, void* workspace, size_t ws_bytes,
                                    hl_stream stream, uint32_t* sflag, uint32_t sval, bool* sent,
                                    const hl_cg_fused* cf, bool compact) {
  *sent = false;
  if (compact && cf && cf->table) return HL_ERR_INVALID_ARG;  // the fused plan's state follows the full layout
  if (cf && cf->table && sample_ids) return HL_ERR_INVALID_ARG;  // the fused plan selects every sample
  hl_status st = check_common(h, codes, bag_ptr, n_samples, bps, n_lookups, sample_ids, n_sel_max, stg_rows);
  if (st != HL_OK) return st;
  if (!workspace) return HL_ERR_INVALID_ARG;
  const int64_t n_bags = (int64_t)n_samples * bps;
  if (ws_bytes < bw_bytes(h, n_lookups, n_bags, compact)) return HL_ERR_CAPACITY;
  hl_ws_note(h, workspace, HL_WSK_OTHER);
  if (n_samples == 0 || n_lookups == 0 || n_sel_max == 0) {
    hl_ws_note(h, workspace, HL_WSK_BWD_PLAN, 0, n_bags, stg_rows);
    hl_ws_find(h, workspace)->compact = compact;
    return HL_OK;
  }
  hipStream_t s = (hipStream_t)stream;
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)n_lookups, n_bags, h->dim, compact);
  const uint8_t* mask = nullptr;
  if (sample_ids) {
    uint32_t gb = hl_div_up(n_samples, 256);
    if (gb > 4096) gb = 4096;
    HL_KERNEL(h, s, "bw_mask", bw_mask, dim3(gb), dim3(256), 0, s, ws.mask, n_samples, sample_ids, n_sel_dev, n_sel_max, 0);
    HL_KERNEL(h, s, "bw_mask", bw_mask, dim3(gb), dim3(256), 0, s, ws.mask, n_samples, sample_ids, n_sel_dev, n_sel_max, 1);
    mask = ws.mask;
  }
  uint32_t *sk, *sv;
  const int bits = bw_key_bits(h, stg_rows);
  if (mask) {
    HL_KERNEL(h, s, "bw_prep", bw_prep, dim3(hl_div_up(n_bags, BP_BAGS)), dim3(256), 0, s, codes, bag_ptr, n_bags,
              bps, mask, h->n_hot, h->k_cap, stg_rows, ws.sort.k0, ws.sort.v0, n_lookups, sflag, sval, h->d_err);
    HL_LAUNCHED();
    *sent = sflag != nullptr;
    st = hl_sort_pairs(h, ws.sort, nullptr, (uint32_t)n_lookups, bits, s, &sk, &sv);
  } else if (hl_group_by_table_ok(h, n_lookups, n_bags)) {
    // one lookup per bag: grouped table by table (hl_group.hip), into the
    // buffers where the sort leaves its result; the others hold the
    // table-major pairs
    if ((uint64_t)n_lookups > ws.sort.n_max) return HL_ERR_CAPACITY;
    uint32_t *rk, *rv;
    hl_sort_result(ws.sort, bits, &rk, &rv);
    uint32_t* tk = rk == ws.sort.k0 ? ws.sort.k1 : ws.sort.k0;
    uint32_t* tv = rv == ws.sort.v0 ? ws.sort.v1 : ws.sort.v0;
    st = hl_group_by_table(h, codes, bag_ptr, n_bags, stg_rows, tk, tv, rk, rv, sflag, sval,
                           cf && cf->table ? cf : nullptr, s);
    *sent = sflag != nullptr;
  } else {
    hl_sort_src src = bw_sort_src(h, stg_rows, codes, bag_ptr, n_bags);
    src.sflag = sflag;
    src.sv = sval;
    if (cf) src.cf = *cf;
    st = hl_sort_codes(h, ws.sort, src, (uint32_t)n_lookups, bits, s, &sk, &sv);
    *sent = st == HL_OK && sflag != nullptr;
  }
  if (st != HL_OK) return st;
  hl_ws_note(h, workspace, HL_WSK_BWD_PLAN, n_lookups, n_bags, stg_rows);
  hl_ws_find(h, workspace)->compact = compact;
  return HL_OK;
}

hl_sort_side_fn hl_fwd_sort_f32();
hl_sort_side_fn hl_fwd_sort_bf16();
hl_sort_side_fn hl_fwd_sort_side(bool bf16, int vec) {
  if (bf16) return vec == 8 ? hl_fwd_sort_bf16() : nullptr;
  return vec == 4 ? hl_fwd_sort_f32() : nullptr;
}

// Lookups per table up to which the sorts beside the forward read the codes
// themselves, which spares gt_prep's launch.  A lane's code lies T codes from its
// neighbour's, from 32 tables on in a cache line of its own, and a compute unit
// takes one line a cycle; but the line lies where the sort goes from 4 to 8 items
// per thread and its registers no longer fit (with 8, 62 spilled at any number of
// tables; gt_prep's keys need no spills).  Back to back, gt_prep and the launch, then the
// launch alone, at 4096 lookups per table of 2, 8, 26 and 64 tables: rows of 16
// 15.4, 15.7, 17.5, 19.9 us and 13.7, 14.0, 14.6, 16.2; rows of 64 15.4, 16.2, 17.9,
// 29.3 and 13.7, 14.5, 15.2, 23.5.  At 8192 of 1, 8, 26 and 64 tables, rows of 16:
// 21.1, 21.9, 23.5, 26.3 and 24.5, 26.9, 29.8, 37.2 (6000: 19.6, 20.1, 21.8, 24.5 and
// 23.0, 24.7, 26.7, 31.0).
#define GT_CODES_E 4096
template <int VEC, bool BF>
static void launch_fwd_gt(hl_handle* h, hipStream_t s, const void* w_hot, const void* stg, int32_t stg_rows,
                          const int32_t* codes, const int32_t* bag_ptr, float* out, eb_geom g, int64_t n_lookups,
                          int64_t n_bags, void* workspace, uint32_t* k_tm, uint32_t* cum, uint32_t* kout,
                          uint32_t* vout) {
  const int32_t T = h->n_tables;
  const uint32_t E = (uint32_t)(n_bags / T);
  // one block per compute unit (each holds the sort's LDS): the tables' sorts
  // and, on the other units, the forward
  const int cus = hl_device_cus(h);
  const uint32_t nf = (uint32_t)std::max(cus > 2 * T ? cus - T : cus, GT_CHECKS);
  const hl_hook hk = hl_hook_take(h);
  gt_src src{};
  if (E <= GT_CODES_E) {
    src.codes = codes;
    src.bag_ptr = bag_ptr;
    src.k_cap = h->k_cap;
    src.stg_rows = stg_rows;
    src.ticket = (uint32_t*)workspace + HL_HDR_GT;
    src.bad = (uint64_t*)((uint32_t*)workspace + HL_HDR_GBAD);
    src.st = (uint64_t*)((uint32_t*)workspace + HL_HDR_GSTAT);
  } else {
    src.keys_tm = k_tm;
    src.cum = cum;
    src.nblk = hl_group_prep(h, const_cast<int32_t*>(codes), bag_ptr, n_bags, stg_rows, k_tm, cum, nullptr, 0, nullptr, s);
  }
#define FGT(I, C)                                                                                                 \
  HL_KERNEL(h, s, "eb_fwd_gt", (eb_fwd_gt<VEC, BF, I, C>), dim3(T + nf), dim3(GT_THREADS), 0, s, w_hot, stg, stg_rows, \
            h->n_hot, h->k_cap, codes, bag_ptr, out, g, n_lookups, n_bags, src, E, T, h->d_tb, kout, vout, h->d_err, \
            h->ballot_ranks, hk)
  static_assert(GT_CODES_E == 4 * GT_THREADS, "items per thread");
  if (E <= GT_THREADS) FGT(1, true);
  else if (E <= 2 * GT_THREADS) FGT(2, true);
  else if (E <= 4 * GT_THREADS) FGT(4, true);
  else FGT(8, false);
#undef FGT
}

extern "C" hl_status hl_embbag_fwd_plan(hl_handle* h, const void* w_hot, const void* staging, int32_t stg_rows,
                                        const int32_t* codes, const int32_t* bag_ptr, int32_t n_samples, int32_t bps,
                                        int64_t n_lookups, float* out, void* workspace, size_t ws_bytes,
                                        hl_stream stream) {
  hl_status st = check_common(h, codes, bag_ptr, n_samples, bps, n_lookups, nullptr, n_samples, stg_rows);
  if (st != HL_OK) return st;
  if (!workspace) return HL_ERR_INVALID_ARG;
  const int64_t n_bags = (int64_t)n_samples * bps;
  const size_t es = h->dtype == HL_F32 ? 4 : 2;
  const int vec = eb_pick_vec(h->dim, es, {w_hot, staging, out});
  const eb_geom g = eb_make_geom(h->dim, vec);
  const bool bf = h->dtype == HL_BF16;
  // (rows of 4 elements per lane: wider rows would spill in blocks of GT_THREADS)
  const bool fused = n_samples > 0 && n_lookups > 0 && n_lookups == n_bags && g.cchunks == 1 && vec == 4 &&
                     hl_group_by_table_ok(h, n_lookups, n_bags);
  const bool by_table = hl_group_by_table_ok(h, n_lookups, n_bags);
  // the general sort: the forward beside its passes, for the lane widths of
  // 16-byte row loads
  hl_sort_side side{};
  side.passes = !fused && !by_table && n_samples > 0 && n_lookups > 0 && g.cchunks == 1 ? hl_fwd_sort_side(bf, vec)
                                                                                        : nullptr;
  if (!fused && !side.passes) {
    // the two calls one after the other
    st = hl_embbag_fwd(h, w_hot, staging, stg_rows, codes, bag_ptr, n_samples, bps, n_lookups, nullptr, nullptr,
                       n_samples, out, stream);
    if (st != HL_OK) return st;
    return hl_embbag_bwd_plan(h, stg_rows, codes, bag_ptr, n_samples, bps, n_lookups, nullptr, nullptr, n_samples,
                              workspace, ws_bytes, stream);
  }
  if (!out || (h->n_hot && !w_hot) || (stg_rows && !staging)) return HL_ERR_INVALID_ARG;
  if (ws_bytes < bw_bytes(h, n_lookups, n_bags, false)) return HL_ERR_CAPACITY;
  hl_ws_note(h, workspace, HL_WSK_OTHER);
  hipStream_t s = (hipStream_t)stream;
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)n_lookups, n_bags, h->dim, false);
  if ((uint64_t)n_lookups > ws.sort.n_max) return HL_ERR_CAPACITY;
  uint32_t *rk, *rv;
  if (side.passes) {
    side.w_hot = w_hot;
    side.stg = staging;
    side.n_samples = n_samples;
    side.bps = bps;
    side.n_lookups = n_lookups;
    side.out = out;
    st = hl_sort_codes(h, ws.sort, bw_sort_src(h, stg_rows, const_cast<int32_t*>(codes), bag_ptr, n_bags),
                       (uint32_t)n_lookups, bw_key_bits(h, stg_rows), s, &rk, &rv, &side);
    if (st != HL_OK) return st;
    hl_ws_note(h, workspace, HL_WSK_BWD_PLAN, n_lookups, n_bags, stg_rows);
    hl_ws_find(h, workspace)->compact = false;
    return HL_OK;
  }
  hl_sort_result(ws.sort, bw_key_bits(h, stg_rows), &rk, &rv);
  uint32_t* tk = rk == ws.sort.k0 ? ws.sort.k1 : ws.sort.k0;
  uint32_t* tv = rv == ws.sort.v0 ? ws.sort.v1 : ws.sort.v0;
#define FG(V, B) launch_fwd_gt<V, B>(h, s, w_hot, staging, stg_rows, codes, bag_ptr, out, g, n_lookups, n_bags, workspace, \
                                     tk, tv, rk, rv)
  if (bf) FG(4, true);
  else FG(4, false);
#undef FG
  HL_LAUNCHED();
  hl_ws_note(h, workspace, HL_WSK_BWD_PLAN, n_lookups, n_bags, stg_rows);
  hl_ws_find(h, workspace)->compact = false;
  return HL_OK;
}

extern "C" hl_status hl_embbag_bwd_apply_part(hl_handle* h, void* w_hot, void* staging, int32_t stg_rows,
                                              int32_t n_samples, int32_t bps, int64_t n_lookups, const float* dY,
                                              float lr, int32_t part, void* workspace, size_t ws_bytes,
                                              hl_stream stream) {
  if (part < 0 || part > 2) return HL_ERR_INVALID_ARG;
  return hl_embbag_bwd_apply_any(h, w_hot, staging, stg_rows, n_samples, bps, n_lookups, dY, lr, part, workspace,
                                 ws_bytes, stream);
}

// parts 0-2 of hl_embbag_bwd_apply_part, and 3: the first half without its
// spanning segments (hl_embbag_finish_cold completes them)
hl_status hl_embbag_bwd_apply_any(hl_handle* h, void* w_hot, void* staging, int32_t stg_rows, int32_t n_samples,
                                  int32_t bps, int64_t n_lookups, const float* dY, float lr, int32_t part,
                                  void* workspace, size_t ws_bytes, hl_stream stream) {
  if (!h || n_samples < 0 || bps < 1 || n_lookups < 0 || stg_rows < 0 || !workspace) return HL_ERR_INVALID_ARG;
  if (part < 0 || part > 3) return HL_ERR_INVALID_ARG;
  const int64_t n_bags = (int64_t)n_samples * bps;
  hl_ws_rec* rec = hl_ws_find(h, workspace);
  if (!rec || rec->n != n_lookups || rec->bags != n_bags || rec->stg != stg_rows)
    return HL_ERR_INVALID_ARG;  // no matching plan is held by this workspace
  if (part == 2 && rec->part1 != 1) return HL_ERR_INVALID_ARG;  // the first half has not run on this plan
  if (part != 0 && rec->compact) return HL_ERR_INVALID_ARG;      // no room for the staging-row sums
  if (n_lookups == 0 || n_samples == 0) {
    if (part == 1 || part == 3) rec->part1 = part == 1 ? 1 : 3;
    return HL_OK;
  }
  if ((part != 2 && (!dY || (h->n_hot && !w_hot))) || (stg_rows && !staging)) return HL_ERR_INVALID_ARG;
  if (ws_bytes < bw_bytes(h, n_lookups, n_bags, rec->compact)) return HL_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)n_lookups, n_bags, h->dim, rec->compact);
  uint32_t *sk, *sv;
  hl_sort_result(ws.sort, bw_key_bits(h, stg_rows), &sk, &sv);
  const uint32_t n = (uint32_t)n_lookups;
  const size_t es = h->dtype == HL_F32 ? 4 : 2;
  const int vec = eb_pick_vec(h->dim, es, {w_hot, staging, part == 2 ? nullptr : dY});
  eb_geom g = eb_make_geom(h->dim, vec);
  const uint32_t te = (uint32_t)(RB_WAVES * g.NG * RB_EN(vec));
  const uint32_t tiles = hl_div_up(n, te);
  if (tiles > ws.tiles) return HL_ERR_CAPACITY;
  const bool bf = h->dtype == HL_BF16;
#define BWD(V, B) launch_bwd<V, B>(h, tiles, s, sk, sv, n, dY, g, w_hot, staging, h->n_hot, lr, ws, part)
  if (vec == 8) BWD(8, true);  // (bf16 only)
  else if (vec == 4) { if (bf) BWD(4, true); else BWD(4, false); }
  else if (vec == 2) { if (bf) BWD(2, true); else BWD(2, false); }
  else { if (bf) BWD(1, true); else BWD(1, false); }
#undef BWD
  HL_LAUNCHED();
  if (part == 1 || part == 3) {
    rec->part1 = part == 1 ? 1 : 3;
    rec->vec = vec;
  }
  return HL_OK;
}

hl_status hl_embbag_fwd_cold_sorted(hl_handle* h, const void* staging, int32_t stg_rows, const int32_t* codes,
                                    const int32_t* bag_ptr, int32_t n_samples, int32_t bps, int64_t n_lookups,
                                    float* out, void* workspace, size_t ws_bytes, hl_stream stream) {
  hl_status st = check_common(h, codes, bag_ptr, n_samples, bps, n_lookups, nullptr, n_samples, stg_rows);
  if (st != HL_OK) return st;
  if (!workspace || !out || (stg_rows && !staging)) return HL_ERR_INVALID_ARG;
  const int64_t n_bags = (int64_t)n_samples * bps;
  hl_ws_rec* rec = hl_ws_find(h, workspace);
  if (!rec || rec->n != n_lookups || rec->bags != n_bags || rec->stg != stg_rows || !rec->part1)
    return HL_ERR_INVALID_ARG;  // the grouping and the first apply half must be in this workspace
  if (n_lookups == 0 || n_samples == 0) return HL_OK;
  if (ws_bytes < bw_bytes(h, n_lookups, n_bags, rec->compact)) return HL_ERR_CAPACITY;
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)n_lookups, n_bags, h->dim, rec->compact);
  uint32_t *sk, *sv;
  hl_sort_result(ws.sort, bw_key_bits(h, stg_rows), &sk, &sv);
  const size_t es = h->dtype == HL_F32 ? 4 : 2;
  const int vec = eb_pick_vec(h->dim, es, {staging, out});
  eb_geom g = eb_make_geom(h->dim, vec);
  const uint32_t n = (uint32_t)n_lookups;
  uint32_t b = hl_div_up(n, 4 * g.NG * FT);
  if (b > 512) b = 512;
  hipStream_t s = (hipStream_t)stream;
  const bool bf = h->dtype == HL_BF16;
#define TAIL(V, B)                                                                                                  \
  HL_KERNEL(h, s, "eb_fwd_tail", (eb_fwd_tail<V, B>), dim3(b, g.cchunks), dim3(256), 0, s, sk, sv, n, ws.bnd, g, \
            staging, stg_rows, h->n_hot, h->k_cap, codes, bag_ptr, out, h->d_err)
  if (vec == 8) TAIL(8, true);  // (bf16 only)
  else if (vec == 4) { if (bf) TAIL(4, true); else TAIL(4, false); }
  else if (vec == 2) { if (bf) TAIL(2, true); else TAIL(2, false); }
  else { if (bf) TAIL(1, true); else TAIL(1, false); }
#undef TAIL
  HL_LAUNCHED();
  return HL_OK;
}

// After apply part 3 and the fetch: the cold half of the forward from the
// sorted tail together with the first half's spanning segments, then the
// staging-row updates (part 2's kernel).
hl_status hl_embbag_finish_cold(hl_handle* h, void* w_hot, void* staging, int32_t stg_rows, const int32_t* codes,
                                const int32_t* bag_ptr, int32_t n_samples, int32_t bps, int64_t n_lookups, float lr,
                                float* out, void* workspace, size_t ws_bytes, hl_stream stream) {
  hl_status st = check_common(h, codes, bag_ptr, n_samples, bps, n_lookups, nullptr, n_samples, stg_rows);
  if (st != HL_OK) return st;
  if (!workspace || !out || (stg_rows && !staging) || (h->n_hot && !w_hot)) return HL_ERR_INVALID_ARG;
  const int64_t n_bags = (int64_t)n_samples * bps;
  hl_ws_rec* rec = hl_ws_find(h, workspace);
  if (!rec || rec->n != n_lookups || rec->bags != n_bags || rec->stg != stg_rows || rec->part1 != 3)
    return HL_ERR_INVALID_ARG;  // the grouping and apply part 3 must be in this workspace
  rec->part1 = 0;  // the plan is used up: no part 2 or second finish on it
  if (n_lookups == 0 || n_samples == 0) return HL_OK;
  if (ws_bytes < bw_bytes(h, n_lookups, n_bags, rec->compact)) return HL_ERR_CAPACITY;
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)n_lookups, n_bags, h->dim, rec->compact);
  uint32_t *sk, *sv;
  hl_sort_result(ws.sort, bw_key_bits(h, stg_rows), &sk, &sv);
  // the first half's vector width (its tile sums' layout); out and the rows must allow it
  const size_t es = h->dtype == HL_F32 ? 4 : 2;
  const int vec = rec->vec;
  if (eb_pick_vec(h->dim, es, {w_hot, staging, out}) < vec) return HL_ERR_INVALID_ARG;
  eb_geom g = eb_make_geom(h->dim, vec);
  const uint32_t n = (uint32_t)n_lookups;
  const uint32_t te = (uint32_t)(RB_WAVES * g.NG * RB_EN(vec));
  const uint32_t tiles = hl_div_up(n, te);
  if (tiles > ws.tiles) return HL_ERR_CAPACITY;
  uint32_t tb = hl_div_up(n, RB_WAVES * g.NG * FT);
  if (tb > 1024) tb = 1024;  // (the tail, cold lookups only, is a part of n the device knows)
  // (as part 2: the tail, cold lookups only, is a part of n the device knows; a
  // grid of a few thousand waves strides over it)
  uint32_t cb = hl_div_up(n, 4 * CW_POS);
  if (cb > 1024) cb = 1024;
  hipStream_t s = (hipStream_t)stream;
  const bool bf = h->dtype == HL_BF16;
  // bags of several lookups: the cold half bag by bag, one bag per row group
  const bool multi = n_lookups > 2 * n_bags;
  const uint32_t fb = (uint32_t)std::min<int64_t>((n_bags + RB_WAVES * g.NG - 1) / (RB_WAVES * g.NG), 1 << 16);
#define FIN(V, B)                                                                                                   \
  do {                                                                                                             \
    if (multi)                                                                                                     \
      HL_KERNEL(h, s, "eb_bags_r2", (eb_bags_r2<V, B>), dim3(bw_r2_blocks(tiles, g) + fb, g.cchunks), dim3(RB_BLOCK), 0, s, tiles,  \
                w_hot, h->n_hot, lr, ws.tfirst, ws.tlast, ws.tflag, ws.tkey, ws.gc, ws.gc_rows, g, staging,        \
                stg_rows, h->k_cap, codes, bag_ptr, bps, n_samples, out, h->d_err);                                \
    else                                                                                                           \
      HL_KERNEL(h, s, "eb_tail_r2", (eb_tail_r2<V, B>), dim3(bw_r2_blocks(tiles, g) + tb, g.cchunks), dim3(RB_BLOCK), 0, s, tiles,  \
                w_hot, h->n_hot, lr, ws.tfirst, ws.tlast, ws.tflag, ws.tkey, ws.gc, ws.gc_rows, sk, sv, n, ws.bnd, \
                g, staging, stg_rows, h->k_cap, codes, bag_ptr, out, h->d_err);                                    \
    HL_KERNEL(h, s, "bw_cold", (bw_cold<V, B>), dim3(cb, g.cchunks), dim3(256), 0, s, sk, n, g, staging, h->n_hot, \
              lr, ws.gc, ws.gc_rows, ws.bnd, hl_hook_take(h));                                                     \
  } while (0)
  if (vec == 8) FIN(8, true);  // (bf16 only)
  else if (vec == 4) { if (bf) FIN(4, true); else FIN(4, false); }
  else if (vec == 2) { if (bf) FIN(2, true); else FIN(2, false); }
  else { if (bf) FIN(1, true); else FIN(1, false); }
#undef FIN
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_embbag_bwd_apply(hl_handle* h, void* w_hot, void* staging, int32_t stg_rows, int32_t n_samples,
                                         int32_t bps, int64_t n_lookups, const float* dY, float lr, void* workspace,
                                         size_t ws_bytes, hl_stream stream) {
  return hl_embbag_bwd_apply_part(h, w_hot, staging, stg_rows, n_samples, bps, n_lookups, dY, lr, 0, workspace,
                                  ws_bytes, stream);
}

extern "C" hl_status hl_embbag_bwd_sgd(hl_handle* h, void* w_hot, void* staging, int32_t stg_rows,
                                       const int32_t* codes, const int32_t* bag_ptr, int32_t n_samples, int32_t bps,
                                       int64_t n_lookups, const int32_t* sample_ids, const int32_t* n_sel_dev,
                                       int32_t n_sel_max, const float* dY, float lr, void* workspace, size_t ws_bytes,
                                       hl_stream stream) {
  hl_status st = check_common(h, codes, bag_ptr, n_samples, bps, n_lookups, sample_ids, n_sel_max, stg_rows);
  if (st != HL_OK) return st;
  if (n_samples == 0 || n_lookups == 0 || n_sel_max == 0) return HL_OK;
  if (!dY || !workspace || (h->n_hot && !w_hot) || (stg_rows && !staging)) return HL_ERR_INVALID_ARG;
  st = hl_embbag_bwd_plan(h, stg_rows, codes, bag_ptr, n_samples, bps, n_lookups, sample_ids, n_sel_dev, n_sel_max,
                          workspace, ws_bytes, stream);
  if (st != HL_OK) return st;
  return hl_embbag_bwd_apply(h, w_hot, staging, stg_rows, n_samples, bps, n_lookups, dY, lr, workspace, ws_bytes,
                             stream);
}

// The grouping that the last hl_embbag_bwd_plan on this workspace left (for
// inspection): the (key, bag) pairs in the order the reduction takes them.
extern "C" hl_status hl_embbag_bwd_grouping(hl_handle* h, int32_t stg_rows, int32_t n_samples, int32_t bps,
                                            int64_t n_lookups, const void* workspace, size_t ws_bytes,
                                            uint32_t* keys_out, uint32_t* bags_out, hl_stream stream) {
  if (!h || !workspace || n_samples < 0 || bps < 1 || n_lookups < 0 || stg_rows < 0) return HL_ERR_INVALID_ARG;
  if (n_lookups > 0 && (!keys_out || !bags_out)) return HL_ERR_INVALID_ARG;
  const int64_t n_bags = (int64_t)n_samples * bps;
  hl_ws_rec* rec = hl_ws_find(h, workspace);
  if (!rec || rec->n != n_lookups || rec->bags != n_bags || rec->stg != stg_rows) return HL_ERR_INVALID_ARG;
  if (n_lookups == 0) return HL_OK;
  if (ws_bytes < bw_bytes(h, n_lookups, n_bags, rec->compact)) return HL_ERR_CAPACITY;
  hl_carver c = hl_carver::after_header(const_cast<void*>(workspace), ws_bytes);
  bw_ws ws;
  bw_carve(c, ws, (uint32_t)n_lookups, n_bags, h->dim, rec->compact);
  uint32_t *sk, *sv;
  hl_sort_result(ws.sort, bw_key_bits(h, stg_rows), &sk, &sv);
  hipStream_t s = (hipStream_t)stream;
  if (hipMemcpyAsync(keys_out, sk, (size_t)n_lookups * 4, hipMemcpyDeviceToDevice, s) != hipSuccess ||
      hipMemcpyAsync(bags_out, sv, (size_t)n_lookups * 4, hipMemcpyDeviceToDevice, s) != hipSuccess)
    return HL_ERR_HIP;
  return HL_OK;
}
