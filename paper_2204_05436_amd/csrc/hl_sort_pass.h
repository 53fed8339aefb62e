// The general sort's pass (hl_sort.hip describes the sort): its block's body and
// the sequence of launches, shared by the sort's own launches and by those that
// run the forward beside the passes (hl_fwd_sort.h).
#pragma once
#include <type_traits>

#include "hl_internal.h"

// Published counts of a group of tiles: two digits in a 64-bit word
// (hl_st_store, hl_st_load), bit 31 of each half telling that it is there.
#define SRT_GRP2 0x8000000080000000ull
// A tile's counts take one 32-bit word per two digits, 15 bits each (a tile has
// fewer than 2^15 items); bit 15 of each half tells that a published count is
// there.  Published words go through relaxed agent-scope atomics: a word carries
// its own value and no other data is published through it.
#define SRT_AGG2 0x80008000u
static_assert(HL_SORT_TILE_MAX < 0x8000, "a tile's digit count must fit 15 bits");
__device__ __forceinline__ void srt_st_store(uint32_t* p, uint32_t w) {
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t srt_st_load(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t srt_n(const uint32_t* n_dev, uint32_t n_host) {
  if (!n_dev) return n_host;
  const uint32_t v = *n_dev;
  return v < n_host ? v : n_host;
}

// passes of b bits, NB bins each
struct srt_plan {
  int passes, b, nb;
};
// the lookups that no bag covers, [0, first) and [covered, n), sort last
__device__ __forceinline__ void srt_uncovered(const hl_sort_src& src, uint32_t n, uint32_t* first, uint32_t* covered) {
  *first = (uint32_t)min((int64_t)max(src.bag_ptr[0], 0), (int64_t)n);
  *covered = max((uint32_t)min((int64_t)max(src.bag_ptr[src.n_bags], 0), (int64_t)n), *first);
}

// Block-wide exclusive scans of two values per digit, two consecutive digits
// per thread, in place.
__device__ __forceinline__ void srt_scan2(uint32_t (&a)[2], uint32_t (&c)[2], uint32_t (*ws)[2]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t sa = a[0] + a[1], sc = c[0] + c[1];
  uint32_t ia = sa, ic = sc;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t ta = __shfl_up(ia, o), tc = __shfl_up(ic, o);
    if (lane >= o) {
      ia += ta;
      ic += tc;
    }
  }
  if (lane == 63) {
    ws[w][0] = ia;
    ws[w][1] = ic;
  }
  __syncthreads();
  uint32_t ra = ia - sa, rc = ic - sc;
  for (int j = 0; j < w; ++j) {
    ra += ws[j][0];
    rc += ws[j][1];
  }
  a[1] = ra + a[0];
  a[0] = ra;
  c[1] = rc + c[0];
  c[0] = rc;
}

// Sums over the tiles' counts of one pass, 64 words (128 digits) per block, 16
// groups of tiles at a time (a wave each).  The digits' totals: of the first
// pass (p = 0) published as flagged 64-bit words with every group's prefix over
// the groups before it, since tile blocks of the same launch wait for them; of a
// later pass stored for its launch.
template <int NB>
__device__ __forceinline__ void srt_sums(uint32_t blk, uint32_t tiles, const uint32_t* __restrict__ row0,
                                         const uint32_t* __restrict__ row1, const uint32_t* __restrict__ row3,
                                         uint64_t* gpre, uint64_t* gtot, uint32_t* __restrict__ tot,
                                         uint32_t (*sum)[128]) {
  constexpr int TW = NB / 2, PB = TW / 64;  // blocks per pass
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = (int)(blk / PB);
  const uint32_t w0 = (blk % PB) * 64, j = w0 + lane;
  const uint32_t* row = p == 0 ? row0 : (p == 1 ? row1 : row3);
  const uint32_t groups = (tiles + HL_SORT_GRP - 1) / HL_SORT_GRP;
  uint32_t a = 0, c = 0;  // (threads 0..63: the two digits of word j over the groups so far)
  for (uint32_t g0 = 0; g0 < groups; g0 += HL_SORT_WAVES) {
    uint32_t x[HL_SORT_GRP], sa = 0, sc = 0;
#pragma unroll
    for (int u = 0; u < HL_SORT_GRP; ++u) {
      const uint32_t t = (g0 + w) * HL_SORT_GRP + u;
      x[u] = t < tiles ? (row + (size_t)t * TW)[j] : 0u;
    }
#pragma unroll
    for (int u = 0; u < HL_SORT_GRP; ++u) {
      sa += x[u] & 0xFFFFu;
      sc += x[u] >> 16;
    }
    sum[w][2 * lane] = sa;
    sum[w][2 * lane + 1] = sc;
    __syncthreads();
    if (w == 0)
      for (uint32_t q = 0; q < HL_SORT_WAVES && g0 + q < groups; ++q) {
        if (p == 0) hl_st_store(gpre + (size_t)(g0 + q) * TW + j, SRT_GRP2 | (uint64_t)c << 32 | a);
        a += sum[q][2 * lane];
        c += sum[q][2 * lane + 1];
      }
    __syncthreads();
  }
  if (w != 0) return;
  if (p == 0) {
    hl_st_store(gtot + j, SRT_GRP2 | (uint64_t)c << 32 | a);
  } else {
    tot[(size_t)p * HL_SORT_MAXNB + 2 * j] = a;
    tot[(size_t)p * HL_SORT_MAXNB + 2 * j + 1] = c;
  }
}

// A flagged 64-bit word, waited for.
__device__ __forceinline__ uint64_t srt_wait(const uint64_t* p, uint32_t* err) {
  uint32_t spins = 0;
  for (;;) {
    const uint64_t x = hl_st_load(p);
    if ((x & SRT_GRP2) == SRT_GRP2) return x & ~SRT_GRP2;
    if (++spins > HL_SPIN_LIMIT) {
      hl_flag(err, HL_DEVERR_STALL);
      return 0;
    }
  }
}

// The bag of each lookup [tb, te) into bag[i - tb] (lookups no bag covers keep
// what is there).  Thread i holds the bounds p, q of bag g0 + i, a window of bags
// around where the first lookup would be if all bags were alike: when it holds
// all of the tile's bags each thread writes its own, else the bag of the first
// lookup is found in it or searched by the whole block, HL_SORT_THREADS probes of
// bag_ptr a round, and each bag from there on writes its lookups.
__device__ __forceinline__ void srt_bag(uint32_t j, int64_t p, int64_t q, uint32_t tb, uint32_t te, uint32_t* bag) {
  const uint32_t lo = (uint32_t)max(p, (int64_t)tb), hi = (uint32_t)min(max(q, (int64_t)0), (int64_t)te);
  for (uint32_t i = lo; i < hi; ++i) bag[i - tb] = j;
}
// (c: the window's bags that start at or before lookup tb, a prefix of it;
// reach: the window's last bag ends at or after te)
__device__ __forceinline__ void srt_bags(const hl_sort_src& src, bool window, int64_t g0, int32_t p, int32_t q, int c,
                                         bool reach, uint32_t tb, uint32_t te, uint32_t* bag) {
  const int64_t mine = g0 + threadIdx.x;
  const bool ends = g0 + HL_SORT_THREADS >= src.n_bags;
  const bool starts = window && (c > 0 || g0 == 0);
  if (starts && (ends || reach)) {
    if (mine < src.n_bags) srt_bag((uint32_t)mine, p, q, tb, te, bag);
    return;
  }
  int64_t a = g0 + (c > 0 ? c - 1 : 0);
  if (!starts || (c == HL_SORT_THREADS && !ends)) {
    int64_t e = src.n_bags;
    for (a = 0; e - a > 1;) {
      const int64_t step = (e - a + HL_SORT_THREADS - 1) / HL_SORT_THREADS;
      const int64_t j = a + threadIdx.x * step;
      const int k = __syncthreads_count(j < e && src.bag_ptr[j] <= (int32_t)tb);
      a += (k > 0 ? k - 1 : 0) * step;
      e = min(a + step, e);
    }
  }
  for (int64_t j = a + threadIdx.x; j < src.n_bags; j += HL_SORT_THREADS) {
    const int32_t jp = src.bag_ptr[j], jq = src.bag_ptr[j + 1];
    if (jp >= (int32_t)te) break;
    srt_bag((uint32_t)j, jp, jq, tb, te, bag);
  }
}

// What one launch of a pass reads and writes.
struct srt_args {
  hl_sort_src src;
  const uint32_t *kin, *vin;
  uint32_t *kout, *vout;
  const uint32_t* n_dev;
  uint32_t n_host, tiles;
  uint32_t sums;                // the first pass: blocks that add up the tiles' counts
  int shift, b;
  const uint32_t *row1, *row3;  // the first pass: the later passes' counts
  uint64_t* gtot;               // the first pass: published totals
  uint32_t* tot;                // digit totals (of the pass; the first pass writes the later ones')
  uint32_t* st;                 // the tiles' counts (of srt_count; a later pass publishes them)
  uint64_t* grp;                // published counts of groups (the first pass: prefixes)
  uint32_t* st_next;            // cleared for the next pass (NULL: nothing)
  uint64_t* grp_next;
  uint32_t *ctr, *err;
};

template <int NB, int ITEMS>
struct srt_lds {
  static constexpr uint32_t TW = NB / 2, SP = HL_SORT_THREADS / TW, TILE = HL_SORT_THREADS * ITEMS;
  uint32_t wcnt[HL_SORT_WAVES][TW];  // per wave, two digits a word (a wave has at most 512 items)
  uint32_t tdex[NB], gbase[NB];
  uint32_t lk[TILE], lv[TILE];
  uint32_t part[SP > 1 ? 4 : 1][SP > 1 ? HL_SORT_THREADS : 1];
  uint32_t scan_ws[HL_SORT_WAVES][2];
  uint32_t tile;
};

// One block of a pass's launch (a.tiles + a.sums of them, by ticket).
template <int NB, int ITEMS, bool FIRST>
__device__ __forceinline__ void srt_pass_body(const srt_args& a, srt_lds<NB, ITEMS>& lds) {
  constexpr uint32_t TILE = HL_SORT_THREADS * ITEMS;
  constexpr uint32_t TW = NB / 2;                // words of two digits
  constexpr uint32_t SP = HL_SORT_THREADS / TW;  // threads per word: each reads every SP-th tile's count
  auto& wcnt = lds.wcnt;
  auto& tdex = lds.tdex;
  auto& gbase = lds.gbase;
  auto& scan_ws = lds.scan_ws;
  auto& lk = lds.lk;
  auto& lv = lds.lv;
  auto& part = lds.part;
  const hl_sort_src& src = a.src;
  const uint32_t *kin = a.kin, *vin = a.vin, *n_dev = a.n_dev, *row1 = a.row1, *row3 = a.row3;
  uint32_t *kout = a.kout, *vout = a.vout, *st = a.st, *st_next = a.st_next, *tot = a.tot, *err = a.err;
  uint64_t *grp = a.grp, *grp_next = a.grp_next, *gtot = a.gtot;
  const uint32_t n_host = a.n_host, tiles = a.tiles, sums = a.sums;
  const int shift = a.shift, b = a.b;
  const uint32_t n = srt_n(n_dev, n_host);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) lds.tile = atomicInc(a.ctr, tiles + sums - 1);
  __syncthreads();
  if (FIRST && lds.tile < sums) {
    static_assert(HL_SORT_WAVES * 128 <= TW * HL_SORT_WAVES, "the sums' LDS");
    srt_sums<NB>(lds.tile, tiles, st, row1, row3, grp, gtot, tot, reinterpret_cast<uint32_t(*)[128]>(&wcnt[0][0]));
    return;
  }
  const uint32_t tile = lds.tile - sums;
  if (!FIRST && st_next)  // this tile's published words of the next pass
    for (uint32_t j = tid; j < TW; j += HL_SORT_THREADS) {
      st_next[(size_t)tile * TW + j] = 0;
      if (tile % HL_SORT_GRP == 0) grp_next[(size_t)(tile / HL_SORT_GRP) * TW + j] = 0;
    }
  const uint64_t tb = (uint64_t)tile * TILE;
  if (tb >= n) return;
  const uint32_t te = (uint32_t)min(tb + TILE, (uint64_t)n);
  const uint32_t mask = (1u << b) - 1u;
  const uint32_t i0 = (uint32_t)tb + w * (ITEMS * 64) + lane;  // item k: i0 + 64 k
  uint32_t key[ITEMS], val[ITEMS];
  const bool from_codes = FIRST && src.codes;
  bool one = from_codes && src.n_bags == (int64_t)n;  // every bag of the tile holds its own lookup alone?
  int32_t lo[ITEMS], hi[ITEMS], gp = 0, gq = 0;
  int64_t g0 = 0;
  uint32_t first = 0, covered = n;
  if (from_codes) srt_uncovered(src, n, &first, &covered);
  if (from_codes && !one) {
    g0 = max((int64_t)(tb * (uint64_t)src.n_bags / n) - HL_SORT_THREADS / 4, (int64_t)0);
    const int64_t j = min(g0 + tid, src.n_bags - 1);
    gp = src.bag_ptr[j];
    gq = src.bag_ptr[j + 1];
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t i = min(i0 + 64 * k, te - 1);
    if (from_codes) {
      key[k] = (uint32_t)src.codes[i];
      if (one) {
        lo[k] = src.bag_ptr[i];
        hi[k] = src.bag_ptr[i + 1];
      }
    } else {
      key[k] = kin[i];
      val[k] = vin[i];
    }
  }
  for (uint32_t j = tid; j < HL_SORT_WAVES * TW; j += HL_SORT_THREADS) (&wcnt[0][0])[j] = 0;
  const uint32_t wd = (uint32_t)tid % TW;
  const uint32_t sp = __builtin_amdgcn_readfirstlane((uint32_t)tid / TW);  // (a wave's words share it)
  // word wd's digits in the earlier tiles of this tile's group of HL_SORT_GRP:
  // the first pass has them from srt_count
  const uint32_t grp0 = tile / HL_SORT_GRP, in_grp = tile % HL_SORT_GRP;
  constexpr int GT = (HL_SORT_GRP - 1 + SP - 1) / SP;
  uint32_t excl[2] = {0, 0};
  uint2 dt = make_uint2(0u, 0u);  // the digits' totals over all tiles
  if (FIRST) {
    uint32_t wv[GT];
#pragma unroll
    for (int q = 0; q < GT; ++q) {
      const uint32_t t = sp + q * SP;
      wv[q] = t < in_grp ? (st + (size_t)(grp0 * HL_SORT_GRP + t) * TW)[wd] : 0u;
    }
#pragma unroll
    for (int q = 0; q < GT; ++q) {
      excl[0] += wv[q] & 0xFFFFu;
      excl[1] += wv[q] >> 16;
    }
    if constexpr (SP > 1) {
      part[2][tid] = excl[0];
      part[3][tid] = excl[1];
    }
  } else if (sp == 0) {
    dt = *reinterpret_cast<const uint2*>(tot + 2 * wd);
  }
  if (from_codes) {
    if (one)
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) {
        const int32_t i = (int32_t)min(i0 + 64 * k, te - 1);
        one = one && lo[k] == i && hi[k] == i + 1;
      }
    // one barrier for what the block has to agree on: whether every bag of the
    // tile is its own lookup's; else how many of the window's bags start by
    // lookup tb, and whether the window reaches te
    const bool window = src.n_bags != (int64_t)n;
    const uint64_t in = __ballot(g0 + tid < src.n_bags && gp <= (int32_t)tb);
    const uint64_t bad = __ballot(!one);
    if (lane == 63) {
      scan_ws[w][0] = (uint32_t)__popcll(in);
      scan_ws[w][1] = (bad ? 1u : 0u) | (w == HL_SORT_WAVES - 1 && gq >= (int32_t)te ? 2u : 0u);
    }
    __syncthreads();  // (wcnt is zero now, too)
    uint32_t c = 0, fl = 0;
#pragma unroll
    for (int q = 0; q < HL_SORT_WAVES; ++q) {
      c += scan_ws[q][0];
      fl |= scan_ws[q][1];
    }
    if (fl & 1u) {
      srt_bags(src, window, g0, gp, gq, (int)c, (fl & 2u) != 0, (uint32_t)tb, te, lk);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) val[k] = lk[w * (ITEMS * 64) + 64 * k + lane];
      // (lk takes the reordered tile after the barriers below)
    } else {
#pragma unroll
      for (int k = 0; k < ITEMS; ++k) val[k] = i0 + 64 * k;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const uint32_t i = i0 + 64 * k;
      key[k] = i >= first && i < covered ? bw_key(key[k], src.n_hot, src.k_cap, src.stg_rows) : EB_SENT;
    }
  } else {
    __syncthreads();  // wcnt is zero
  }
  // ranking, stable by construction: for each item slot the lanes holding the
  // same digit find one another with one ballot per digit bit (their peer
  // mask); the lowest peer adds the group's size to the wave's counter of that
  // digit (one atomic per distinct digit, so no two lanes of an instruction
  // touch one digit's count) and the others take its old value by a lane
  // shuffle; a lane's rank is that value plus its peers on lower lanes.  A
  // wave's LDS instructions execute in issue order, so the counters advance in
  // item order: ranks follow (item, lane) order, which is index order.  The
  // peer masks, the atomics and the shuffles of all items are issued as three
  // groups, so that an item's latency hides behind the others'.
  uint32_t lr[ITEMS];
  {
    uint64_t peers[ITEMS];
    uint32_t old[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
      peers[k] = hl_match_digit((key[k] >> shift) & mask, b, i0 + 64 * k < te);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const uint32_t d = (key[k] >> shift) & mask;
      old[k] = 0;
      if (peers[k] && lane == __ffsll((unsigned long long)peers[k]) - 1)
        old[k] = atomicAdd(&wcnt[w][d >> 1], (uint32_t)__popcll(peers[k]) << (16 * (d & 1)));
    }
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const uint32_t d = (key[k] >> shift) & mask;
      const int leader = __ffsll((unsigned long long)peers[k]) - 1;
      const uint32_t x = __shfl(old[k], leader < 0 ? 0 : leader);
      lr[k] = ((x >> (16 * (d & 1))) & 0xFFFFu) + (uint32_t)__popcll(peers[k] & lt);
    }
  }
  __syncthreads();
  // wave-exclusive offsets of word wd's digits (both at once: a tile has fewer
  // than 2^15 items); the totals are the tile's counts, which a later pass
  // publishes at once for the later tiles
  uint32_t tx[2] = {0, 0}, gx[2] = {0, 0}, mine[2] = {0, 0};
  if (sp == 0) {
    uint32_t run = 0;
#pragma unroll
    for (int q = 0; q < HL_SORT_WAVES; ++q) {
      const uint32_t c = wcnt[q][wd];
      wcnt[q][wd] = run;
      run += c;
    }
    if (!FIRST) srt_st_store(st + (size_t)tile * TW + wd, SRT_AGG2 | run);
    tx[0] = mine[0] = run & 0xFFFFu;
    tx[1] = mine[1] = run >> 16;
    if constexpr (FIRST) {
      if constexpr (SP > 1)
        for (uint32_t q = 1; q < SP; ++q) {
          excl[0] += part[2][tid + q * TW];
          excl[1] += part[3][tid + q * TW];
        }
      // from the launch's first blocks, which wait for nothing
      const uint64_t gt = srt_wait(gtot + wd, err), gp0 = srt_wait(grp + (size_t)grp0 * TW + wd, err);
      dt = make_uint2((uint32_t)gt, (uint32_t)(gt >> 32));
      excl[0] += (uint32_t)gp0;
      excl[1] += (uint32_t)(gp0 >> 32);
    }
    gx[0] = dt.x;
    gx[1] = dt.y;
  }
  srt_scan2(tx, gx, scan_ws);
  if (sp == 0)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      tdex[2 * wd + j] = tx[j];
      if (FIRST) gbase[2 * wd + j] = gx[j] + excl[j] - tx[j];
    }
  __syncthreads();
  // the tile in digit order in LDS (its own offsets are known now; a later
  // pass reads the earlier tiles' counts below)
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (i0 + 64 * k < te) {
      const uint32_t d = (key[k] >> shift) & mask;
      const uint32_t p = tdex[d] + ((wcnt[w][d >> 1] >> (16 * (d & 1))) & 0xFFFFu) + lr[k];
      lk[p] = key[k];
      lv[p] = val[k];
    }
  }
  if (!FIRST) {
    // counts of word wd's digits in all earlier tiles, in two steps of loads that
    // are all in flight together (no chain through inclusive prefixes): the
    // earlier tiles of this tile's group of HL_SORT_GRP, then the earlier groups,
    // whose counts their last tiles publish; a step with an unpublished word is
    // read again
    constexpr int GC = 16;
    uint32_t spins = 0;
    for (bool again = in_grp > sp; again;) {
      uint32_t wv[GT], ready = SRT_AGG2, s0 = 0, s1 = 0;
#pragma unroll
      for (int q = 0; q < GT; ++q) {
        const uint32_t t = sp + q * SP;
        wv[q] = t < in_grp ? srt_st_load(st + (size_t)(grp0 * HL_SORT_GRP + t) * TW + wd) : SRT_AGG2;
      }
#pragma unroll
      for (int q = 0; q < GT; ++q) {
        ready &= wv[q];
        s0 += wv[q] & 0x7FFFu;
        s1 += (wv[q] >> 16) & 0x7FFFu;
      }
      again = ready != SRT_AGG2;
      if (!again) {
        excl[0] = s0;
        excl[1] = s1;
      } else if (++spins > HL_SPIN_LIMIT) {
        hl_flag(err, HL_DEVERR_STALL);
        again = false;
      }
    }
    if constexpr (SP > 1) {
      part[2][tid] = excl[0];
      part[3][tid] = excl[1];
      __syncthreads();
      if (sp == 0)
        for (uint32_t q = 1; q < SP; ++q) {
          excl[0] += part[2][tid + q * TW];
          excl[1] += part[3][tid + q * TW];
        }
      else
        excl[0] = excl[1] = 0;
    }
    if (in_grp == HL_SORT_GRP - 1 && sp == 0)
      hl_st_store(grp + (size_t)grp0 * TW + wd,
                  SRT_GRP2 | (uint64_t)(excl[1] + mine[1]) << 32 | (excl[0] + mine[0]));
    for (uint32_t q0 = sp; q0 < grp0; q0 += SP * GC) {
      for (;;) {
        uint64_t wv[GC], ready = SRT_GRP2;
        uint32_t s0 = 0, s1 = 0;
#pragma unroll
        for (int q = 0; q < GC; ++q) {
          const uint32_t t = q0 + q * SP;
          wv[q] = t < grp0 ? hl_st_load(grp + (size_t)t * TW + wd) : SRT_GRP2;
        }
#pragma unroll
        for (int q = 0; q < GC; ++q) {
          ready &= wv[q];
          s0 += (uint32_t)wv[q] & 0x7FFFFFFFu;
          s1 += (uint32_t)(wv[q] >> 32) & 0x7FFFFFFFu;
        }
        if ((ready & SRT_GRP2) == SRT_GRP2) {
          excl[0] += s0;
          excl[1] += s1;
          break;
        }
        if (++spins > HL_SPIN_LIMIT) {
          hl_flag(err, HL_DEVERR_STALL);
          break;
        }
      }
    }
    if constexpr (SP > 1) {
      part[0][tid] = excl[0];
      part[1][tid] = excl[1];
      __syncthreads();
      if (sp == 0)
        for (uint32_t q = 1; q < SP; ++q) {
          excl[0] += part[0][tid + q * TW];
          excl[1] += part[1][tid + q * TW];
        }
    }
    if (sp == 0)
#pragma unroll
      for (int j = 0; j < 2; ++j) gbase[2 * wd + j] = gx[j] + excl[j] - tx[j];
  }
  __syncthreads();
  // (gbase: an item's place less its place in the tile)
  const uint32_t nv = te - (uint32_t)tb;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t i = tid + k * HL_SORT_THREADS;
    if (i >= nv) break;
    const uint32_t kk = lk[i];
    const uint32_t p = gbase[(kk >> shift) & mask] + i;
    if (p < n) {  // (always, for counts of the same keys)
      kout[p] = kk;
      vout[p] = lv[i];
    }
  }
}

// The launches of a sort after srt_count: launch(first, args, hook) makes one.
template <int NB, int ITEMS, typename L>
static void srt_passes(hl_handle* h, hl_sort_ws& ws, const hl_sort_src& src, const uint32_t* n_dev, uint32_t n_host,
                       const srt_plan& pl, const hl_hook& hk, L launch) {
  srt_args a{};
  a.src = src;
  a.kin = ws.k0;
  a.vin = ws.v0;
  a.kout = ws.k1;
  a.vout = ws.v1;
  a.n_dev = n_dev;
  a.n_host = n_host;
  a.tiles = hl_div_up(n_host, HL_SORT_THREADS * ITEMS);
  a.sums = (uint32_t)pl.passes * (NB / 128);
  a.b = pl.b;
  a.row1 = ws.row[1];
  a.row3 = ws.row[3];
  a.gtot = ws.gtot;
  a.tot = ws.tot;
  a.st = ws.row[0];
  a.grp = ws.grp[1];
  a.ctr = ws.ctr;
  a.err = h->d_err;
  launch(std::true_type{}, a, hk);  // (the hook: srt_count's writes are complete then)
  // the published counts of the second pass go to row[2], of the third to row[0]
  // (the first pass's counts, done with by then; cleared by the second pass)
  a.sums = 0;
  for (int p = 1; p < pl.passes; ++p) {
    const uint32_t *k = a.kin, *v = a.vin;
    a.kin = a.kout;
    a.vin = a.vout;
    a.kout = const_cast<uint32_t*>(k);
    a.vout = const_cast<uint32_t*>(v);
    a.shift = pl.b * p;
    a.tot = ws.tot + (size_t)p * HL_SORT_MAXNB;
    a.st = ws.row[p == 1 ? 2 : 0];
    a.grp = ws.grp[p - 1];
    a.st_next = p == 1 && pl.passes > 2 ? ws.row[0] : nullptr;
    a.grp_next = ws.grp[1];
    a.ctr = ws.ctr + p;
    launch(std::false_type{}, a, hl_hook{});
  }
}

// The launches for the digit width and the tile size of a sort:
// f(std::integral_constant<int, NB>, std::integral_constant<int, ITEMS>).
template <typename F>
static void srt_dispatch(int nb, int items, F f) {
  auto by_items = [&](auto NB) {
    if (items == 1) f(NB, std::integral_constant<int, 1>{});
    else if (items == 2) f(NB, std::integral_constant<int, 2>{});
    else if (items == 4) f(NB, std::integral_constant<int, 4>{});
    else f(NB, std::integral_constant<int, 8>{});
  };
  if (nb == 256) by_items(std::integral_constant<int, 256>{});
  else if (nb == 512) by_items(std::integral_constant<int, 512>{});
  else if (nb == 1024) by_items(std::integral_constant<int, 1024>{});
  else by_items(std::integral_constant<int, 2048>{});
}
