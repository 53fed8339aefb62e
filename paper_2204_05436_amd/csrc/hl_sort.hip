// Stable LSD radix sort of (key, value) uint32 pairs, of the backward's (key,
// bag) pairs read from the slot codes, or of the access logger's (set, id) pairs
// read from the ids.
//
// A sort of `bits` bits takes P = ceil(bits / 11) passes of b = ceil(bits / P)
// bits (two passes of 10 bits for 20-bit keys), in P + 1 launches over the same
// tiles of consecutive items:
//
//   srt_count -- each tile's digit counts of every pass in one read of the keys
//                (from slot codes: it forms them, points the fused plan's cold
//                codes at their staging rows, and nothing is written per item;
//                from ids: it forms and writes the pairs).
//   srt_pass  -- one per digit.  A block ranks its tile's items by digit with
//                per-wave LDS counters that the lanes of one digit advance
//                together (their peer mask found by ballots), reorders the tile
//                in LDS so that each digit's run is contiguous, and writes the
//                runs at their global offsets: the digit's offset (exclusive
//                scan of its total over all tiles) plus the digit's count in the
//                earlier tiles.  The first pass's tiles are srt_count's: a few
//                blocks of its launch (the first by ticket, which wait for
//                nothing) add up the counts and publish the totals and each
//                group of 8 tiles' prefix, which a tile needs only once it has
//                ranked its items.  A later pass's tiles hold other items: each
//                publishes its counts, the last tile of a group the group's, and
//                a tile reads its group's earlier tiles and the earlier groups,
//                two rounds of loads (a chain of inclusive prefixes, or a read of
//                every earlier tile's counts, takes rounds that grow with the
//                tiles).  Tiles come from a ticket, so every lower one is already
//                running.
//
// Item order inside a tile is wave-major, then item, then lane, which is index
// order, so the sort is stable.  A pass is bound by latency (its dependent
// phases; a tile's bytes take a microsecond): at 328,000 pairs and 10-bit
// digits, 81 tiles of 4096, a later pass's are the ticket 1.0, loads and ranking
// 3.1, offsets 1.6, LDS reorder 0.4, earlier counts 2.2, scatter 0.8 us.  With
// 16 histogram blocks before the passes, 512-thread tiles and every earlier
// tile's counts read, the three launches took 9.5 + 19.2 + 19.2 us; now 4.9 +
// 13.3 + 11.2 (852,000 pairs, 11-bit digits: 19.3 + 34.7 + 34.7, now 6.4 + 23.6 +
// 17.6; 64,500 pairs, 9-bit: 6.6 + 11.6 + 11.6, now 3.5 + 7.5 + 7.6).
#include <algorithm>
#include <atomic>

#include "hl_sort_pass.h"

void hl_sort_ws_carve(hl_carver& c, hl_sort_ws& ws, uint32_t n_max) {
  hl_sort_ws_carve_pairs(c, ws, n_max);
  hl_sort_ws_carve_counts(c, ws);
}

void hl_sort_ws_carve_pairs(hl_carver& c, hl_sort_ws& ws, uint32_t n_max) {
  ws.n_max = n_max;
  // (fewer items per thread than 8 only up to HL_SORT_TILES_AIM tiles)
  ws.tiles_max = std::max({std::min(hl_div_up(n_max, HL_SORT_TILE_MIN), (uint32_t)HL_SORT_TILES_AIM),
                           hl_div_up(n_max, HL_SORT_TILE_MAX), 1u});
  ws.k0 = c.take<uint32_t>(n_max);
  ws.v0 = c.take<uint32_t>(n_max);
  ws.k1 = c.take<uint32_t>(n_max);
  ws.v1 = c.take<uint32_t>(n_max);
  ws.ctr = c.base ? c.header() + HL_HDR_SORT : nullptr;
}

void hl_sort_ws_carve_counts(hl_carver& c, hl_sort_ws& ws) {
  ws.tot = c.take<uint32_t>((size_t)HL_SORT_MAXPASS * HL_SORT_MAXNB);
  for (int i = 0; i < 4; ++i) ws.row[i] = c.take<uint32_t>((size_t)ws.tiles_max * (HL_SORT_MAXNB / 2));
  for (int i = 0; i < 2; ++i)
    ws.grp[i] = c.take<uint64_t>((size_t)hl_div_up(ws.tiles_max, HL_SORT_GRP) * (HL_SORT_MAXNB / 2));
  ws.gtot = c.take<uint64_t>(HL_SORT_MAXNB / 2);
}

static srt_plan srt_make_plan(int bits) {
  if (bits < 1) bits = 1;
  srt_plan p;
  p.passes = (bits + 10) / 11;
  p.b = (bits + p.passes - 1) / p.passes;
  p.nb = p.b <= 8 ? 256 : (p.b <= 9 ? 512 : (p.b <= 10 ? 1024 : 2048));
  return p;
}

// Digit counts of tile blockIdx.x for every pass (row[0], row[1], row[3]; the
// words the first two passes publish, row[2], grp and gtot, are cleared).
template <int NB>
__global__ void __launch_bounds__(HL_SORT_THREADS)
srt_count(hl_sort_src src, const uint32_t* n_dev, uint32_t n_host, int passes, int b, uint32_t tile,
          uint32_t* __restrict__ row0, uint32_t* __restrict__ row1, uint32_t* __restrict__ row2,
          uint32_t* __restrict__ row3, uint64_t* __restrict__ grp0, uint64_t* __restrict__ grp1,
          uint64_t* __restrict__ gtot, uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, uint32_t* err) {
  __shared__ uint32_t h[HL_SORT_MAXPASS][NB];
  bw_start_signal(src.sflag, src.sv);
  const uint32_t n = srt_n(n_dev, n_host);
  const uint32_t tb = blockIdx.x * tile, te = min(tb + tile, n);
  const int tid = threadIdx.x;
  for (int j = tid; j < HL_SORT_MAXPASS * NB; j += HL_SORT_THREADS) (&h[0][0])[j] = 0;
  uint32_t first = 0, covered = n;
  bool fits = false;
  if (src.codes) {
    srt_uncovered(src, n, &first, &covered);
    fits = src.cf.table && *src.cf.ncold <= (uint32_t)src.cf.cap;
    if (blockIdx.x == 0 && tid == 0) {
      if (src.bag_ptr[src.n_bags] != (int64_t)n) hl_flag(err, HL_DEVERR_SHAPE);
      if (src.cf.table && !fits) hl_flag(err, HL_DEVERR_CAPACITY);
    }
  }
  __syncthreads();
  const uint32_t mask = (1u << b) - 1u;
  bool bad = false;
  for (uint32_t i0 = tb + tid; i0 < te; i0 += 4 * HL_SORT_THREADS) {
    uint32_t k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t i = i0 + u * HL_SORT_THREADS;
      k[u] = i < te ? (src.codes ? (uint32_t)src.codes[i] : (src.ids ? src.ids[i] : src.k[i])) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t i = i0 + u * HL_SORT_THREADS;
      if (i >= te) continue;
      uint32_t key = k[u];
      if (src.codes) {
        if (i < first || i >= covered) {
          key = EB_SENT;
        } else {
          if (src.cf.table && key == 0xFFFFFFFFu) {
            const uint32_t sl = src.cf.slotof[i];
            key = (uint32_t)bw_fused_code(-1, i, src.cf, src.k_cap, fits);
            if (key != 0xFFFFFFFFu) src.codes[i] = (int32_t)key;
            if (sl < src.cf.S) src.cf.table[sl] = 0;
          }
          key = bw_key(key, src.n_hot, src.k_cap, src.stg_rows);
          bad = bad || key == EB_SENT;
        }
      } else if (src.ids) {
        vout[i] = key;
        key = hl_set_of(key, src.n_sets);
        kout[i] = key;
      }
      for (int p = 0; p < passes; ++p) atomicAdd(&h[p][(key >> (b * p)) & mask], 1u);
    }
  }
  if (bad) hl_flag(err, HL_DEVERR_BAD_CODE);
  __syncthreads();
  constexpr int TW = NB / 2;
  for (int j = tid; j < TW; j += HL_SORT_THREADS) {
    const size_t o = (size_t)blockIdx.x * TW + j;
    row0[o] = h[0][2 * j] | (h[0][2 * j + 1] << 16);
    const bool lead = blockIdx.x % HL_SORT_GRP == 0;
    const size_t go = (size_t)(blockIdx.x / HL_SORT_GRP) * TW + j;
    if (lead) grp1[go] = 0;
    if (blockIdx.x == 0) gtot[j] = 0;
    if (passes > 1) {
      row1[o] = h[1][2 * j] | (h[1][2 * j + 1] << 16);
      row2[o] = 0;
      if (lead) grp0[go] = 0;
    }
    if (passes > 2) row3[o] = h[2][2 * j] | (h[2][2 * j + 1] << 16);
  }
}

void hl_sort_result(const hl_sort_ws& ws, int bits, uint32_t** out_k, uint32_t** out_v) {
  const bool odd = srt_make_plan(bits).passes & 1;
  *out_k = odd ? ws.k1 : ws.k0;
  *out_v = odd ? ws.v1 : ws.v0;
}

int hl_device_cus(const hl_handle* h) {
  static std::atomic<int> cus[64];
  const int d = h->device >= 0 && h->device < 64 ? h->device : 0;
  int v = cus[d].load(std::memory_order_relaxed);
  if (v <= 0) {
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess || v <= 0) v = 1;
    cus[d].store(v, std::memory_order_relaxed);
  }
  return v;
}

// (reading a mask costs the host most of a microsecond; the default stream has none)
int hl_stream_cus(const hl_handle* h, hipStream_t s) {
  if (!s) return hl_device_cus(h);
  uint32_t m[16] = {0};
  if (hipExtStreamGetCUMask(s, 16, m) != hipSuccess) return 0;
  int c = 0;
  for (uint32_t w : m) c += __builtin_popcount(w);
  return c;
}

// items per thread of a tile: the fewest that keep a sort to HL_SORT_TILES_AIM
// tiles and to the stream's compute units (one tile per unit, one round)
static int srt_items(uint32_t n_host, int cus) {
  const uint32_t aim = cus > 0 && cus < HL_SORT_TILES_AIM ? (uint32_t)cus : HL_SORT_TILES_AIM;
  for (int it : {1, 2, 4})
    if (hl_div_up(n_host, HL_SORT_THREADS * it) <= aim) return it;
  return 8;
}

template <int NB, int ITEMS, bool FIRST>
__global__ void __launch_bounds__(HL_SORT_THREADS)
srt_pass(srt_args a, hl_hook hk) {
  __shared__ srt_lds<NB, ITEMS> lds;
  hl_hook_head(hk);
  srt_pass_body<NB, ITEMS, FIRST>(a, lds);
}

// The counts' launch, and with side the forward beside the passes.
static hl_status srt_run(hl_handle* h, hl_sort_ws& ws, const hl_sort_src& src, const uint32_t* n_dev, uint32_t n_host,
                         int bits, hipStream_t s, uint32_t** out_k, uint32_t** out_v, const hl_sort_side* side) {
  *out_k = ws.k0;
  *out_v = ws.v0;
  if (n_host == 0) return HL_OK;
  if (n_host > ws.n_max || n_host >= (1u << 30)) return HL_ERR_CAPACITY;
  if (bits > 32) return HL_ERR_UNSUPPORTED;
  const srt_plan pl = srt_make_plan(bits);
  const int cus = hl_stream_cus(h, s), items = srt_items(n_host, cus);
  const hl_hook hk = hl_hook_take(h);
  const uint32_t tile = (uint32_t)(HL_SORT_THREADS * items), tiles = hl_div_up(n_host, tile);
#define CNT(NB)                                                                                                      \
  HL_KERNEL(h, s, "srt_count", srt_count<NB>, dim3(tiles), dim3(HL_SORT_THREADS), 0, s, src, n_dev, n_host, pl.passes, \
            pl.b, tile, ws.row[0], ws.row[1], ws.row[2], ws.row[3], ws.grp[0], ws.grp[1], ws.gtot, ws.k0, ws.v0, h->d_err)
  if (pl.nb == 256) CNT(256);
  else if (pl.nb == 512) CNT(512);
  else if (pl.nb == 1024) CNT(1024);
  else CNT(2048);
#undef CNT
  if (side) {
    side->passes(h, ws, src, n_host, pl.passes, pl.b, pl.nb, items, cus, s, hk, *side);
  } else {
    srt_dispatch(pl.nb, items, [&](auto NB, auto IT) {
      constexpr int nb = decltype(NB)::value, it = decltype(IT)::value;
      srt_passes<nb, it>(h, ws, src, n_dev, n_host, pl, hk, [&](auto first, const srt_args& a, const hl_hook& k) {
        HL_KERNEL(h, s, "srt_pass", (srt_pass<nb, it, decltype(first)::value>), dim3(a.tiles + a.sums),
                  dim3(HL_SORT_THREADS), 0, s, a, k);
      });
    });
  }
  HL_LAUNCHED();
  hl_sort_result(ws, bits, out_k, out_v);
  return HL_OK;
}

hl_status hl_sort_pairs(hl_handle* h, hl_sort_ws& ws, const uint32_t* n_dev, uint32_t n_host, int bits,
                        hipStream_t s, uint32_t** out_k, uint32_t** out_v) {
  hl_sort_src src{};
  src.k = ws.k0;
  return srt_run(h, ws, src, n_dev, n_host, bits, s, out_k, out_v, nullptr);
}

hl_status hl_sort_ids_by_set(hl_handle* h, hl_sort_ws& ws, const uint32_t* ids, uint32_t n_sets, uint32_t n,
                             hipStream_t s, uint32_t** out_k, uint32_t** out_v) {
  hl_sort_src src{};
  src.ids = ids;
  src.n_sets = n_sets;
  return srt_run(h, ws, src, nullptr, n, hl_bit_width(n_sets), s, out_k, out_v, nullptr);
}

hl_status hl_sort_codes(hl_handle* h, hl_sort_ws& ws, const hl_sort_src& src, uint32_t n, int bits, hipStream_t s,
                        uint32_t** out_k, uint32_t** out_v, const hl_sort_side* side) {
  return srt_run(h, ws, src, nullptr, n, bits, s, out_k, out_v, side);
}
