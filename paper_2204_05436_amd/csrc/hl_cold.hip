// Cold-row gather of a mu-batch: the distinct non-hot rows its lookups need,
// in order of first occurrence in the mini-batch's lookup order, fetched from
// the pinned host table by the GPU over the host link, with the lookups'
// codes pointed at the staging rows.
//
//   insert : each cold lookup (code -1) of a selected sample enters an
//            open-addressing hash table keyed by row id with one CAS (a 64-bit
//            atomic min keeps the smallest lookup index per id); a thread per
//            lookup, or with a sample list 8 to 256 threads per listed sample
//            (a long one by whole blocks)
//   rank   : a scan over all lookups in index order (tiles of 2048, their counts
//            published and read by the whole block) numbers the first
//            occurrences: staging row u of each id
//   codes  : the selected cold lookups again: capacity check, code rewrite, the
//            cold id list, and the clearing of the table slots this call used
//   copy   : the row copy between the pinned host table and the staging rows,
//            in either direction (fetch before the mu-batch runs, write-back
//            of the updated rows after it)
// The hash table belongs to the handle (cleared once, then left clean by every
// call); the rest lives in the workspace.  The copy reads only the cold id
// list and count, so it can run on a stream of its own while the popular
// mu-batch and the backward's grouping proceed (the overlap of the paper's
// pipeline, Sec. IV and Fig. "hotlinepipe").
#include <algorithm>

#include "hl_internal.h"

#define CG_C_NCOLD 1
#define CG_C_RTILE 2
#define CG_RT_THREADS 512
#define CG_RT (CG_RT_THREADS * 4)  // lookups per rank tile

struct cg_ws {
  uint32_t* ctr;      // header counters
  uint32_t* uidx;     // [S] staging row of the id in the slot
  uint32_t* slotof;   // [n_max] slot of a cold lookup
  uint32_t* fst;      // [n_max] id of staging row u
  uint64_t* rstat;    // [rtiles] look-back status of the rank scan
  uint32_t S, rtiles;
};

static uint32_t cg_table_slots(uint32_t n_max) {
  uint32_t s = 1024;
  while (s < 2u * n_max) s <<= 1;
  return s;
}

static void cg_carve(hl_carver& c, cg_ws& ws, uint32_t n_max) {
  ws.S = cg_table_slots(n_max);
  ws.rtiles = n_max ? hl_div_up(n_max, CG_RT) : 1;
  ws.ctr = c.base ? c.header() + HL_HDR_COLD : nullptr;
  ws.uidx = c.take<uint32_t>(ws.S);
  ws.slotof = c.take<uint32_t>(n_max);
  ws.fst = c.take<uint32_t>(n_max);
  ws.rstat = c.take<uint64_t>(ws.rtiles);
}

size_t hl_cold_ws_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags, int32_t max_samples) {
  (void)h;
  hl_carver c = hl_carver::after_header(nullptr, 0);
  cg_ws ws;
  cg_carve(c, ws, (uint32_t)max_lookups);
  return c.off;
}

// The handle's hash table, (id + 1) << 32 | smallest lookup index per slot, 0
// = empty; grown (and zeroed) when a call needs more slots.  The growth
// allocates, so a caller that captures calls into a graph reserves the largest
// size first (hl_cold_reserve).
static hl_status cg_table(hl_handle* h, uint32_t S, hipStream_t s, uint64_t** out) {
  if (h->cg_slots < S) {
    if (h->cg_table) {
      if (hipFree(h->cg_table) != hipSuccess) return HL_ERR_HIP;
      h->cg_table = nullptr;
      h->cg_slots = 0;
    }
    if (hipMalloc(&h->cg_table, (size_t)S * 8) != hipSuccess) return HL_ERR_HIP;
    h->cg_slots = S;
    hl_status st = hl_fill32((uint32_t*)h->cg_table, (uint64_t)S * 2, 0, s);
    if (st != HL_OK) return st;
  }
  *out = h->cg_table;
  return HL_OK;
}

// The selected lookups: of the first sel_bags bags (ids NULL), one per thread of
// a flat grid, or of the listed samples, tps threads (8 to 256, about as many as a
// sample has lookups) per sample; a sample of more than CG_LONG tps lookups by the
// whole block, four per thread at a time, and by gridDim.y blocks where samples
// are that long on average (then its lookups are its blocks' share and more).
// f(i, g) takes a lookup with code -1 and, when `gids` is given, its id.  One
// lookup per thread keeps each thread to one chain of dependent accesses (probe,
// slot, code): four per thread took 7.6 and 5.3 us (insert, codes; 212,992
// lookups) against 4.6 and 3.3, and blocks that first compacted their cold lookups
// in LDS 5.7 and 4.0.  A list marked in a mask over the samples by two launches of
// its own and searched by bag: 16.7 us for the insert of 328,000 lookups in bags
// of 20, 5.6 by the listed samples.  Long samples by a sample's own threads alone,
// one lookup at a time (whole calls, a fifth of the lookups cold): one of 320,000
// lookups 2184 us against 283, 4 of 80,000 529 against 283, one of 40,000 among
// 2047 of 40 923 against 309.
#define CG_LONG 4
struct cg_sel {
  const int32_t* ids;     // the listed samples (NULL: every sample up to sel_bags / bps)
  const int32_t* n_dev;   // their number on the device (NULL: n_max)
  int32_t n_max, n_samples, bps, tps;
  int64_t sel_bags;
};
template <typename F>
__device__ __forceinline__ void cg_lookups(const cg_sel& sel, const int32_t* __restrict__ bag_ptr,
                                           const int32_t* codes, const uint32_t* gids, uint32_t n_lookups, uint32_t* err,
                                           F f) {
  auto end = [&](int64_t bag) { return (uint32_t)min(max((int64_t)bag_ptr[bag], (int64_t)0), (int64_t)n_lookups); };
  if (!sel.ids) {
    const uint32_t t = blockIdx.x * 256 + threadIdx.x, lo = end(0), hi = end(sel.sel_bags);
    if (t < n_lookups) {
      const int32_t c = codes[t];
      const uint32_t g = gids ? gids[t] : 0u;
      if (c == -1 && t >= lo && t < hi) f(t, g);
    }
    return;
  }
  // (the grid covers a list of every sample; a longer one, which names samples
  // again, in turns: n_max is only a bound and may be any number)
  __shared__ uint32_t l_lo[32], l_hi[32], l_n;
  const uint32_t tps = (uint32_t)sel.tps, per = 256 / tps, r = threadIdx.x % tps;
  const int64_t n = sel.n_dev ? min(max(*sel.n_dev, 0), sel.n_max) : sel.n_max;
  for (int64_t q0 = (int64_t)blockIdx.x * per; q0 < n; q0 += (int64_t)gridDim.x * per) {
    const int64_t q = q0 + threadIdx.x / tps;
    uint32_t lo = 0, hi = 0;
    if (q < n) {
      const int32_t s = sel.ids[q];
      if (s >= 0 && s < sel.n_samples) {
        const int64_t b0 = (int64_t)s * sel.bps;
        lo = end(b0);
        hi = end(b0 + sel.bps);
      } else if (r == 0) {
        hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
      }
    }
    const bool lng = hi > lo && hi - lo > CG_LONG * tps;
    if (!lng && blockIdx.y == 0)
      for (uint32_t i = lo + r; i < hi; i += tps) {
        const int32_t c = codes[i];
        const uint32_t g = gids ? gids[i] : 0u;
        if (c == -1) f(i, g);
      }
    if (threadIdx.x == 0) l_n = 0;
    if (!__syncthreads_or(lng)) continue;
    if (lng && r == 0) {
      const uint32_t k = atomicAdd(&l_n, 1u);
      l_lo[k] = lo;
      l_hi[k] = hi;
    }
    __syncthreads();
    for (uint32_t k = 0; k < l_n; ++k)
      for (uint32_t i0 = l_lo[k] + blockIdx.y * 1024 + threadIdx.x; i0 < l_hi[k]; i0 += gridDim.y * 1024) {
        int32_t c[4];
        uint32_t g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t i = i0 + u * 256;
          c[u] = i < l_hi[k] ? codes[i] : 0;
          g[u] = gids && i < l_hi[k] ? gids[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (c[u] == -1) f(i0 + u * 256, g[u]);
      }
    __syncthreads();  // (the list is reused)
  }
}

__global__ void __launch_bounds__(256)
cg_insert(const uint32_t* __restrict__ gids, const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr,
          cg_sel sel, uint32_t n_lookups, uint64_t n_rows, uint64_t* table, cg_ws ws, uint32_t* err) {
  // the rank scan's status words, cleared for the kernel that follows
  if (blockIdx.y == 0)
    for (uint32_t j = blockIdx.x * 256 + threadIdx.x; j < ws.rtiles; j += gridDim.x * 256) ws.rstat[j] = 0;
  cg_lookups(sel, bag_ptr, codes, gids, n_lookups, err, [&](uint32_t i, uint32_t g) {
    if (g >= n_rows) {
      hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
      ws.slotof[i] = 0xFFFFFFFFu;
    } else {
      ws.slotof[i] = hl_cg_insert(table, ws.S - 1, g, i);
    }
  });
}

// Lookup i is a first occurrence iff it is a cold lookup of this call whose
// slot holds (its id, i); the running count of first occurrences numbers the
// staging rows.  In the fused plan (fused = 1) the ids of staging rows below
// cap go straight to the cold id list.
__global__ void __launch_bounds__(CG_RT_THREADS)
cg_rank(const uint32_t* __restrict__ gids, const int32_t* __restrict__ codes, uint32_t n_lookups,
        const uint64_t* __restrict__ table, cg_ws ws, int32_t* n_cold_dev, uint32_t epoch, uint32_t* cold_ids,
        int32_t cap, int fused, uint32_t* err) {
  __shared__ uint32_t s_tile, wt[CG_RT_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) s_tile = atomicInc(ws.ctr + CG_C_RTILE, gridDim.x - 1);
  __syncthreads();
  const uint32_t tile = s_tile;
  if (n_lookups == 0) {
    if (tile == 0 && tid == 0) {
      ws.ctr[CG_C_NCOLD] = 0;
      *n_cold_dev = 0;
    }
    return;
  }
  const uint64_t tb = (uint64_t)tile * CG_RT;
  if (tb >= n_lookups) return;
  const uint64_t lt = (1ull << lane) - 1ull;
  int32_t cd[4];
  uint32_t slot[4], g[4];
  bool first[4];
  // codes, slots and ids loaded together (the slot and id only matter for code -1)
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t i = tb + w * 256 + k * 64 + lane;
    const bool in = i < n_lookups;
    cd[k] = in ? codes[i] : 0;
    slot[k] = in ? ws.slotof[i] : 0xFFFFFFFFu;
    g[k] = in ? gids[i] : 0u;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (cd[k] != -1) slot[k] = 0xFFFFFFFFu;
  uint32_t wsum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t i = tb + w * 256 + k * 64 + lane;
    bool f = false;
    if (slot[k] < ws.S)  // a slot left by an earlier call fails the test below
      f = table[slot[k]] == (((uint64_t)(g[k] + 1) << 32) | (uint32_t)i);
    first[k] = f;
    wsum += (uint32_t)__popcll(__ballot(f));
  }
  if (lane == 0) wt[w] = wsum;
  __syncthreads();
  uint32_t before = 0, tc = 0;
  for (int q = 0; q < CG_RT_THREADS / 64; ++q) {
    if (q < w) before += wt[q];
    tc += wt[q];
  }
  const bool direct = gridDim.x <= HL_DIRECT_TILES;  // (else a look-back through inclusive prefixes)
  if (tid == 0) hl_st_store(ws.rstat + tile, hl_st_pack(epoch, tile == 0 && !direct ? HL_ST_PRE : HL_ST_AGG, tc));
  uint32_t ex = 0;
  if (direct) ex = hl_block_before(ws.rstat, tile, epoch, err);
  else if (tile > 0) ex = hl_block_lookback(ws.rstat, tile, epoch, err);
  if (!direct && tid == 0 && tile > 0) hl_st_store(ws.rstat + tile, hl_st_pack(epoch, HL_ST_PRE, ex + tc));
  uint32_t run = ex + before;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t i = tb + w * 256 + k * 64 + lane;
    const uint64_t m = __ballot(first[k]);
    if (first[k]) {
      const uint32_t u = run + (uint32_t)__popcll(m & lt);
      ws.uidx[slot[k]] = u;
      if (!fused) ws.fst[u] = g[k];
      else if (u < (uint32_t)cap) cold_ids[u] = g[k];
    }
    run += (uint32_t)__popcll(m);
    if (i == (uint64_t)n_lookups - 1) {
      ws.ctr[CG_C_NCOLD] = run;
      *n_cold_dev = (int32_t)run;
    }
  }
}

// The selected cold lookups point their codes at their staging rows and free
// their table slots; cold_ids[u] = id of staging row u.  When the rows do not
// fit: only the capacity bit and the slot clearing.  (A sample listed twice is
// done twice: the second time its codes are no longer -1, or are left alone.)
__global__ void __launch_bounds__(256)
cg_codes(const int32_t* __restrict__ bag_ptr, cg_sel sel, uint32_t n_lookups, uint64_t* table, cg_ws ws, int32_t cap,
         uint32_t k_cap, int32_t* codes, uint32_t* __restrict__ cold_ids, uint32_t* err) {
  const uint32_t ncold = ws.ctr[CG_C_NCOLD];
  const bool fits = ncold <= (uint32_t)cap;
  if (blockIdx.x == 0 && threadIdx.x == 0 && !fits) hl_flag(err, HL_DEVERR_CAPACITY);
  cg_lookups(sel, bag_ptr, codes, nullptr, n_lookups, err, [&](uint32_t i, uint32_t) {
    const uint32_t sl = ws.slotof[i];
    if (sl >= ws.S) return;
    if (fits) codes[i] = (int32_t)(k_cap + ws.uidx[sl]);
    table[sl] = 0;
  });
  if (!fits) return;
  const uint32_t gs = gridDim.x * gridDim.y * blockDim.x;
  for (uint32_t u = (blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; u < ncold; u += gs)
    cold_ids[u] = ws.fst[u];
}

// Row copy between host table and staging rows: TO_HOST = 0 copies
// staging[u] = host[ids[u]], TO_HOST = 1 copies host[ids[u]] = staging[u], for
// u < *n_dev.  A count above cap copies nothing and sets the capacity bit; an
// id >= n_rows is skipped and sets the range bit.  Each thread keeps 4 units in
// flight.  64 blocks already hold enough reads in flight to fill the host link
// (measured: fewer blocks lose bandwidth, more gain none); more blocks only fill
// the shared memory pipeline with slow host reads, which then stall the HBM
// traffic of kernels running beside the copy on other streams (a concurrent
// streaming kernel ran 5.5x slower beside 512 copy blocks, 1.5x beside 64).
template <typename V, bool TO_HOST>
__global__ void __launch_bounds__(256)
cg_copy(const uint32_t* __restrict__ ids, const int32_t* n_dev, int32_t cap, uint64_t n_rows, V* host, V* stg,
        uint32_t upr, uint32_t* err, hl_hook hk) {
  // a handover: block 0 signals as the copy starts (the copy before it on the
  // stream is complete), and every block waits for its inputs first
  hl_hook_head(hk);
  hl_hook_gate(hk);
  if (hk.gate) __syncthreads();
  const int32_t nd = *n_dev;
  if (nd < 0 || nd > cap) {
    if (blockIdx.x == 0 && threadIdx.x == 0) hl_flag(err, nd < 0 ? HL_DEVERR_OUT_OF_RANGE : HL_DEVERR_CAPACITY);
    return;
  }
  const uint64_t total = (uint64_t)nd * upr, gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t0 < total; t0 += 4 * gs) {
    V v[4];
    uint64_t dst[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t t = t0 + k * gs;
      dst[k] = ~0ull;
      if (t < total) {
        const uint32_t u = (uint32_t)(t / upr), c = (uint32_t)(t - (uint64_t)u * upr);
        const uint32_t g = ids[u];
        if (g < n_rows) {
          const uint64_t hp = (uint64_t)g * upr + c, sp = (uint64_t)u * upr + c;
          v[k] = TO_HOST ? stg[sp] : host[hp];
          dst[k] = TO_HOST ? hp : sp;
        } else if (c == 0) {
          hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (dst[k] != ~0ull) {
        if (TO_HOST) host[dst[k]] = v[k];
        else stg[dst[k]] = v[k];
      }
    }
  }
}

static hl_status cg_launch_copy(hl_handle* h, const uint32_t* ids, const int32_t* n_dev, int32_t cap, void* host,
                                void* stg, bool to_host, hipStream_t s) {
  const uint32_t rb = h->row_bytes;
  uint64_t units = (uint64_t)(cap > 0 ? cap : 1) * (rb / 4);
  uint32_t g = (uint32_t)((units + 1023) / 1024);
  g = g < 1 ? 1 : (g > 64 ? 64 : g);
  const hl_hook hk = to_host ? hl_hook{} : hl_hook_take(h);  // (the fetch carries the pipeline's handover)
#define CG_COPY(V)                                                                                             \
  if (to_host)                                                                                                 \
    HL_KERNEL(h, s, "cg_scatter", (cg_copy<V, true>), dim3(g), dim3(256), 0, s, ids, n_dev, cap, h->n_rows,     \
              (V*)host, (V*)stg, (uint32_t)(rb / sizeof(V)), h->d_err, hl_hook{});                             \
  else                                                                                                         \
    HL_KERNEL(h, s, "cg_fetch", (cg_copy<V, false>), dim3(g), dim3(256), 0, s, ids, n_dev, cap, h->n_rows,      \
              (V*)host, (V*)stg, (uint32_t)(rb / sizeof(V)), h->d_err, hk);
  if (rb % 16 == 0 && ((uintptr_t)host | (uintptr_t)stg) % 16 == 0) { CG_COPY(uint4) }
  else if (rb % 8 == 0 && ((uintptr_t)host | (uintptr_t)stg) % 8 == 0) { CG_COPY(uint2) }
  else if (rb % 4 == 0 && ((uintptr_t)host | (uintptr_t)stg) % 4 == 0) { CG_COPY(uint32_t) }
  else { CG_COPY(uint16_t) }
#undef CG_COPY
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_cold_plan(hl_handle* h, const uint32_t* gids, int32_t* codes, const int32_t* bag_ptr,
                                  int32_t n_samples, int32_t bps, int64_t n_lookups, const int32_t* sample_ids,
                                  const int32_t* n_sel_dev, int32_t n_sel_max, int32_t cap, uint32_t* cold_ids_out,
                                  int32_t* n_cold_dev, void* workspace, size_t ws_bytes, hl_stream stream) {
  if (!h || n_samples < 0 || bps < 1 || n_lookups < 0 || n_sel_max < 0 || cap < 0) return HL_ERR_INVALID_ARG;
  if (!n_cold_dev || !bag_ptr || !workspace) return HL_ERR_INVALID_ARG;
  if (!sample_ids && n_sel_max > n_samples) return HL_ERR_INVALID_ARG;
  if (n_lookups > 0 && (!gids || !codes || (cap > 0 && !cold_ids_out))) return HL_ERR_INVALID_ARG;
  if (n_lookups >= (1ll << 30) || (uint64_t)h->k_cap + (uint64_t)cap >= (1ull << 31)) return HL_ERR_UNSUPPORTED;
  if ((int64_t)n_samples * bps >= (1ll << 31)) return HL_ERR_UNSUPPORTED;
  const int64_t n_bags = (int64_t)n_samples * bps;
  if (ws_bytes < hl_cold_ws_bytes(h, n_lookups, n_bags, n_samples)) return HL_ERR_CAPACITY;
  hl_ws_note(h, workspace, HL_WSK_OTHER);
  hipStream_t s = (hipStream_t)stream;
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  cg_ws ws;
  cg_carve(c, ws, (uint32_t)n_lookups);
  uint64_t* table = nullptr;
  hl_status st = cg_table(h, ws.S, s, &table);
  if (st != HL_OK) return st;
  const uint32_t n = (uint32_t)n_lookups;
  // selection: the first n_sel_max samples (no list) or the listed ones; an
  // empty selection inserts nothing
  int32_t tps = 8;
  while (tps < 256 && (int64_t)tps * n_samples < n_lookups) tps *= 2;
  uint32_t parts = 1;  // blocks per listed sample: 1024 lookups each on average, at most 1024 of them
  if (sample_ids && n_samples > 0) parts = (uint32_t)std::min<int64_t>(1 + n_lookups / (1024ll * n_samples), 1024);
  const cg_sel sel{sample_ids, n_sel_dev, n_sel_max, n_samples, bps, tps, (int64_t)n_sel_max * bps};
  uint32_t ib = 0;
  if (n_sel_max > 0) {
    const uint64_t listed = std::min(n_sel_max, std::max(n_samples, 1));  // (a longer list: cg_lookups)
    // (a list is looked through for ids that name no sample also where there are no lookups)
    ib = sample_ids ? std::min(hl_div_up(listed * tps, 256), 1u << 16) : hl_div_up(n, 256);
  }
  if (ib > 0)
    HL_KERNEL(h, s, "cg_insert", cg_insert, dim3(ib, parts), dim3(256), 0, s, gids, codes, bag_ptr, sel, n, h->n_rows, table, ws,
              h->d_err);
  // the insert kernel cleared the status words, so one fixed tag serves every
  // call (and every replay of a captured graph)
  const uint32_t epoch = 1;
  HL_KERNEL(h, s, "cg_rank", cg_rank, dim3(ws.rtiles), dim3(CG_RT_THREADS), 0, s, gids, codes, ib > 0 ? n : 0u, table, ws,
            n_cold_dev, epoch, nullptr, 0, 0, h->d_err);
  if (ib > 0 && n > 0)
    HL_KERNEL(h, s, "cg_codes", cg_codes, dim3(ib, parts), dim3(256), 0, s, bag_ptr, sel, n, table, ws, cap, h->k_cap, codes,
              cold_ids_out, h->d_err);
  HL_LAUNCHED();
  return HL_OK;
}

// The fused plan's cold state: the cold regions carved after the grouping's
// region of the workspace.
static hl_carver cg_fused_carver(const hl_handle* h, void* workspace, size_t ws_bytes, int64_t n_lookups,
                                 int64_t n_bags) {
  hl_carver c = hl_carver::after_header(workspace, ws_bytes);
  c.off = hl_bwd_ws_bytes(h, n_lookups, n_bags);
  return c;
}

size_t hl_plan_ws_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags, int32_t max_samples) {
  hl_carver c = cg_fused_carver(h, nullptr, 0, max_lookups, max_bags);
  cg_ws ws;
  cg_carve(c, ws, (uint32_t)max_lookups);
  return c.off;
}

hl_status hl_cold_fused_begin(hl_handle* h, int64_t n_lookups, int64_t n_bags, int32_t n_samples, int32_t cap,
                              void* workspace, size_t ws_bytes, hipStream_t s, hl_cg_fused* out) {
  *out = hl_cg_fused{};
  if (!h || !workspace || n_lookups <= 0 || n_bags <= 0 || n_samples <= 0 || cap < 0) return HL_ERR_INVALID_ARG;
  if (n_lookups >= (1ll << 30) || (uint64_t)h->k_cap + (uint64_t)cap >= (1ull << 31)) return HL_ERR_UNSUPPORTED;
  if (ws_bytes < hl_plan_ws_bytes(h, n_lookups, n_bags, n_samples)) return HL_ERR_CAPACITY;
  hl_carver c = cg_fused_carver(h, workspace, ws_bytes, n_lookups, n_bags);
  cg_ws ws;
  cg_carve(c, ws, (uint32_t)n_lookups);
  // no growth here: a larger table is allocated by a plain cold plan, after
  // its waits (the table is shared with the steps still in flight)
  if (h->cg_slots < ws.S || !h->cg_table) return HL_ERR_CAPACITY;
  (void)s;
  out->table = h->cg_table;
  out->S = ws.S;
  out->slotof = ws.slotof;
  out->uidx = ws.uidx;
  out->rstat = ws.rstat;
  out->rtiles = ws.rtiles;
  out->ncold = ws.ctr + CG_C_NCOLD;
  out->cap = cap;
  return HL_OK;
}

hl_status hl_cold_rank_fused(hl_handle* h, const uint32_t* gids, const int32_t* codes, int64_t n_lookups,
                             uint32_t* cold_ids, int32_t* n_cold_dev, void* workspace, const hl_cg_fused& cf,
                             hipStream_t s) {
  if (!h || !gids || !codes || !n_cold_dev || !workspace || !cf.table || n_lookups <= 0) return HL_ERR_INVALID_ARG;
  if (cf.cap > 0 && !cold_ids) return HL_ERR_INVALID_ARG;
  cg_ws ws{};
  ws.ctr = reinterpret_cast<uint32_t*>(workspace) + HL_HDR_COLD;
  ws.S = cf.S;
  ws.uidx = cf.uidx;
  ws.slotof = cf.slotof;
  ws.rstat = cf.rstat;
  ws.rtiles = cf.rtiles;
  // the dispatch kernel cleared the status words
  const uint32_t epoch = 1;
  HL_KERNEL(h, s, "cg_rank", cg_rank, dim3(cf.rtiles), dim3(CG_RT_THREADS), 0, s, gids, codes, (uint32_t)n_lookups,
            cf.table, ws, n_cold_dev, epoch, cold_ids, cf.cap, 1, h->d_err);
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_cold_reserve(hl_handle* h, int64_t max_lookups, hl_stream stream) {
  if (!h || max_lookups < 0) return HL_ERR_INVALID_ARG;
  if (max_lookups >= (1ll << 30)) return HL_ERR_UNSUPPORTED;
  uint64_t* t = nullptr;
  return cg_table(h, cg_table_slots((uint32_t)max_lookups), (hipStream_t)stream, &t);
}

extern "C" hl_status hl_cold_fetch(hl_handle* h, const uint32_t* cold_ids, const int32_t* n_cold_dev, int32_t cap,
                                   const void* w_host, void* staging, hl_stream stream) {
  if (!h || cap < 0 || !n_cold_dev) return HL_ERR_INVALID_ARG;
  if (cap > 0 && (!cold_ids || !w_host || !staging)) return HL_ERR_INVALID_ARG;
  if (cap == 0) return HL_OK;
  return cg_launch_copy(h, cold_ids, n_cold_dev, cap, const_cast<void*>(w_host), staging, false, (hipStream_t)stream);
}

extern "C" hl_status hl_cold_scatter(hl_handle* h, const uint32_t* cold_ids, const int32_t* n_cold_dev, int32_t cap,
                                     const void* staging, void* w_host, hl_stream stream) {
  if (!h || cap < 0 || !n_cold_dev) return HL_ERR_INVALID_ARG;
  if (cap > 0 && (!cold_ids || !w_host || !staging)) return HL_ERR_INVALID_ARG;
  if (cap == 0) return HL_OK;
  return cg_launch_copy(h, cold_ids, n_cold_dev, cap, w_host, const_cast<void*>(staging), true, (hipStream_t)stream);
}

extern "C" hl_status hl_cold_gather(hl_handle* h, const uint32_t* gids, int32_t* codes, const int32_t* bag_ptr,
                                    int32_t n_samples, int32_t bps, int64_t n_lookups,
                                    const int32_t* sample_ids, const int32_t* n_sel_dev, int32_t n_sel_max,
                                    const void* w_host, void* staging, int32_t cap, uint32_t* cold_ids_out,
                                    int32_t* n_cold_dev, void* workspace, size_t ws_bytes,
                                    hl_stream stream) {
  if (h && n_lookups > 0 && cap > 0 && (!w_host || !staging)) return HL_ERR_INVALID_ARG;
  hl_status st = hl_cold_plan(h, gids, codes, bag_ptr, n_samples, bps, n_lookups, sample_ids, n_sel_dev, n_sel_max,
                              cap, cold_ids_out, n_cold_dev, workspace, ws_bytes, stream);
  if (st != HL_OK || n_lookups == 0) return st;
  return hl_cold_fetch(h, cold_ids_out, n_cold_dev, cap, w_host, staging, stream);
}
