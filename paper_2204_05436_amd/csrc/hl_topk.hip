// Hot-set selection from access counts: exact top-K by (count desc, id asc)
// among rows accessed at least once, and installation of an explicit hot set.
//
// A row is hot iff count > tau, or count == tau and fewer than need_tau rows
// with count == tau have a smaller id, tau being the K-th largest count (when
// K rows or fewer were accessed: iff it was accessed).
//
//   tk_hist   -- the only pass over every count: a bit per accessed row goes to
//                the bitmap (the later passes follow it and read a count only
//                where a 64-row word holds an accessed row: 0.4% of 9.9e7 rows
//                are, after 16 mini-batches), and the accessed counts go into a
//                histogram of 896 bins, exact below 64 and of 32 bins per power
//                of two above.  Its last block finds the bin of tau.
//   tk_refine -- x2: the histogram of the counts inside that bin, 2^13 bins at
//                a time until a bin holds one value (nothing to do once it does:
//                for a tau below 64 at once, below 2^19 after the first).
//   tk_tiles  -- per tile of 16384 rows the counts above and equal to tau; its
//                last block scans them.
//   tk_emit   -- the hot ids in ascending order, so hot slots are ascending-id
//                ranks by construction, the membership bitmap, the rank
//                directory, and (on request) the counts of the accessed rows
//                back to zero.
//
// tk_hist is bound by HBM (reads every count), the others by latency and the
// sparse counts.  9.9e7 rows, 423k accessed: 1000 us with a radix select of
// four passes over all counts, a serial merge of its 1024 blocks' histograms
// and a rewrite of every count; 128 us like this.
#include "hl_internal.h"

#define HL_TRY_ST(x)                  \
  do {                                \
    const hl_status _st = (x);        \
    if (_st != HL_OK) return _st;     \
  } while (0)

#define TK_THREADS 1024
#define TK_BLOCKS 512     // blocks of the pass over all rows: two per compute unit
#define TK_BLOCKS_SPARSE 256
#define TK_BINS 896       // tk_hist: 64 + 26 * 32
#define TK_RBITS 13
#define TK_RBINS (1 << TK_RBITS)
#define TK_TILE 16384     // rows per tk_emit block: 256 words, one per thread when they are placed
#define TK_TWORDS (TK_TILE / 64)
// scratch words: the state, then the histogram (left zero by every call), then
// the tiles' counts
#define S_LO 0        // the candidates: counts of [lo, lo + 2^lg)
#define S_LG 1
#define S_NEED 2      // of them are hot
#define S_ALL 3       // every accessed row is hot
#define S_NHOT 4
#define S_CTR 8       // blocks done, per kernel (wraps to 0)
#define TK_STATE 16
#define TK_HIST TK_STATE
#define TK_TILES (TK_STATE + TK_RBINS)

static uint64_t tk_n_tiles(uint64_t n_rows) { return (n_rows + TK_TILE - 1) / TK_TILE; }

size_t hl_topk_scratch_bytes(uint64_t n_rows) { return 4 * (TK_TILES + 2 * (size_t)tk_n_tiles(n_rows) + 64); }

// State that crosses blocks inside a launch (histogram bins, tile counts) is
// written by agent-scope atomics whose old value is waited for before the block
// counts itself done, and read by agent-scope loads in the last block: no fence
// (a fence at agent scope writes back the L2).
// odd: an impossible property of this thread's old values; it is always false,
// and testing it is what makes the block wait for them.
__device__ __forceinline__ bool tk_last_block(uint32_t* ctr, bool odd) {
  __shared__ uint32_t s_last;
  const uint32_t any = __syncthreads_or(odd) ? 1u : 0u;
  if (threadIdx.x == 0) s_last = atomicInc(ctr, gridDim.x - 1) + any == gridDim.x - 1 ? 1u : 0u;
  __syncthreads();
  return s_last != 0;
}
__device__ __forceinline__ uint32_t tk_load(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Adds the block's LDS histogram to the global one; returns tk_last_block's odd
// (a bin never holds 2^32 - 1 rows).
template <int NB>
__device__ __forceinline__ bool tk_add_hist(const uint32_t* h, uint32_t* g) {
  bool odd = false;
  for (int j = threadIdx.x; j < NB; j += TK_THREADS)
    if (h[j]) odd = odd || atomicAdd(g + j, h[j]) == 0xFFFFFFFFu;
  return odd;
}

// The bin, from the top, where the running count reaches `need` (1 <= need <=
// the bins' total): *bin, and *above = the count of the bins over it.  NB / 1024
// consecutive bins per thread; leaves the global histogram zero.
template <int NB>
__device__ __forceinline__ void tk_select(uint32_t* g, uint32_t need, uint32_t* bin, uint32_t* above,
                                          uint32_t* total) {
  constexpr int PER = (NB + TK_THREADS - 1) / TK_THREADS;
  __shared__ uint32_t ws[TK_THREADS / 64], s_bin, s_above;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t c[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = NB - 1 - (threadIdx.x * PER + j);  // descending bins
    c[j] = b >= 0 ? tk_load(g + b) : 0u;
    sum += c[j];
  }
  uint32_t x = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) ws[w] = x;
  __syncthreads();
  uint32_t before = x - sum, tot = 0;
  for (int q = 0; q < TK_THREADS / 64; ++q) {
    if (q < w) before += ws[q];
    tot += ws[q];
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = NB - 1 - (threadIdx.x * PER + j);
    if (b >= 0 && before < need && before + c[j] >= need) {
      s_bin = (uint32_t)b;
      s_above = before;
    }
    before += c[j];
    if (b >= 0 && c[j]) g[b] = 0;
  }
  __syncthreads();
  *bin = s_bin;
  *above = s_above;
  *total = tot;
}

// bins of tk_hist: counts below 64 one each, then 32 per power of two
__device__ __forceinline__ uint32_t tk_bin(uint32_t c) {
  if (c < 64) return c;
  const uint32_t e = 31 - __clz(c);
  return 64 + (e - 6) * 32 + ((c >> (e - 5)) & 31u);
}

// A wave takes 1024 consecutive rows at a time: 16 coalesced loads in flight
// per lane, one ballot per 64-row word.
__global__ void __launch_bounds__(TK_THREADS)
tk_hist(const uint32_t* __restrict__ counts, uint64_t n, uint64_t n_words, uint64_t* __restrict__ bitmap,
        uint32_t* st, uint32_t k) {
  __shared__ uint32_t hist[TK_BINS];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int j = threadIdx.x; j < TK_BINS; j += TK_THREADS) hist[j] = 0;
  __syncthreads();
  constexpr int WV = TK_THREADS / 64;
  for (uint64_t w0 = ((uint64_t)blockIdx.x * WV + w) * 16; w0 < n_words; w0 += (uint64_t)gridDim.x * WV * 16) {
    const uint64_t base = w0 * 64;
    uint32_t c[16];
    if (base + 1024 <= n) {
#pragma unroll
      for (int j = 0; j < 16; ++j) c[j] = counts[base + j * 64 + lane];
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) c[j] = base + j * 64 + lane < n ? counts[base + j * 64 + lane] : 0u;
    }
    uint64_t mine = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const uint64_t m = __ballot(c[j] != 0);
      if (lane == j) mine = m;
      if (c[j]) atomicAdd(&hist[tk_bin(c[j])], 1u);
    }
    if (lane < 16 && w0 + lane < n_words) bitmap[w0 + lane] = mine;
  }
  __syncthreads();
  if (!tk_last_block(st + S_CTR, tk_add_hist<TK_BINS>(hist, st + TK_HIST))) return;
  uint32_t bin, above, total;
  tk_select<TK_BINS>(st + TK_HIST, k ? k : 1, &bin, &above, &total);
  if (threadIdx.x != 0) return;
  const bool all = total <= k;
  st[S_ALL] = all;
  st[S_NEED] = all || k == 0 ? 0u : k - above;
  st[S_LO] = all ? 0u : (k == 0 ? 0xFFFFFFFFu : (bin < 64 ? bin : (32u + (bin & 31u)) << ((bin - 64) / 32 + 1)));
  st[S_LG] = all || k == 0 || bin < 64 ? 0u : (bin - 64) / 32 + 1;
}

// Visits the accessed rows of words [w0, w0 + 64) with a wave: f(j, word of
// accessed rows, this lane's count), eight words' counts in flight.  word: lane
// j's is word w0 + j.
template <typename F>
__device__ __forceinline__ void tk_visit(const uint32_t* __restrict__ counts, uint64_t n, uint64_t w0, uint64_t word,
                                         F f) {
  const int lane = threadIdx.x & 63;
  uint64_t todo = __ballot(word != 0);
  while (todo) {
    int j[8];
    uint32_t c[8];
    uint64_t t = todo;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      j[q] = t ? __ffsll((unsigned long long)t) - 1 : -1;
      t &= t - 1;
      const uint64_t g = (w0 + (uint64_t)(j[q] < 0 ? 0 : j[q])) * 64 + lane;
      c[q] = j[q] >= 0 && g < n ? counts[g] : 0u;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (j[q] >= 0) f(j[q], c[q]);
    todo = t;
  }
}

__global__ void __launch_bounds__(TK_THREADS)
tk_refine(const uint32_t* __restrict__ counts, uint64_t n, uint64_t n_words, const uint64_t* __restrict__ bitmap,
          uint32_t* st) {
  const uint32_t lg = st[S_LG], lo = st[S_LO];
  if (lg == 0) return;
  __shared__ uint32_t hist[TK_RBINS];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int j = threadIdx.x; j < TK_RBINS; j += TK_THREADS) hist[j] = 0;
  __syncthreads();
  const uint32_t sh = lg > TK_RBITS ? lg - TK_RBITS : 0;
  constexpr int WV = TK_THREADS / 64;
  for (uint64_t w0 = ((uint64_t)blockIdx.x * WV + w) * 64; w0 < n_words; w0 += (uint64_t)gridDim.x * WV * 64)
    tk_visit(counts, n, w0, w0 + lane < n_words ? bitmap[w0 + lane] : 0ull, [&](int, uint32_t c) {
      if (c >= lo && ((c - lo) >> lg) == 0) atomicAdd(&hist[(c - lo) >> sh], 1u);
    });
  __syncthreads();
  const uint32_t need = st[S_NEED];
  if (!tk_last_block(st + S_CTR + 1, tk_add_hist<TK_RBINS>(hist, st + TK_HIST))) return;
  uint32_t bin, above, total;
  tk_select<TK_RBINS>(st + TK_HIST, need, &bin, &above, &total);
  if (threadIdx.x != 0) return;
  st[S_NEED] = need - above;
  st[S_LO] = lo + (bin << sh);
  st[S_LG] = sh;
}

// This lane's word of the tile (word w0 + lane) split into rows above tau and
// equal to it; all: every accessed row counts as above.
__device__ __forceinline__ void tk_split(const uint32_t* __restrict__ counts, uint64_t n, uint64_t w0, uint64_t word,
                                         bool all, uint32_t tau, uint64_t* above, uint64_t* equal) {
  const int lane = threadIdx.x & 63;
  *above = all ? word : 0ull;
  *equal = 0;
  if (all) return;
  uint64_t a = 0, e = 0;
  tk_visit(counts, n, w0, word, [&](int j, uint32_t c) {
    const uint64_t ma = __ballot(c > tau), me = __ballot(c == tau && c != 0);
    if (lane == j) {
      a = ma;
      e = me;
    }
  });
  *above = a;
  *equal = e;
}

// Rows above and equal to tau per tile: a block takes TK_SUB tiles at a time,
// 4 waves of 64 words each.  (Every block ends with an atomic on one counter,
// and these complete one after another: a block per tile took 91 us for 6057
// tiles, 21 like this.)  The last block turns both arrays into exclusive
// prefixes, each thread a run of consecutive tiles, and stores the number of
// hot rows.
#define TK_SUB (TK_THREADS / 256)
__global__ void __launch_bounds__(TK_THREADS)
tk_tiles(const uint32_t* __restrict__ counts, uint64_t n, uint64_t n_words, const uint64_t* __restrict__ bitmap,
         uint32_t* st, uint32_t n_tiles, uint32_t* rank_last) {
  constexpr int WV = TK_THREADS / 64;
  __shared__ uint32_t rs[WV], re[WV];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t* ts = st + TK_TILES;
  uint32_t* te = ts + n_tiles;
  const bool all = st[S_ALL] != 0;
  const uint32_t tau = st[S_LO];
  bool odd = false;
  for (uint32_t t0 = blockIdx.x * TK_SUB; t0 < n_tiles; t0 += gridDim.x * TK_SUB) {
    const uint64_t w0 = (uint64_t)t0 * TK_TWORDS + w * 64;
    uint64_t a, e;
    tk_split(counts, n, w0, w0 + lane < n_words ? bitmap[w0 + lane] : 0ull, all, tau, &a, &e);
    uint32_t s = (uint32_t)__popcll(a), q = (uint32_t)__popcll(e);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s += __shfl_xor(s, o);
      q += __shfl_xor(q, o);
    }
    if (lane == 0) {
      rs[w] = s;
      re[w] = q;
    }
    __syncthreads();
    if (threadIdx.x < 2 * TK_SUB) {
      const uint32_t j = threadIdx.x >> 1;
      const uint32_t* r = (threadIdx.x & 1 ? re : rs) + 4 * j;
      if (t0 + j < n_tiles)
        odd = odd || __hip_atomic_exchange((threadIdx.x & 1 ? te : ts) + t0 + j, r[0] + r[1] + r[2] + r[3],
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0xFFFFFFFFu;
    }
    __syncthreads();  // (rs and re are reused)
  }
  if (!tk_last_block(st + S_CTR + 2, odd)) return;
  const uint32_t per = (n_tiles + TK_THREADS - 1) / TK_THREADS, t0 = threadIdx.x * per;
  uint32_t ss = 0, se = 0;
  for (uint32_t j = 0; j < per; j += 8) {
    uint32_t vs[8], ve[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t t = t0 + j + u;
      const bool in = j + u < per && t < n_tiles;
      vs[u] = in ? tk_load(ts + t) : 0u;
      ve[u] = in ? tk_load(te + t) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      ss += vs[u];
      se += ve[u];
    }
  }
  uint32_t is = ss, ie = se;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t x = __shfl_up(is, o), y = __shfl_up(ie, o);
    if (lane >= o) {
      is += x;
      ie += y;
    }
  }
  __syncthreads();
  if (lane == 63) {
    rs[w] = is;
    re[w] = ie;
  }
  __syncthreads();
  uint32_t ps = is - ss, pe = ie - se, tots = 0, tote = 0;
  for (int x = 0; x < WV; ++x) {
    if (x < w) {
      ps += rs[x];
      pe += re[x];
    }
    tots += rs[x];
    tote += re[x];
  }
  for (uint32_t j = 0; j < per; j += 8) {
    uint32_t vs[8], ve[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t t = t0 + j + u;
      const bool in = j + u < per && t < n_tiles;
      vs[u] = in ? tk_load(ts + t) : 0u;
      ve[u] = in ? tk_load(te + t) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t t = t0 + j + u;
      if (j + u < per && t < n_tiles) {
        ts[t] = ps;
        te[t] = pe;
      }
      ps += vs[u];
      pe += ve[u];
    }
  }
  if (threadIdx.x == 0) {
    const uint32_t need = st[S_NEED];
    const uint32_t nh = tots + (tote < need ? tote : need);
    st[S_NHOT] = nh;
    *rank_last = nh;
  }
}

// Output pass, a tile per block: each thread places one 64-row word, its hot
// rows after the hot rows of the words before it (the rank directory takes the
// first of every four words' places).
__global__ void __launch_bounds__(256)
tk_emit(uint32_t* __restrict__ counts, uint64_t n, uint64_t n_words, uint64_t* __restrict__ bitmap,
        const uint32_t* st, uint32_t n_tiles, uint32_t* __restrict__ hot_ids, uint32_t* __restrict__ rank, int reset) {
  __shared__ uint32_t wsum[4], wequ[4];
  const uint32_t need = st[S_NEED];
  const uint32_t* ts = st + TK_TILES;
  const uint32_t* te = ts + n_tiles;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t w0 = (uint64_t)blockIdx.x * TK_TWORDS + w * 64;
  const uint64_t word = w0 + lane < n_words ? bitmap[w0 + lane] : 0ull;
  uint64_t a, e;
  tk_split(counts, n, w0, word, st[S_ALL] != 0, st[S_LO], &a, &e);
  const uint32_t ns = (uint32_t)__popcll(a), ne = (uint32_t)__popcll(e);
  uint32_t is = ns, ie = ne;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t x = __shfl_up(is, o), y = __shfl_up(ie, o);
    if (lane >= o) {
      is += x;
      ie += y;
    }
  }
  if (lane == 63) {
    wsum[w] = is;
    wequ[w] = ie;
  }
  __syncthreads();
  uint32_t sb = ts[blockIdx.x] + is - ns, eb = te[blockIdx.x] + ie - ne;
  for (int j = 0; j < w; ++j) {
    sb += wsum[j];
    eb += wequ[j];
  }
  const uint32_t pos = sb + (eb < need ? eb : need);
  // the first need - eb equal rows of the word are hot
  uint32_t take = eb < need ? need - eb : 0u;
  uint64_t sel = a;
  if (take >= ne) {
    sel |= e;
  } else {
    for (; take; --take) {
      sel |= e & (~e + 1);
      e &= e - 1;
    }
  }
  if (w0 + lane < n_words) {
    bitmap[w0 + lane] = sel;
    if ((lane & 3) == 0) rank[(w0 + lane) >> 2] = pos;
  }
  const uint64_t g0 = (w0 + lane) * 64;
  uint32_t p = pos;
  for (uint64_t m = sel; m; m &= m - 1) hot_ids[p++] = (uint32_t)(g0 + __ffsll((unsigned long long)m) - 1);
  if (reset)
    for (uint64_t todo = __ballot(word != 0); todo; todo &= todo - 1) {
      const int j = __ffsll((unsigned long long)todo) - 1;
      const uint64_t m = __shfl((unsigned long long)word, j);
      if ((m >> lane) & 1ull) counts[(w0 + j) * 64 + lane] = 0;
    }
}

extern "C" hl_status hl_profile_topk(hl_handle* h, uint32_t k, uint32_t* hot_ids_out, uint32_t* n_hot_out,
                                     int reset_counts, hl_stream stream) {
  if (!h || !hot_ids_out) return HL_ERR_INVALID_ARG;
  if (k > h->k_cap) return HL_ERR_OUT_OF_RANGE;
  hipStream_t s = (hipStream_t)stream;
  // (the bitmap's words cover n_tiles4k * 4096 rows; those past n_rows stay 0)
  const uint64_t n = h->n_rows, words = h->n_tiles4k * 64;
  const uint32_t tiles = hl_div_up(words, TK_TWORDS);
  uint32_t nb = hl_div_up(words, 16 * (TK_THREADS / 64)), nr = hl_div_up(words, 64 * (TK_THREADS / 64));
  if (nb > TK_BLOCKS) nb = TK_BLOCKS;
  if (nr > TK_BLOCKS_SPARSE) nr = TK_BLOCKS_SPARSE;
  HL_KERNEL(h, s, "tk_hist", tk_hist, dim3(nb), dim3(TK_THREADS), 0, s, h->d_counts, n, words, h->d_bitmap, h->d_tk, k);
  for (int r = 0; r < 2; ++r)  // (a bin of tk_hist holds at most 2^26 values)
    HL_KERNEL(h, s, "tk_refine", tk_refine, dim3(nr), dim3(TK_THREADS), 0, s, h->d_counts, n, words, h->d_bitmap,
              h->d_tk);
  HL_KERNEL(h, s, "tk_tiles", tk_tiles, dim3(nr), dim3(TK_THREADS), 0, s, h->d_counts, n, words, h->d_bitmap, h->d_tk, tiles,
            h->d_rank + h->n_tiles4k * 16);
  HL_KERNEL(h, s, "tk_emit", tk_emit, dim3(tiles), dim3(256), 0, s, h->d_counts, n, words, h->d_bitmap, h->d_tk, tiles,
            hot_ids_out, h->d_rank, reset_counts);
  HL_LAUNCHED();
  HL_TRY_ST(hl_table_bounds(h, s));
  uint32_t nh = 0;
  HL_HIP(hipMemcpyAsync(&nh, h->d_tk + S_NHOT, 4, hipMemcpyDeviceToHost, s));
  HL_HIP(hipStreamSynchronize(s));
  h->n_hot = nh;
  if (n_hot_out) *n_hot_out = nh;
  return HL_OK;
}

// ----------------------------------------------------------------------------- explicit hot set
__global__ void __launch_bounds__(256)
sh_bits(const uint32_t* __restrict__ ids, uint32_t n_hot, uint64_t n_rows, uint64_t* bitmap, uint32_t* err) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_hot; i += gridDim.x * blockDim.x) {
    const uint32_t g = ids[i];
    const bool ok = g < n_rows && (i == 0 || ids[i - 1] < g);
    if (!ok) { hl_flag(err, HL_DEVERR_BAD_HOTSET); continue; }
    atomicOr((unsigned long long*)(bitmap + (g >> 6)), 1ull << (g & 63));
  }
}

__global__ void __launch_bounds__(256)
sh_rank(const uint32_t* __restrict__ ids, uint32_t n_hot, uint64_t n_entries, uint32_t* rank) {
  for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_entries;
       j += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t key = j * 256;
    uint32_t a = 0, b = n_hot;  // first index with ids[idx] >= key
    while (a < b) {
      uint32_t m = (a + b) >> 1;
      if ((uint64_t)ids[m] < key) a = m + 1; else b = m;
    }
    rank[j] = a;
  }
}

extern "C" hl_status hl_set_hot(hl_handle* h, const uint32_t* hot_ids, uint32_t n_hot, hl_stream stream) {
  if (!h || (n_hot && !hot_ids)) return HL_ERR_INVALID_ARG;
  if (n_hot > h->k_cap || n_hot > h->n_rows) return HL_ERR_OUT_OF_RANGE;
  hipStream_t s = (hipStream_t)stream;
  const uint64_t tiles = h->n_tiles4k;
  hl_status st = hl_fill32((uint32_t*)h->d_bitmap, tiles * 128, 0, s);
  if (st != HL_OK) return st;
  if (n_hot) {
    uint32_t g = hl_div_up(n_hot, 256);
    if (g > 4096) g = 4096;
    HL_KERNEL(h, s, "sh_bits", sh_bits, dim3(g), dim3(256), 0, s, hot_ids, n_hot, h->n_rows, h->d_bitmap, h->d_err);
  }
  const uint64_t ne = tiles * 16 + 1;
  uint32_t g2 = hl_div_up(ne, 256);
  if (g2 > 4096) g2 = 4096;
  HL_KERNEL(h, s, "sh_rank", sh_rank, dim3(g2), dim3(256), 0, s, hot_ids, n_hot, ne, h->d_rank);
  HL_LAUNCHED();
  HL_TRY_ST(hl_table_bounds(h, s));
  h->n_hot = n_hot;
  return HL_OK;
}
