// The Embedding Access Logger with SRRIP replacement (Sec. V-B): instead of a
// counter per row, a set-associative cache of row ids with a 2-bit
// re-reference prediction value (RRPV) per way.  Id g lives in set
// mix(g) % n_sets (mix: the 32-bit finalizer of MurmurHash3); a hit sets its
// RRPV to 0; a miss takes the first way whose RRPV is 3, ageing the set by one
// until one is, and enters with RRPV 2.  Empty ways hold 0xFFFFFFFF and RRPV 3.
// The hot set the logger yields is every id it holds, ascending.
//
// Sets are independent, so the stream-order semantics hold per set: a batch's
// (set, id) pairs are sorted by set with the library's stable radix sort
// (ties keep lookup order), and each set's run is replayed in order (eal_runs).
#include "hl_internal.h"

#define EAL_MAX_WAYS 16
#define EAL_EMPTY 0xFFFFFFFFu

struct hl_eal {
  hl_handle* h;
  uint32_t n_sets;
  int32_t ways;
  int64_t max_n;    // lookups per call
  uint32_t* tag;    // [n_sets * ways]
  uint8_t* rrpv;    // [n_sets * ways]
  uint32_t* cnt;    // [1] held ids (extraction)
  void* ws;         // sort workspace, zero-filled once
  size_t ws_bytes;
  uint32_t sort_n;  // the sort's capacity: max(max_n, n_sets * ways)
};

__global__ void eal_init(uint32_t* tag, uint8_t* rrpv, uint64_t m) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
    tag[i] = EAL_EMPTY;
    rrpv[i] = 3;
  }
}

// The RRPVs of a set's ways as two bit planes (way w: bit w of hi and lo), all
// ways at once per operation.
struct eal_rr {
  uint32_t hi, lo;
  __device__ __forceinline__ void hit(uint32_t ways_hit) {
    hi &= ~ways_hit;
    lo &= ~ways_hit;
  }
  // the way a miss takes: the first at 3, the set aged by one until some way is
  // (three times at most); it enters at 2
  __device__ __forceinline__ int take(uint32_t all) {
    for (int age = 0; age < 3 && !(hi & lo); ++age) {
      hi ^= lo;
      lo = ~lo & all;
    }
    const int v = __ffs((int)(hi & lo)) - 1;
    lo &= ~(1u << v);
    return v;
  }
};

// Replays each set's run.  A run's first EAL_SHORT accesses are replayed by 16
// lanes, one per way, so a wave replays four runs at once (the block's heads
// listed and its positions held in LDS): a step is a compare, a ballot and, on a
// miss, three ballots that find the way to take.  The rest of a longer run is
// replayed by the whole wave, 64 accesses at a time: if they name at most
// EAL_FEW ids, all held, those ways' RRPVs are cleared and that is all (the order
// of hits does not matter); else lane w holds way w's id and the mask of the
// accesses that name it, so all accesses up to the first miss are one step, and a
// miss is a step of scalar work.  Bound by the latency of the steps (11 of 15.5
// us without the long runs) and by the longest run: a popular row gives its set
// two thousand.  212,992 accesses on 26,436 sets of 16: 634 us with a thread per
// run; 22 with the first 8 accesses by a thread; 15.5 like this (EAL_SHORT 8, 12,
// 16: 15.5, 15.8, 16.4).  Whole calls with 4, 8, 12 and 16, Zipf 1.1: 212,992
// accesses 86.1, 86.8, 86.6, 87.8; a million 324, 324, 324, 327; ids of equal
// weight, which give no set a long run: 39.5, 36.0, 35.1, 34.8 and 125, 119, 112, 105.
#define EAL_THREADS 256
#define EAL_SHORT 8
#define EAL_AHEAD 4  // times 64 accesses of a long run loaded at once
#define EAL_FEW 4    // ids of 64 accesses looked up one by one first
#define EAL_LDS (EAL_THREADS + EAL_SHORT + 64)  // positions in LDS: the first 64 past EAL_SHORT of every run
__global__ void __launch_bounds__(EAL_THREADS)
eal_runs(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint32_t n, uint32_t n_sets,
         int32_t ways, uint32_t* __restrict__ tag, uint8_t* __restrict__ rrpv) {
  __shared__ uint32_t lk[EAL_LDS + 1], lv[EAL_LDS];
  __shared__ uint32_t heads[EAL_THREADS], wc[EAL_THREADS / 64];
  const uint32_t b0 = blockIdx.x * EAL_THREADS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t j = threadIdx.x; j < EAL_LDS + 1; j += EAL_THREADS) {
    const uint32_t q = b0 + j;  // lk[j] is position b0 - 1 + j
    lk[j] = q > 0 && q - 1 < n ? keys[q - 1] : EAL_EMPTY;  // (past n: no set)
    if (j < EAL_LDS) lv[j] = q < n ? vals[q] : 0u;
  }
  __syncthreads();
  const uint32_t all = (1u << ways) - 1u;
  // the positions where a run begins
  const uint32_t key = lk[threadIdx.x + 1];
  const bool head = key < n_sets && lk[threadIdx.x] != key;
  const uint64_t hm = __ballot(head);
  if (lane == 0) wc[wave] = (uint32_t)__popcll(hm);
  __syncthreads();
  uint32_t before = 0, nh = 0;
#pragma unroll
  for (int q = 0; q < EAL_THREADS / 64; ++q) {
    before += q < wave ? wc[q] : 0u;
    nh += wc[q];
  }
  if (head) heads[before + (uint32_t)__popcll(hm & ((1ull << lane) - 1ull))] = threadIdx.x;
  __syncthreads();
  const int grp = lane & ~15, way = lane & 15;  // (the group's first lane)
  auto mask16 = [&](bool x) {  // the group's ballot
    const uint64_t m = __ballot(x);
    return ((grp & 32 ? (uint32_t)(m >> 32) : (uint32_t)m) >> (grp & 16)) & 0xFFFFu;
  };
  for (uint32_t h0 = wave * 4; h0 < nh; h0 += EAL_THREADS / 16) {
    const uint32_t h = h0 + (uint32_t)grp / 16;
    bool live = h < nh;  // (then: this step's access is the run's)
    const bool holds = live && way < ways;  // (a lane that holds a way)
    const uint32_t q0 = live ? heads[h] : 0u, s = lk[q0 + 1];
    uint32_t t = EAL_EMPTY, rv = 0;
    if (holds) {
      t = tag[(uint64_t)s * ways + way];
      rv = rrpv[(uint64_t)s * ways + way];
    }
    // the run's accesses here (a prefix of EAL_SHORT positions)
    static_assert(EAL_SHORT <= 16, "a lane looks at one position");
    const int len = __popc(mask16(live && way < EAL_SHORT && lk[q0 + way + 1] == s));
    uint32_t g = lv[q0];
    for (int k = 0; __ballot(k < len); ++k) {
      const uint32_t gk = g;
      g = lv[q0 + k + 1];  // (in flight during the step)
      live = k < len;
      const bool hit = live && holds && t == gk;
      const uint32_t who = mask16(hit);
      const bool miss = live && who == 0;
      if (hit) rv = 0;
      if (!__ballot(miss)) continue;
      uint32_t m3 = mask16(holds && rv == 3);
      if (__ballot(miss && m3 == 0)) {
        const uint32_t m2 = mask16(holds && rv == 2), m1 = mask16(holds && rv == 1);
        if (miss && m3 == 0) {
          rv += m2 ? 1u : (m1 ? 2u : 3u);
          m3 = m2 ? m2 : (m1 ? m1 : all);
        }
      }
      if (miss && way == __ffs((int)m3) - 1) {
        t = gk;
        rv = 2;
      }
    }
    const bool more = len == EAL_SHORT && lk[q0 + EAL_SHORT + 1] == s;  // the run goes on
    if (holds && !more) {
      tag[(uint64_t)s * ways + way] = t;
      rrpv[(uint64_t)s * ways + way] = (uint8_t)rv;
    }
    // the longer of the wave's runs, one after another
    for (uint64_t todo = __ballot(more && way == 0); todo; todo &= todo - 1) {
      const int src = __ffsll((unsigned long long)todo) - 1;
      const uint32_t ss = __builtin_amdgcn_readlane(s, src);
      eal_rr r;
      r.hi = (uint32_t)(__ballot(holds && (rv & 2)) >> src) & 0xFFFFu;
      r.lo = (uint32_t)(__ballot(holds && (rv & 1)) >> src) & 0xFFFFu;
      uint32_t tw = __shfl(t, src + way);  // lane w: way w's id
      if (lane >= ways) tw = EAL_EMPTY;
      uint32_t p = b0 + __builtin_amdgcn_readlane(q0, src) + EAL_SHORT;
      // replays the 64 accesses gc, those of `in` (a prefix of the lanes)
      auto replay = [&](uint64_t in, uint32_t gc) {
        // a chunk of a popular row's run names few ids: all hits, in any order?
        uint64_t left = in;
        uint32_t named = 0;
        for (int c = 0; c < EAL_FEW && left; ++c) {
          const uint32_t x = __builtin_amdgcn_readlane(gc, __ffsll((unsigned long long)left) - 1);
          const uint32_t at = (uint32_t)__ballot(tw == x);
          if (!at) break;
          named |= at;
          left &= ~__ballot(gc == x);
        }
        if (!left) {
          r.hit(named);
          return;
        }
        uint64_t mine = 0, hits = 0;  // lane w: the accesses that name way w's id; their union
#pragma unroll
        for (int w = 0; w < EAL_MAX_WAYS; ++w) {  // (a way past the set's holds EAL_EMPTY, which no access names)
          const uint64_t m = __ballot(gc == (uint32_t)__builtin_amdgcn_readlane(tw, w)) & in;
          mine = lane == w ? m : mine;
          hits |= m;
        }
        for (uint64_t rem = in; rem;) {
          const uint64_t miss = rem & ~hits;
          const uint64_t seg = miss ? rem & ((miss & (~miss + 1)) - 1) : rem;  // up to the first miss
          r.hit((uint32_t)__ballot((mine & seg) != 0));
          if (!miss) break;
          const int a = __ffsll((unsigned long long)miss) - 1;
          const uint32_t ga = __builtin_amdgcn_readlane(gc, a);
          const int v = r.take(all);
          // way v: its old id's later accesses miss now, the new id's hit
          const uint64_t old = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(mine >> 32), v) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((uint32_t)mine, v);
          const uint64_t m = __ballot(gc == ga) & in;
          hits = (hits & ~old) | m;
          if (lane == v) {
            tw = ga;
            mine = m;
          }
          rem = a == 63 ? 0ull : rem & ~((2ull << a) - 1);
        }
      };
      // the first 64 from LDS, then EAL_AHEAD times 64, loaded while those before
      // are replayed
      uint32_t kk[EAL_AHEAD], g[EAL_AHEAD];
      auto load = [&](uint32_t q) {
#pragma unroll
        for (int c = 0; c < EAL_AHEAD; ++c, q += 64) {
          kk[c] = q + lane < n ? keys[q + lane] : EAL_EMPTY;
          g[c] = q + lane < n ? vals[q + lane] : 0u;
        }
      };
      const uint64_t in0 = __ballot(lk[p - b0 + lane + 1] == ss);  // (past n: EAL_EMPTY, no set)
      bool full = in0 == ~0ull;
      if (full) load(p + 64);
      if (in0) replay(in0, lv[p - b0 + lane]);
      for (p += 64; full;) {
        uint64_t in[EAL_AHEAD];
        uint32_t gc[EAL_AHEAD];
#pragma unroll
        for (int c = 0; c < EAL_AHEAD; ++c) {
          in[c] = __ballot(kk[c] == ss);
          gc[c] = g[c];
        }
        full = in[EAL_AHEAD - 1] == ~0ull;
        p += 64 * EAL_AHEAD;
        if (full) load(p);
#pragma unroll
        for (int c = 0; c < EAL_AHEAD; ++c)
          if (in[c]) replay(in[c], gc[c]);
      }
      if (lane < ways) {
        tag[(uint64_t)ss * ways + lane] = tw;
        rrpv[(uint64_t)ss * ways + lane] = (uint8_t)(((r.hi >> lane) & 1u) * 2 + ((r.lo >> lane) & 1u));
      }
    }
  }
}

__global__ void eal_compact(const uint32_t* __restrict__ tag, uint64_t m, uint32_t* __restrict__ out,
                            uint32_t* __restrict__ vals, uint32_t* cnt) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t g = tag[i];
    if (g != EAL_EMPTY) {
      const uint32_t k = atomicAdd(cnt, 1u);
      out[k] = g;
      vals[k] = g;
    }
  }
}

static uint32_t eal_grid(uint64_t n) {
  uint64_t b = (n + 255) / 256;
  return (uint32_t)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

extern "C" hl_status hl_eal_destroy(hl_eal* e) {
  if (!e) return HL_ERR_INVALID_ARG;
  hl_status st = HL_OK;
  for (void* p : {(void*)e->tag, (void*)e->rrpv, (void*)e->cnt, e->ws})
    if (p && hipFree(p) != hipSuccess) st = HL_ERR_HIP;
  delete e;
  return st;
}

extern "C" hl_status hl_eal_reset(hl_eal* e, hl_stream stream) {
  if (!e) return HL_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const uint64_t m = (uint64_t)e->n_sets * e->ways;
  HL_KERNEL(e->h, s, "eal_init", eal_init, dim3(eal_grid(m)), dim3(256), 0, s, e->tag, e->rrpv, m);
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_eal_create(hl_handle* h, uint32_t n_sets, int32_t ways, int64_t max_lookups, hl_eal** out) {
  if (!h || !out || n_sets < 1 || ways < 1 || ways > EAL_MAX_WAYS || max_lookups < 0) return HL_ERR_INVALID_ARG;
  const uint64_t m = (uint64_t)n_sets * ways;
  if (m >= (1ull << 30) || max_lookups >= (1ll << 30)) return HL_ERR_UNSUPPORTED;
  hl_eal* e = new hl_eal();
  e->h = h;
  e->n_sets = n_sets;
  e->ways = ways;
  e->max_n = max_lookups;
  e->sort_n = (uint32_t)((uint64_t)max_lookups > m ? (uint64_t)max_lookups : m);
  hl_carver c = hl_carver::after_header(nullptr, 0);
  hl_sort_ws sw;
  hl_sort_ws_carve(c, sw, e->sort_n);
  e->ws_bytes = c.off;
  hl_status st = HL_OK;
  if (hipMalloc(&e->tag, m * 4) != hipSuccess || hipMalloc(&e->rrpv, m) != hipSuccess ||
      hipMalloc(&e->cnt, 4) != hipSuccess || hipMalloc(&e->ws, e->ws_bytes) != hipSuccess ||
      hipMemset(e->ws, 0, e->ws_bytes) != hipSuccess)
    st = HL_ERR_HIP;
  if (st == HL_OK) st = hl_eal_reset(e, nullptr);
  if (st == HL_OK && hipDeviceSynchronize() != hipSuccess) st = HL_ERR_HIP;
  if (st != HL_OK) {
    hl_eal_destroy(e);
    return st;
  }
  *out = e;
  return HL_OK;
}

extern "C" hl_status hl_eal_access(hl_eal* e, const uint32_t* gids, int64_t n, hl_stream stream) {
  if (!e || n < 0 || (n > 0 && !gids)) return HL_ERR_INVALID_ARG;
  if (n > e->max_n) return HL_ERR_CAPACITY;
  if (n == 0) return HL_OK;
  hipStream_t s = (hipStream_t)stream;
  hl_carver c = hl_carver::after_header(e->ws, e->ws_bytes);
  hl_sort_ws sw;
  hl_sort_ws_carve(c, sw, e->sort_n);
  const uint32_t nn = (uint32_t)n;
  uint32_t *sk, *sv;
  const hl_status st = hl_sort_ids_by_set(e->h, sw, gids, e->n_sets, nn, s, &sk, &sv);
  if (st != HL_OK) return st;
  HL_KERNEL(e->h, s, "eal_runs", eal_runs, dim3(hl_div_up(nn, EAL_THREADS)), dim3(EAL_THREADS), 0, s, sk, sv, nn, e->n_sets,
            e->ways, e->tag, e->rrpv);
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_eal_hot(hl_eal* e, uint32_t* hot_ids_out, uint32_t* n_hot_out, hl_stream stream) {
  if (!e || !hot_ids_out || !n_hot_out) return HL_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const uint64_t m = (uint64_t)e->n_sets * e->ways;
  hl_carver c = hl_carver::after_header(e->ws, e->ws_bytes);
  hl_sort_ws sw;
  hl_sort_ws_carve(c, sw, e->sort_n);
  HL_HIP(hipMemsetAsync(e->cnt, 0, 4, s));
  HL_KERNEL(e->h, s, "eal_compact", eal_compact, dim3(eal_grid(m)), dim3(256), 0, s, e->tag, m, sw.k0, sw.v0, e->cnt);
  HL_LAUNCHED();
  uint32_t *sk, *sv;
  hl_status st = hl_sort_pairs(e->h, sw, e->cnt, (uint32_t)m, hl_bit_width(e->h->n_rows), s, &sk, &sv);
  if (st != HL_OK) return st;
  uint32_t n = 0;
  HL_HIP(hipMemcpyAsync(&n, e->cnt, 4, hipMemcpyDeviceToHost, s));
  HL_HIP(hipStreamSynchronize(s));
  if (n) HL_HIP(hipMemcpy(hot_ids_out, sk, (size_t)n * 4, hipMemcpyDeviceToDevice));
  *n_hot_out = n;
  return HL_OK;
}

extern "C" hl_status hl_eal_state(const hl_eal* e, uint32_t* tags_out, uint8_t* rrpv_out, hl_stream stream) {
  if (!e || !tags_out || !rrpv_out) return HL_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const uint64_t m = (uint64_t)e->n_sets * e->ways;
  HL_HIP(hipMemcpyAsync(tags_out, e->tag, m * 4, hipMemcpyDeviceToDevice, s));
  HL_HIP(hipMemcpyAsync(rrpv_out, e->rrpv, m, hipMemcpyDeviceToDevice, s));
  return HL_OK;
}
