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

__device__ __forceinline__ uint32_t eal_mix(uint32_t x) {
  x ^= x >> 16;
  x *= 0x85EBCA6Bu;
  x ^= x >> 13;
  x *= 0xC2B2AE35u;
  x ^= x >> 16;
  return x;
}

__global__ void eal_init(uint32_t* tag, uint8_t* rrpv, uint64_t m) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
    tag[i] = EAL_EMPTY;
    rrpv[i] = 3;
  }
}

// (set, id) of every lookup; an invalid id (0xFFFFFFFF) gets the key n_sets,
// which sorts after every set and is skipped
__global__ void eal_keys(const uint32_t* __restrict__ gids, uint32_t n, uint32_t n_sets, uint32_t* __restrict__ keys,
                         uint32_t* __restrict__ vals) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const uint32_t g = gids[i];
    keys[i] = g == EAL_EMPTY ? n_sets : eal_mix(g) % n_sets;
    vals[i] = g;
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

// Replays each set's run.  The first EAL_SHORT accesses of a run are replayed
// by the thread of its first position (ways in registers, every index into them
// a compile-time constant; the block's positions in LDS); the rest of a longer
// run by the whole wave, 64 accesses at a time: lane w holds way w's id and the
// mask of the 64 accesses that name it, so all accesses up to the first miss
// are one step (their ways' RRPVs cleared by a ballot), and a miss is a step of
// scalar work.  The runs are what bounds the kernel: a popular row gives its
// set a run of thousands, and one thread replaying it took 634 us for 212,992
// accesses on 26,436 sets of 16; 24 us like this (4, 8, 12
// accesses by the thread: 25, 24, 24; 16 and 32 with a looped compare: 41, 47).
#define EAL_THREADS 256
#define EAL_SHORT 8
__global__ void __launch_bounds__(EAL_THREADS)
eal_runs(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint32_t n, uint32_t n_sets,
         int32_t ways, uint32_t* __restrict__ tag, uint8_t* __restrict__ rrpv) {
  __shared__ uint32_t lk[EAL_THREADS + EAL_SHORT + 1], lv[EAL_THREADS + EAL_SHORT];
  const uint32_t b0 = blockIdx.x * EAL_THREADS, i = b0 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  for (uint32_t j = threadIdx.x; j < EAL_THREADS + EAL_SHORT + 1; j += EAL_THREADS) {
    const uint32_t q = b0 + j;  // lk[j] is position b0 - 1 + j
    lk[j] = q > 0 && q - 1 < n ? keys[q - 1] : EAL_EMPTY;
    if (j < EAL_THREADS + EAL_SHORT) lv[j] = q < n ? vals[q] : 0u;
  }
  __syncthreads();
  const uint32_t all = (1u << ways) - 1u;
  const uint32_t s = lk[threadIdx.x + 1];
  const bool head = i < n && s < n_sets && (i == 0 || lk[threadIdx.x] != s);
  uint32_t t[EAL_MAX_WAYS];
  eal_rr rr{0, 0};
  bool more = false;  // the run goes on past EAL_SHORT accesses
  if (head) {
#pragma unroll
    for (int w = 0; w < EAL_MAX_WAYS; ++w) {
      t[w] = EAL_EMPTY;  // (matches no access)
      if (w < ways) {
        t[w] = tag[(uint64_t)s * ways + w];
        const uint32_t r = rrpv[(uint64_t)s * ways + w];
        rr.hi |= (r >> 1) << w;
        rr.lo |= (r & 1u) << w;
      }
    }
    more = true;
    for (int k = 0; k < EAL_SHORT; ++k) {
      if (lk[threadIdx.x + 1 + k] != s) {
        more = false;
        break;
      }
      const uint32_t g = lv[threadIdx.x + k];
      uint32_t m = 0;
#pragma unroll
      for (int w = 0; w < EAL_MAX_WAYS; ++w) m |= t[w] == g ? 1u << w : 0u;
      if (m) {
        rr.hit(m);
        continue;
      }
      const int v = rr.take(all);
#pragma unroll
      for (int w = 0; w < EAL_MAX_WAYS; ++w) t[w] = w == v ? g : t[w];
    }
    if (!more) {
#pragma unroll
      for (int w = 0; w < EAL_MAX_WAYS; ++w)
        if (w < ways) {
          tag[(uint64_t)s * ways + w] = t[w];
          rrpv[(uint64_t)s * ways + w] = (uint8_t)(((rr.hi >> w) & 1u) * 2 + ((rr.lo >> w) & 1u));
        }
    }
  }
  // the long runs of the wave, one after another
  for (uint64_t todo = __ballot(more); todo; todo &= todo - 1) {
    const int src = __ffsll((unsigned long long)todo) - 1;
    const uint32_t ss = __builtin_amdgcn_readlane(s, src);
    eal_rr r;
    r.hi = __builtin_amdgcn_readlane(rr.hi, src);
    r.lo = __builtin_amdgcn_readlane(rr.lo, src);
    uint32_t tw = EAL_EMPTY;  // lane w: way w's id
#pragma unroll
    for (int w = 0; w < EAL_MAX_WAYS; ++w) {
      const uint32_t x = __builtin_amdgcn_readlane(t[w], src);
      tw = lane == w ? x : tw;
    }
    uint32_t p = __builtin_amdgcn_readlane(i, src) + EAL_SHORT;
    uint32_t g = 0, kk = EAL_EMPTY;
    if (p + lane < n) {
      kk = keys[p + lane];
      g = vals[p + lane];
    }
    for (;;) {
      const uint64_t in = __ballot(kk == ss);  // (a prefix of the lanes)
      if (!in) break;
      const uint32_t gc = g;
      // the next 64, loaded while these are replayed
      p += 64;
      kk = EAL_EMPTY;
      if (in == ~0ull && p + lane < n) {
        kk = keys[p + lane];
        g = vals[p + lane];
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
    }
    if (lane < ways) {
      tag[(uint64_t)ss * ways + lane] = tw;
      rrpv[(uint64_t)ss * ways + lane] = (uint8_t)(((r.hi >> lane) & 1u) * 2 + ((r.lo >> lane) & 1u));
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
  HL_KERNEL(e->h, s, "eal_keys", eal_keys, dim3(eal_grid(nn)), dim3(256), 0, s, gids, nn, e->n_sets, sw.k0, sw.v0);
  HL_LAUNCHED();
  uint32_t *sk, *sv;
  hl_status st = hl_sort_pairs(e->h, sw, nullptr, nn, hl_bit_width(e->n_sets), s, &sk, &sv);
  if (st != HL_OK) return st;
  HL_KERNEL(e->h, s, "eal_runs", eal_runs, dim3(hl_div_up(nn, EAL_THREADS)), dim3(EAL_THREADS), 0, s, sk, sv, nn, e->n_sets, e->ways,
            e->tag, e->rrpv);
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
