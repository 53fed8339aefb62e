// Handle, workspace, errors, pinned host memory, address generation, access
// counting and the bitwise row gather.
#include <stdlib.h>
#include <string.h>

#include <vector>

#include <cstring>

#include "hl_internal.h"

size_t hl_topk_scratch_bytes(uint64_t n_rows);
size_t hl_partition_ws_bytes(int32_t max_samples);
size_t hl_cold_ws_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags, int32_t max_samples);
size_t hl_bwd_ws_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags);
size_t hl_plan_ws_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags, int32_t max_samples);

extern "C" const char* hl_status_string(int32_t s) {
  switch (s) {
    case HL_OK: return "ok";
    case HL_ERR_INVALID_ARG: return "invalid argument";
    case HL_ERR_OUT_OF_RANGE: return "out of range";
    case HL_ERR_CAPACITY: return "capacity exceeded";
    case HL_ERR_HIP: return "HIP runtime error";
    case HL_ERR_UNSUPPORTED: return "unsupported";
    case HL_ERR_DEVICE: return "device error word set";
  }
  return "unknown status";
}

// ----------------------------------------------------------------------------- fill
__global__ void hl_k_fill32(uint32_t* p, uint64_t n, uint32_t v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

static hl_status fill32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return HL_OK;
  uint32_t g = hl_div_up(n, 256);
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(hl_k_fill32, dim3(g), dim3(256), 0, s, p, n, v);
  HL_LAUNCHED();
  return HL_OK;
}

hl_status hl_fill32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) { return fill32(p, n, v, s); }

// ----------------------------------------------------------------------------- tracing
// name is one of the comma-separated names of list
static bool trace_listed(const char* list, const char* name) {
  const size_t n = strlen(name);
  for (const char* p = list; *p;) {
    const char* e = strchr(p, ',');
    const size_t m = e ? (size_t)(e - p) : strlen(p);
    if (m == n && strncmp(p, name, n) == 0) return true;
    if (!e) break;
    p = e + 1;
  }
  return false;
}

int hl_trace_take(const hl_handle* h, const char* name, hipEvent_t* a, hipEvent_t* b) {
  hl_trace* t = h ? h->trace : nullptr;
  if (!t || t->n >= t->cap) return -1;
  if (t->only[0] && !trace_listed(t->only, name)) return -1;
  const int i = t->n++;
  t->rec[i].name = name;
  *a = t->rec[i].a;
  *b = t->rec[i].b;
  return i;
}

static void trace_free(hl_trace* t) {
  for (int i = 0; i < t->cap; ++i) {
    (void)hipEventDestroy(t->rec[i].a);
    (void)hipEventDestroy(t->rec[i].b);
  }
  free(t->rec);
  t->rec = nullptr;
  t->cap = t->n = 0;
}

extern "C" hl_status hl_trace_enable(hl_handle* h, int32_t cap) {
  if (!h || cap < 0) return HL_ERR_INVALID_ARG;
  HL_HIP(hipDeviceSynchronize());
  trace_free(h->trace);
  if (cap == 0) return HL_OK;
  h->trace->rec = (hl_trace_rec*)calloc((size_t)cap, sizeof(hl_trace_rec));
  if (!h->trace->rec) return HL_ERR_CAPACITY;
  for (int i = 0; i < cap; ++i) {
    // timing only: no system-scope fence (cache write-back and invalidate) at
    // each record, which would lengthen and perturb what is measured
    if (hipEventCreateWithFlags(&h->trace->rec[i].a, hipEventDisableSystemFence) != hipSuccess ||
        hipEventCreateWithFlags(&h->trace->rec[i].b, hipEventDisableSystemFence) != hipSuccess) {
      h->trace->cap = i + 1;
      trace_free(h->trace);
      return HL_ERR_HIP;
    }
  }
  h->trace->cap = cap;
  return HL_OK;
}

extern "C" hl_status hl_trace_only(hl_handle* h, const char* name) {
  if (!h || (name && strlen(name) >= sizeof(h->trace->only))) return HL_ERR_INVALID_ARG;
  strcpy(h->trace->only, name ? name : "");
  return HL_OK;
}

extern "C" int32_t hl_trace_count(const hl_handle* h) { return h ? h->trace->n : 0; }

extern "C" hl_status hl_trace_read(const hl_handle* h, int32_t i, const char** name, float* ms) {
  if (!h || i < 0 || i >= h->trace->n || !name || !ms) return HL_ERR_INVALID_ARG;
  HL_HIP(hipEventSynchronize(h->trace->rec[i].b));
  HL_HIP(hipEventElapsedTime(ms, h->trace->rec[i].a, h->trace->rec[i].b));
  *name = h->trace->rec[i].name;
  return HL_OK;
}

extern "C" hl_status hl_trace_read_at(const hl_handle* h, int32_t i, const char** name, float* start_ms,
                                      float* ms) {
  if (!h || i < 0 || i >= h->trace->n || !name || !start_ms || !ms) return HL_ERR_INVALID_ARG;
  const hl_status st = hl_trace_read(h, i, name, ms);
  if (st != HL_OK) return st;
  HL_HIP(hipEventSynchronize(h->trace->rec[0].a));
  HL_HIP(hipEventElapsedTime(start_ms, h->trace->rec[0].a, h->trace->rec[i].a));
  return HL_OK;
}

extern "C" hl_status hl_trace_reset(hl_handle* h) {
  if (!h) return HL_ERR_INVALID_ARG;
  HL_HIP(hipDeviceSynchronize());
  h->trace->n = 0;
  return HL_OK;
}

// ----------------------------------------------------------------------------- handle
// ----------------------------------------------------------------------------- table bounds
__global__ void hl_k_tbounds(const uint32_t* __restrict__ base, int32_t n_tables, const uint64_t* __restrict__ bm,
                             const uint32_t* __restrict__ rank, uint64_t n_entries, uint32_t* __restrict__ tb) {
  for (int32_t t = threadIdx.x; t <= n_tables; t += blockDim.x)
    tb[t] = t < n_tables ? hl_hot_below(bm, rank, base[t]) : rank[n_entries - 1];
}

hl_status hl_table_bounds(hl_handle* h, hipStream_t s) {
  HL_KERNEL(h, s, "hl_k_tbounds", hl_k_tbounds, dim3(1), dim3(256), 0, s, h->d_base, h->n_tables, h->d_bitmap,
            h->d_rank, h->n_tiles4k * 16 + 1, h->d_tb);
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_create(hl_handle** out, int32_t n_tables, const uint32_t* rows_per_table,
                               int32_t dim, int32_t dtype, uint32_t k_cap) {
  if (!out || n_tables < 1 || !rows_per_table || dim < 1 || dim > 8192 || k_cap < 1)
    return HL_ERR_INVALID_ARG;
  if (dtype != HL_F32 && dtype != HL_BF16) return HL_ERR_INVALID_ARG;
  uint64_t total = 0;
  std::vector<uint32_t> base(n_tables);
  for (int32_t t = 0; t < n_tables; ++t) {
    if (rows_per_table[t] == 0) return HL_ERR_INVALID_ARG;
    base[t] = (uint32_t)total;
    total += rows_per_table[t];
    if (total >= 0xFFFFFFFFull) return HL_ERR_OUT_OF_RANGE;
  }
  hl_handle* h = (hl_handle*)calloc(1, sizeof(hl_handle));
  if (!h) return HL_ERR_CAPACITY;
  h->n_tables = n_tables;
  h->n_rows = total;
  h->dim = dim;
  h->dtype = (hl_dtype)dtype;
  h->k_cap = k_cap;
  h->row_bytes = (uint32_t)dim * (dtype == HL_F32 ? 4u : 2u);
  h->n_tiles4k = (total + 4095) / 4096;
  h->tk_bytes = hl_topk_scratch_bytes(total);
  h->trace = new hl_trace();
  hl_status st = HL_OK;
  if (hipGetDevice(&h->device) != hipSuccess) st = HL_ERR_HIP;
  // the allocation-free backward's static workspace on this device
  if (st == HL_OK) st = hl_scratch_setup(h->device);
  auto dm = [&](void** p, size_t bytes) {
    if (st == HL_OK && hipMalloc(p, bytes) != hipSuccess) st = HL_ERR_HIP;
  };
  dm((void**)&h->d_base, sizeof(uint32_t) * n_tables);
  dm((void**)&h->d_rows, sizeof(uint32_t) * n_tables);
  dm((void**)&h->d_counts, sizeof(uint32_t) * total);
  dm((void**)&h->d_bitmap, sizeof(uint64_t) * h->n_tiles4k * 64);
  dm((void**)&h->d_rank, sizeof(uint32_t) * (h->n_tiles4k * 16 + 1));
  dm((void**)&h->d_tb, sizeof(uint32_t) * (n_tables + 1));
  dm((void**)&h->d_err, sizeof(uint32_t));
  dm((void**)&h->d_tk, h->tk_bytes);
  if (st == HL_OK) {
    if (hipMemcpy(h->d_base, base.data(), sizeof(uint32_t) * n_tables, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(h->d_rows, rows_per_table, sizeof(uint32_t) * n_tables, hipMemcpyHostToDevice) != hipSuccess)
      st = HL_ERR_HIP;
  }
  if (st == HL_OK) st = fill32(h->d_counts, total, 0, 0);
  if (st == HL_OK) st = fill32((uint32_t*)h->d_bitmap, h->n_tiles4k * 128, 0, 0);
  if (st == HL_OK) st = fill32(h->d_rank, h->n_tiles4k * 16 + 1, 0, 0);
  if (st == HL_OK) st = fill32(h->d_tb, n_tables + 1, 0, 0);
  if (st == HL_OK) st = fill32(h->d_err, 1, 0, 0);
  if (st == HL_OK) st = fill32(h->d_tk, h->tk_bytes / 4, 0, 0);
  if (st == HL_OK && hipDeviceSynchronize() != hipSuccess) st = HL_ERR_HIP;
  if (st != HL_OK) {
    hl_destroy(h);
    return st;
  }
  *out = h;
  return HL_OK;
}

extern "C" hl_status hl_destroy(hl_handle* h) {
  if (!h) return HL_ERR_INVALID_ARG;
  void* ps[] = {h->d_base, h->d_rows, h->d_counts, h->d_bitmap, h->d_rank, h->d_tb, h->d_err, h->d_tk, h->cg_table};
  hl_status st = HL_OK;
  if (h->trace) {
    trace_free(h->trace);
    delete h->trace;
  }
  for (void* p : ps)
    if (p && hipFree(p) != hipSuccess) st = HL_ERR_HIP;
  free(h);
  return st;
}

extern "C" hl_status hl_debug_ballot_ranks(hl_handle* h, int32_t on) {
  if (!h) return HL_ERR_INVALID_ARG;
  h->ballot_ranks = on != 0;
  return HL_OK;
}

extern "C" uint64_t hl_n_rows(const hl_handle* h) { return h ? h->n_rows : 0; }
extern "C" uint32_t hl_n_hot(const hl_handle* h) { return h ? h->n_hot : 0; }
extern "C" uint32_t hl_k_cap(const hl_handle* h) { return h ? h->k_cap : 0; }

extern "C" size_t hl_workspace_bytes(const hl_handle* h, int64_t max_lookups, int64_t max_bags,
                                     int32_t max_samples) {
  if (!h || max_lookups < 0 || max_bags < 0 || max_samples < 0) return 0;
  size_t a = hl_partition_ws_bytes(max_samples);
  size_t b = hl_cold_ws_bytes(h, max_lookups, max_bags, max_samples);
  size_t c = hl_bwd_ws_bytes(h, max_lookups, max_bags);
  size_t d = hl_plan_ws_bytes(h, max_lookups, max_bags, max_samples);
  size_t m = a > b ? a : b;
  m = m > c ? m : c;
  m = m > d ? m : d;
  return (m + 4095) & ~(size_t)4095;
}

extern "C" hl_status hl_workspace_init(void* ws, size_t bytes, hl_stream stream) {
  if (!ws || (bytes & 3)) return HL_ERR_INVALID_ARG;
  return fill32((uint32_t*)ws, bytes / 4, 0, (hipStream_t)stream);
}

extern "C" hl_status hl_last_device_error(hl_handle* h, uint32_t* err_out) {
  if (!h || !err_out) return HL_ERR_INVALID_ARG;
  HL_HIP(hipDeviceSynchronize());
  uint32_t e = 0;
  HL_HIP(hipMemcpy(&e, h->d_err, 4, hipMemcpyDeviceToHost));
  uint32_t z = 0;
  HL_HIP(hipMemcpy(h->d_err, &z, 4, hipMemcpyHostToDevice));
  *err_out = e;
  return e ? HL_ERR_DEVICE : HL_OK;
}

extern "C" hl_status hl_host_alloc(size_t bytes, void** host, void** dev) {
  if (!host || bytes == 0) return HL_ERR_INVALID_ARG;
  void* p = nullptr;
  HL_HIP(hipHostMalloc(&p, bytes, hipHostMallocMapped | hipHostMallocPortable));
  if (dev) {
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, p, 0) != hipSuccess) {
      (void)hipHostFree(p);
      return HL_ERR_HIP;
    }
    *dev = d;
  }
  *host = p;
  return HL_OK;
}

extern "C" hl_status hl_host_free(void* host) {
  if (!host) return HL_ERR_INVALID_ARG;
  HL_HIP(hipHostFree(host));
  return HL_OK;
}

// ----------------------------------------------------------------------------- gids
// A group of GIDS_BAGS consecutive bags, whose lookups are contiguous, by one
// wave or by several in turn: lane j holds the offset of bag j, and each lookup's
// bag is found by binary search over the lanes' offsets (shuffles; no LDS, no
// barrier), four lookups per lane at a time with their row loads issued together.
// The call knows bags, not lookups: groups of 32 bags give a wave of one-lookup
// bags half its lanes, one of 20-lookup bags ten rounds of lanes, and where there
// are few groups up to GIDS_PARTS waves share each (GIDS_WAVES in all), since then
// the bags may be of any length.  Bound by latency: offsets, rows, ids.  A block
// of 256 threads per 64 bags took 4.5 us for 212,992 single lookups and 7.2 for
// 328,000 in bags of 20, a wave per group 4.2 and 6.7.  Back to back: 4 bags of
// 20,000 135 us with the block, 400 with one wave, 9 with several; one bag of
// 200,000 237, 998 and 20; 320 bags of 3000 517, 502 and 11.
#define GIDS_BAGS 32
#define GIDS_PARTS 64
#define GIDS_WAVES 2048
__global__ void __launch_bounds__(256)
hl_k_gids(const uint32_t* __restrict__ rows, const int32_t* __restrict__ bag_ptr, int64_t n_bags, int32_t parts,
          const uint32_t* __restrict__ base, const uint32_t* __restrict__ nrow, int32_t n_tables,
          uint32_t* __restrict__ gids, uint32_t* err) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b0 = wave / parts * GIDS_BAGS;
  const int32_t part = (int32_t)(wave % parts);
  if (b0 >= n_bags) return;
  const int nb = (int)min((int64_t)GIDS_BAGS, n_bags - b0);
  const int32_t off = bag_ptr[b0 + min(lane, nb)];  // (lanes past nb: the end)
  const uint32_t t0 = (uint32_t)(b0 % n_tables);
  // lane j's table, its base and size
  const uint32_t tj = (t0 + (uint32_t)lane) % (uint32_t)n_tables;
  const uint32_t bj = base[tj], nj = nrow[tj];
  const int32_t lo = __shfl(off, 0), hi = __shfl(off, nb);
  // 4 lookups per lane at a time, their row loads issued together
  for (int64_t i0 = (int64_t)lo + part * 256; i0 < hi; i0 += parts * 256) {
    uint32_t r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = i0 + k * 64 + lane;
      r[k] = i < hi ? rows[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k * 64 >= hi) break;  // (the same for every lane)
      const int64_t i = i0 + k * 64 + lane;
      int a = 0;  // the last bag that starts at or before lookup i
#pragma unroll
      for (int s = GIDS_BAGS / 2; s > 0; s >>= 1) {
        const int32_t o = __shfl(off, a + s);
        if (a + s < nb && o <= i) a += s;
      }
      const uint32_t b = __shfl(bj, a), n = __shfl(nj, a);
      if (i < hi) {
        gids[i] = r[k] < n ? b + r[k] : 0xFFFFFFFFu;
        if (r[k] >= n) hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
      }
    }
  }
}

extern "C" hl_status hl_lookup_gids(const hl_handle* h, const uint32_t* rows, const int32_t* bag_ptr,
                                    int64_t n_bags, uint32_t* gids, hl_stream stream) {
  if (!h || n_bags < 0 || (n_bags > 0 && (!rows || !bag_ptr || !gids))) return HL_ERR_INVALID_ARG;
  if (n_bags == 0) return HL_OK;
  if (n_bags >= (1ll << 31)) return HL_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  const uint32_t groups = hl_div_up(n_bags, GIDS_BAGS);
  const uint32_t parts = groups >= GIDS_WAVES ? 1 : (GIDS_WAVES / groups < GIDS_PARTS ? GIDS_WAVES / groups : GIDS_PARTS);
  HL_KERNEL(h, s, "hl_k_gids", hl_k_gids, dim3(hl_div_up((uint64_t)groups * parts, 4)), dim3(256), 0, s, rows, bag_ptr, n_bags,
            (int32_t)parts, h->d_base, h->d_rows, h->n_tables, gids, h->d_err);
  HL_LAUNCHED();
  return HL_OK;
}

// ----------------------------------------------------------------------------- counting
// A block takes THREADS * CT_ITEMS lookups and adds up equal ids in an LDS table
// first (open addressing, CT_PROBES probes; an id that finds no slot goes to
// memory directly); the thread that put an id into its slot then adds the slot's
// count with one atomic.  The kernel is bound by atomics that meet on one cache
// line (the popular rows, and every row of a small table): they complete one
// after another.  So the blocks walk the lookups with stride n_tables, which in
// the one-lookup-per-bag layout gives a block one table's lookups (any order
// counts the same): a row then meets about as many atomics as its table has
// blocks.  1024 lookups a block, so that they reach every compute unit; 2048 where
// 256 such blocks are too few, since then the meetings count.  Back to back, one
// atomic per lookup, then blocks of 2048 in LDS with every slot looked through at
// the end, then this: 212,992 lookups of 1e6 rows in 26 tables 49.3, 9.1 and 8.4
// us (Zipf 1.2) or 9.8, 12.6 and 11.0 (rows of equal weight: the LDS table then
// finds little to add up), 852,000 (Zipf) 192, 25.3 and 24.2 (blocks of 1024
// there 28.0).
#define CT_ITEMS 2
#define CT_PROBES 4
#define CT_BLOCKS 256
template <int THREADS>
__global__ void __launch_bounds__(THREADS)
hl_k_count(const uint32_t* __restrict__ gids, uint32_t n, uint32_t stride, uint32_t* __restrict__ counts,
           uint64_t n_rows, uint32_t* err) {
  constexpr int SLOTS = 2 * THREADS * CT_ITEMS;
  __shared__ uint4 key4[SLOTS / 4], cnt4[SLOTS / 4];
  uint32_t *key = reinterpret_cast<uint32_t*>(key4), *cnt = reinterpret_cast<uint32_t*>(cnt4);
  const uint32_t q0 = blockIdx.x * (THREADS * CT_ITEMS) + threadIdx.x;
  // position q of the walk is lookup (q % per) stride + q / per
  const uint32_t per = (n + stride - 1) / stride;
  uint32_t g[CT_ITEMS];
  bool in[CT_ITEMS];
#pragma unroll
  for (int k = 0; k < CT_ITEMS; ++k) {
    const uint32_t q = q0 + k * THREADS, t = q / per;
    const uint64_t i = (uint64_t)(q - t * per) * stride + t;
    in[k] = t < stride && i < n;
    g[k] = in[k] ? gids[i] : 0u;
  }
  for (int j = threadIdx.x; j < SLOTS / 4; j += THREADS) {
    key4[j] = make_uint4(~0u, ~0u, ~0u, ~0u);  // (no row's id)
    cnt4[j] = make_uint4(0u, 0u, 0u, 0u);
  }
  __syncthreads();
  uint32_t slot[CT_ITEMS], old[CT_ITEMS];
  bool mine[CT_ITEMS];  // this thread put the id into its slot, and adds the slot's count
#pragma unroll
  for (int k = 0; k < CT_ITEMS; ++k) {
    if (in[k] && g[k] >= n_rows) {
      hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
      in[k] = false;
    }
    slot[k] = hl_cg_hash(g[k]) % SLOTS;
    old[k] = in[k] ? atomicCAS(&key[slot[k]], 0xFFFFFFFFu, g[k]) : 0u;
  }
#pragma unroll
  for (int k = 0; k < CT_ITEMS; ++k) {
    mine[k] = false;
    if (!in[k]) continue;
    bool held = old[k] == 0xFFFFFFFFu || old[k] == g[k];
    for (int p = 1; p < CT_PROBES && !held; ++p) {
      slot[k] = (slot[k] + 1) % SLOTS;
      old[k] = atomicCAS(&key[slot[k]], 0xFFFFFFFFu, g[k]);
      held = old[k] == 0xFFFFFFFFu || old[k] == g[k];
    }
    mine[k] = old[k] == 0xFFFFFFFFu;
    if (held) atomicAdd(&cnt[slot[k]], 1u);
    else atomicAdd(counts + g[k], 1u);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < CT_ITEMS; ++k)
    if (mine[k]) atomicAdd(counts + g[k], cnt[slot[k]]);
}

extern "C" hl_status hl_profile_count(hl_handle* h, const uint32_t* gids, int64_t n, hl_stream stream) {
  if (!h || n < 0 || (n > 0 && !gids)) return HL_ERR_INVALID_ARG;
  if (n == 0) return HL_OK;
  hipStream_t s = (hipStream_t)stream;
  // (positions stay below 2^31: at most 2^30 lookups a launch, and as many of the walk's gaps)
  const int64_t most = 1ll << 30;
  for (int64_t i = 0; i < n; i += most) {
    const uint32_t m = (uint32_t)(n - i < most ? n - i : most);
    const uint32_t stride = (uint32_t)h->n_tables < m ? (uint32_t)h->n_tables : m;
    const uint64_t walk = (uint64_t)hl_div_up(m, stride) * stride;
#define CNT(T)                                                                                                     \
  HL_KERNEL(h, s, "hl_k_count", hl_k_count<T>, dim3(hl_div_up(walk, T * CT_ITEMS)), dim3(T), 0, s, gids + i, m, stride, \
            h->d_counts, h->n_rows, h->d_err)
    if (walk <= CT_BLOCKS * 512 * CT_ITEMS) CNT(512);
    else CNT(1024);
#undef CNT
  }
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_profile_counts(const hl_handle* h, uint32_t* counts_out, hl_stream stream) {
  if (!h || !counts_out) return HL_ERR_INVALID_ARG;
  HL_HIP(hipMemcpyAsync(counts_out, h->d_counts, sizeof(uint32_t) * h->n_rows, hipMemcpyDeviceToDevice,
                        (hipStream_t)stream));
  return HL_OK;
}

// ----------------------------------------------------------------------------- gather
// dst[r] = src[ids[r]], bit for bit.  Lanes copy U-byte units of a row; for a
// 256-byte row and U = 16, 16 lanes cover a row and a wave moves 4 rows.
// Ids >= n_src_rows are skipped and flagged (the source is never read out of
// bounds).
template <typename V>
__global__ void __launch_bounds__(256)
hl_k_gather(const uint32_t* __restrict__ ids, const int32_t* n_dev, uint32_t n_host,
            const V* __restrict__ src, uint64_t n_src_rows, V* __restrict__ dst, uint32_t upr,
            uint32_t* err) {
  const uint32_t n = n_dev ? (uint32_t)max((int64_t)0, min((int64_t)*n_dev, (int64_t)n_host)) : n_host;
  const uint64_t total = (uint64_t)n * upr;
  for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
       t += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t r = (uint32_t)(t / upr), c = (uint32_t)(t - (uint64_t)r * upr);
    const uint32_t id = ids[r];
    if (id < n_src_rows) dst[(uint64_t)r * upr + c] = src[(uint64_t)id * upr + c];
    else if (c == 0) hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
  }
}

hl_status hl_launch_gather(const hl_handle* h, const uint32_t* ids, const int32_t* n_dev, uint32_t n_host,
                           const void* src, uint64_t n_src_rows, void* dst, uint32_t row_bytes, uint32_t* err,
                           hipStream_t s) {
  if (n_host == 0) return HL_OK;
  uint64_t total;
  uint32_t g;
#define HL_GATHER_LAUNCH(V)                                                                       \
  total = (uint64_t)n_host * (row_bytes / sizeof(V));                                             \
  g = hl_div_up(total, 256);                                                                      \
  if (g > 16384) g = 16384;                                                                       \
  HL_KERNEL(h, s, "hl_k_gather", hl_k_gather<V>, dim3(g), dim3(256), 0, s, ids, n_dev, n_host, (const V*)src, \
                     n_src_rows, (V*)dst, (uint32_t)(row_bytes / sizeof(V)), err);
  if (row_bytes % 16 == 0) { HL_GATHER_LAUNCH(uint4) }
  else if (row_bytes % 8 == 0) { HL_GATHER_LAUNCH(uint2) }
  else if (row_bytes % 4 == 0) { HL_GATHER_LAUNCH(uint32_t) }
  else { HL_GATHER_LAUNCH(uint16_t) }
#undef HL_GATHER_LAUNCH
  HL_LAUNCHED();
  return HL_OK;
}

extern "C" hl_status hl_hot_fill(const hl_handle* h, const uint32_t* hot_ids, const void* w_host,
                                 void* w_hot, hl_stream stream) {
  if (!h || (h->n_hot && (!hot_ids || !w_host || !w_hot))) return HL_ERR_INVALID_ARG;
  return hl_launch_gather(h, hot_ids, nullptr, h->n_hot, w_host, h->n_rows, w_hot, h->row_bytes, h->d_err,
                          (hipStream_t)stream);
}

// ----------------------------------------------------------------------------- streams
extern "C" hl_status hl_stream_create(int32_t first_cu, int32_t n_cu, int32_t complement, hl_stream* out) {
  if (!out || first_cu < 0 || n_cu < 0) return HL_ERR_INVALID_ARG;
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return HL_ERR_HIP;
  if (n_cu == 0) {  // no mask
    hipStream_t s;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return HL_ERR_HIP;
    *out = (hl_stream)s;
    return HL_OK;
  }
  if (first_cu + n_cu > ncu || (complement && n_cu >= ncu)) return HL_ERR_INVALID_ARG;
  const int words = (ncu + 31) / 32;
  std::vector<uint32_t> mask((size_t)words, 0u);
  for (int c = 0; c < ncu; ++c) {
    const bool in = c >= first_cu && c < first_cu + n_cu;
    if (in != (complement != 0)) mask[(size_t)c / 32] |= 1u << (c % 32);
  }
  hipStream_t s;
  if (hipExtStreamCreateWithCUMask(&s, (uint32_t)words, mask.data()) != hipSuccess) return HL_ERR_HIP;
  *out = (hl_stream)s;
  return HL_OK;
}

extern "C" hl_status hl_stream_destroy(hl_stream s) {
  if (!s) return HL_ERR_INVALID_ARG;
  return hipStreamDestroy((hipStream_t)s) == hipSuccess ? HL_OK : HL_ERR_HIP;
}
