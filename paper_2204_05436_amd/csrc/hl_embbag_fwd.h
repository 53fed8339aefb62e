// EmbeddingBag sum pooling: row I/O, the lane layout and the forward's bodies,
// shared by the forward's own launches (hl_embbag.hip) and by the launches that
// run it beside the grouping's sorts (hl_embbag.hip, hl_fwd_sort.h).  The lane
// layout and the summation order are described in hl_embbag.hip.
#pragma once
#include <initializer_list>

#include "hl_internal.h"

// ----------------------------------------------------------------------------- row I/O
template <int VEC, bool BF>
struct RowIO;

// A row slice of VEC elements: load() gives it as floats; load_raw() keeps the
// loaded bytes (Raw) and unpack() converts them when they are used, so a row
// in flight holds only its bytes' registers (bf16: half of the floats').
template <>
struct RowIO<4, false> {
  typedef float T;
  typedef float4 Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *reinterpret_cast<const float4*>(p); }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) {
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  }
  static __device__ __forceinline__ void load(const T* p, float* v) { unpack(load_raw(p), v); }
  static __device__ __forceinline__ void store(T* p, const float* v) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <>
struct RowIO<2, false> {
  typedef float T;
  typedef float2 Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *reinterpret_cast<const float2*>(p); }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) {
    v[0] = x.x; v[1] = x.y;
  }
  static __device__ __forceinline__ void load(const T* p, float* v) { unpack(load_raw(p), v); }
  static __device__ __forceinline__ void store(T* p, const float* v) {
    *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
  }
};
template <>
struct RowIO<8, false> {
  typedef float T;
  struct Raw {
    float4 a, b;
  };
  static __device__ __forceinline__ Raw load_raw(const T* p) {
    return Raw{*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)};
  }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) {
    RowIO<4, false>::unpack(x.a, v);
    RowIO<4, false>::unpack(x.b, v + 4);
  }
  static __device__ __forceinline__ void load(const T* p, float* v) { unpack(load_raw(p), v); }
  static __device__ __forceinline__ void store(T* p, const float* v) {
    RowIO<4, false>::store(p, v);
    RowIO<4, false>::store(p + 4, v + 4);
  }
};
template <>
struct RowIO<1, false> {
  typedef float T;
  typedef float Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *p; }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) { v[0] = x; }
  static __device__ __forceinline__ void load(const T* p, float* v) { v[0] = *p; }
  static __device__ __forceinline__ void store(T* p, const float* v) { *p = v[0]; }
};

__device__ __forceinline__ float bf2f(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint32_t f2bf(float f) {  // round to nearest even (finite values)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

template <>
struct RowIO<4, true> {
  typedef uint16_t T;
  typedef uint2 Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *reinterpret_cast<const uint2*>(p); }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) {
    v[0] = bf2f(x.x & 0xFFFFu); v[1] = bf2f(x.x >> 16); v[2] = bf2f(x.y & 0xFFFFu); v[3] = bf2f(x.y >> 16);
  }
  static __device__ __forceinline__ void load(const T* p, float* v) { unpack(load_raw(p), v); }
  static __device__ __forceinline__ void store(T* p, const float* v) {
    *reinterpret_cast<uint2*>(p) = make_uint2(f2bf(v[0]) | (f2bf(v[1]) << 16), f2bf(v[2]) | (f2bf(v[3]) << 16));
  }
};
template <>
struct RowIO<8, true> {
  typedef uint16_t T;
  typedef uint4 Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *reinterpret_cast<const uint4*>(p); }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) {
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = bf2f(w[i] & 0xFFFFu);
      v[2 * i + 1] = bf2f(w[i] >> 16);
    }
  }
  static __device__ __forceinline__ void load(const T* p, float* v) { unpack(load_raw(p), v); }
  static __device__ __forceinline__ void store(T* p, const float* v) {
    *reinterpret_cast<uint4*>(p) = make_uint4(f2bf(v[0]) | (f2bf(v[1]) << 16), f2bf(v[2]) | (f2bf(v[3]) << 16),
                                              f2bf(v[4]) | (f2bf(v[5]) << 16), f2bf(v[6]) | (f2bf(v[7]) << 16));
  }
};
template <>
struct RowIO<2, true> {
  typedef uint16_t T;
  typedef uint32_t Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *reinterpret_cast<const uint32_t*>(p); }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) {
    v[0] = bf2f(x & 0xFFFFu); v[1] = bf2f(x >> 16);
  }
  static __device__ __forceinline__ void load(const T* p, float* v) { unpack(load_raw(p), v); }
  static __device__ __forceinline__ void store(T* p, const float* v) {
    *reinterpret_cast<uint32_t*>(p) = f2bf(v[0]) | (f2bf(v[1]) << 16);
  }
};
template <>
struct RowIO<1, true> {
  typedef uint16_t T;
  typedef uint16_t Raw;
  static __device__ __forceinline__ Raw load_raw(const T* p) { return *p; }
  static __device__ __forceinline__ void unpack(const Raw& x, float* v) { v[0] = bf2f(x); }
  static __device__ __forceinline__ void load(const T* p, float* v) { v[0] = bf2f(*p); }
  static __device__ __forceinline__ void store(T* p, const float* v) { *p = (uint16_t)f2bf(v[0]); }
};

template <int VEC>
__device__ __forceinline__ void ld_f32(const float* p, float* v) { RowIO<VEC, false>::load(p, v); }
template <int VEC>
__device__ __forceinline__ void st_f32(float* p, const float* v) { RowIO<VEC, false>::store(p, v); }

// Pooled outputs are written once per launch and not read again by it: the
// non-temporal hint marks their lines for early eviction, so they do not push
// the hot rows out of the caches (the forward's hot half measured ~20% faster
// alone on the GPU; the same hint on the backward's gradient-row loads was
// slower, and they keep plain loads).
typedef float hl_f4 __attribute__((ext_vector_type(4)));
template <int VEC>
__device__ __forceinline__ void st_f32_nt(float* p, const float* v) {
  if constexpr (VEC == 4 || VEC == 8) {
#pragma unroll
    for (int i = 0; i < VEC; i += 4) {
      const hl_f4 x = {v[i], v[i + 1], v[i + 2], v[i + 3]};
      __builtin_nontemporal_store(x, reinterpret_cast<hl_f4*>(p + i));
    }
  } else {
    RowIO<VEC, false>::store(p, v);
  }
}

struct eb_geom {
  int32_t D, vpr, G, NG, cchunks, VEC;
};

static inline eb_geom eb_make_geom(int32_t D, int vec) {
  eb_geom g;
  g.D = D;
  g.VEC = vec;
  g.vpr = D / vec;
  g.G = g.vpr < 64 ? g.vpr : 64;
  g.NG = 64 / g.G;
  g.cchunks = (g.vpr + 63) / 64;
  return g;
}

// bf16 rows take 8 elements per lane (16-byte loads), fp32 rows 4; fewer
// when the dimension or a pointer's alignment does not allow them
static inline int eb_pick_vec(int32_t D, size_t esize, std::initializer_list<const void*> ptrs) {
  int vec = (esize == 2 && D % 8 == 0) ? 8 : (D % 4 == 0 ? 4 : (D % 2 == 0 ? 2 : 1));
  for (;;) {
    bool ok = true;
    for (const void* p : ptrs)
      if (p && ((uintptr_t)p % (vec * esize) != 0 || (uintptr_t)p % (vec * 4) != 0)) ok = false;
    if (ok || vec == 1) return vec;
    vec >>= 1;
  }
}

// selected-sample count
__device__ __forceinline__ int32_t eb_nsel(const int32_t* ids, const int32_t* n_dev, int32_t n_max) {
  if (ids && n_dev) return min(max(*n_dev, 0), n_max);
  return n_max;
}

// ----------------------------------------------------------------------------- forward
// A row group takes FC (bags of about one lookup) or 1 (multi-hot bags)
// consecutive bag slots of the selection (slot q = bag j of selected sample
// q / bps) and issues the loads of all of them before using any: offsets,
// then codes, then rows, so FC rows per lane are in flight.  When every bag of
// the chunk holds one lookup (one-hot features) that is the whole work;
// otherwise bags are pooled one by one (eb_bag).
//
// A bag's sum is the sum of its hot rows plus the sum of its staging (cold)
// rows, each in CSR order, so that the two halves can run apart with
// identical results: PART 0 does both, PART 1 only the hot rows (writing the
// partial sum), PART 2 adds the cold rows' sum onto the stored partial sum
// (bags without cold rows are left alone).  The hot half needs no fetched row,
// so it runs while the working parameters still travel over the host link.
#ifndef FC
#define FC 4  // bag slots per row group of the forward (4 measured fastest of 4, 6, 8, 12, 16)
#endif
// bags of several lookups each (multi-hot): one bag per row group, so that
// more groups pool at once; bags of about one lookup: FC per group
static inline int32_t eb_bags_per_group(int64_t n_lookups, int64_t n_bags) { return n_lookups > 2 * n_bags ? 1 : FC; }
__device__ __forceinline__ bool eb_code_row(uint32_t cu, uint32_t n_hot, uint32_t k_cap, int32_t stg_rows,
                                            int64_t* row, bool* stg) {
  if (cu < n_hot) {
    *row = cu;
    *stg = false;
    return true;
  }
  if (cu >= k_cap && cu - k_cap < (uint32_t)stg_rows) {
    *row = cu - k_cap;
    *stg = true;
    return true;
  }
  return false;
}

enum { EB_HOT_ROWS, EB_STG_ROWS, EB_ANY_ROWS };

// The narrow form (row groups of fewer than 8 lanes), 4 codes and then their 4
// rows at a time: the bag's rows of the kind asked for, hot ones added to acc_h,
// staging ones to acc_c, each in CSR order; *anyc: some staging row was found
// (for EB_HOT_ROWS: some hot one).  Codes that name no row are flagged except by
// the staging pass.
template <int VEC, bool BF, int KIND>
__device__ __forceinline__ void eb_pass4(float* acc_h, float* acc_c, bool* anyc,
                                         const typename RowIO<VEC, BF>::T* w_hot,
                                         const typename RowIO<VEC, BF>::T* stg, int32_t stg_rows, uint32_t n_hot,
                                         uint32_t k_cap, const int32_t* __restrict__ codes, int32_t lo, int32_t hi,
                                         eb_geom g, int64_t col, bool cact, int gl, uint32_t* err) {
  for (int32_t i = lo; i < hi; i += 4) {
    uint32_t cc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) cc[k] = i + k < hi ? (uint32_t)codes[i + k] : 0u;
    float v[4][VEC];
    bool use[4], cold[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      int64_t r = 0;
      bool st = false;
      const bool in = i + k < hi;
      const bool ok = in && eb_code_row(cc[k], n_hot, k_cap, stg_rows, &r, &st);
      use[k] = ok && (KIND == EB_ANY_ROWS || st == (KIND == EB_STG_ROWS));
      cold[k] = st;
      *anyc = *anyc || (use[k] && (KIND == EB_HOT_ROWS || st));
      if (use[k] && cact)
        RowIO<VEC, BF>::load((KIND == EB_STG_ROWS || (KIND == EB_ANY_ROWS && st) ? stg : w_hot) + r * g.D + col, v[k]);
      if (KIND != EB_STG_ROWS && in && !ok && gl == 0) hl_flag(err, HL_DEVERR_BAD_CODE);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (use[k] && cact) {
        if (KIND == EB_STG_ROWS || (KIND == EB_ANY_ROWS && cold[k])) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc_c[e] += v[k][e];
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc_h[e] += v[k][e];
        }
      }
  }
}

#ifndef EB_SEG_ROWS
#define EB_SEG_ROWS 8  // rows in flight per lane in the passes' wide form
#endif

// The wide form's segment: lane gl's lookup b0 + gl of [b0, hi) as the address of
// its row with EB_USED (a row of the kind asked for: hot, staging, or any) and
// EB_STG (a staging row) in bits no address has, 0 for none (past hi, another
// kind, or a code that names no row: flagged when `flag`).  Worked out once per
// lookup, by its own lane, and passed to the group's lanes by shuffles.
#define EB_USED (1ull << 63)
#define EB_STG (1ull << 62)
template <int VEC, bool BF, int KIND>
__device__ __forceinline__ uint64_t eb_seg_addr(const typename RowIO<VEC, BF>::T* w_hot,
                                                const typename RowIO<VEC, BF>::T* stg,
                                                const int32_t* __restrict__ codes, int32_t b0, int32_t hi, int gl,
                                                uint32_t n_hot, uint32_t k_cap, int32_t stg_rows, eb_geom g, bool flag,
                                                uint32_t* err) {
  const int32_t i = b0 + gl;
  if (i >= hi) return 0;
  int64_t r = 0;
  bool st = false;
  if (!eb_code_row((uint32_t)codes[i], n_hot, k_cap, stg_rows, &r, &st)) {
    if (flag) hl_flag(err, HL_DEVERR_BAD_CODE);
    return 0;
  }
  if (KIND == EB_HOT_ROWS ? st : (KIND == EB_STG_ROWS ? !st : false)) return 0;
  return (uint64_t)((KIND == EB_STG_ROWS || (KIND == EB_ANY_ROWS && st) ? stg : w_hot) + r * g.D) | EB_USED |
         (st ? EB_STG : 0ull);
}

// The rows of a segment's lookups k0 .. k0 + EB_SEG_ROWS - 1 for this lane:
// addresses from the group's lanes (first lane g0), all loads in flight
// together.  An address past the segment's n lookups repeats the last one's
// and is not used.
template <int VEC, bool BF>
__device__ __forceinline__ void eb_seg_rows(uint64_t mine, int g0, int k0, int n, int64_t col, bool cact,
                                            uint32_t (&fl)[EB_SEG_ROWS],
                                            typename RowIO<VEC, BF>::Raw (&rv)[EB_SEG_ROWS]) {
  typedef typename RowIO<VEC, BF>::T T;
#pragma unroll
  for (int k = 0; k < EB_SEG_ROWS; ++k) {
    const int src = g0 + min(k0 + k, n - 1);
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)mine, src), hi = (uint32_t)__shfl((int)(mine >> 32), src);
    fl[k] = k0 + k < n && cact ? hi : 0u;
    if (fl[k] & (uint32_t)(EB_USED >> 32))
      rv[k] = RowIO<VEC, BF>::load_raw(
          reinterpret_cast<const T*>(((uint64_t)(hi & ~(uint32_t)((EB_USED | EB_STG) >> 32)) << 32) | lo) + col);
  }
}

// acc += the bag's rows of one kind (hot, or staging when COLD), in CSR order;
// *any: some row of that kind was found (on lanes that hold columns).  Invalid
// codes are flagged by the hot pass only.  Called by a whole row group at once
// (its G lanes in the same control flow).  Row groups of 8 lanes or more take the
// wide form's segments of G lookups, 8 rows in flight; narrower groups load 4
// codes, then 4 rows, at a time.  Either way each lane adds the rows in CSR
// order.
template <int VEC, bool BF, bool COLD>
__device__ __forceinline__ void eb_pass(float* acc, const typename RowIO<VEC, BF>::T* w_hot,
                                        const typename RowIO<VEC, BF>::T* stg, int32_t stg_rows, uint32_t n_hot,
                                        uint32_t k_cap, const int32_t* __restrict__ codes, int32_t lo, int32_t hi,
                                        eb_geom g, int64_t col, bool cact, int gl, uint32_t* err, bool* any) {
  if (g.G < EB_SEG_ROWS) {
    float other[VEC];
    bool some = false;
    eb_pass4<VEC, BF, COLD ? EB_STG_ROWS : EB_HOT_ROWS>(COLD ? other : acc, COLD ? acc : other, &some, w_hot, stg,
                                                        stg_rows, n_hot, k_cap, codes, lo, hi, g, col, cact, gl, err);
    *any = *any || some;
    return;
  }
  const int g0 = (int)(threadIdx.x & 63) - gl;  // the group's first lane
  for (int32_t b0 = lo; b0 < hi; b0 += g.G) {
    const uint64_t mine = eb_seg_addr<VEC, BF, COLD ? EB_STG_ROWS : EB_HOT_ROWS>(w_hot, stg, codes, b0, hi, gl, n_hot,
                                                                                 k_cap, stg_rows, g, !COLD, err);
    const int n = min(g.G, hi - b0);
    for (int k0 = 0; k0 < n; k0 += EB_SEG_ROWS) {
      uint32_t fl[EB_SEG_ROWS];
      typename RowIO<VEC, BF>::Raw rv[EB_SEG_ROWS];
      eb_seg_rows<VEC, BF>(mine, g0, k0, n, col, cact, fl, rv);
#pragma unroll
      for (int k = 0; k < EB_SEG_ROWS; ++k)
        if (fl[k] & (uint32_t)(EB_USED >> 32)) {
          *any = true;
          float v[VEC];
          RowIO<VEC, BF>::unpack(rv[k], v);
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[e] += v[e];
        }
    }
  }
}

// Both kinds at once, into separate sums (hot into acc_h, staging into acc_c,
// each in CSR order: the sums the two single-kind passes give), with one code
// load per segment.  *anyc: some staging row was found.  The vector instructions
// per row bound it as much as the loads' latency does, so a row's kind is a
// branch that all lanes usually take the same way, not a select per element:
// 328,000 lookups in bags of 20, bf16 rows of 128, beside the sort's
// passes: 23 + 25 -> 16.6 + 17.2 us.
template <int VEC, bool BF>
__device__ __forceinline__ void eb_pass_both(float* acc_h, float* acc_c, bool* anyc,
                                             const typename RowIO<VEC, BF>::T* w_hot,
                                             const typename RowIO<VEC, BF>::T* stg, int32_t stg_rows, uint32_t n_hot,
                                             uint32_t k_cap, const int32_t* __restrict__ codes, int32_t lo, int32_t hi,
                                             eb_geom g, int64_t col, bool cact, int gl, uint32_t* err) {
  if (g.G < EB_SEG_ROWS) {
    eb_pass4<VEC, BF, EB_ANY_ROWS>(acc_h, acc_c, anyc, w_hot, stg, stg_rows, n_hot, k_cap, codes, lo, hi, g, col, cact,
                                   gl, err);
    return;
  }
  const int g0 = (int)(threadIdx.x & 63) - gl;
  for (int32_t b0 = lo; b0 < hi; b0 += g.G) {
    const uint64_t mine = eb_seg_addr<VEC, BF, EB_ANY_ROWS>(w_hot, stg, codes, b0, hi, gl, n_hot, k_cap, stg_rows, g,
                                                            true, err);
    const int n = min(g.G, hi - b0);
    for (int k0 = 0; k0 < n; k0 += EB_SEG_ROWS) {
      uint32_t fl[EB_SEG_ROWS];
      typename RowIO<VEC, BF>::Raw rv[EB_SEG_ROWS];
      eb_seg_rows<VEC, BF>(mine, g0, k0, n, col, cact, fl, rv);
#pragma unroll
      for (int k = 0; k < EB_SEG_ROWS; ++k) {
        const bool used = fl[k] & (uint32_t)(EB_USED >> 32), cold = fl[k] & (uint32_t)(EB_STG >> 32);
        if (used && !cold) {
          float v[VEC];
          RowIO<VEC, BF>::unpack(rv[k], v);
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc_h[e] += v[e];
        }
        if (__ballot(cold) != 0) {  // (rare: most rows are hot)
          if (cold) {
            *anyc = true;
            float v[VEC];
            RowIO<VEC, BF>::unpack(rv[k], v);
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc_c[e] += v[e];
          }
        }
      }
    }
  }
}

// One bag pooled into *o (the row group's slice of the bag's output row):
// PART 0 sums the hot rows and the staging rows apart (each in CSR order) and
// stores their sum (the hot sum alone when no staging row is in the bag);
// PART 1 stores the hot sum; PART 2 adds the staging rows' sum onto the stored
// hot sum (bags without staging rows are left alone).  So PART 1 then PART 2
// store what PART 0 does.
template <int VEC, bool BF, int PART>
__device__ __forceinline__ void eb_bag(float* o, const typename RowIO<VEC, BF>::T* w_hot,
                                       const typename RowIO<VEC, BF>::T* stg, int32_t stg_rows, uint32_t n_hot,
                                       uint32_t k_cap, const int32_t* __restrict__ codes, int32_t lo, int32_t hi,
                                       eb_geom g, int64_t col, bool cact, int gl, uint32_t* err) {
  float acc[VEC], accc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    acc[e] = 0.f;
    accc[e] = 0.f;
  }
  bool anyc = false;
  if (PART == 0) {
    eb_pass_both<VEC, BF>(acc, accc, &anyc, w_hot, stg, stg_rows, n_hot, k_cap, codes, lo, hi, g, col, cact, gl,
                          err);
  } else if (PART == 1) {
    bool anyh = false;
    eb_pass<VEC, BF, false>(acc, w_hot, stg, stg_rows, n_hot, k_cap, codes, lo, hi, g, col, cact, gl, err, &anyh);
  } else {
    eb_pass<VEC, BF, true>(accc, w_hot, stg, stg_rows, n_hot, k_cap, codes, lo, hi, g, col, cact, gl, err, &anyc);
    if (!anyc) return;
    if (cact) ld_f32<VEC>(o, acc);
  }
  if (anyc)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] += accc[e];
  if (cact) st_f32_nt<VEC>(o, acc);
}

// The forward's work of block bid of nblk (each of blockDim.x / 64 waves) on the
// chunks [c0, c1) of nbg bags.
template <int VEC, bool BF, int PART>
__device__ __forceinline__ void eb_fwd_body(uint32_t bid, uint32_t nblk, const void* w_hot_, const void* stg_,
                                            int32_t stg_rows, uint32_t n_hot, uint32_t k_cap,
                                            const int32_t* __restrict__ codes, const int32_t* __restrict__ bag_ptr,
                                            int32_t bps, const int32_t* __restrict__ sample_ids,
                                            const int32_t* n_sel_dev, int32_t n_sel_max, float* __restrict__ out,
                                            eb_geom g, int32_t n_samples, int32_t nbg, uint32_t* err,
                                            int64_t c0 = 0, int64_t c1 = INT64_MAX) {
  typedef typename RowIO<VEC, BF>::T T;
  const T* w_hot = (const T*)w_hot_;
  const T* stg = (const T*)stg_;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  if (gi >= g.NG) return;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  const int64_t total = (int64_t)eb_nsel(sample_ids, n_sel_dev, n_sel_max) * bps;
  const int64_t chunks = min((total + nbg - 1) / nbg, c1);
  const int64_t stride = (int64_t)nblk * nw * g.NG;
  for (int64_t c = c0 + ((int64_t)bid * nw + w) * g.NG + gi; c < chunks; c += stride) {
    const int64_t q0 = c * nbg;
    int64_t si = q0 / bps, j = q0 - si * bps;
    int64_t bag[FC];
    bool val[FC];
#pragma unroll
    for (int u = 0; u < FC; ++u) {
      val[u] = u < nbg && q0 + u < total;
      int64_t smp = si;
      if (val[u] && sample_ids) smp = sample_ids[si];
      if (val[u] && (smp < 0 || smp >= n_samples)) {
        if (gl == 0 && PART != 2) hl_flag(err, HL_DEVERR_OUT_OF_RANGE);
        val[u] = false;
      }
      bag[u] = smp * bps + j;
      if (++j == bps) {
        j = 0;
        ++si;
      }
    }
    int32_t lo[FC], hi[FC];
    bool one = true;
#pragma unroll
    for (int u = 0; u < FC; ++u) {
      lo[u] = val[u] ? bag_ptr[bag[u]] : 0;
      hi[u] = val[u] ? bag_ptr[bag[u] + 1] : 1;
    }
#pragma unroll
    for (int u = 0; u < FC; ++u) one = one && (hi[u] - lo[u] == 1);
    if (one) {
      uint32_t cu[FC];
#pragma unroll
      for (int u = 0; u < FC; ++u) cu[u] = val[u] ? (uint32_t)codes[lo[u]] : 0u;
      float v[FC][VEC];
      bool wr[FC];
#pragma unroll
      for (int u = 0; u < FC; ++u) {
        int64_t r = 0;
        bool st = false;
        const bool ok = val[u] && eb_code_row(cu[u], n_hot, k_cap, stg_rows, &r, &st);
        // PART 0 and 1 write every valid bag (PART 1 a zero for a cold row); PART 2 only cold ones
        const bool take = ok && (PART == 0 || (PART == 1 ? !st : st));
        wr[u] = val[u] && (PART == 2 ? take : true);
        if (take && cact) RowIO<VEC, BF>::load((st ? stg : w_hot) + r * g.D + col, v[u]);
        else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[u][e] = 0.f;
        }
        if (PART != 2 && val[u] && !ok && gl == 0) hl_flag(err, HL_DEVERR_BAD_CODE);
      }
      // the sum starts from 0 (PART 2: from the stored hot partial sum, which is 0)
#pragma unroll
      for (int u = 0; u < FC; ++u)
        if (wr[u] && cact) {
          float o[VEC];
          if (PART == 2) ld_f32<VEC>(out + bag[u] * g.D + col, o);
          else
#pragma unroll
            for (int e = 0; e < VEC; ++e) o[e] = 0.f;
#pragma unroll
          for (int e = 0; e < VEC; ++e) o[e] += v[u][e];
          st_f32_nt<VEC>(out + bag[u] * g.D + col, o);
        }
      continue;
    }
    for (int u = 0; u < FC; ++u) {
      if (!val[u]) continue;
      eb_bag<VEC, BF, PART>(out + bag[u] * g.D + col, w_hot, stg, stg_rows, n_hot, k_cap, codes, lo[u], hi[u], g,
                            col, cact, gl, err);
    }
  }
}

// The forward of a one-hot mini-batch over every sample (as many lookups as
// bags: bag j is expected to hold lookup j alone), PART 0 or 1, wave by wave:
// a wave takes a unit of NG * OH_RPG consecutive bags (OH_RPG per row group,
// at most 256 bags), loads their offsets and codes one bag per lane and
// passes the codes to the row groups through LDS; when every bag of the unit
// holds exactly its own lookup, each row group issues its rows' loads all at
// once, then stores them, so a unit costs two dependent rounds of loads.  A
// unit with a bag that is not one-hot is pooled bag by bag as eb_fwd does.
// Same sums, same outputs: the row itself (PART 1: its hot rows only, zero
// for a staging row; zero for a code that names no row).
#define OH_RPG(VEC) ((VEC) >= 8 ? 8 : 16)  // rows per row group per unit (at most): up to 64 floats per lane in flight
#define OH_UNIT 256                // bags per unit (at most)
#define OH_MAXW 16                 // waves per block (at most)

static inline int64_t eb_oh_units(const eb_geom& g, int vec, int64_t n_bags) {
  const int64_t rpg = g.NG * OH_RPG(vec) <= OH_UNIT ? OH_RPG(vec) : OH_UNIT / g.NG, ub = g.NG * rpg;
  return (n_bags + ub - 1) / ub;
}

// The work of block bid of nblk (each of blockDim.x / 64 waves) on the units
// [u0, u1); s_code: a row of OH_UNIT words in LDS per wave.  strict: a bag that
// is not one-hot is also an error of the call (HL_DEVERR_SHAPE).
template <int VEC, bool BF, int PART>
__device__ __forceinline__ void eb_fwd_oh_body(uint32_t bid, uint32_t nblk, const void* w_hot_, const void* stg_,
                                               int32_t stg_rows, uint32_t n_hot, uint32_t k_cap,
                                               const int32_t* __restrict__ codes,
                                               const int32_t* __restrict__ bag_ptr, float* __restrict__ out,
                                               eb_geom g, int64_t n_lookups, int64_t n_bags, uint32_t* err,
                                               uint32_t (*s_code)[OH_UNIT], int64_t u0 = 0,
                                               int64_t u1 = INT64_MAX, bool strict = false) {
  static_assert(PART == 0 || PART == 1, "whole forward or its hot half");
  typedef typename RowIO<VEC, BF>::T T;
  const T* w_hot = (const T*)w_hot_;
  const T* stg = (const T*)stg_;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int gi = lane / g.G, gl = lane - gi * g.G;
  if (bid == 0 && blockIdx.y == 0 && threadIdx.x == 0 && bag_ptr[n_bags] != n_lookups)
    hl_flag(err, HL_DEVERR_SHAPE);
  const bool gact = gi < g.NG;
  const int32_t colv = blockIdx.y * 64 + gl;
  const bool cact = gact && colv < g.vpr;
  const int64_t col = (int64_t)colv * VEC;
  constexpr int RPG = OH_RPG(VEC);
  const int rpg = g.NG * RPG <= OH_UNIT ? RPG : OH_UNIT / g.NG;
  const int64_t ub = (int64_t)g.NG * rpg;  // bags per unit
  const int64_t units = min((n_bags + ub - 1) / ub, u1);
  uint32_t* sc = s_code[w];
  for (int64_t u = u0 + (int64_t)bid * nw + w; u < units; u += (int64_t)nblk * nw) {
    const int64_t b0 = u * ub;
    // offsets and codes, one bag per lane
    bool bad = false;
#pragma unroll
    for (int k = 0; k < OH_UNIT / 64; ++k) {
      const int64_t q = (int64_t)k * 64 + lane, b = b0 + q;
      if (q < ub && b < n_bags) {
        const int32_t lo = bag_ptr[b], hi = bag_ptr[b + 1];
        const uint32_t cu = (uint32_t)codes[b];
        sc[q] = cu;
        bad = bad || lo != b || hi != b + 1;
        if (!bad && !(cu < n_hot || (cu >= k_cap && cu - k_cap < (uint32_t)stg_rows))) hl_flag(err, HL_DEVERR_BAD_CODE);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (__ballot(bad)) {
      if (strict && lane == 0) hl_flag(err, HL_DEVERR_SHAPE);
      // some bag of the unit is not one-hot: bag by bag, its hot rows then
      // (PART 0) its staging rows, in CSR order
      if (gact)
        for (int i = 0; i < rpg; ++i) {
          const int64_t b = b0 + (int64_t)gi * rpg + i;
          if (b >= n_bags) break;
          eb_bag<VEC, BF, PART>(out + b * g.D + col, w_hot, stg, stg_rows, n_hot, k_cap, codes, bag_ptr[b],
                                bag_ptr[b + 1], g, col, cact, gl, err);
        }
    } else if (gact) {
      float v[RPG][VEC];
#pragma unroll
      for (int i = 0; i < RPG; ++i) {
        const int64_t b = b0 + (int64_t)gi * rpg + i;
        const uint32_t cu = i < rpg ? sc[gi * rpg + i] : 0u;
        const bool in = i < rpg && b < n_bags && cact;
        const bool hot = cu < n_hot;
        const bool cold = PART == 0 && cu >= k_cap && cu - k_cap < (uint32_t)stg_rows;
        if (in && (hot || cold)) {
          const T* p = hot ? w_hot + (int64_t)cu * g.D : stg + (int64_t)(cu - k_cap) * g.D;
          RowIO<VEC, BF>::load(p + col, v[i]);
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[i][e] = 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < RPG; ++i) {
        const int64_t b = b0 + (int64_t)gi * rpg + i;
        if (i < rpg && b < n_bags && cact) st_f32_nt<VEC>(out + b * g.D + col, v[i]);
      }
    }
    // (the next unit's codes overwrite sc: every lane has read this one's)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}
