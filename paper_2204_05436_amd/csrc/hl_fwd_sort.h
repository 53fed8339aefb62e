// The forward over every sample beside the general sort's passes (the grouping
// of mini-batches that are not grouped table by table: multi-hot bags, more than
// 8192 lookups per table).  A pass is bound by latency and takes one block per
// tile (about 100 of 1024 threads, with most of a compute unit's LDS); the
// forward is bound by its row loads and needs only the codes.  So each pass's
// launch holds the pass's blocks first, then blocks that pool that launch's share
// of the bags: on the compute units the pass leaves free, then on all of them.
// The forward's registers allow 16 to 20 waves per compute unit in its own
// launch and 16 here.  Nothing one side writes is read by the other.
// Batch 32768 of 26 tables (852,000 lookups, f32 rows of 64): the forward 56.0 and
// the passes 23.6 + 17.5 us apart, 38 + 33 together; 328,000 lookups in bags of
// 20 (bf16 rows of 128): 25.7, 13.3 and 11.2 apart, 23 + 25 together (16 + 17 with
// the forward's fewer instructions per row, its own launch then 19).
#pragma once
#include "hl_embbag_fwd.h"
#include "hl_sort_pass.h"

struct eb_side {
  const void *w_hot, *stg;
  int32_t stg_rows;
  uint32_t n_hot, k_cap;
  const int32_t *codes, *bag_ptr;
  float* out;
  eb_geom g;
  int64_t n_lookups, n_bags;
  int32_t n_samples, bps, nbg;
  int one_hot;         // as many lookups as bags: wave units (eb_fwd_oh_body), else chunks of nbg bags
  int64_t from, to;    // this launch's units or chunks
};

template <int VEC, bool BF, int NB, int ITEMS, bool FIRST>
__global__ void __launch_bounds__(HL_SORT_THREADS)
eb_fwd_srt(srt_args a, eb_side f, hl_hook hk) {
  __shared__ srt_lds<NB, ITEMS> lds;
  hl_hook_head(hk);
  const uint32_t sort_blocks = a.tiles + a.sums;
  if (blockIdx.x < sort_blocks) {
    srt_pass_body<NB, ITEMS, FIRST>(a, lds);
    return;
  }
  const uint32_t bid = blockIdx.x - sort_blocks, nblk = gridDim.x - sort_blocks;
  static_assert(HL_SORT_WAVES <= OH_MAXW, "the one-hot forward's waves");
  static_assert(sizeof(lds) >= sizeof(uint32_t) * HL_SORT_WAVES * OH_UNIT, "the one-hot forward's LDS");
  if (f.one_hot)
    eb_fwd_oh_body<VEC, BF, 0>(bid, nblk, f.w_hot, f.stg, f.stg_rows, f.n_hot, f.k_cap, f.codes, f.bag_ptr, f.out, f.g,
                               f.n_lookups, f.n_bags, a.err, reinterpret_cast<uint32_t(*)[OH_UNIT]>(&lds), f.from, f.to);
  else
    eb_fwd_body<VEC, BF, 0>(bid, nblk, f.w_hot, f.stg, f.stg_rows, f.n_hot, f.k_cap, f.codes, f.bag_ptr, f.bps, nullptr,
                            nullptr, f.n_samples, f.out, f.g, f.n_samples, f.nbg, a.err, f.from, f.to);
}

template <int VEC, bool BF>
static void eb_fwd_srt_passes(hl_handle* h, hl_sort_ws& ws, const hl_sort_src& src, uint32_t n, int npasses, int b,
                              int nb, int items, int cus, hipStream_t s, const hl_hook& hk, const hl_sort_side& side) {
  eb_side f{};
  f.w_hot = side.w_hot;
  f.stg = side.stg;
  f.stg_rows = src.stg_rows;
  f.n_hot = src.n_hot;
  f.k_cap = src.k_cap;
  f.codes = src.codes;
  f.bag_ptr = src.bag_ptr;
  f.out = side.out;
  f.g = eb_make_geom(h->dim, VEC);
  f.n_lookups = side.n_lookups;
  f.n_bags = src.n_bags;
  f.n_samples = side.n_samples;
  f.bps = side.bps;
  f.nbg = eb_bags_per_group(side.n_lookups, src.n_bags);
  f.one_hot = side.n_lookups == src.n_bags;
  // units (of a wave) or chunks (of a row group), split evenly over the passes;
  // bags that fit the compute units beside the first pass all at once go there
  // together, since each launch would last as long as its longest bag (3 bags of
  // 80,000 lookups: 26.7 ms shared, 13.0 together)
  const int64_t total = f.one_hot ? eb_oh_units(f.g, VEC, src.n_bags) : (src.n_bags + f.nbg - 1) / f.nbg;
  const int64_t per_block = f.one_hot ? HL_SORT_WAVES : HL_SORT_WAVES * f.g.NG;
  const srt_plan pl{npasses, b, nb};
  int p = 0;
  bool together = false;
  srt_dispatch(nb, items, [&](auto NB, auto IT) {
    constexpr int nbins = decltype(NB)::value, it = decltype(IT)::value;
    srt_passes<nbins, it>(h, ws, src, nullptr, n, pl, hk, [&](auto first, const srt_args& a, const hl_hook& k) {
      if (p == 0) together = !f.one_hot && (total + per_block - 1) / per_block <= cus - (int64_t)(a.tiles + a.sums);
      f.from = together ? (p == 0 ? 0 : total) : total * p / npasses;
      f.to = together ? total : total * (p + 1) / npasses;
      ++p;
      int64_t blocks = (f.to - f.from + per_block - 1) / per_block;
      if (blocks > 4096) blocks = 4096;
      HL_KERNEL(h, s, "eb_fwd_srt", (eb_fwd_srt<VEC, BF, nbins, it, decltype(first)::value>),
                dim3(a.tiles + a.sums + (uint32_t)blocks), dim3(HL_SORT_THREADS), 0, s, a, f, k);
    });
  });
}
