"""The allocation-free backward (hl_embbag_bwd_sgd_noalloc, its workspace a
static device array) against hl_embbag_bwd_sgd with a caller's workspace, on
the same inputs, through the C ABI: the updated hot and staging rows bit for
bit (same kernels, same grouping), on two calls in a row, the second with a
smaller mini-batch (the array keeps the first call's contents), mini-batches
that nearly fill the array, and one too large for it refused with
HL_ERR_CAPACITY."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2204_05436_amd import configs, hotline as hl, workload as W
from paper_2204_05436_amd.runner import HotPath, to_device
from parity_lib import log, make_table

pytestmark = pytest.mark.gpu


def _prefix(mb, n_samples):
    """The first n_samples samples of a host batch."""
    ptr = np.asarray(mb.bag_ptr)[: n_samples * mb.bags_per_sample + 1].copy()
    return dataclasses.replace(mb, rows=np.asarray(mb.rows)[: int(ptr[-1])].copy(), bag_ptr=ptr,
                               n_samples=n_samples)


@pytest.mark.parametrize("name", ["dlrm-large", "multi-hot"])
def test_noalloc_matches_workspace_backward(name):
    w = configs.scaled(configs.WORKLOADS[name], batch=2048, row_scale=0.02, name=name + "-noalloc")
    rows = W.table_rows(w)
    n_rows = int(rows.sum(dtype=np.int64))
    prof = [W.make_batch(w, rows, i) for i in range(4)]
    full = W.make_batch(w, rows, 4)
    cases = [full, _prefix(full, 777)]  # two calls in a row, the second smaller
    table = make_table(w, n_rows)
    hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + cases), w.batch)
    h = hp.h
    try:
        hp.learn([to_device(p, "cuda") for p in prof])
        n_hot = hp.n_hot
        for ci, mb in enumerate(cases):
            dY = W.make_dy(w, 4 + ci, mb.n_bags)
            b = to_device(mb, "cuda", dY)
            B, bps, L = b.n_samples, b.bps, b.n_lookups
            log(f"[noalloc] {name} call {ci}: B={B} L={L}")
            # codes and staging rows as a step makes them
            hl.hl_dispatch(h, b.rows, b.bag_ptr, B, bps, L, hp.gids, hp.codes, hp.flags, hp.pop, hp.nonpop,
                           hp.counts, hp.ws)
            hl.hl_cold_gather(h, hp.gids, hp.codes, b.bag_ptr, B, bps, L, hp.nonpop, hp.counts[1:], B,
                              table.dev, hp.staging, hp.staging_cap, hp.cold_ids, hp.n_cold, hp.ws)
            torch.cuda.synchronize()
            n_cold = int(hp.n_cold.item())
            w_a, w_b = hp.w_hot.clone(), hp.w_hot.clone()
            s_a, s_b = hp.staging.clone(), hp.staging.clone()
            hl.hl_embbag_bwd_sgd(h, w_a, s_a, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B, b.dY,
                                 w.lr, hp.ws)
            hl.hl_embbag_bwd_sgd_noalloc(h, w_b, s_b, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B,
                                         b.dY, w.lr)
            torch.cuda.synchronize()
            assert hp.device_error() == 0, f"call {ci}"
            assert np.array_equal(w_a[:n_hot].cpu().numpy().view(np.uint8), w_b[:n_hot].cpu().numpy().view(np.uint8)), \
                f"call {ci}: hot rows differ"
            assert np.array_equal(s_a[:n_cold].cpu().numpy().view(np.uint8),
                                  s_b[:n_cold].cpu().numpy().view(np.uint8)), f"call {ci}: staging rows differ"
            changed = int((w_a[:n_hot] != hp.w_hot[:n_hot]).any(dim=1).sum())
            assert changed > 0, "the step changed no hot row"
            log(f"[noalloc] {name} call {ci}: {changed} hot rows and {n_cold} staging rows equal")
        # a mini-batch whose plan exceeds the array is refused before any work
        big = hl.hl_noalloc_scratch_bytes() // 16
        with pytest.raises(hl.HotlineError) as e:
            hl.hl_embbag_bwd_sgd_noalloc(h, hp.w_hot, hp.staging, hp.staging_cap, hp.codes, hp.pop, 1, big, big,
                                         None, None, 1, hp.out, w.lr)
        assert e.value.status == 3
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("dim,n", [(192, 215_604), (256, 168_756), (320, 138_648), (384, 117_632), (1024, 46_784)])
def test_noalloc_largest(dim, n):
    """Mini-batches of one lookup per bag that nearly fill the 32 MiB: accepted,
    with the same rows as the workspace form, twice in a row (the second call
    finds the first one's tile sums where its sort keeps counts)."""
    rng = np.random.default_rng(dim)
    n_hot, n_stg = 1000, 700
    h = hl.hl_create(np.array([5000], np.uint32), dim, "f32", n_hot)
    try:
        hl.hl_set_hot(h, torch.arange(n_hot, dtype=torch.int32, device="cuda"), n_hot)
        g = rng.zipf(1.2, n) % (n_hot + n_stg)
        codes = torch.from_numpy(g.astype(np.int32)).cuda()  # (k_cap = n_hot: row g of the two together)
        ptr = torch.arange(n + 1, dtype=torch.int32, device="cuda")
        dY = torch.randn((n, dim), device="cuda")
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n, n), dtype=torch.uint8, device="cuda")
        a = torch.randn((n_hot + n_stg, dim), device="cuda")
        b = a.clone()
        for _ in range(2):
            hl.hl_embbag_bwd_sgd(h, a[:n_hot], a[n_hot:], n_stg, codes, ptr, n, 1, n, None, None, n, dY, 0.01, ws)
            hl.hl_embbag_bwd_sgd_noalloc(h, b[:n_hot], b[n_hot:], n_stg, codes, ptr, n, 1, n, None, None, n, dY, 0.01)
            assert hl.hl_last_device_error(h) == 0
            assert torch.equal(a, b)
    finally:
        h.close()
