"""The cold plan's selections against the oracle: every sample, the first ones,
a list of samples (8 to 256 threads or whole blocks each; out of order,
repeated, counted on the device), and enough lookups that the rank scan goes back to a look-back."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2204_05436_amd import hotline as hl
from parity_lib import u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,bps,mean,how", [
    (1, 1, 1, "all"), (333, 5, 1, "all"), (333, 5, 3, "first"), (257, 3, 2, "list"), (257, 3, 2, "dup"),
    (64, 8, 20, "list"), (65, 8, 20, "dup"), (1000, 26, 1, "list"), (70, 4, 0, "all"), (8_400_001, 1, 1, "all")])
def test_cold_plan_selection(B, bps, mean, how):
    rng = np.random.default_rng(B + bps)
    n_bags = B * bps
    lens = np.ones(n_bags, np.int64) if mean == 1 else rng.poisson(mean, n_bags)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(ptr[-1])
    n_rows, k_cap = 50_000, 9_000
    hot = np.sort(rng.permutation(n_rows)[:k_cap]).astype(np.uint32)
    gids = (rng.zipf(1.2, n) % n_rows).astype(np.uint32)
    codes = O.remap(hot, gids)
    if how == "all":
        sel, n_max, dev = np.arange(B, dtype=np.int32), B, None
    elif how == "first":
        sel, n_max, dev = np.arange(B // 2, dtype=np.int32), B // 2, None
    else:
        sel = np.sort(rng.permutation(B)[:max(1, B // 2)]).astype(np.int32)
        n_max, dev = B, sel.size
    want_cold, want_codes = O.cold_plan(gids, codes.copy(), ptr, sel, sel.size, bps, k_cap)
    listed = sel
    if how == "dup":
        listed = rng.permutation(np.concatenate([sel, sel[: B - sel.size]])).astype(np.int32)
        dev = listed.size
    h = hl.hl_create(np.array([n_rows], np.uint32), 4, "f32", k_cap)
    try:
        d = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).cuda()
        dg, dc, dp = d(gids), d(codes.astype(np.int32)), d(ptr)
        ids = cnt = None
        if how in ("list", "dup"):
            ids = d(np.concatenate([listed, np.full(B - listed.size, -7, np.int32)]))
            cnt = torch.tensor([dev], dtype=torch.int32, device="cuda")
        cap = max(1, n)
        cold, nc = torch.zeros(cap, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n_bags, B), dtype=torch.uint8, device="cuda")
        for _ in range(2):  # (the table is left clean)
            dc.copy_(d(codes.astype(np.int32)))
            hl.hl_cold_plan(h, dg, dc, dp, B, bps, n, ids, cnt, n_max, cap, cold, nc, ws)
            assert int(nc.item()) == want_cold.size
            assert np.array_equal(u32(cold[:want_cold.size]), want_cold)
            assert np.array_equal(dc.cpu().numpy(), want_codes)
        assert hl.hl_last_device_error(h) == 0
    finally:
        h.close()


@pytest.mark.parametrize("B,bps,base,long", [
    (1, 1, 33, 0), (3, 2, 4000, 0), (40, 3, 11, 40), (64, 2, 0, 17), (300, 1, 1, 33), (200, 1, 1, 6000), (9, 2, 600, 9000)])
def test_cold_plan_long_samples(B, bps, base, long):
    """Listed samples of very different lengths: about 8 to 256 threads a sample,
    samples past 4 lookups per thread by the block, several blocks a sample."""
    rng = np.random.default_rng(B + base)
    n_bags, n_rows, k_cap = B * bps, 20_000, 2_000
    lens = np.full(n_bags, base)
    lens[::7] = np.maximum(lens[::7], long)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(ptr[-1])
    hot = np.sort(rng.permutation(n_rows)[:k_cap]).astype(np.uint32)
    gids = rng.integers(0, n_rows, n).astype(np.uint32)
    gids[rng.random(n) < 0.5] = 7
    codes = O.remap(hot, gids).astype(np.int32)
    sel = np.sort(rng.permutation(B)[:max(1, (2 * B) // 3)]).astype(np.int32)
    want_cold, want_codes = O.cold_plan(gids, codes.copy(), ptr, sel, sel.size, bps, k_cap)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).cuda()
    h = hl.hl_create(np.array([n_rows], np.uint32), 4, "f32", k_cap)
    try:
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n_bags, B), dtype=torch.uint8, device="cuda")
        cold, nc = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        for _ in range(2):
            dc = d(codes)
            hl.hl_cold_plan(h, d(gids), dc, d(ptr), B, bps, n, d(sel), None, sel.size, n, cold, nc, ws)
            assert int(nc.item()) == want_cold.size
            assert np.array_equal(u32(cold[:want_cold.size]), want_cold)
            assert np.array_equal(dc.cpu().numpy(), want_codes)
        assert hl.hl_last_device_error(h) == 0
    finally:
        h.close()


@pytest.mark.parametrize("n_max", [200, 1 << 26, 2**31 - 1])
@pytest.mark.parametrize("mean", [1, 120])
def test_cold_plan_loose_bound(n_max, mean):
    """A list counted on the device, under bounds far above the number of samples
    (n_sel_max only limits the count), shorter and (samples named again) longer
    than the samples; a listed id that is no sample is reported."""
    rng = np.random.default_rng(mean)
    B, bps, n_rows, k_cap = 37, 3, 5000, 900
    lens = rng.poisson(mean, B * bps)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(ptr[-1])
    hot = np.sort(rng.permutation(n_rows)[:k_cap]).astype(np.uint32)
    gids = (rng.zipf(1.2, n) % n_rows).astype(np.uint32)
    codes = O.remap(hot, gids).astype(np.int32)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).cuda()
    h = hl.hl_create(np.array([n_rows], np.uint32), 4, "f32", k_cap)
    try:
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, B * bps, B), dtype=torch.uint8, device="cuda")
        cold, nc = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        for listed in (5, B, 190):
            sel = np.resize(rng.permutation(B), listed).astype(np.int32)
            cnt = torch.tensor([listed], dtype=torch.int32, device="cuda")
            uniq = np.unique(sel).astype(np.int32)
            want_cold, want_codes = O.cold_plan(gids, codes.copy(), ptr, uniq, uniq.size, bps, k_cap)
            dc = d(codes)
            hl.hl_cold_plan(h, d(gids), dc, d(ptr), B, bps, n, d(sel), cnt, n_max, n, cold, nc, ws)
            assert int(nc.item()) == want_cold.size
            assert np.array_equal(u32(cold[:want_cold.size]), want_cold)
            assert np.array_equal(dc.cpu().numpy(), want_codes)
            assert hl.hl_last_device_error(h) == 0
        sel[189] = B
        hl.hl_cold_plan(h, d(gids), d(codes), d(ptr), B, bps, n, d(sel), cnt, n_max, n, cold, nc, ws)
        assert hl.hl_last_device_error(h) == hl.DEVERR["OUT_OF_RANGE"]
    finally:
        h.close()


def test_cold_plan_list_without_lookups():
    """A mini-batch of empty bags: no cold rows, and a listed id that names no
    sample is still reported."""
    h = hl.hl_create(np.array([10], np.uint32), 4, "f32", 4)
    try:
        z = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")
        ws = torch.zeros(hl.hl_workspace_bytes(h, 1, 6, 3), dtype=torch.uint8, device="cuda")
        for ids, err in (([0, 2], 0), ([2, 3], hl.DEVERR["OUT_OF_RANGE"]), ([-1, 0], hl.DEVERR["OUT_OF_RANGE"])):
            nc = torch.full((1,), 5, dtype=torch.int32, device="cuda")
            sel = torch.tensor(ids, dtype=torch.int32, device="cuda")
            hl.hl_cold_plan(h, z(1), z(1), z(7), 3, 2, 0, sel, None, 2, 0, None, nc, ws)
            assert int(nc.item()) == 0
            assert hl.hl_last_device_error(h) == err
    finally:
        h.close()
