"""The general grouping's sort at the sizes and layouts where its branches
switch: tiles of 1, 2, 4 and 8 items per thread (128 tiles of each), the last
tile and the last group of 8 tiles full or nearly empty, digit widths on either
side of each bin count, two and three passes, and the ways a tile finds its
lookups' bags (one lookup per bag, a window of bags around the average position,
a search over all bags).  Checked against numpy's stable order of the keys."""
import numpy as np
import pytest
import torch

from paper_2204_05436_amd import hotline as hl
from parity_lib import check_grouping

pytestmark = pytest.mark.gpu


def _lens(rng, layout, n):
    """Bag lengths that add up to n."""
    if layout == "even":  # about 3 lookups a bag
        nb = max(1, n // 3)
        return rng.multinomial(n, np.full(nb, 1.0 / nb))
    if layout == "one":
        return np.ones(n, np.int64)
    if layout == "as_many":  # as many lookups as bags, not one each
        lens = np.ones(n, np.int64)
        lens[n // 2], lens[n // 2 + 1:n // 2 + 4] = 4, 0
        return lens
    if layout == "head":  # nearly all lookups in the first bag, thousands of empty bags, then single lookups
        k = min(5, n - 1)
        return np.concatenate([[n - k], np.zeros(9000, np.int64), np.ones(k, np.int64)])
    if layout == "tail":  # the other way round
        k = min(5, n - 1)
        return np.concatenate([np.ones(k, np.int64), np.zeros(9000, np.int64), [n - k]])
    raise ValueError(layout)


SIZES = [
    (1, "even", 10), (1023, "even", 9), (1025, "tail", 17), (8 * 1024, "head", 16), (8 * 1024 + 1, "even", 18),
    (9001, "one", 19), (9002, "as_many", 20), (20000, "head", 22), (20000, "tail", 24),
    (128 * 1024, "even", 18), (128 * 1024 + 1, "even", 20), (128 * 2048 + 1, "tail", 21), (128 * 2048, "one", 22),
    (128 * 4096, "head", 17), (128 * 4096 + 1, "even", 23), (128 * 4096 + 3, "as_many", 22),
    (128 * 8192 + 5, "even", 12)]


@pytest.mark.parametrize("n,layout,bits", SIZES)
def test_grouping_sort(n, layout, bits):
    rng = np.random.default_rng(n + bits)
    lens = _lens(rng, layout, n)
    nb = lens.size
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert ptr[-1] == n
    n_hot, k_cap = 300, 400
    cap = (1 << bits) - 1 - n_hot  # the keys' width: bit length of n_hot + cap
    h = hl.hl_create(np.array([1000], np.uint32), 4, "f32", k_cap)
    try:
        hl.hl_set_hot(h, torch.arange(n_hot, dtype=torch.int32, device="cuda"), n_hot)
        hot = rng.zipf(1.3, n) % n_hot
        cold = k_cap + np.where(rng.random(n) < 0.5, rng.integers(0, cap, n), rng.zipf(1.2, n) % cap)
        codes = np.where(rng.random(n) < 0.6, hot, cold).astype(np.int32)
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, nb, nb), dtype=torch.uint8, device="cuda")
        dc, dp = torch.from_numpy(codes).cuda(), torch.from_numpy(ptr).cuda()
        keys, bags = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
        bag_of = np.repeat(np.arange(nb, dtype=np.uint32), lens)
        for again in range(2):  # (the counters and published words of a call must not outlive it)
            hl.hl_embbag_bwd_plan(h, cap, dc, dp, nb, 1, n, None, None, nb, ws)
            hl.hl_embbag_bwd_grouping(h, cap, nb, 1, n, ws, keys, bags)
            check_grouping(keys.cpu().numpy().view(np.uint32), bags.cpu().numpy().view(np.uint32), codes, bag_of, n_hot,
                           k_cap, f"{layout} {n}")
        assert hl.hl_last_device_error(h) == 0
    finally:
        h.close()


@pytest.mark.parametrize("dim,dtype", [(16, "f32"), (64, "f32"), (64, "bf16")])
@pytest.mark.parametrize("n,layout,bits", SIZES)
def test_forward_beside_sort(n, layout, bits, dim, dtype):
    """hl_embbag_fwd_plan where the forward runs beside the sort's passes: bags of
    any layout, tiles of every size, one to three passes to share the bags among;
    rows of fewer than 8 lanes and of more.  Pooled outputs bit for bit those of
    hl_embbag_fwd, the grouping that of hl_embbag_bwd_plan."""
    rng = np.random.default_rng(n + bits)
    lens = _lens(rng, layout, n)
    nb = lens.size
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n_hot, k_cap = 300, 400
    cap = (1 << bits) - 1 - n_hot
    h = hl.hl_create(np.array([1000], np.uint32), dim, dtype, k_cap)
    try:
        hl.hl_set_hot(h, torch.arange(n_hot, dtype=torch.int32, device="cuda"), n_hot)
        hot = rng.zipf(1.3, n) % n_hot
        cold = k_cap + np.where(rng.random(n) < 0.5, rng.integers(0, cap, n), rng.zipf(1.2, n) % cap)
        dc = torch.from_numpy(np.where(rng.random(n) < 0.6, hot, cold).astype(np.int32)).cuda()
        dp = torch.from_numpy(ptr).cuda()
        tt = torch.float32 if dtype == "f32" else torch.bfloat16
        w, s = (torch.randn((k, dim), device="cuda", dtype=tt) for k in (n_hot, cap))
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, nb, nb), dtype=torch.uint8, device="cuda")
        i32 = lambda: torch.zeros(n, dtype=torch.int32, device="cuda")
        k1, b1, k2, b2 = i32(), i32(), i32(), i32()
        want, out = (torch.full((nb, dim), v, device="cuda") for v in (7.0, 8.0))
        hl.hl_embbag_fwd(h, w, s, cap, dc, dp, nb, 1, n, None, None, nb, want)
        hl.hl_embbag_bwd_plan(h, cap, dc, dp, nb, 1, n, None, None, nb, ws)
        hl.hl_embbag_bwd_grouping(h, cap, nb, 1, n, ws, k1, b1)
        for again in range(2):
            hl.hl_embbag_fwd_plan(h, w, s, cap, dc, dp, nb, 1, n, out, ws)
            hl.hl_embbag_bwd_grouping(h, cap, nb, 1, n, ws, k2, b2)
            assert torch.equal(out, want)
            assert torch.equal(k1, k2) and torch.equal(b1, b2)
        assert hl.hl_last_device_error(h) == 0
    finally:
        h.close()


@pytest.mark.parametrize("B,T", [(1, 1), (1, 64), (333, 64), (1023, 3), (1024, 2), (1025, 3), (2048, 2), (2049, 2),
                                 (4096, 2), (4097, 2), (8191, 1)])
def test_forward_with_table_sorts(B, T):
    """The forward with the tables' sorts in its launch (hl_embbag_fwd_plan) at
    the edges of its items per thread and of where the sorts read the codes
    themselves: every pooled row, the grouping, and a mini-batch of as many
    lookups as bags that is not one-hot (HL_DEVERR_SHAPE); called several times,
    since the tables' published counts are told apart by an epoch."""
    rng = np.random.default_rng(B * 100 + T)
    dim, per, n = 8, 50, B * T
    h = hl.hl_create(np.full(T, per, np.uint32), dim, "f32", per * T)
    try:
        hot = np.sort(rng.permutation(per * T)[:max(1, per * T // 3)]).astype(np.int32)
        n_hot, k_cap, n_stg = hot.size, per * T, per * T
        hl.hl_set_hot(h, torch.from_numpy(hot).cuda(), n_hot)
        ptr = np.arange(n + 1, dtype=np.int32)
        dp = torch.from_numpy(ptr).cuda()
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n, B), dtype=torch.uint8, device="cuda")
        w = torch.randn((n_hot + n_stg, dim), device="cuda")
        out = torch.zeros((n, dim), device="cuda")
        keys, bags = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
        for again in range(3):
            gid = (rng.zipf(1.3, n) % per) + per * (np.arange(n) % T)
            at = np.minimum(np.searchsorted(hot, gid), n_hot - 1)
            codes = np.where(hot[at] == gid, at, k_cap + gid).astype(np.int32)
            dc = torch.from_numpy(codes).cuda()
            hl.hl_embbag_fwd_plan(h, w[:n_hot], w[n_hot:], n_stg, dc, dp, B, T, n, out, ws)
            hl.hl_embbag_bwd_grouping(h, n_stg, B, T, n, ws, keys, bags)
            row = np.where(codes < n_hot, codes, n_hot + codes - k_cap)
            assert torch.equal(out, w[torch.from_numpy(row).cuda()])
            check_grouping(keys.cpu().numpy().view(np.uint32), bags.cpu().numpy().view(np.uint32), codes,
                           np.arange(n, dtype=np.uint32), n_hot, k_cap, f"{B}x{T}")
            assert hl.hl_last_device_error(h) == 0
        if -(-B // 32) * (T + 1) <= n:  # (else: the general sort, which takes any bags)
            ptr[1] = 2  # the first bag holds two lookups, the second none
            hl.hl_embbag_fwd_plan(h, w[:n_hot], w[n_hot:], n_stg, dc, torch.from_numpy(ptr).cuda(), B, T, n, out, ws)
            assert hl.hl_last_device_error(h) & hl.DEVERR["SHAPE"]
    finally:
        h.close()


@pytest.mark.parametrize("B,T", [(33, 3), (1024, 2), (1500, 5), (2049, 2), (4096, 2), (4097, 2)])
def test_misfit_bags_are_skipped(B, T):
    """As many lookups as bags, but some bags of two lookups or none: the
    grouping that hl_embbag_fwd_plan leaves is the one of hl_embbag_bwd_plan,
    which skips the lookups of such bags (and a code that names no row), with
    the same errors reported."""
    rng = np.random.default_rng(B + T)
    dim, n, n_hot, n_stg = 8, B * T, 40 * T, 100
    h = hl.hl_create(np.full(T, 50, np.uint32), dim, "f32", 50 * T)
    try:
        k_cap = 50 * T
        hot = (np.arange(n_hot) // 40 * 50 + np.arange(n_hot) % 40).astype(np.int32)  # 40 hot rows a table
        hl.hl_set_hot(h, torch.from_numpy(hot).cuda(), n_hot)
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n, B), dtype=torch.uint8, device="cuda")
        w = torch.randn((n_hot + n_stg, dim), device="cuda")
        out = torch.zeros((n, dim), device="cuda")
        codes = np.where(rng.random(n) < 0.8, rng.integers(0, 40, n) + 40 * (np.arange(n) % T),
                         k_cap + rng.integers(0, n_stg, n)).astype(np.int32)
        codes[n // 3] = k_cap + n_stg
        ptr = np.arange(n + 1, dtype=np.int32)
        ptr[[1, n // 2, n // 2 + 1, n - 1]] += 1
        dc, dp = torch.from_numpy(codes).cuda(), torch.from_numpy(ptr).cuda()
        i32 = lambda: torch.zeros(n, dtype=torch.int32, device="cuda")
        k1, b1, k2, b2 = i32(), i32(), i32(), i32()
        hl.hl_embbag_bwd_plan(h, n_stg, dc, dp, B, T, n, None, None, B, ws)
        e1 = hl.hl_last_device_error(h)
        hl.hl_embbag_bwd_grouping(h, n_stg, B, T, n, ws, k1, b1)
        hl.hl_embbag_fwd_plan(h, w[:n_hot], w[n_hot:], n_stg, dc, dp, B, T, n, out, ws)
        e2 = hl.hl_last_device_error(h)
        hl.hl_embbag_bwd_grouping(h, n_stg, B, T, n, ws, k2, b2)
        assert e1 == e2 == hl.DEVERR["SHAPE"] | hl.DEVERR["BAD_CODE"]
        assert torch.equal(k1, k2)
        used = k1 != -1
        assert torch.equal(b1[used], b2[used])
        good = (ptr[:-1] == np.arange(n)) & (ptr[1:] == np.arange(1, n + 1)) & (codes != k_cap + n_stg)
        assert int(used.sum()) == int(good.sum())
    finally:
        h.close()


def test_tickets_past_the_launch():
    """A workspace header that is not as the calls keep it (here: tickets handed
    out past the launch's blocks) is reported, and nothing is indexed by such a
    ticket; after a zero fill the workspace serves again."""
    B, T, dim = 512, 4, 8
    n = B * T
    h = hl.hl_create(np.full(T, 50, np.uint32), dim, "f32", 50 * T)
    try:
        i32 = lambda k: torch.zeros(k, dtype=torch.int32, device="cuda")
        hl.hl_set_hot(h, torch.arange(50 * T, dtype=torch.int32, device="cuda"), 50 * T)
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n, B), dtype=torch.uint8, device="cuda")
        ptr = torch.arange(n + 1, dtype=torch.int32, device="cuda")
        rows, w, out = i32(n), torch.ones((50 * T, dim), device="cuda"), torch.zeros((n, dim), device="cuda")
        gids, codes, flags, pop, non, cnt = i32(n), i32(n), torch.zeros(B, dtype=torch.uint8, device="cuda"), i32(B), i32(B), i32(2)
        dispatch = lambda: hl.hl_dispatch(h, rows, ptr, B, T, n, gids, codes, flags, pop, non, cnt, ws)
        forward = lambda: hl.hl_embbag_fwd_plan(h, w, None, 0, codes, ptr, B, T, n, out, ws)
        dispatch()
        forward()
        assert hl.hl_last_device_error(h) == 0
        for word, call in ((64, dispatch), (72, forward)):
            ws.view(torch.int32)[word] = 5000
            call()
            assert hl.hl_last_device_error(h) == hl.DEVERR["INTERNAL"]
            hl.hl_workspace_init(ws)
            for _ in range(2):
                call()
                assert hl.hl_last_device_error(h) == 0
        assert int(cnt[0]) == B and bool((out == 1).all())
    finally:
        h.close()
