"""The address generation over bags of any length, and the dispatch at the sizes
where its blocks change: more than 2048 lookups a block, and mini-batches for
which one sizing or both would take more blocks than its published words have
room for.  Whether it is one launch is the same on a
stream of the whole GPU and on one of few compute units."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2204_05436_amd import hotline as hl
from parity_lib import u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,fused", [(32768, 26, True), (150_000, 26, True), (155_000, 26, True), (192_308, 26, True),
                                       (301_440, 26, True), (301_441, 26, False), (500_000, 16, False)])
def test_dispatch_block_sizes(B, T, fused):
    rng = np.random.default_rng(B + T)
    n = B * T
    rows_per = rng.integers(50, 5000, T).astype(np.uint32)
    n_rows = int(rows_per.sum())
    hot = np.sort(rng.permutation(n_rows)[:int(0.9 * n_rows)]).astype(np.uint32)
    rows = (rng.integers(0, 1 << 30, n) % np.tile(rows_per, B)).astype(np.uint32)
    ptr = np.arange(n + 1, dtype=np.int32)
    gids, _ = O.gids(rows_per, rows, ptr)
    flags = O.classify(hot, gids, ptr, B, T)
    pop, nonpop = O.partition(flags)
    codes = O.remap(hot, gids)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).cuda()
    i32 = lambda k: torch.full((k,), -9, dtype=torch.int32, device="cuda")
    h = hl.hl_create(rows_per, 4, "f32", hot.size)
    few = hl.hl_stream_create(0, 64)
    try:
        hl.hl_set_hot(h, d(hot), hot.size)
        dr, dp = d(rows), d(ptr)
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n, B), dtype=torch.uint8, device="cuda")
        hl.hl_trace_enable(h, 64)
        for stream in (None, few):
            g, c, po, no, cnt = i32(n), i32(n), i32(B), i32(B), i32(2)
            fl = torch.zeros(B, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            hl.hl_trace_reset(h)
            hl.hl_dispatch(h, dr, dp, B, T, n, g, c, fl, po, no, cnt, ws, stream)
            torch.cuda.synchronize()
            names = [hl.hl_trace_read(h, i)[0] for i in range(hl.hl_trace_count(h))]
            assert (names == ["ds_kernel"]) == fused, names
            assert cnt.tolist() == [len(pop), len(nonpop)]
            assert np.array_equal(u32(g), gids) and np.array_equal(c.cpu().numpy(), codes)
            assert np.array_equal(fl.cpu().numpy(), flags)
            assert np.array_equal(po[:len(pop)].cpu().numpy(), pop)
            assert np.array_equal(no[:len(nonpop)].cpu().numpy(), nonpop)
            assert hl.hl_last_device_error(h) == 0
    finally:
        hl.hl_trace_enable(h, 0)
        hl.hl_stream_destroy(few)
        h.close()


@pytest.mark.parametrize("T,lens", [
    (1, [70_001]), (3, [0, 33_000, 0, 0, 7, 20_000, 0]), (5, [1000] * 31 + [0, 999]), (26, [1] * 2600),
    (4, [300] * 33 + [0] * 40 + [5000] * 3), (2, [0, 0]), (7, [1, 2, 0] * 21_846), (3, [1, 0, 3] * 22_000)])
def test_lookup_gids_bag_lengths(T, lens):
    """The row-to-id kernel where several waves share 32 bags (fewer than 65,536
    bags) and where each has its own, bags of any length; a row past its table is
    reported and gets no id."""
    rng = np.random.default_rng(len(lens))
    lens = np.array(lens)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(ptr[-1])
    rows_per = rng.integers(50, 5000, T).astype(np.uint32)
    base = np.concatenate([[0], np.cumsum(rows_per)[:-1]])
    t = np.repeat(np.arange(lens.size) % T, lens)
    rows = rng.integers(0, 1 << 30, n) % rows_per[t]
    want = (base[t] + rows).astype(np.uint32)
    h = hl.hl_create(rows_per, 4, "f32", 10)
    try:
        d = lambda a: torch.from_numpy(np.ascontiguousarray(a).astype(np.int32)).cuda()
        gids = torch.zeros(n + 5, dtype=torch.int32, device="cuda")
        for bad in ([], [0, n // 2, n - 1]):
            if bad and not n:
                continue
            for i in bad:
                rows[i], want[i] = rows_per[t[i]], 0xFFFFFFFF
            hl.hl_lookup_gids(h, d(np.append(rows, 0)), d(ptr), lens.size, gids)
            assert np.array_equal(u32(gids[:n]), want) and not gids[n:].any()
            assert hl.hl_last_device_error(h) == (hl.DEVERR["OUT_OF_RANGE"] if bad else 0)
    finally:
        h.close()
