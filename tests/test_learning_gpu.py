"""GPU parity of the learning phase's kernels at the sizes where they can go
wrong: access counting and the top-K selection against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2204_05436_amd import hotline as hl
from parity_lib import u32

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint32).view(np.int32)).cuda()


@pytest.mark.parametrize("n_rows,tables", [(1, 1), (63, 2), (4096, 3), (16384, 1), (16385, 26), (70001, 5),
                                           (1_100_003, 7)])
def test_count_and_topk(n_rows, tables):
    """Counts on either side of every regime of the selection's bins (exact
    below 64, 32 bins per power of two, up to three levels of them), ties at
    the boundary, sparse and dense rows, at row counts around the 64-row words,
    the 4096-row blocks and the 16384-row tiles; the lookups in an order that
    mixes hot and rare ids, fed in calls of odd lengths; the rows past the last
    call's hot set forgotten, the counts zeroed by reset."""
    rng = np.random.default_rng(n_rows)
    want = np.zeros(n_rows, np.int64)
    some = rng.permutation(n_rows)[:max(1, n_rows // 40)]
    want[some] = rng.integers(1, 5, some.size)
    # (a bin of 2^19 and above holds more values than one level below it parts)
    edge = [1, 2, 62, 63, 64, 65, 66, 127, 128, 129, 130, 1000, 1001, 2047, 2048, 2049, 4095, 4096, 70000, 70001,
            (1 << 17) + 5, (1 << 17) + 6, (1 << 17) + 9, (1 << 17) + 9, (1 << 20) + 2, (1 << 20) + 3, (1 << 20) + 7]
    at = rng.permutation(n_rows)[:len(edge)]
    want[at] = edge[:at.size]
    if n_rows > 5000:  # a dense stretch with many ties
        want[1000:1400] = rng.integers(60, 70, 400)
    ids = rng.permutation(np.repeat(np.arange(n_rows, dtype=np.uint32), want))
    rows = np.full(tables, max(1, n_rows // tables), np.uint32)
    rows[-1] = n_rows - rows[:-1].sum(dtype=np.int64)
    h = hl.hl_create(rows, 4, "f32", n_rows)
    try:
        acc = int((want > 0).sum())
        ks = sorted({0, 1, 2, 3, 4, 5, 7, 9, 12, 20, acc // 2, acc - 1, acc, n_rows} & set(range(n_rows + 1)))
        out = torch.zeros(n_rows, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(n_rows, dtype=torch.int32, device="cuda")
        d = _dev(ids)
        for a, b in zip([0, 1, 2050, 9001], [1, 2050, 9001, ids.size]):
            b = min(b, ids.size)
            if a < b:
                hl.hl_profile_count(h, d[a:b].clone(), b - a)
        hl.hl_profile_counts(h, cnt)
        assert np.array_equal(u32(cnt), want.astype(np.uint32)), "counts"
        probe = np.arange(n_rows, dtype=np.uint32)
        codes = torch.zeros(n_rows, dtype=torch.int32, device="cuda")
        for k in reversed(ks):
            n = hl.hl_profile_topk(h, k, out, reset_counts=k == ks[0])
            hot = O.topk(want.astype(np.uint32), k)
            assert n == hot.size == h.n_hot, f"k={k}"
            assert np.array_equal(u32(out[:n]), hot), f"k={k}"
            # the bitmap and the rank directory, through the slot of every row
            hl.hl_remap(h, _dev(probe), n_rows, codes)
            assert np.array_equal(codes.cpu().numpy(), O.remap(hot, probe)), f"k={k}"
        hl.hl_profile_counts(h, cnt)
        assert not u32(cnt).any(), "reset"
        assert hl.hl_last_device_error(h) == 0
    finally:
        h.close()


@pytest.mark.parametrize("n", [1, 1023, 1025, 2049, 262_144, 262_145, 300_001])
@pytest.mark.parametrize("tables", [1, 7])
def test_count_block_sizes(n, tables):
    """Access counting where its blocks change size (256 blocks of 1024 lookups),
    on one id, a few, and so many that a block's LDS table refuses some; ids that
    are no row's are reported and not counted."""
    rng = np.random.default_rng(n + tables)
    n_rows = 7 * 300_000
    h = hl.hl_create(np.full(tables, n_rows // tables, np.uint32), 4, "f32", 10)
    try:
        cnt = torch.zeros(n_rows, dtype=torch.int32, device="cuda")
        want = np.zeros(n_rows, np.int64)
        for wide in (1, 40, n_rows):
            ids = rng.integers(0, wide, n).astype(np.uint32)
            if wide == 40:
                ids[[0, n // 2, n - 1]] = [n_rows, 0xFFFFFFFF, n_rows + 5]
            hl.hl_profile_count(h, _dev(ids), n)
            want += np.bincount(ids[ids < n_rows], minlength=n_rows)
            assert hl.hl_last_device_error(h) == (hl.DEVERR["OUT_OF_RANGE"] if wide == 40 else 0)
        hl.hl_profile_counts(h, cnt)
        assert np.array_equal(u32(cnt), want.astype(np.uint32))
    finally:
        h.close()


@pytest.mark.parametrize("n_sets,ways,n", [(1, 16, 7), (1, 16, 8), (1, 5, 9), (1, 16, 71), (2, 1, 81), (1, 16, 72),
                                           (1, 16, 137), (3, 16, 5000), (7, 3, 9000), (40, 16, 20011), (300, 2, 3000),
                                           (1, 16, 328), (1, 16, 336), (1, 7, 700)])
def test_logger_long_runs(n_sets, ways, n):
    """The access logger's replay of runs around the lengths where it changes
    form (8 accesses by 16 lanes, then 64 at a time by a wave): few sets, so
    that every batch gives each a long run; ids from all hits to all misses;
    every entry against the oracle after each batch."""
    rng = np.random.default_rng(n * 31 + ways)
    h = hl.hl_create(np.array([1 << 20], np.uint32), 4, "f32", 16)
    e, oe = hl.EAL(h, n_sets, ways, n), O.EAL(n_sets, ways)
    tags = torch.zeros(n_sets * ways, dtype=torch.int32, device="cuda")
    rr = torch.zeros(n_sets * ways, dtype=torch.uint8, device="cuda")
    try:
        for b, spread in enumerate([n_sets * ways // 2 + 1, 2 * n_sets * ways + 3, 1 << 20, n_sets * ways + 1, 1]):
            g = rng.integers(0, spread, n).astype(np.uint32)
            hot = rng.random(n) < 0.6  # a few ids that keep hitting among the rest
            g[hot] = rng.integers(0, max(1, n_sets * ways // 3), int(hot.sum()))
            g[rng.random(n) < 0.02] = np.uint32(0xFFFFFFFF)  # not logged
            hl.hl_eal_access(e, _dev(g), n)
            oe.access(g)
            hl.hl_eal_state(e, tags, rr)
            torch.cuda.synchronize()
            assert np.array_equal(u32(tags), oe.tag), f"batch {b}: ids"
            assert np.array_equal(rr.cpu().numpy(), oe.rrpv), f"batch {b}: values"
    finally:
        e.close()
        h.close()
