"""The update's runs of one row over several tiles of the sorted lookups, at the
lengths where their sums change hands: within a row group, a block, up to 8 tiles
(by a row group of the second launch) and more (by whole blocks that look for
them), one row group to a wave (dim >= 256) and columns in two parts, the last
run ending on the last tile's edge or inside it.  Small whole numbers, so that
every order of summation gives the same exact rows."""
import numpy as np
import pytest
import torch

from paper_2204_05436_amd import hotline as hl

pytestmark = pytest.mark.gpu


def _tile(dim, dtype):
    """Sorted lookups per tile: two waves of row groups, 6 or 8 lookups each."""
    vec = 8 if dtype == "bf16" and dim % 8 == 0 else next(v for v in (4, 2, 1) if dim % v == 0)
    return 2 * (64 // min(dim // vec, 64)) * (6 if vec >= 4 else 8)


@pytest.mark.parametrize("part", ["whole", "halves"])
@pytest.mark.parametrize("last", ["edge", "inside", "short"])
@pytest.mark.parametrize("dim,dtype", [(1, "f32"), (16, "f32"), (64, "f32"), (256, "f32"), (260, "f32"), (130, "f32"),
                                       (128, "bf16"), (512, "bf16")])
def test_runs_over_tiles(dim, dtype, last, part):
    rng = np.random.default_rng(dim + len(last))
    te = _tile(dim, dtype)
    lens, at = [], 0

    def run(start, pieces, end):
        """Fill up to position `start` of a tile, then a run over `pieces` tiles
        that ends at position `end` (1 to te) of the last of them."""
        nonlocal at
        while at % te != start:
            k = min(int(rng.integers(1, 9)), (start - at) % te)
            lens.append(k)
            at += k
        lens.append((pieces - 1) * te + end - start)
        at += lens[-1]

    for p in (1, 2, 3, 7, 8, 9, 10, 15, 16, 17, 33, 150):
        run(te // 2, p, te)
        run(0, p, te // 3 + 1)
        run(te - 1, p + 1, 1)
    if last == "edge":
        run(te // 3, 20, te)
    elif last == "inside":
        run(te // 3, 20, te // 2)
    else:
        run(te - 1, 2, 3)
    n_rows = len(lens)
    n_hot = n_rows * 3 // 5  # (the later runs are of staging rows)
    n_stg = n_rows - n_hot
    n = sum(lens)
    codes = np.repeat(np.arange(n_rows, dtype=np.int32), lens)  # (k_cap = n_hot)
    rng.shuffle(codes)
    h = hl.hl_create(np.array([n_rows], np.uint32), dim, dtype, n_hot)
    try:
        hl.hl_set_hot(h, torch.arange(n_hot, dtype=torch.int32, device="cuda"), n_hot)
        tt = torch.float32 if dtype == "f32" else torch.bfloat16
        w = torch.randint(-8, 9, (n_rows, dim), device="cuda").to(tt)
        dY = torch.randint(-3, 4, (n, dim), device="cuda").float()
        dc = torch.from_numpy(codes).cuda()
        g = torch.zeros((n_rows, dim), dtype=torch.float64, device="cuda").index_add_(0, dc.long(), dY.double())
        want = (w.double() - g / 64).float().to(tt)
        ptr = torch.arange(n + 1, dtype=torch.int32, device="cuda")
        ws = torch.zeros(hl.hl_workspace_bytes(h, n, n, n), dtype=torch.uint8, device="cuda")
        hot, stg = w[:n_hot].clone(), w[n_hot:].clone()
        hl.hl_embbag_bwd_plan(h, n_stg, dc, ptr, n, 1, n, None, None, n, ws)
        if part == "whole":
            hl.hl_embbag_bwd_apply(h, hot, stg, n_stg, n, 1, n, dY, 1 / 64, ws)
        else:
            for q in (1, 2):
                hl.hl_embbag_bwd_apply_part(h, hot, stg, n_stg, n, 1, n, dY if q == 1 else None, 1 / 64, q, ws)
        assert hl.hl_last_device_error(h) == 0
        assert torch.equal(torch.cat([hot, stg]), want)
    finally:
        h.close()
