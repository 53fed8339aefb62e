"""GPU parity: every stage of the HIP path against the oracle on the same seeded
inputs, through the C ABI.  Bit-exact for counts, hot set, gids, flags,
partition, remap, cold ids/codes and gathered rows; within tolerance for pooled
outputs (1e-5 of the summation scale) and updated rows (1e-5 fp32, 1e-2 bf16
of |row| + lr*sum|dY|); untouched rows bitwise unchanged."""
import numpy as np
import pytest
import torch

from paper_2204_05436_amd import configs, hotline as hl, workload as W
from paper_2204_05436_amd.runner import HotPath, to_device
from parity_lib import as_f64, compare, log, make_table, run_gpu_stages, run_oracle

pytestmark = pytest.mark.gpu


def parity_case(w, n_prof=16, idx=16, k=None, hot_ids=None, batches=None, split=False, staging_cap=None):
    rows = W.table_rows(w)
    n_rows = int(rows.sum(dtype=np.int64))
    k_cap = w.k_cap(n_rows)
    if batches is None:
        prof = [W.make_batch(w, rows, i) for i in range(n_prof)]
        mb = W.make_batch(w, rows, idx)
    else:
        prof, mb = batches
    dY = W.make_dy(w, idx, mb.n_bags)
    log(f"[parity] {w.name}: rows={n_rows} B={mb.n_samples} L={mb.n_lookups} k_cap={k_cap} dim={w.dim} {w.dtype}")
    table = make_table(w, n_rows)
    max_l = max([p.n_lookups for p in prof] + [mb.n_lookups, 1])
    hp = HotPath(w, rows, table, max_l, max(1, mb.n_samples), staging_cap=staging_cap)
    try:
        g = run_gpu_stages(hp, prof, mb, dY, k=k, hot_ids=hot_ids, split=split)
        o = run_oracle(w, rows, prof, mb, dY, table.array, k_cap, k=k, hot_ids=hot_ids)
        compare(w, g, o, k_cap, check_counts=hot_ids is None)
        log(f"[parity] {w.name}: n_hot={len(o['hot'])} pop={len(o['pop'])} cold={len(o['cold'])} ok")
    finally:
        hp.close()
        table.close()
    return g, o


@pytest.mark.parametrize("name", configs.ORDER)
def test_full_size(name):
    """Each workload at its full size, through the entry points the benchmark's
    pipelined step calls (cold plan + fetch, backward plan + apply, on side
    streams)."""
    parity_case(configs.WORKLOADS[name], split=True)


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("name", configs.ORDER)
def test_scaled_ragged(name, split):
    """Smaller tables and a batch that is not a multiple of any tile size."""
    w = configs.WORKLOADS[name]
    w = configs.scaled(w, batch=777, row_scale=0.003 if name != "tiny" else 0.5, name=name + "-ragged")
    parity_case(w, n_prof=4, idx=5, split=split)


@pytest.mark.parametrize("k", [0, 1, 7, 10**9])
def test_k_extremes(k):
    w = configs.scaled(configs.WORKLOADS["tiny"], batch=300, row_scale=0.05, name="tiny-k")
    rows = W.table_rows(w)
    kk = min(k, w.k_cap(int(rows.sum())))
    parity_case(w, n_prof=3, idx=3, k=kk)


def test_all_rows_hot():
    w = configs.scaled(configs.WORKLOADS["tbsm"], batch=200, row_scale=0.001, hot_frac=1.0, name="tbsm-allhot")
    rows = W.table_rows(w)
    g, o = parity_case(w, n_prof=2, idx=2, hot_ids=np.arange(int(rows.sum()), dtype=np.uint32))
    assert len(o["nonpop"]) == 0 and len(o["cold"]) == 0


def test_stale_hot_set():
    """Profile one stream, run a batch from another seed: misclassification never changes results."""
    w = configs.scaled(configs.WORKLOADS["dlrm-small"], batch=512, row_scale=0.01, name="small-stale")
    rows = W.table_rows(w)
    prof = [W.make_batch(w, rows, i) for i in range(3)]
    other = configs.scaled(w, seed=w.seed + 99, name="small-other")
    mb = W.make_batch(other, rows, 0)
    parity_case(w, batches=(prof, mb))


def _random_batch(rng, rows_per_table, B, steps, max_len, zero_frac=0.2):
    T = len(rows_per_table)
    bps = T * steps
    lens = rng.integers(1, max_len + 1, B * bps)
    lens[rng.random(B * bps) < zero_frac] = 0
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows = np.empty(int(ptr[-1]), np.uint32)
    for j in range(B * bps):
        t = j % T
        # skewed draws so that rows repeat inside and across bags
        r = (rng.zipf(1.3, lens[j]) - 1) % rows_per_table[t]
        rows[ptr[j]:ptr[j + 1]] = r
    return W.Batch(0, rows, ptr, B, bps)


@pytest.mark.parametrize("seed", range(12))
def test_random_shapes(seed):
    rng = np.random.default_rng(1000 + seed)
    dim = [1, 2, 3, 4, 6, 16, 64, 128, 136, 260, 24, 8][seed]
    dtype = "bf16" if seed % 3 == 2 else "f32"
    T = int(rng.integers(1, 5))
    rows = rng.integers(1, 400, T).astype(np.uint32)
    w = configs.Workload(name=f"rand{seed}", n_tables=T, dim=dim, dtype=dtype, batch=int(rng.integers(1, 300)),
                         steps=int(rng.integers(1, 3)), rows_fixed=tuple(int(r) for r in rows),
                         hot_frac=float(rng.uniform(0.05, 0.6)), seed=seed, lr=0.05)
    prof = [_random_batch(rng, rows, w.batch, w.steps, 64) for _ in range(2)]
    mb = _random_batch(rng, rows, w.batch, w.steps, 64)
    parity_case(w, batches=(prof, mb))


@pytest.mark.parametrize("bits", [9, 10, 11, 12, 17, 19, 20, 21, 22, 23])
def test_backward_key_widths(bits):
    """The backward's sort keys span n_hot + staging rows: the staging capacity
    sets their width, and with it the digit width and pass count of the sort
    (one pass of 9-11 bits; two of 6, 9, 10 or 11; three of 8).  Heavily
    repeated rows over many tiles."""
    rng = np.random.default_rng(bits)
    rows = np.array([64, 40, 100], np.uint32)
    w = configs.Workload(name=f"keys{bits}", n_tables=3, dim=16, dtype="f32", batch=3000, steps=1,
                         rows_fixed=tuple(int(r) for r in rows), hot_frac=0.05, seed=bits, lr=0.05)
    mb = _random_batch(rng, rows, w.batch, 1, 8)
    hot = np.arange(0, 16, 2, dtype=np.uint32)
    cap = (1 << (bits - 1)) - len(hot)
    parity_case(w, batches=([], mb), hot_ids=hot, split=bits % 2 == 0, staging_cap=cap)


@pytest.mark.parametrize("n", [1024 * 128, 1024 * 128 + 1, 2048 * 128, 2048 * 128 + 1, 3072 * 128 + 1, 4096 * 128,
                               4096 * 128 + 1])
def test_sort_tile_sizes(n):
    """The general radix sort takes 1, 2, 4 or 8 items per thread of its
    1024-thread tiles, the fewest that keep a sort to 128 tiles: mini-batches of
    exactly n lookups on either side of each switch, in multi-hot bags (so the
    grouping by table does not apply), against the oracle (the grouping
    against the stable order of the keys)."""
    rng = np.random.default_rng(n)
    rows = np.array([5000, 3000], np.uint32)
    T, B = len(rows), 2048
    nb = B * T
    lens = 1 + rng.multinomial(n - nb, np.full(nb, 1.0 / nb))
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert int(ptr[-1]) == n
    ids = np.empty(n, np.uint32)
    for j in range(nb):
        ids[ptr[j]:ptr[j + 1]] = (rng.zipf(1.2, lens[j]) - 1) % rows[j % T]
    mb = W.Batch(0, ids, ptr, B, T)
    w = configs.Workload(name=f"tiles{n}", n_tables=T, dim=16, dtype="f32", batch=B, steps=1,
                         rows_fixed=tuple(int(r) for r in rows), hot_frac=0.05, seed=n % 997, lr=0.05)
    hot = np.arange(0, 400, 3, dtype=np.uint32)
    parity_case(w, batches=([], mb), hot_ids=hot, split=n % 2 == 1)


def test_determinism_and_split_equals_unsplit():
    w = configs.scaled(configs.WORKLOADS["multi-hot"], batch=300, row_scale=0.002, name="mh-det")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    prof = [to_device(W.make_batch(w, rows, i), "cuda") for i in range(3)]
    mb = W.make_batch(w, rows, 3)
    dY = W.make_dy(w, 3, mb.n_bags)
    results = []
    for mode, split in (("sequential", True), ("sequential", False), ("pipelined", True)):
        hp = HotPath(w, rows, table, max(p.n_lookups for p in prof + [to_device(mb, "cuda")]), w.batch)
        hp.learn(prof)
        b = to_device(mb, "cuda", dY)
        hp.step(b, mode=mode, split_fwd=split)
        torch.cuda.synchronize()
        results.append((hp.out[:mb.n_bags].cpu().numpy().copy(), hp.w_hot[:hp.n_hot].cpu().numpy().copy(),
                        hp.staging.cpu().numpy().copy(), hp.device_error()))
        hp.close()
    table.close()
    o1, w1, s1, e1 = results[0]
    for i, (o2, w2, s2, e2) in enumerate(results[1:]):
        assert e1 == 0 and e2 == 0
        assert np.array_equal(o1.view(np.uint32), o2.view(np.uint32)), f"pooled output differs (run {i + 1})"
        assert np.array_equal(w1.view(np.uint8), w2.view(np.uint8)), f"hot rows differ (run {i + 1})"
        assert np.array_equal(s1.view(np.uint8), s2.view(np.uint8)), f"staging rows differ (run {i + 1})"


def test_sample_list_backward():
    """Backward over one mu-batch (a sample list) against the oracle's selected update."""
    import oracle as O
    w = configs.scaled(configs.WORKLOADS["tbsm"], batch=256, row_scale=0.01, hot_frac=0.5, name="tbsm-sel")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    mb = W.make_batch(w, rows, 0)
    dY = W.make_dy(w, 0, mb.n_bags)
    hp = HotPath(w, rows, table, mb.n_lookups, w.batch)
    try:
        hot = np.arange(0, n_rows, 3, dtype=np.uint32)
        hp.set_hot(torch.from_numpy(hot.view(np.int32)).cuda())
        b = to_device(mb, "cuda", dY)
        B, bps, L = b.n_samples, b.bps, b.n_lookups
        sel = np.sort(np.random.default_rng(0).choice(B, B // 3, replace=False)).astype(np.int32)
        dsel = torch.from_numpy(sel).cuda()
        nsel = torch.tensor([len(sel)], dtype=torch.int32, device="cuda")
        hl.hl_lookup_gids(hp.h, b.rows, b.bag_ptr, b.n_bags, hp.gids)
        hl.hl_remap(hp.h, hp.gids, L, hp.codes)
        hl.hl_cold_gather(hp.h, hp.gids, hp.codes, b.bag_ptr, B, bps, L, None, None, B, table.dev, hp.staging,
                          hp.staging_cap, hp.cold_ids, hp.n_cold, hp.ws)
        codes = hp.codes[:L].cpu().numpy().copy()
        n_cold = int(hp.n_cold.item())
        w0 = hp.w_hot[:len(hot)].cpu().numpy().copy()
        s0 = hp.staging[:n_cold].cpu().numpy().copy()
        hl.hl_embbag_bwd_sgd(hp.h, hp.w_hot, hp.staging, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, dsel, nsel,
                             B, b.dY, w.lr, hp.ws)
        gw = hp.w_hot[:len(hot)].cpu().numpy()
        gs = hp.staging[:n_cold].cpu().numpy()
        assert hp.device_error() == 0
        ow, os_ = w0.copy(), s0.copy()
        uniq, sc, rc = O.embbag_bwd_sgd(w.dtype, ow, hp.k_cap, os_, codes, mb.bag_ptr, sel, len(sel), bps, dY, w.lr,
                                        want_scale=True)
        assert rc == 0
        from parity_lib import check_close
        th = uniq[uniq < hp.k_cap]
        ts = uniq[uniq >= hp.k_cap] - hp.k_cap
        check_close(gw[th], ow[th], sc[uniq < hp.k_cap], 1e-5, "selected update (hot)")
        check_close(gs[ts], os_[ts], sc[uniq >= hp.k_cap], 1e-5, "selected update (staging)")
        assert np.array_equal(np.delete(gw, th, axis=0), np.delete(w0, th, axis=0))
    finally:
        hp.close()
        table.close()


def test_capacity_and_range_errors():
    w = configs.scaled(configs.WORKLOADS["tiny"], batch=64, row_scale=0.1, name="tiny-err")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    mb = W.make_batch(w, rows, 0)
    hp = HotPath(w, rows, table, mb.n_lookups, w.batch, staging_cap=2)
    try:
        hp.set_hot(torch.arange(0, 5, dtype=torch.int32, device="cuda"))
        b = to_device(mb, "cuda")
        B, bps, L = b.n_samples, b.bps, b.n_lookups
        hl.hl_lookup_gids(hp.h, b.rows, b.bag_ptr, b.n_bags, hp.gids)
        hl.hl_remap(hp.h, hp.gids, L, hp.codes)
        before = hp.codes[:L].clone()
        stg_before = hp.staging.clone()
        hl.hl_cold_gather(hp.h, hp.gids, hp.codes, b.bag_ptr, B, bps, L, None, None, B, table.dev, hp.staging,
                          hp.staging_cap, hp.cold_ids, hp.n_cold, hp.ws)
        err = hp.device_error()
        assert err & hl.DEVERR["CAPACITY"]
        assert int(hp.n_cold.item()) > 2                       # the count needed is reported
        assert torch.equal(hp.codes[:L], before)               # nothing else written
        assert torch.equal(hp.staging, stg_before)
        # a row outside its table
        bad = mb.rows.copy()
        bad[3] = rows[3 % w.n_tables] + 5
        db = to_device(W.Batch(0, bad, mb.bag_ptr, B, bps), "cuda")
        hl.hl_lookup_gids(hp.h, db.rows, db.bag_ptr, db.n_bags, hp.gids)
        assert hp.device_error() & hl.DEVERR["OUT_OF_RANGE"]
        assert int(hp.gids[3].item()) == -1
        # a code naming no row
        hp.codes[:L] = -1
        hl.hl_embbag_fwd(hp.h, hp.w_hot, hp.staging, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B,
                         hp.out)
        assert hp.device_error() & hl.DEVERR["BAD_CODE"]
        # shape mismatch between bag_ptr and n_lookups
        hl.hl_classify(hp.h, hp.gids, b.bag_ptr, B, bps, L + 1, hp.flags)
        assert hp.device_error() & hl.DEVERR["SHAPE"]
        # unsorted explicit hot set
        hl.hl_set_hot(hp.h, torch.tensor([5, 3], dtype=torch.int32, device="cuda"), 2)
        assert hp.device_error() & hl.DEVERR["BAD_HOTSET"]
    finally:
        hp.close()
        table.close()


def test_plan_apply_contract():
    """The backward's apply needs its plan in the workspace: refused without one,
    after another call on that workspace, or with other sizes; calls on another
    workspace leave it; applying one plan twice is two SGD steps (against the
    oracle run twice)."""
    import oracle as O
    from parity_lib import check_close
    w = configs.scaled(configs.WORKLOADS["tiny"], batch=128, row_scale=0.2, name="tiny-contract")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    mb = W.make_batch(w, rows, 0)
    dY = W.make_dy(w, 0, mb.n_bags)
    hp = HotPath(w, rows, table, mb.n_lookups, w.batch)
    try:
        hot = np.arange(0, n_rows, 2, dtype=np.uint32)[:hp.k_cap]
        hp.set_hot(torch.from_numpy(hot.view(np.int32)).cuda())
        b = to_device(mb, "cuda", dY)
        B, bps, L = b.n_samples, b.bps, b.n_lookups
        h = hp.h
        with pytest.raises(hl.HotlineError):
            hl.hl_embbag_bwd_apply(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L, b.dY, w.lr, hp.ws)
        hl.hl_lookup_gids(h, b.rows, b.bag_ptr, b.n_bags, hp.gids)
        hl.hl_remap(h, hp.gids, L, hp.codes)
        hl.hl_embbag_bwd_plan(h, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B, hp.ws)
        with pytest.raises(hl.HotlineError):   # other sizes
            hl.hl_embbag_bwd_apply(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L - 1, b.dY, w.lr, hp.ws)
        # the cold lookups still have code -1 here: the plan reports them
        assert hp.device_error() & hl.DEVERR["BAD_CODE"]
        hl.hl_cold_plan(h, hp.gids, hp.codes, b.bag_ptr, B, bps, L, None, None, B, hp.staging_cap, hp.cold_ids,
                        hp.n_cold, hp.ws)
        with pytest.raises(hl.HotlineError):   # the cold plan reused the workspace
            hl.hl_embbag_bwd_apply(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L, b.dY, w.lr, hp.ws)
        hl.hl_cold_fetch(h, hp.cold_ids, hp.n_cold, hp.staging_cap, table.dev, hp.staging)
        codes = hp.codes[:L].cpu().numpy().copy()
        n_cold = int(hp.n_cold.item())
        w0 = hp.w_hot[:len(hot)].cpu().numpy().copy()
        s0 = hp.staging[:n_cold].cpu().numpy().copy()
        hl.hl_embbag_bwd_plan(h, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B, hp.ws)
        # calls on another workspace (a plan of its own included) leave this plan intact
        ws2 = torch.zeros_like(hp.ws)
        hl.hl_embbag_bwd_plan(h, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B, ws2)
        hl.hl_partition(h, hp.flags, B, hp.pop, hp.nonpop, hp.counts, ws2)
        for _ in range(2):
            hl.hl_embbag_bwd_apply(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L, b.dY, w.lr, hp.ws)
        assert hp.device_error() == 0
        ow, os_ = w0.copy(), s0.copy()
        sc = None
        for _ in range(2):
            uniq, s1, rc = O.embbag_bwd_sgd(w.dtype, ow, hp.k_cap, os_, codes, mb.bag_ptr, None, B, bps, dY, w.lr,
                                            want_scale=True)
            assert rc == 0
            sc = s1 if sc is None else sc + s1
        th = uniq[uniq < hp.k_cap]
        ts = uniq[uniq >= hp.k_cap] - hp.k_cap
        check_close(hp.w_hot[:len(hot)].cpu().numpy()[th], ow[th], sc[uniq < hp.k_cap], 1e-5, "two applies (hot)")
        check_close(hp.staging[:n_cold].cpu().numpy()[ts], os_[ts], sc[uniq >= hp.k_cap], 1e-5,
                    "two applies (staging)")
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("B,T,max_len", [(1, 3, 4), (777, 26, 1), (5000, 26, 1), (100_000, 1, 1), (3000, 8, 40),
                                         (1_300_000, 1, 1), (60_000, 26, 1)])
def test_dispatch_shapes(B, T, max_len):
    """The dispatch kernel against the oracle's ids, classify, partition and remap:
    one tile to several hundred, ragged tails and multi-hot bags (the sizes where
    its blocks change: test_dispatch_gpu.py); three calls in a row
    (the device-side epoch advances)."""
    import oracle as O
    rng = np.random.default_rng(B + T)
    rows = rng.integers(50, 5000, T).astype(np.uint32)
    w = configs.Workload(name=f"disp{B}", n_tables=T, dim=4, dtype="f32", batch=B, steps=1,
                         rows_fixed=tuple(int(r) for r in rows), hot_frac=0.3, seed=B)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    batches = [_random_batch(rng, rows, B, 1, max_len, zero_frac=0.05 if max_len > 1 else 0.0) for _ in range(3)]
    hp = HotPath(w, rows, table, max(b.n_lookups for b in batches), B)
    try:
        hot = np.sort(rng.choice(n_rows, int(0.7 * n_rows), replace=False)).astype(np.uint32)[:hp.k_cap]
        hp.set_hot(torch.from_numpy(hot.view(np.int32)).cuda())
        for mb in batches:
            b = to_device(mb, "cuda")
            L = b.n_lookups
            hl.hl_dispatch(hp.h, b.rows, b.bag_ptr, B, T, L, hp.gids, hp.codes, hp.flags, hp.pop, hp.nonpop,
                           hp.counts, hp.ws)
            g, _ = O.gids(rows, mb.rows, mb.bag_ptr)
            flags = O.classify(hot, g, mb.bag_ptr, B, T)
            pop, nonpop = O.partition(flags)
            c = hp.counts.cpu().numpy()
            assert np.array_equal(hp.gids[:L].cpu().numpy().view(np.uint32), g)
            assert np.array_equal(hp.codes[:L].cpu().numpy(), O.remap(hot, g))
            assert np.array_equal(hp.flags[:B].cpu().numpy(), flags)
            assert c[0] == len(pop) and c[1] == len(nonpop)
            assert np.array_equal(hp.pop[:c[0]].cpu().numpy(), pop)
            assert np.array_equal(hp.nonpop[:c[1]].cpu().numpy(), nonpop)
            assert hp.device_error() == 0
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("seed", range(6))
def test_halves_equal_whole(seed):
    """Forward part 1 + part 2 == part 0 and backward apply part 1 + part 2 ==
    part 0, bit for bit, on random shapes (multi-hot bags mixing hot and staging
    rows, empty bags, fp32 and bf16, dims needing every vector width); and the
    staging rows are not read by the halves that run before the fetch (they are
    poisoned with NaN meanwhile)."""
    rng = np.random.default_rng(500 + seed)
    dim = int(rng.choice([1, 3, 16, 64, 130]))
    dtype = "bf16" if seed % 2 else "f32"
    T = int(rng.integers(1, 4))
    rows = rng.integers(20, 300, T).astype(np.uint32)
    w = configs.Workload(name=f"halves{seed}", n_tables=T, dim=dim, dtype=dtype, batch=int(rng.integers(50, 400)),
                         steps=1, rows_fixed=tuple(int(r) for r in rows), hot_frac=0.4, seed=seed, lr=0.05)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    mb = _random_batch(rng, rows, w.batch, 1, 12)
    dY = W.make_dy(w, seed, mb.n_bags)
    hp = HotPath(w, rows, table, mb.n_lookups, w.batch)
    try:
        hot = np.sort(rng.choice(n_rows, hp.k_cap, replace=False)).astype(np.uint32)
        hp.set_hot(torch.from_numpy(hot.view(np.int32)).cuda())
        b = to_device(mb, "cuda", dY)
        B, bps, L, h = b.n_samples, b.bps, b.n_lookups, hp.h
        hl.hl_dispatch(h, b.rows, b.bag_ptr, B, bps, L, hp.gids, hp.codes, hp.flags, hp.pop, hp.nonpop, hp.counts,
                       hp.ws)
        hl.hl_cold_gather(h, hp.gids, hp.codes, b.bag_ptr, B, bps, L, None, None, B, table.dev, hp.staging,
                          hp.staging_cap, hp.cold_ids, hp.n_cold, hp.ws)
        w0, s0 = hp.w_hot.clone(), hp.staging.clone()
        args = (h, hp.w_hot, hp.staging, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B)
        hl.hl_embbag_fwd_part(*args, hp.out, 0)
        whole = hp.out[:mb.n_bags].clone()
        hp.out.fill_(7.0)
        poison = torch.full_like(hp.staging, -1) if dtype == "bf16" else torch.full_like(hp.staging, float("nan"))
        hp.staging.copy_(poison)
        hl.hl_embbag_fwd_part(*args, hp.out, 1)
        hp.staging.copy_(s0)
        hl.hl_embbag_fwd_part(*args, hp.out, 2)
        assert torch.equal(hp.out[:mb.n_bags].view(torch.int32), whole.view(torch.int32)), "forward halves differ"
        hl.hl_embbag_bwd_sgd(h, hp.w_hot, hp.staging, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B,
                             b.dY, w.lr, hp.ws)
        w1, s1 = hp.w_hot.clone(), hp.staging.clone()
        hp.w_hot.copy_(w0)
        hl.hl_embbag_bwd_plan(h, hp.staging_cap, hp.codes, b.bag_ptr, B, bps, L, None, None, B, hp.ws)
        with pytest.raises(hl.HotlineError):  # part 2 needs part 1
            hl.hl_embbag_bwd_apply_part(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L, b.dY, w.lr, 2, hp.ws)
        hp.staging.copy_(poison)
        hl.hl_embbag_bwd_apply_part(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L, b.dY, w.lr, 1, hp.ws)
        torch.cuda.synchronize()
        assert torch.equal(hp.staging.view(torch.int16), poison.view(torch.int16)), "part 1 touched staging rows"
        hp.staging.copy_(s0)
        hl.hl_embbag_bwd_apply_part(h, hp.w_hot, hp.staging, hp.staging_cap, B, bps, L, b.dY, w.lr, 2, hp.ws)
        assert torch.equal(hp.w_hot.view(torch.int16), w1.view(torch.int16)), "hot rows differ"
        assert torch.equal(hp.staging.view(torch.int16), s1.view(torch.int16)), "staging rows differ"
        assert hp.device_error() == 0
    finally:
        hp.close()
        table.close()


def test_empty_batch():
    w = configs.scaled(configs.WORKLOADS["tiny"], batch=0, row_scale=0.1, name="tiny-empty")
    rows = W.table_rows(w)
    table = make_table(w, int(rows.sum()))
    hp = HotPath(w, rows, table, 1, 1)
    try:
        ptr = torch.zeros(1, dtype=torch.int32, device="cuda")
        hl.hl_classify(hp.h, hp.gids, ptr, 0, w.bags_per_sample, 0, hp.flags)
        hl.hl_partition(hp.h, hp.flags, 0, hp.pop, hp.nonpop, hp.counts, hp.ws)
        hl.hl_cold_gather(hp.h, hp.gids, hp.codes, ptr, 0, w.bags_per_sample, 0, hp.nonpop, hp.counts[1:], 0,
                          table.dev, hp.staging, hp.staging_cap, hp.cold_ids, hp.n_cold, hp.ws)
        hl.hl_embbag_fwd(hp.h, hp.w_hot, hp.staging, hp.staging_cap, hp.codes, ptr, 0, w.bags_per_sample, 0, None,
                         None, 0, hp.out)
        assert hp.counts.cpu().tolist() == [0, 0] and int(hp.n_cold.item()) == 0
        assert hp.device_error() == 0
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 4096, 4097, 8192, 16384, 16385, 200_003, 1_300_007])
def test_partition_sizes(n):
    """One block for up to 16K samples (the flags in registers), then 1K
    tiles, and more than 1M samples (64K tiles)."""
    w = configs.scaled(configs.WORKLOADS["tiny"], batch=1, row_scale=0.1, name="tiny-part")
    rows = W.table_rows(w)
    table = make_table(w, int(rows.sum()))
    hp = HotPath(w, rows, table, 1, n)
    try:
        f = (np.random.default_rng(n).random(n) < 0.3).astype(np.uint8)
        hp.flags.copy_(torch.from_numpy(f))
        hl.hl_partition(hp.h, hp.flags, n, hp.pop, hp.nonpop, hp.counts, hp.ws)
        c = hp.counts.cpu().numpy()
        assert c[0] == f.sum() and c[1] == n - f.sum()
        assert np.array_equal(hp.pop[:c[0]].cpu().numpy(), np.flatnonzero(f))
        assert np.array_equal(hp.nonpop[:c[1]].cpu().numpy(), np.flatnonzero(f == 0))
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("name,writeback", [("dlrm-large", False), ("multi-hot", True), ("tbsm", True)])
def test_graph_replay(name, writeback):
    """A HIP graph of the pipelined step (the benchmark's timed unit) replays to
    the eager step's results bit for bit, three times, with eager steps on
    another batch and synchronizations between the replays."""
    w = configs.scaled(configs.WORKLOADS[name], batch=600, row_scale=0.004, name=name + "-graph")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    table = make_table(w, n_rows)
    prof = [W.make_batch(w, rows, i) for i in range(3)]
    mba, mbb = W.make_batch(w, rows, 3), W.make_batch(w, rows, 4)
    da = to_device(mba, "cuda", W.make_dy(w, 3, mba.n_bags))
    db = to_device(mbb, "cuda", W.make_dy(w, 4, mbb.n_bags))
    hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + [mba, mbb]), w.batch, writeback=writeback)
    try:
        hp.learn([to_device(p, "cuda") for p in prof])
        torch.cuda.synchronize()
        w0, tab0 = hp.w_hot.clone(), table.array.copy()

        def state(bufs):
            torch.cuda.synchronize()
            n = int(bufs.n_cold.item())
            return dict(out=hp.out[:mba.n_bags].cpu().numpy().copy(), w_hot=hp.w_hot[:hp.n_hot].cpu().numpy().copy(),
                        stg=bufs.staging[:n].cpu().numpy().copy(), cold=bufs.cold_ids[:n].cpu().numpy().copy(),
                        codes=bufs.codes[:mba.n_lookups].cpu().numpy().copy(), tab=table.array.copy())

        def reset():
            torch.cuda.synchronize()
            hp.w_hot.copy_(w0)
            table.array[:] = tab0
            torch.cuda.synchronize()

        hp.step(da)
        ref = state(hp)
        assert hp.device_error() == 0
        reset()
        g, bufs = hp.capture(da)
        for rep in range(3):
            reset()
            g.replay()
            torch.cuda.synchronize()
            got = state(bufs)
            assert hp.device_error() == 0, f"replay {rep}"
            for k in ref:
                assert np.array_equal(got[k].view(np.uint8), ref[k].view(np.uint8)), f"replay {rep}: {k} differs"
            hp.step(db)  # eager work between replays
            torch.cuda.synchronize()
            assert hp.device_error() == 0
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("mode,writeback", [("pipelined", True), ("pipelined", False), ("sequential", True),
                                           ("lookahead", True), ("lookahead", False)])
@pytest.mark.parametrize("name", ["dlrm-large", "multi-hot", "tbsm"])
def test_multi_step(name, mode, writeback):
    """Several consecutive steps with one workspace and one hot cache (the hot
    cache carries the updates from step to step).  Every step is checked against
    the oracle run from the same pre-step state (the oracle's hot cache, and with
    write-back its host table, take the GPU's after each comparison), to the
    single-step tolerances.  With write-back, the host table after a step holds
    the step's updated staging rows bit for bit at the cold ids and is unchanged
    elsewhere.  "lookahead": each step also plans the next batch, whose
    dispatch and cold plan run on the plan stream while the step trains."""
    import oracle as O
    from parity_lib import check_close
    w = configs.scaled(configs.WORKLOADS[name], batch=600, row_scale=0.004, name=name + "-steps")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    k_cap = w.k_cap(n_rows)
    rtol = {"f32": 1e-5, "bf16": 1e-2}[w.dtype]
    table = make_table(w, n_rows)
    prof = [W.make_batch(w, rows, i) for i in range(4)]
    steps = [W.make_batch(w, rows, 4 + s) for s in range(4)]
    hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + steps), w.batch, writeback=writeback)
    try:
        hp.learn([to_device(p, "cuda") for p in prof])
        counts = np.zeros(n_rows, np.uint32)
        for p in prof:
            O.count(n_rows, [O.gids(rows, p.rows, p.bag_ptr)[0]], counts)
        hot = O.topk(counts, k_cap)
        assert np.array_equal(hp.hot_ids[:hp.n_hot].cpu().numpy().view(np.uint32), hot)
        w_hot = O.gather(table.array, hot)
        dYs = [W.make_dy(w, 4 + si, mb.n_bags) for si, mb in enumerate(steps)]
        dbs = [to_device(mb, "cuda", dY) for mb, dY in zip(steps, dYs)]
        if mode == "lookahead":
            hl.hl_trace_enable(hp.h, 4096)
        for si, mb in enumerate(steps):
            pre = hp.w_hot[:len(hot)].cpu().numpy().copy()
            assert si > 0 or np.array_equal(pre.view(np.uint8), w_hot.view(np.uint8))
            w_hot = pre.copy()
            tab_pre = table.array.copy()
            dY = dYs[si]
            if mode == "lookahead":
                hp.step(dbs[si], next=dbs[si + 1] if si + 1 < len(dbs) else None)
            else:
                hp.step(dbs[si], mode=mode)
            torch.cuda.synchronize()
            assert hp.device_error() == 0, f"step {si}"
            B, bps, L = mb.n_samples, mb.bags_per_sample, mb.n_lookups
            g, _ = O.gids(rows, mb.rows, mb.bag_ptr)
            flags = O.classify(hot, g, mb.bag_ptr, B, bps)
            pop, nonpop = O.partition(flags)
            cold, codes = O.cold_plan(g, O.remap(hot, g), mb.bag_ptr, nonpop, len(nonpop), bps, k_cap)
            stg = O.gather(tab_pre, cold)
            out, sc, _ = O.embbag_fwd(w.dtype, w_hot, k_cap, stg, codes, mb.bag_ptr, None, B, bps, B * bps,
                                      want_scale=True)
            assert np.array_equal(hp.flags[:B].cpu().numpy(), flags), f"step {si} flags"
            assert np.array_equal(hp.codes[:L].cpu().numpy(), codes), f"step {si} codes"
            n_cold = int(hp.n_cold.item())
            assert np.array_equal(hp.cold_ids[:n_cold].cpu().numpy().view(np.uint32), cold), f"step {si} cold ids"
            check_close(hp.out[:B * bps].cpu().numpy(), out, sc, 1e-5, f"step {si} pooled output")
            uniq, usc, _ = O.embbag_bwd_sgd(w.dtype, w_hot, k_cap, stg, codes, mb.bag_ptr, None, B, bps, dY, w.lr,
                                            want_scale=True)
            hu = uniq < k_cap
            gw = hp.w_hot[:len(hot)].cpu().numpy()
            gst = hp.staging[:n_cold].cpu().numpy()
            check_close(as_f64(gw[uniq[hu]], w.dtype), as_f64(w_hot[uniq[hu]], w.dtype), usc[hu], rtol,
                        f"step {si} hot rows")
            ts = uniq[~hu] - k_cap
            check_close(as_f64(gst[ts], w.dtype), as_f64(stg[ts], w.dtype), usc[~hu], rtol, f"step {si} staging rows")
            untouched = np.setdiff1d(np.arange(len(hot)), uniq[hu])
            assert np.array_equal(gw[untouched].view(np.uint8), pre[untouched].view(np.uint8)), f"step {si}"
            tab = table.array
            if writeback:
                ref_tab = tab_pre.copy()
                O.scatter(ref_tab, cold, gst)
                assert np.array_equal(tab.view(np.uint8), ref_tab.view(np.uint8)), f"step {si} write-back"
            else:
                assert np.array_equal(tab.view(np.uint8), tab_pre.view(np.uint8)), f"step {si} host table changed"
        if mode == "lookahead":
            # every step is planned ahead, and the plans take the fused form: the
            # dispatch kernel inserts the cold lookups and the grouping's first
            # kernel writes their codes (no cold-plan insert or codes kernel)
            names = [hl.hl_trace_read(hp.h, i)[0] for i in range(hl.hl_trace_count(hp.h))]
            hl.hl_trace_enable(hp.h, 0)
            assert names.count("cg_insert") == 0 and names.count("cg_codes") == 0, names
            assert names.count("cg_rank") == len(steps) and names.count("ds_kernel") == len(steps), names
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("writeback", [False, True])
@pytest.mark.parametrize("name", ["dlrm-large", "multi-hot"])
def test_lookahead_chain(name, writeback):
    """Six untied back-to-back steps, each planning the next batch ahead, with
    one sync at the end: the hot cache (and with write-back the host table) ends
    bit for bit where six plain pipelined steps leave it, and within the
    single-step tolerance, compounded, of the oracle's six steps in order."""
    import oracle as O
    from parity_lib import check_close
    w = configs.scaled(configs.WORKLOADS[name], batch=700, row_scale=0.004, name=name + "-chain")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    k_cap = w.k_cap(n_rows)
    prof = [W.make_batch(w, rows, i) for i in range(4)]
    steps = [W.make_batch(w, rows, 4 + s) for s in range(6)]
    dYs = [W.make_dy(w, 4 + si, mb.n_bags) for si, mb in enumerate(steps)]
    finals = {}
    for variant in ("plain", "lookahead"):
        table = make_table(w, n_rows)
        hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + steps), w.batch, writeback=writeback)
        try:
            hp.learn([to_device(p, "cuda") for p in prof])
            hot = hp.hot_ids[:hp.n_hot].cpu().numpy().view(np.uint32).copy()
            w0 = hp.w_hot[:len(hot)].cpu().numpy().copy()
            tab0 = table.array.copy()
            dbs = [to_device(mb, "cuda", dY) for mb, dY in zip(steps, dYs)]
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                for si in range(len(dbs)):
                    if variant == "plain":
                        hp.step(dbs[si], untied=True)
                    else:
                        hp.step(dbs[si], untied=True, next=dbs[si + 1] if si + 1 < len(dbs) else None)
                hp.sync()
            torch.cuda.synchronize()
            assert hp.device_error() == 0, variant
            finals[variant] = (hp.w_hot[:len(hot)].cpu().numpy().copy(), table.array.copy())
        finally:
            hp.close()
            table.close()
    assert np.array_equal(finals["plain"][0].view(np.uint8), finals["lookahead"][0].view(np.uint8)), "hot cache"
    assert np.array_equal(finals["plain"][1].view(np.uint8), finals["lookahead"][1].view(np.uint8)), "host table"
    # the oracle's six steps in order, updating its hot cache and staging rows in
    # place (a step's staging rows are dropped after it unless written back)
    w_hot, tab = np.ascontiguousarray(w0.copy()), tab0.copy()
    B, bps = w.batch, w.bags_per_sample
    for mb, dY in zip(steps, dYs):
        g, _ = O.gids(rows, mb.rows, mb.bag_ptr)
        flags = O.classify(hot, g, mb.bag_ptr, B, bps)
        _, nonpop = O.partition(flags)
        cold, codes = O.cold_plan(g, O.remap(hot, g), mb.bag_ptr, nonpop, len(nonpop), bps, k_cap)
        stg = np.ascontiguousarray(O.gather(tab, cold))
        _, _, rc = O.embbag_bwd_sgd(w.dtype, w_hot, k_cap, stg, codes, mb.bag_ptr, None, B, bps, dY, w.lr)
        assert rc == 0
        if writeback:
            O.scatter(tab, cold, stg)
    rtol = {"f32": 1e-5, "bf16": 1e-2}[w.dtype] * len(steps)
    got = finals["lookahead"][0]
    scale = np.maximum(np.abs(as_f64(w0, w.dtype)), 1e-3)
    check_close(as_f64(got, w.dtype), as_f64(w_hot, w.dtype), scale, rtol, "hot cache after the chain")
    if writeback:
        check_close(as_f64(finals["lookahead"][1], w.dtype), as_f64(tab, w.dtype),
                    np.maximum(np.abs(as_f64(tab0, w.dtype)), 1e-3), rtol, "host table after the chain")


@pytest.mark.parametrize("writeback", [False, True])
def test_mixed_plain_and_planned(writeback):
    """Plain steps (their own dispatch and cold plan on the main stream) and
    planned ones (look-ahead plans on the plan stream) interleaved in one untied
    chain: a plan after a plain step waits for it with a launch of its own (the
    plain step's cold plan leaves the shared hash table, which the plan reads),
    the others wait inside the dispatch kernel.  The hot cache and the host
    table end bit for bit where plain steps alone leave them."""
    w = configs.scaled(configs.WORKLOADS["dlrm-large"], batch=640, row_scale=0.004, name="dlrm-large-mixed")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    prof = [W.make_batch(w, rows, i) for i in range(4)]
    steps = [W.make_batch(w, rows, 4 + s) for s in range(8)]
    dYs = [W.make_dy(w, 4 + si, mb.n_bags) for si, mb in enumerate(steps)]
    # which steps plan ahead: step i plans batch i + 1 when ahead[i]
    ahead = [False, True, True, False, False, True, False, False]
    finals = {}
    for variant in ("plain", "mixed"):
        table = make_table(w, n_rows)
        hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + steps), w.batch, writeback=writeback)
        try:
            hp.learn([to_device(p, "cuda") for p in prof])
            dbs = [to_device(mb, "cuda", dY) for mb, dY in zip(steps, dYs)]
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                for si in range(len(dbs)):
                    nxt = dbs[si + 1] if variant == "mixed" and ahead[si] and si + 1 < len(dbs) else None
                    hp.step(dbs[si], untied=True, next=nxt)
                hp.sync()
            torch.cuda.synchronize()
            assert hp.device_error() == 0, variant
            finals[variant] = (hp.w_hot[:hp.n_hot].cpu().numpy().copy(), table.array.copy())
        finally:
            hp.close()
            table.close()
    assert np.array_equal(finals["plain"][0].view(np.uint8), finals["mixed"][0].view(np.uint8)), "hot cache"
    assert np.array_equal(finals["plain"][1].view(np.uint8), finals["mixed"][1].view(np.uint8)), "host table"


@pytest.mark.parametrize("name", ["dlrm-large", "multi-hot"])
def test_relearn_migration(name):
    """Re-learning after training steps (with write-back): the new hot set is
    the oracle's top-K over drifted sample batches (another rank-to-row map);
    the hot cache and the host table after the migration equal the oracle's
    migration of the GPU's state before it, bit for bit (so the table the path
    reads is unchanged); a step on the new hot set matches the oracle run from
    that state (flags, codes, cold ids, pooled output)."""
    import oracle as O
    from parity_lib import check_close
    w = configs.scaled(configs.WORKLOADS[name], batch=600, row_scale=0.004, name=name + "-relearn")
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    k_cap = w.k_cap(n_rows)
    table = make_table(w, n_rows)
    prof = [W.make_batch(w, rows, i) for i in range(4)]
    steps = [W.make_batch(w, rows, 4 + s) for s in range(2)]
    drift = [W.make_batch(w, rows, 8 + i, phase=1) for i in range(4)]
    mb = W.make_batch(w, rows, 12, phase=1)
    hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + steps + drift + [mb]), w.batch, writeback=True)
    try:
        hp.learn([to_device(p, "cuda") for p in prof])
        for si, sb in enumerate(steps):
            hp.step(to_device(sb, "cuda", W.make_dy(w, 4 + si, sb.n_bags)))
        torch.cuda.synchronize()
        assert hp.device_error() == 0
        n_old = hp.n_hot
        old = hp.hot_ids[:n_old].cpu().numpy().view(np.uint32).copy()
        w_old = hp.w_hot[:n_old].cpu().numpy().copy()
        host0 = table.array.copy()
        n_new = hp.relearn([to_device(b, "cuda") for b in drift])
        torch.cuda.synchronize()
        assert hp.device_error() == 0
        counts = np.zeros(n_rows, np.uint32)
        for b in drift:
            O.count(n_rows, [O.gids(rows, b.rows, b.bag_ptr)[0]], counts)
        new = O.topk(counts, k_cap)
        assert np.array_equal(hp.hot_ids[:n_new].cpu().numpy().view(np.uint32), new)
        leave, enter = np.setdiff1d(old, new), np.setdiff1d(new, old)
        log(f"[relearn] {name}: {n_old} -> {n_new} hot rows, {len(leave)} leave, {len(enter)} enter")
        assert len(leave) > 0 and len(enter) > 0
        host_ref = host0.copy()
        w_ref, n_wb = O.migrate(old, w_old, new, host_ref)
        assert n_wb == len(leave)
        assert np.array_equal(hp.w_hot[:n_new].cpu().numpy().view(np.uint8), w_ref.view(np.uint8)), "hot cache"
        assert np.array_equal(table.array.view(np.uint8), host_ref.view(np.uint8)), "host table"
        # a step on the new hot set
        dY = W.make_dy(w, 12, mb.n_bags)
        hp.step(to_device(mb, "cuda", dY))
        torch.cuda.synchronize()
        assert hp.device_error() == 0
        B, bps, L = mb.n_samples, mb.bags_per_sample, mb.n_lookups
        g, _ = O.gids(rows, mb.rows, mb.bag_ptr)
        flags = O.classify(new, g, mb.bag_ptr, B, bps)
        pop, nonpop = O.partition(flags)
        cold, codes = O.cold_plan(g, O.remap(new, g), mb.bag_ptr, nonpop, len(nonpop), bps, k_cap)
        stg = O.gather(host_ref, cold)
        out, sc, _ = O.embbag_fwd(w.dtype, w_ref, k_cap, stg, codes, mb.bag_ptr, None, B, bps, B * bps,
                                  want_scale=True)
        assert np.array_equal(hp.flags[:B].cpu().numpy(), flags)
        assert np.array_equal(hp.codes[:L].cpu().numpy(), codes)
        n_cold = int(hp.n_cold.item())
        assert np.array_equal(hp.cold_ids[:n_cold].cpu().numpy().view(np.uint32), cold)
        check_close(hp.out[:B * bps].cpu().numpy(), out, sc, 1e-5, "pooled output after re-learning")
    finally:
        hp.close()
        table.close()


@pytest.mark.parametrize("name,geom", [("tiny", None), ("tbsm", None), ("multi-hot", None), ("dlrm-small", (7, 3)),
                                       ("dlrm-large", (4096, 16))])
def test_eal_srrip(name, geom):
    """The SRRIP access logger against the oracle's, bit for bit: every entry
    (id and 2-bit value) after each profiling batch, fed through the GPU's own
    gids (with a few rows out of range), and the hot set it yields.  Default
    geometry: 16 ways and K / 16 sets (as many entries as the hot cache); the
    others force evictions in every set."""
    import oracle as O
    w0 = configs.WORKLOADS[name]
    w = configs.scaled(w0, batch=min(w0.batch, 1024), row_scale=0.02, name=name + "-eal") \
        if name in ("dlrm-small", "dlrm-large", "multi-hot") else w0
    rows = W.table_rows(w)
    n_rows = int(rows.sum())
    k_cap = w.k_cap(n_rows)
    n_sets, ways = geom if geom else (max(1, k_cap // 16), 16)
    batches = [W.make_batch(w, rows, i) for i in range(6)]
    batches[2].rows[::97] = np.uint32(0xFFFFFFFF)  # rows out of range: ids 0xFFFFFFFF, not logged
    h = hl.hl_create(rows, w.dim, w.dtype, k_cap)
    e = hl.EAL(h, n_sets, ways, max(b.n_lookups for b in batches))
    oe = O.EAL(n_sets, ways)
    try:
        gids = torch.zeros(max(b.n_lookups for b in batches), dtype=torch.int32, device="cuda")
        tags = torch.zeros(n_sets * ways, dtype=torch.int32, device="cuda")
        rr = torch.zeros(n_sets * ways, dtype=torch.uint8, device="cuda")
        for bi, b in enumerate(batches):
            db = to_device(b, "cuda")
            hl.hl_lookup_gids(h, db.rows, db.bag_ptr, db.n_bags, gids)
            hl.hl_eal_access(e, gids, b.n_lookups)
            g, _ = O.gids(rows, b.rows, b.bag_ptr)
            oe.access(g)
            hl.hl_eal_state(e, tags, rr)
            torch.cuda.synchronize()
            assert np.array_equal(tags.cpu().numpy().view(np.uint32), oe.tag), f"batch {bi}: ids"
            assert np.array_equal(rr.cpu().numpy(), oe.rrpv), f"batch {bi}: values"
        hot = torch.zeros(n_sets * ways, dtype=torch.int32, device="cuda")
        n = hl.hl_eal_hot(e, hot)
        assert np.array_equal(hot[:n].cpu().numpy().view(np.uint32), oe.hot())
        log(f"[eal] {name}: {n_sets}x{ways}: holds {n} ids")
    finally:
        e.close()
        hl.hl_destroy(h)


@pytest.mark.parametrize("name", ["dlrm-large", "tbsm", "tiny"])
def test_grouping_ranks_fallback(name):
    """The grouping's radix passes rank equal digits with one counter update per
    item, check the order they kept, and redo a pass with ballot ranks if an
    order broke.  With the ballot ranks forced (hl_debug_ballot_ranks) the
    grouping is the same bit for bit, and the parity holds."""
    w = configs.scaled(configs.WORKLOADS[name], batch=1500, row_scale=0.01 if name != "tiny" else 0.5,
                       name=name + "-ranks")
    rows = W.table_rows(w)
    n_rows = int(rows.sum(dtype=np.int64))
    k_cap = w.k_cap(n_rows)
    prof = [W.make_batch(w, rows, i) for i in range(4)]
    mb = W.make_batch(w, rows, 5)
    dY = W.make_dy(w, 5, mb.n_bags)
    groupings = []
    for forced in (False, True):
        table = make_table(w, n_rows)
        hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + [mb]), mb.n_samples)
        try:
            hl.hl_debug_ballot_ranks(hp.h, forced)
            g = run_gpu_stages(hp, prof, mb, dY, split=True)
            o = run_oracle(w, rows, prof, mb, dY, table.array, k_cap)
            compare(w, g, o, k_cap)
            groupings.append(g["grouping"])
        finally:
            hp.close()
            table.close()
    assert np.array_equal(groupings[0][0], groupings[1][0]) and np.array_equal(groupings[0][1], groupings[1][1])


@pytest.mark.parametrize("name,full", [("dlrm-large", True), ("dlrm-large", False), ("dlrm-small", False),
                                       ("tbsm", False), ("tiny", False), ("multi-hot", False)])
def test_fwd_plan(name, full):
    """hl_embbag_fwd_plan (the forward over every sample with the backward's
    plan; for one-hot mini-batches the tables' sorts run in the forward's
    launch) then the apply: pooled outputs, the grouping and the updated rows
    bit for bit those of hl_embbag_fwd then hl_embbag_bwd_sgd, and within
    tolerance of the oracle."""
    w = configs.WORKLOADS[name]
    if not full:
        w = configs.scaled(w, batch=700 if name != "tiny" else 1024, row_scale=0.004 if name != "tiny" else 1.0,
                           name=name + "-fp")
    rows = W.table_rows(w)
    n_rows = int(rows.sum(dtype=np.int64))
    k_cap = w.k_cap(n_rows)
    prof = [W.make_batch(w, rows, i) for i in range(4 if not full else w.profile_batches)]
    mb = W.make_batch(w, rows, w.profile_batches)
    dY = W.make_dy(w, w.profile_batches, mb.n_bags)
    table = make_table(w, n_rows)
    res = []
    try:
        for fp in (False, True):
            hp = HotPath(w, rows, table, max(b.n_lookups for b in prof + [mb]), mb.n_samples)
            try:
                res.append(run_gpu_stages(hp, prof, mb, dY, fwd_plan=fp))
            finally:
                hp.close()
        o = run_oracle(w, rows, prof, mb, dY, table.array, k_cap)
    finally:
        table.close()
    a, b = res
    assert a["deverr"] == 0 and b["deverr"] == 0
    for key in ("codes", "cold", "out", "w_hot_new", "staging_new"):
        assert np.array_equal(np.asarray(a[key]).view(np.uint8), np.asarray(b[key]).view(np.uint8)), key
    assert np.array_equal(a["grouping"][0], b["grouping"][0]) and np.array_equal(a["grouping"][1], b["grouping"][1])
    compare(w, b, o, k_cap)
