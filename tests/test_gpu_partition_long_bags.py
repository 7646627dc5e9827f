"""Partition where a tile of samples holds far more lookups than its share, which then go to the kernel
that takes lookups whoever owns them: one long history among short ones, few samples, runs of empty
bags longer than a round of lookups, tables whose offsets fit LDS only a few at a time; 32- and 64-bit
ids, beside one-hot tables, and what must be refused there.  Against the definition in numpy."""
import time

import numpy as np
import pytest
import torch

from paper_2103_00686_amd import binding as B

pytestmark = pytest.mark.gpu

ONE = None


def _call(S, lengths, idx, remap, bits=32, offsets=None):
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(t).cuda()  # noqa: E731
    if offsets is None:
        offsets = [None if ln is None else np.concatenate([[0], np.cumsum(ln)]) for ln in lengths]
    t_idx = [dev(i, torch.int64 if bits == 64 else torch.int32) for i in idx]
    t_off = [None if o is None else dev(o, torch.int32) for o in offsets]
    batch = B.Batch(S, t_idx, t_off, [len(i) for i in idx], bits)
    ctx, tables = B.Context(0, None), B.Tables([len(m) for m in remap], 4)
    new = lambda n: torch.full((n,), -7, dtype=torch.int32, device="cuda")  # noqa: E731
    out = [new(S), new(S), [new(max(len(i), 1)) for i in idx], [new(S + 1) for _ in remap]]
    ws = torch.empty(B.fae_partition_workspace_bytes(tables, S), dtype=torch.uint8, device="cuda")
    t_map = [dev(m, torch.int32) for m in remap]
    run = lambda: B.fae_partition_batch(ctx, tables, batch, t_map, out[0], out[1], out[2], out[3], ws)  # noqa: E731
    return run, out


def _lengths(kind, rng):
    """(samples, lengths per table, share of cold rows)"""
    if kind == "one_sample":
        return 1, [np.array([9000]), ONE, np.array([0])], 0.0
    if kind == "few":
        return 16, [np.full(16, 4001), rng.integers(0, 3000, 16)], 2e-5
    if kind == "one_long":  # a tile of 16 samples with a bag of 300 000 beside tiles of short ones
        ln = rng.integers(0, 6, 3000)
        ln[1501] = 300_000
        return 3000, [ln, ONE, rng.integers(0, 4, 3000)], 1e-6
    if kind == "cold_long":
        ln = rng.integers(0, 6, 700)
        ln[[3, 4, 699]] = 20_000, 8191, 40_000
        return 700, [ONE, ln], 1e-4
    if kind == "empty_runs":  # rounds that reach over thousands of empty bags
        ln = np.zeros(20_001, dtype=np.int64)
        ln[[0, 7, 9000, 9001, 20_000]] = 5, 9500, 8700, 1, 12_345
        return 20_001, [ln, rng.integers(0, 2, 20_001)], 1e-5
    if kind == "many_tables":
        return 40, [rng.integers(0, 90, 40) for _ in range(63)] + [ONE], 1e-6
    if kind == "tables_in_turn":  # tiles of 64 samples: 35 of the 50 tables at a time
        return 100_000, [rng.integers(0, 2, 100_000) for _ in range(50)], 1e-4
    if kind == "tables_in_turn_long":
        ls = [rng.integers(0, 2, 530_000) for _ in range(9)]  # tiles of 256 samples: eight tables at a time
        ls[8][[100, 300_000]] = 30_000, 9000
        return 530_000, ls + [ONE], 1e-4
    assert kind == "all_hot"
    return 50, [np.full(50, 700), np.full(50, 1000)], 0.0


@pytest.mark.parametrize("kind,bits", [("one_sample", 32), ("few", 64), ("one_long", 32), ("cold_long", 64), ("empty_runs", 32), ("many_tables", 32),
                                       ("tables_in_turn", 32), ("tables_in_turn_long", 64), ("all_hot", 32)])
def test_partition_of_long_bags(kind, bits):
    rng = np.random.default_rng(len(kind))
    S, lengths, cold = _lengths(kind, rng)
    rows = [int(r) for r in rng.integers(20_000, 200_000, len(lengths))]
    remap = [np.where(rng.random(r) < cold, -1, rng.integers(0, 1 << 20, r)).astype(np.int32) for r in rows]
    idx = [rng.integers(0, r, S if ln is None else int(ln.sum())) for r, ln in zip(rows, lengths)]
    run, (hot, coldl, slots, hoff) = _call(S, lengths, idx, remap, bits)
    owner = [np.arange(S) if ln is None else np.repeat(np.arange(S), ln) for ln in lengths]
    is_hot = np.ones(S, dtype=bool)
    for i, m, s in zip(idx, remap, owner):
        is_hot[s[m[i] < 0]] = False
    want = np.flatnonzero(is_hot)
    for _ in range(2):  # the second call finds the first one's states in the workspace
        n_hot, nl = run()
        assert n_hot == want.size
        assert np.array_equal(hot.cpu().numpy(), np.concatenate([want, np.full(S - want.size, -7)]))
        assert np.array_equal(coldl.cpu().numpy(), np.concatenate([np.flatnonzero(~is_hot), np.full(want.size, -7)]))
        for z in range(len(rows)):
            keep = is_hot[owner[z]]
            ref = remap[z][idx[z][keep]]
            lens = np.bincount(owner[z], minlength=S)[is_hot]
            got = slots[z].cpu().numpy()
            assert int(nl[z]) == ref.size
            assert np.array_equal(got[:ref.size], ref) and (got[ref.size:] == -7).all()
            assert np.array_equal(hoff[z].cpu().numpy()[:want.size + 1], np.concatenate([[0], np.cumsum(lens)]))


@pytest.mark.parametrize("what", ["id", "wide_id", "falls", "first", "past", "last"])
def test_a_bad_long_bag_is_refused(what):
    S, rows = 40, 1000
    lengths = np.full(S, 1500)
    idx = np.zeros(int(lengths.sum()), dtype=np.int64)
    off = np.concatenate([[0], np.cumsum(lengths)])
    if what == "id":
        idx[31_234] = rows
    elif what == "wide_id":
        idx[31_234] = 1 << 32
    elif what == "falls":
        off[20] = off[22]
    elif what == "first":
        off[0] = 1
    elif what == "past":
        off[21] = len(idx) + 1
    else:
        off[S] = len(idx) - 1
    run, _ = _call(S, [lengths, ONE], [idx, np.zeros(S, dtype=np.int64)], [np.arange(rows, dtype=np.int32)] * 2,
                   64 if what == "wide_id" else 32, [off, None])
    with pytest.raises(B.FaeError, match="out of range or a malformed CSR"):
        run()


@pytest.mark.parametrize("over", [0, 1])  # lookups above the most that a tile walks itself
@pytest.mark.parametrize("S,bits", [(5, 32), (2047, 64), (40_000, 32), (131_073, 64)])
def test_a_lone_table_of_bags(S, bits, over):
    rng = np.random.default_rng(S)
    n_cu, log = torch.cuda.get_device_properties(0).multi_processor_count, 4
    while (S + (1 << log) - 1) >> log > 8 * n_cu:
        log += 1
    tiles, tile = (S + (1 << log) - 1) >> log, (S // 2) >> log << log
    ln = rng.integers(0, 7, S)

    def above(n):  # lookups of the tile beyond its limit, with a bag of n in it
        ln[tile] = n
        share = int(ln.sum()) // tiles
        limit = max(int(ln.sum()) // (2 * n_cu), 4096)
        return int(ln[tile:tile + (1 << log)].sum()) - (limit if share > limit else limit + 2 * share)
    lo, hi = 0, 100_000
    if above(hi) > over:
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if above(mid) <= over else (lo, mid)
    above(lo)
    idx, remap = [rng.integers(0, 5000, int(ln.sum()))], [np.where(rng.random(5000) < 0.01, -1, np.arange(5000)).astype(np.int32)]
    run, out = _call(S, [ln], idx, remap, bits)
    owner = np.repeat(np.arange(S), ln)
    is_hot = np.ones(S, dtype=bool)
    is_hot[owner[remap[0][idx[0]] < 0]] = False
    ref = remap[0][idx[0][is_hot[owner]]]
    for _ in range(2):
        n_hot, nl = run()
        assert n_hot == is_hot.sum() and int(nl[0]) == ref.size
        assert np.array_equal(out[0].cpu().numpy()[:n_hot], np.flatnonzero(is_hot))
        assert np.array_equal(out[1].cpu().numpy()[:S - n_hot], np.flatnonzero(~is_hot))
        assert np.array_equal(out[2][0].cpu().numpy()[:ref.size], ref)
        assert np.array_equal(out[3][0].cpu().numpy()[:n_hot + 1], np.concatenate([[0], np.cumsum(ln[is_hot])]))


@pytest.mark.parametrize("what", ["id", "falls", "first", "past", "last"])
def test_a_bad_short_bag_of_a_lone_table_is_refused(what):
    S, rows = 3000, 1000
    ln = np.full(S, 3)
    idx, off = np.zeros(3 * S, dtype=np.int64), np.arange(S + 1) * 3
    if what == "id":
        idx[4321] = -1
    elif what == "falls":
        off[1600] = off[1602]
    elif what == "first":
        off[0] = -1
    elif what == "past":
        off[1601] = 3 * S + 1
    else:
        off[S] = 3 * S - 1
    run, _ = _call(S, [ln], [idx], [np.arange(rows, dtype=np.int32)], 32, [off])
    with pytest.raises(B.FaeError, match="out of range or a malformed CSR"):
        run()


def test_time_goes_by_the_lookups_and_not_by_who_owns_them():
    """Four million lookups: in equal bags, in sixteen bags, and nearly all in one bag.  A workgroup that
    walks a long bag by itself takes a hundred times as long."""
    rng = np.random.default_rng(1)
    n, rows = 4_000_000, 50_000
    idx, remap = rng.integers(0, rows, n), np.arange(rows, dtype=np.int32)
    times = {}
    for name, ln in (("equal", np.full(40_000, 100)), ("few", np.full(16, n // 16)), ("one", np.concatenate([np.ones(39_999, dtype=np.int64), [n - 39_999]]))):
        run, _ = _call(len(ln), [ln], [idx], [remap])
        took = []
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            run()
            took.append(time.perf_counter() - t)
        times[name] = min(took)
    assert times["few"] < 10 * times["equal"] and times["one"] < 10 * times["equal"], times
