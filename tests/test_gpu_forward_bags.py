"""Forward over bags whose lengths sit at the edges of what one load of slots covers (a lane group's
lanes, a wave's 64) and of the plain sum (128 lookups per lane group), mixed with one-hot tables in
one launch, against fp64."""
import numpy as np
import pytest
import torch

from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

pytestmark = pytest.mark.gpu

SHORT = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17]
LONG = [0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257, 300]


@pytest.mark.parametrize("pooling", [B.FAE_POOL_SUM, B.FAE_POOL_MEAN])
@pytest.mark.parametrize("dim", [2, 3, 4, 8, 20, 50, 64, 100, 128, 260])
def test_bag_lengths_at_the_edges(dim, pooling):
    rng = np.random.default_rng(dim)
    rows, S = [700, 90, 50, 33], 77
    lengths = [rng.permutation(np.resize(LONG, S)), rng.permutation(np.resize(SHORT, S)), None, rng.permutation(np.resize(LONG + SHORT, S))]
    slots, offs, nl = [], [], []
    for r, ln in zip(rows, lengths):
        n = S if ln is None else int(ln.sum())
        slots.append(torch.from_numpy(rng.integers(0, r, n, dtype=np.int32)).cuda())
        offs.append(None if ln is None else torch.from_numpy(np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)).cuda())
        nl.append(n)
    hp = HotPath(rows, dim)
    hp.alloc_counts()
    hp.build([0] * len(rows), rows, seed=3)
    out = torch.full((S, len(rows), dim), float("nan"), device="cuda")
    hp.forward(HotBatch(S, slots, offs, nl), out, pooling)
    hp.sync()
    for z, ln in enumerate(lengths):
        ln = np.ones(S, dtype=np.int64) if ln is None else ln.astype(np.int64)
        w = hp.hotW[z].double()[slots[z].long()]
        seg = torch.from_numpy(np.repeat(np.arange(S), ln)).cuda()
        ref = torch.zeros((S, dim), dtype=torch.float64, device="cuda").index_add_(0, seg, w)
        mag = torch.zeros((S, dim), dtype=torch.float64, device="cuda").index_add_(0, seg, w.abs())
        if pooling == B.FAE_POOL_MEAN:
            scale = torch.from_numpy(1.0 / np.maximum(ln, 1)).cuda()[:, None]
            ref, mag = ref * scale, mag * scale
        # at most 128 plain additions in a row, six more across lane groups and the scaling: 136 * 2^-24
        assert bool(((out[:, z].double() - ref).abs() <= 136 * 2.0 ** -24 * mag).all()), f"table {z}"


@pytest.mark.parametrize("variant", [1, 2])  # a lane group per bag, a wave per bag
@pytest.mark.parametrize("dim", [4, 64])
def test_bags_at_the_end_of_the_longest_list(dim, variant):
    """A list of the most lookups that a call takes: the chunk behind the last bag's end lies past 2^31.
    Only the last 300 entries belong to a bag and are read."""
    n, rows = (1 << 31) - 2, 1000
    slots = torch.empty(n, dtype=torch.int32, device="cuda")
    tail = torch.randint(0, rows, (300,), dtype=torch.int32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    slots[-300:] = tail
    off = torch.tensor([n - 300, n - 129, n - 3, n], dtype=torch.int32, device="cuda")
    hp = HotPath([rows], dim)
    hp.alloc_counts()
    hp.build([0], [rows], seed=3)
    B.fae_set_option(hp.ctx, "fwd_variant", variant)
    out = hp.forward(HotBatch(3, [slots], [off], [n]))
    hp.sync()
    w = hp.hotW[0].double()[tail.long()]
    for s, (b, e) in enumerate([(0, 171), (171, 297), (297, 300)]):
        # up to 171 terms: 136 * 2^-24 covers the plain sum's 128 and what a compensated one leaves
        assert bool(((out[s, 0].double() - w[b:e].sum(0)).abs() <= 136 * 2.0 ** -24 * w[b:e].abs().sum(0)).all())


@pytest.mark.parametrize("dim", [1, 2, 4, 8, 16, 64, 128, 256])
@pytest.mark.parametrize("variant", [1, 2])
def test_an_infinite_last_row_stays_infinite(dim, variant):
    """The sum of a long bag (more than 128 lookups per lane group, so the rounding error is carried
    along) whose last row is infinite: nothing may be added behind it, not even a zero."""
    rows = 100
    ncols = dim // 4 if dim % 4 == 0 else dim
    lpr = 1
    while lpr < min(ncols, 64):
        lpr *= 2
    groups = 64 // lpr if variant == 2 else 1
    ln = np.array([128 * groups + x for x in (1, 2, 3, 5, 7, 11, 13, 30, 37, 63)])
    off = np.concatenate([[0], np.cumsum(ln)])
    slots = np.random.default_rng(dim).integers(0, rows - 1, off[-1], dtype=np.int32)
    slots[off[1:] - 1] = rows - 1
    hp = HotPath([rows], dim)
    hp.alloc_counts()
    hp.build([0], [rows], seed=3)
    hp.hotW[0][rows - 1] = float("inf")
    B.fae_set_option(hp.ctx, "fwd_variant", variant)
    out = hp.forward(HotBatch(len(ln), [torch.from_numpy(slots).cuda()], [torch.from_numpy(off.astype(np.int32)).cuda()], [int(off[-1])]))
    hp.sync()
    assert bool((out == float("inf")).all())


@pytest.mark.parametrize("dim", [1, 2, 4, 8, 12])
def test_narrow_rows(dim):
    """Rows of one, two and four lanes, whose slots come eight at a time (the first two) from any entry on:
    every length up to two such loads and around the plain sum's limit; a slot that no row has is reported
    and adds nothing, and a bag does not see the ones of the bags behind it."""
    rng = np.random.default_rng(dim)
    ln = np.concatenate([rng.permutation(np.repeat(np.arange(18), 5)), [127, 128, 129, 136, 137, 7]])
    off = np.concatenate([[0], np.cumsum(ln)])
    rows, n = 200, int(off[-1])
    slots = rng.integers(0, rows, n, dtype=np.int32)
    bad = rng.permutation(n)[:40]
    wrong = slots.copy()
    wrong[bad] = rng.choice([-1, rows, 1 << 30], 40)
    hp = HotPath([rows], dim)
    hp.alloc_counts()
    hp.build([0], [rows], seed=3)
    B.fae_set_option(hp.ctx, "fwd_variant", 1)
    w = hp.hotW[0].double().cpu().numpy()
    for s, keep in ((slots, np.ones(n, dtype=bool)), (wrong, ~np.isin(np.arange(n), bad))):
        out = hp.forward(HotBatch(len(ln), [torch.from_numpy(s).cuda()], [torch.from_numpy(off.astype(np.int32)).cuda()], [n]))
        if keep.all():
            hp.sync()
        else:
            with pytest.raises(B.FaeError, match="out of range"):
                hp.sync()
        seg = np.repeat(np.arange(len(ln)), ln)[keep]
        ref, mag = np.zeros((len(ln), dim)), np.zeros((len(ln), dim))
        np.add.at(ref, seg, w[slots[keep]])
        np.add.at(mag, seg, np.abs(w[slots[keep]]))
        assert (np.abs(out[:, 0].double().cpu().numpy() - ref) <= 128 * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("S", [131072, 131071])  # 768 MiB of one-hot rows: a launch of their own; less: one for all
def test_large_one_hot_tables_beside_bags(S):
    rows, dim = [500, 60_000, 9, 3000], 512
    gen = torch.Generator(device="cuda").manual_seed(S)
    ln = torch.randint(0, 4, (S,), device="cuda", generator=gen)
    off = torch.zeros(S + 1, dtype=torch.int32, device="cuda")
    off[1:] = ln.cumsum(0)
    nl = [S, S, int(off[-1]), S]
    slots = [torch.randint(0, r, (n,), dtype=torch.int32, device="cuda", generator=gen) for r, n in zip(rows, nl)]
    hp = HotPath(rows, dim)
    hp.alloc_counts()
    hp.build([0] * 4, rows, seed=3)
    out = torch.full((S, 4, dim), float("nan"), device="cuda")
    hp.forward(HotBatch(S, slots, [None, None, off, None], nl), out)
    hp.sync()
    for z in (0, 1, 3):
        assert torch.equal(out[:, z], hp.hotW[z][slots[z].long()])
    w = hp.hotW[2][slots[2].long()]
    pooled = torch.zeros((S, dim), device="cuda")
    for k in range(3):  # the same additions in the same order
        has = ln > k
        pooled[has] += w[(off[:-1].long() + k)[has]]
    assert torch.equal(out[:, 2], pooled)


@pytest.mark.parametrize("dim", [4, 8, 16, 32, 64])
def test_a_long_bag_among_short_ones_is_as_accurate(dim):
    """A table of short bags is summed by a lane group per bag.  Its rare long bags must not lose to that:
    120 times one row drifts by up to 30 units of the last place if added one after the other."""
    rng = np.random.default_rng(dim)
    S, rows, n = 4000, 3000, 120
    ln = rng.integers(1, 4, S)
    ln[::40] = n
    off = np.concatenate([[0], np.cumsum(ln)])
    slots = rng.integers(0, rows, off[-1], dtype=np.int32)
    for s in range(0, S, 40):
        slots[off[s]:off[s + 1]] = slots[off[s]]
    hp = HotPath([rows], dim)
    hp.alloc_counts()
    hp.build([0], [rows], seed=3)
    out = hp.forward(HotBatch(S, [torch.from_numpy(slots).cuda()], [torch.from_numpy(off.astype(np.int32)).cuda()], [int(off[-1])]))
    hp.sync()
    row = hp.hotW[0].double()[torch.from_numpy(slots[off[:-1][::40]]).cuda().long()]
    # pairs of pairs (2 roundings) or of eight (3), up to 16 rows to a part (3 more), the parts: 120 / 16, with
    # eight lanes per row 120 / 8
    assert bool(((out[::40, 0].double() - n * row).abs() <= (6 + n // (8 if dim == 32 else 16) + 1) * 2.0 ** -24 * n * row.abs()).all())


@pytest.mark.parametrize("S", [5120, 5121])  # with two tables the last count with a wave from one and a half rounds on
@pytest.mark.parametrize("dim", [16, 20, 64])  # 16 and 8 lane groups; 4 keep two rounds
def test_bags_of_one_and_a_half_rounds(dim, S):
    groups = {16: 16, 20: 8, 64: 4}[dim]
    rng = np.random.default_rng(S)
    # one table of exactly 1.5 lookups for each lane group a bag, one of a single lookup less
    lengths = [rng.integers(0, 3 * groups + 1, S) for _ in range(2)]
    for ln, n in zip(lengths, [(3 * groups * S + 1) // 2, (3 * groups * S + 1) // 2 - 1]):
        while ln.sum() != n:
            d = int(np.sign(n - ln.sum()))
            i = rng.integers(0, S, abs(int(n - ln.sum())))
            ln[np.unique(i)] += d
            np.clip(ln, 0, 3 * groups, out=ln)
    slots = [torch.from_numpy(rng.integers(0, 900, int(ln.sum()), dtype=np.int32)).cuda() for ln in lengths]
    offs = [torch.from_numpy(np.concatenate([[0], np.cumsum(ln)]).astype(np.int32)).cuda() for ln in lengths]
    hp = HotPath([900, 900], dim)
    hp.alloc_counts()
    hp.build([0, 0], [900, 900], seed=3)
    out = hp.forward(HotBatch(S, slots, offs, [int(ln.sum()) for ln in lengths]))
    hp.sync()
    for z, ln in enumerate(lengths):
        w = hp.hotW[z].double()[slots[z].long()]
        seg = torch.from_numpy(np.repeat(np.arange(S), ln)).cuda()
        ref = torch.zeros((S, dim), dtype=torch.float64, device="cuda").index_add_(0, seg, w)
        mag = torch.zeros((S, dim), dtype=torch.float64, device="cuda").index_add_(0, seg, w.abs())
        # at most 3 * groups rows to a bag, added in no more than that many roundings
        assert bool(((out[:, z].double() - ref).abs() <= (3 * groups + 1) * 2.0 ** -24 * mag).all()), f"table {z}"
