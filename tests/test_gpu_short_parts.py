"""The LDS sort around the length up to which a part's places are counted outright (256 keys of one
part): distinct slots, multiplicities and weights against fp64, with one slot that owns most of a
list (a part past the limit beside short ones), every lookup on one slot, and bags; and the order of
the lookups inside a slot's run, which decides the last bits of the sums, against the global passes."""
import numpy as np
import pytest
import torch

from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 63, 64, 127, 129, 255, 256, 257, 511, 1023, 1024, 2049, 4096])
@pytest.mark.parametrize("bags", [False, True])
def test_short_lists(S, bags):
    rng = np.random.default_rng(S)
    rows, dim, lr = [100_000, 40_000, 3, 1], 4, 0.05
    slots, offs = [], []
    for z, r in enumerate(rows):
        s = rng.integers(0, r, S)
        if z == 1:
            s[rng.random(S) < 0.6] = r // 2
        slots.append(torch.from_numpy(s.astype(np.int32)).cuda())
        cuts = np.sort(rng.integers(0, S + 1, S - 1))
        offs.append(torch.from_numpy(np.concatenate([[0], cuts, [S]]).astype(np.int32)).cuda() if bags else None)
    hp = HotPath(rows, dim)
    hp.alloc_counts()
    hp.build([0] * len(rows), rows, seed=3)
    before = [w.double() for w in hp.hotW]
    gout = torch.randn((S, len(rows), dim), device="cuda", generator=torch.Generator(device="cuda").manual_seed(S))
    uniq, runs = hp.backward_sgd(HotBatch(S, slots, offs, [S] * len(rows)), gout, lr, debug=True)
    hp.sync()
    for z, s in enumerate(slots):
        u, c = torch.unique(s, return_counts=True)
        assert torch.equal(uniq[z], u) and torch.equal(runs[z], c.int())
        sample = torch.arange(S, device="cuda") if offs[z] is None else torch.repeat_interleave(torch.arange(S, device="cuda"), offs[z].diff().long())
        up = gout[sample, z].double()
        grad = torch.zeros_like(before[z]).index_add_(0, s.long(), up)
        mag = torch.zeros_like(before[z]).index_add_(0, s.long(), up.abs())
        # a sum of up to S terms in fp32, then one multiply and one subtraction
        bound = lr * mag * (S + 2) * 2.0 ** -24 + (before[z].abs() + lr * grad.abs()) * 2.0 ** -23
        assert bool(((hp.hotW[z].double() - (before[z] - float(np.float32(lr)) * grad)).abs() <= bound).all()), f"table {z}"


@pytest.mark.parametrize("S", [64, 255, 256, 257, 1023, 4096])
@pytest.mark.parametrize("bags", [False, True])
def test_lookups_of_a_slot_stay_in_order(S, bags):
    """The same bytes as from the stable global passes (sort_variant 1): few slots, so that every run
    is long and another order inside it gives other sums."""
    rng = np.random.default_rng(S + bags)
    rows, dim = [100_000, 40_000, 3, 12], 4
    slots, offs = [], []
    for z, r in enumerate(rows):
        s = rng.integers(0, 40, S) * (r // 40) if r > 40 else rng.integers(0, r, S)
        if z == 1:
            s[rng.random(S) < 0.6] = r // 2  # a part past the limit
        slots.append(torch.from_numpy(s.astype(np.int32)).cuda())
        cuts = np.sort(rng.integers(0, S + 1, S - 1))
        offs.append(torch.from_numpy(np.concatenate([[0], cuts, [S]]).astype(np.int32)).cuda() if bags else None)
    gout = torch.randn((S, len(rows), dim), device="cuda", generator=torch.Generator(device="cuda").manual_seed(S))
    got = []
    for variant in (0, 1):
        hp = HotPath(rows, dim)
        B.fae_set_option(hp.ctx, "sort_variant", variant)
        hp.alloc_counts()
        hp.build([0] * len(rows), rows, seed=3)
        hp.backward_sgd(HotBatch(S, slots, offs, [S] * len(rows)), gout, 0.05)
        hp.sync()
        got.append([w.clone() for w in hp.hotW])
    assert all(torch.equal(a, b) for a, b in zip(*got))
