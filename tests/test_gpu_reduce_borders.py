"""Runs that cross span borders, at the counts of spans where the wave that closes a run changes what
it does (64 pieces at a time, fetched eight per lane group), and launches of more spans than the chip
holds at once, where the reduce kernel's tiles run as a loop (rows of 36 to 64 floats).  Gradients and
weights are whole numbers and lr is a power of two, so every sum is exact in fp32 whatever its order."""
import numpy as np
import pytest
import torch

from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

pytestmark = pytest.mark.gpu


def _step(dim, lists, rows, span):
    S = max(len(x) for x in lists)
    hp = HotPath(rows, dim)
    B.fae_set_option(hp.ctx, "reduce_span", span)
    hp.alloc_counts()
    hp.build([0] * len(rows), rows, seed=3)
    gen = torch.Generator(device="cuda").manual_seed(dim)
    for w in hp.hotW:
        w.copy_(torch.randint(-8, 9, w.shape, device="cuda", generator=gen).float())
    before = [w.double() for w in hp.hotW]
    gout = torch.randint(-4, 5, (S, len(rows), dim), device="cuda", generator=gen).float()
    slots = [torch.from_numpy(x.astype(np.int32)).cuda() for x in lists]
    offs = [torch.arange(S + 1, device="cuda").clamp(max=len(x)).int() for x in lists]
    hp.backward_sgd(HotBatch(S, slots, offs, [len(x) for x in lists]), gout, 0.125)
    hp.sync()
    for z, s in enumerate(slots):
        grad = torch.zeros_like(before[z]).index_add_(0, s.long(), gout[:len(lists[z]), z].double())
        assert torch.equal(hp.hotW[z].double(), before[z] - 0.125 * grad), f"table {z}"


@pytest.mark.parametrize("dim", [1, 4, 8, 20, 64, 100, 256])
@pytest.mark.parametrize("pieces", [1, 7, 8, 9, 63, 64, 65, 128, 129, 200])
def test_runs_over_many_spans(dim, pieces):
    rng = np.random.default_rng(pieces)
    lists, n = [], pieces * 64
    for lead, tail in ((0, 5), (1, 63), (63, 200), (64, 0)):  # lookups of other slots before and behind the long run
        s = np.concatenate([rng.integers(0, 50, lead), np.full(n, 50), rng.integers(51, 300, tail)])
        lists.append(rng.permutation(s))
    _step(dim, lists, [300] * len(lists), 64)


@pytest.mark.parametrize("dim", [36, 64])
@pytest.mark.parametrize("spans", [4096, 4097, 5120, 5121, 9000])
def test_more_spans_than_the_chip_holds(dim, spans):
    rng = np.random.default_rng(spans)
    n = spans * 64 // 2
    lists = [np.where(rng.random(n) < 0.1, 17, rng.integers(0, 4000, n)), rng.integers(0, 100_000, n)]
    _step(dim, lists, [4000, 100_000], 64)
