"""The LDS sort of lists that are split by a sample of their lookups (beyond 10 240, up to 128 K): the same bytes
as from the radix passes (sort_variant 1) at the edges of its rules, with slots that own several parts,
neighbouring popular slots, samples that mislead, offsets beyond what LDS holds, slots out of range and a
list that does not start on 16 bytes."""
import numpy as np
import pytest
import torch

from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

pytestmark = pytest.mark.gpu
ROWS = 300_000  # three radix passes: beyond 16 384 lookups the LDS sort takes only these by itself


def _slots(kind, n, rng):
    if kind == "uniform":
        return rng.integers(0, ROWS, n)
    if kind == "one":
        return np.full(n, ROWS - 1)
    if kind == "ordered":  # popular slots next to each other
        return (rng.random(n) ** 8 * ROWS).astype(np.int64)
    if kind == "heavy":  # two neighbours own a third each
        s = rng.integers(0, ROWS, n)
        pick = rng.random(n)
        s[pick < 0.66] = 1234
        s[pick < 0.33] = 1235
        return s
    if kind == "misled":  # every sampled lookup is on slot 7, hardly any other
        s = rng.integers(1000, ROWS, n)
        s[np.arange(1024, dtype=np.int64) * n // 1024] = 7
        return s
    return np.where(rng.random(n) < 0.5, rng.integers(0, 3, n), rng.integers(0, ROWS, n))  # "few": three own half


def _step(variant, slots, offs, S, lengths, fused=False, rows=ROWS, dim=4):
    nt = len(slots)
    hp = HotPath([rows] * nt, dim)
    B.fae_set_option(hp.ctx, "sort_variant", variant)
    hp.alloc_counts()
    hp.build([0] * nt, [rows] * nt, seed=3)
    hb = HotBatch(S, slots, offs, lengths)
    gout = torch.randn((S, nt, dim), device="cuda", generator=torch.Generator(device="cuda").manual_seed(S))
    out = hp.forward_presort(hb) if fused else None
    uniq, runs = hp.backward_sgd(hb, gout, 0.05, debug=True)
    return hp, list(uniq) + list(runs) + [w.clone() for w in hp.hotW] + ([out.clone()] if fused else [])


KINDS = ["uniform", "one", "ordered", "heavy", "misled", "few"]


@pytest.mark.parametrize("n", [7168, 7169, 10_240, 10_241, 16384, 16385, 40_003, 100_000, 131_071])
@pytest.mark.parametrize("kind", KINDS)
def test_long_lists_as_the_radix_passes(n, kind):
    rng = np.random.default_rng(n)
    one = [torch.from_numpy(_slots(kind, n, rng).astype(np.int32)).cuda(), torch.from_numpy(_slots("uniform", n, rng).astype(np.int32)).cuda()]
    want = _step(1, one, [None] * 2, n, [n] * 2, fused=True)[1]
    got = _step(0, one, [None] * 2, n, [n] * 2, fused=True)[1]
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    for S in (500, 9001):  # bags, empty ones among them; offsets of more than LDS holds
        offs = [torch.from_numpy(np.concatenate([[0], np.sort(rng.integers(0, n + 1, S - 1)), [n]]).astype(np.int32)).cuda() for _ in one]
        want = _step(1, one, offs, S, [n] * 2)[1]
        got = _step(0, one, offs, S, [n] * 2)[1]
        assert all(torch.equal(a, b) for a, b in zip(want, got))


@pytest.mark.parametrize("kind", ["uniform", "ordered", "heavy"])
@pytest.mark.parametrize("n", [11_000, 50_001])
def test_slots_out_of_range_and_unaligned_lists(n, kind):
    rng = np.random.default_rng(n)
    s = _slots(kind, n, rng).astype(np.int32)
    s[rng.random(n) < 0.1] = -1
    s[rng.random(n) < 0.1] = ROWS
    s[rng.random(n) < 0.01] = 2**31 - 1
    buf = torch.empty(n + 1, dtype=torch.int32, device="cuda")
    buf[1:] = torch.from_numpy(s).cuda()
    slots = [buf[1:]]
    weights = []
    for variant in (1, 0):
        hp, res = _step(variant, slots, [None], n, [n])
        with pytest.raises(B.FaeError):
            hp.sync()
        weights.append(res[2])
    assert torch.equal(*weights)


def test_many_samples_with_empty_bags():
    """More samples than the LDS sort numbers: the passes take the list, whatever its length."""
    rng = np.random.default_rng(3)
    n, S = 9000, 140_000
    slots = [torch.from_numpy(_slots("few", n, rng).astype(np.int32)).cuda()]
    offs = [torch.from_numpy(np.concatenate([[0], np.sort(rng.integers(0, n + 1, S - 1)), [n]]).astype(np.int32)).cuda()]
    want, got = (_step(v, slots, offs, S, [n])[1] for v in (1, 0))
    assert all(torch.equal(a, b) for a, b in zip(want, got))


@pytest.mark.parametrize("nt,n", [(1, 1), (1, 31), (1, 33), (2, 511), (2, 513), (26, 5120), (26, 5121), (26, 10_753)])
@pytest.mark.parametrize("dim", [4, 60, 64, 128, 260])
def test_row_copies_beside_the_sort(nt, n, dim):
    """Pieces of 32 samples per wave, and both sides of the rule on how many copies run beside the sorts."""
    rng = np.random.default_rng(n + dim)
    one = [torch.from_numpy(rng.integers(0, 999, n).astype(np.int32)).cuda() for _ in range(nt)]
    want = _step(1, one, [None] * nt, n, [n] * nt, fused=True, rows=999, dim=dim)[1]
    got = _step(0, one, [None] * nt, n, [n] * nt, fused=True, rows=999, dim=dim)[1]
    assert all(torch.equal(a, b) for a, b in zip(want, got))
