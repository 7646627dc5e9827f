"""The forms of the backward's radix passes give the same stable order: with tiles that add up their
table's digit counts themselves (the rule's choice here), with chained tiles and with separate
histogram kernels, distinct slots, multiplicities and updated weights are the same bytes.  List
lengths sit at the edges of a tile (1024), of the LDS sort (16 384) and of the direct form (128
tiles per table), of the tiles that the direct form takes in all (one per compute unit, most of them in
a few tables) and of small tiles (1024); one slot may own most of a list; slots take one to four digits."""
import numpy as np
import pytest
import torch

from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

pytestmark = pytest.mark.gpu


CHIP = 256 * 1024  # lookups in one tile per compute unit
KINDS = {
    "one_digit": ([200, 255, 3], [17 * 1024, 3000, 500], True),
    "two_digits": ([40_000, 255], [40 * 1024 + 5, 20_000], True),
    "four_digits": ([17_000_000, 1000], [30 * 1024, 17_000], True),
    "chip": ([70_000, 9000], [CHIP // 2, CHIP // 2], True),
    "chip_and_one": ([70_000, 9000, 800], [CHIP // 2, CHIP // 2, 1], True),
    "six_equal": ([5000] * 6, [18 * 1024] * 6, True),
    "seven_equal": ([5000] * 7, [18 * 1024] * 7, True),
    "small_tiles": ([90_000] * 8, [128 * 1024] * 8, True),
    "small_tiles_and_one": ([90_000] * 8 + [70], [128 * 1024] * 8 + [1], True),
}
DIRECT = {"one_digit", "two_digits", "four_digits", "chip", "six_equal", "edges", "most", "one_hot"}


def _lists(kind, seed):
    rng = np.random.default_rng(seed)
    S = 4100
    rows, lengths, bags = KINDS[kind] if kind in KINDS else {
        "edges": ([3_000_000, 300, 70_000, 5, 1], [16385, 17 * 1024, 1023, 1025, 1], True),
        "most": ([200_000, 65_535, 900], [128 * 1024, 127 * 1024 + 1, 0], True),
        "beyond": ([200_000, 4000], [128 * 1024 + 1, 20_000], True),
        "one_hot": ([1 << 20, 256, 257, 100_000], None, False),
    }[kind]
    if not bags:
        S = 50_001
        lengths = [S] * len(rows)
    slots, offs = [], []
    for z, (r, n) in enumerate(zip(rows, lengths)):
        s = rng.integers(0, r, n)
        s[rng.random(n) < (0.0, 0.7, 0.2)[z % 3]] = r - 1  # a slot that owns much of the list
        slots.append(torch.from_numpy(s.astype(np.int32)).cuda())
        cuts = np.sort(rng.integers(0, n + 1, S - 1))  # empty bags among them
        offs.append(torch.from_numpy(np.concatenate([[0], cuts, [n]]).astype(np.int32)).cuda() if bags else None)
    return rows, S, slots, offs, lengths


@pytest.mark.parametrize("kind", ["edges", "most", "beyond", "one_hot"] + list(KINDS))
def test_every_form_of_pass_gives_the_same_step(kind):
    rows, S, slots, offs, lengths = _lists(kind, 11)
    dim = 8 if max(rows) < 1 << 24 else 2
    gen = torch.Generator(device="cuda").manual_seed(5)
    gout = torch.randn((S, len(rows), dim), device="cuda", generator=gen)
    hb = HotBatch(S, slots, offs, [int(n) for n in lengths])
    want = None
    for variant in (0, 3, 1):
        hp = HotPath(rows, dim)
        B.fae_set_option(hp.ctx, "sort_variant", variant)
        hp.alloc_counts()
        hp.build([0] * len(rows), rows, seed=3)
        got = []
        B.fae_timing_enable(hp.ctx, True)
        for _ in range(2):  # the second step runs over a workspace that holds the first one's counts
            uniq, runs = hp.backward_sgd(hb, gout, 0.05, debug=True)
            got += list(uniq) + list(runs) + [w.clone() for w in hp.hotW]
        hp.sync()
        if variant == 0 and torch.cuda.get_device_properties(0).multi_processor_count == 256:
            fills = [B.fae_timing_read(hp.ctx, k)[1] for k in range(B.FAE_K_COUNT) if "fill" in B.fae_kernel_name(k)]
            assert (fills[0] == 0) == (kind in DIRECT)  # only the direct form clears nothing by a launch of its own
        if want is None:
            want = got
            for z, s in enumerate(slots):
                u, c = torch.unique(s, return_counts=True)
                assert torch.equal(uniq[z], u) and torch.equal(runs[z], c.int())
        assert all(torch.equal(a, b) for a, b in zip(want, got)), f"sort_variant {variant}"
