"""Seeded random shapes through the library against the oracle: table counts from 1 to 64, row
widths that are and are not multiples of four, batches on both sides of the tile and tier limits,
one-lookup and multi-lookup tables mixed, uniform to heavily skewed slots, a very long bag now and
then, every call sequence of the step and random settings of the kernel options.  The cases are
fixed by their seeds; each prints what it is before it runs."""
import numpy as np
import pytest
import torch

from oracle import fae_oracle as O
from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd import synth as S
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

import fae_testlib as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return torch.device("cuda", 0)


@pytest.mark.parametrize("case", range(24))
def test_random_step(dev, case):
    """Three steps of forward + backward + SGD on one random batch, through HotPath.prepare_steps in a
    random mode, compared in full after every step; then distinct slots and multiplicities."""
    rng = np.random.default_rng(41000 + case)
    nt = int(rng.choice([1, 2, 3, 5, 8, 13, 26, 40, 64]))
    dim = int(rng.choice([1, 2, 4, 6, 8, 12, 16, 20, 32, 48, 64, 96, 128, 200, 256, 260]))
    S_ = int(rng.choice([1, 2, 63, 64, 65, 127, 300, 1000, 2048, 4097, 8192, 16384, 16385, 20000]))
    if nt * S_ * dim > 20_000_000:
        S_ = max(1, 20_000_000 // (nt * dim))
    kinds = str(rng.choice(["one", "multi", "mix"], p=[0.4, 0.3, 0.3]))
    skew = float(rng.choice([0.0, 0.8, 1.2, 2.0]))
    n_hot = [int(x) for x in np.exp(rng.uniform(0, np.log(300_000), nt)).astype(np.int64) + 1]
    lr = float(rng.choice([0.01, 0.05, 0.5]))
    slots, offs = [], []
    for n in n_hot:
        if kinds == "one" or (kinds == "mix" and rng.random() < 0.5):
            nl = S_
            offs.append(None)
        else:
            lens = rng.integers(0, int(rng.choice([2, 5, 30, 120])) + 1, S_)
            if rng.random() < 0.2 and S_ > 3:
                lens[rng.integers(0, S_)] = int(rng.integers(200, 3000))     # one very long bag
            o = np.zeros(S_ + 1, dtype=np.int32)
            o[1:] = np.cumsum(lens)
            nl = int(o[-1])
            offs.append(o)
        if skew == 0.0:
            s_ = rng.integers(0, n, nl)
        else:
            s_ = ((rng.zipf(1.0 + skew, nl) - 1) * (int(rng.integers(1, 1 << 30)) | 1)) % n
        slots.append(s_.astype(np.int32))
    mode = str(rng.choice(["auto", "none", "fused", "ahead"]))
    opts = {}
    for name, values, p_ in (("reduce_span", [0, 64, 128, 256], 0.5), ("sort_variant", [0, 1, 2, 3, 4], 0.3),
                             ("reduce_variant", [1, 2], 0.3), ("fixup_variant", [0, 1], 0.3), ("reduce_unroll", [0, 2, 4], 0.3),
                             ("reduce_wg_waves", [0, 1, 2, 4], 0.3), ("fwd_variant", [0, 1, 2], 0.3)):
        if rng.random() < p_:
            opts[name] = int(rng.choice(values))
    print(f"case {case}: tables={nt} dim={dim} samples={S_} kinds={kinds} skew={skew} lookups={sum(x.size for x in slots)} "
          f"mode={mode} options={opts}", flush=True)
    hp = HotPath(n_hot, dim, 0)
    for k, v in opts.items():
        B.fae_set_option(hp.ctx, k, v)
    hp.n_hot = n_hot
    Wref = [(rng.random((n, dim), dtype=np.float32) - 0.5) for n in n_hot]
    hp.hotW = [torch.from_numpy(x.copy()).to(dev) for x in Wref]
    wtol = [np.zeros_like(x) for x in Wref]
    hb = HotBatch(S_, [torch.from_numpy(x).to(dev) for x in slots],
                  [None if o is None else torch.from_numpy(o).to(dev) for o in offs], [x.size for x in slots])
    n_steps = 3
    g_np = [rng.standard_normal((S_, nt, dim)).astype(np.float32) for _ in range(n_steps)]
    gouts = [torch.from_numpy(g).to(dev) for g in g_np]
    outs = [torch.full((S_, nt, dim), 7.0, dtype=torch.float32, device=dev) for _ in range(n_steps)]
    one_hot_fits = all(o is None for o in offs) and S_ <= 16384
    if mode == "fused" and not one_hot_fits:
        mode = "auto"                                    # the fused launch takes one-lookup tables of up to 16 384 samples
    steps, _ = hp.prepare_steps([hb] * n_steps, gouts, outs, lr, presort=mode)
    for k in range(n_steps):
        steps[k]()
        hp.sync()
        ref, mag = O.embbag_fwd(Wref, S_, slots, offs, want_mag=True)
        inherited = O.embbag_fwd(wtol, S_, slots, offs).astype(np.float64) * 1.001
        T.assert_close_sum(outs[k].cpu().numpy(), ref, mag, f"step {k}: forward", inherited)
        before = [x.copy() for x in Wref]
        uniq, runlen, mg = O.embbag_bwd_sgd(Wref, S_, slots, offs, g_np[k], lr, want_mag=True)
        for z in range(nt):
            got = hp.hotW[z].cpu().numpy()
            if uniq[z].size:
                inh = wtol[z][uniq[z]].astype(np.float64)
                T.assert_close_sum(got[uniq[z]], Wref[z][uniq[z]], mg[z], f"step {k}: table {z}", inh)
                wtol[z][uniq[z]] = (inh + T.RTOL * mg[z]).astype(np.float32) * np.float32(1.001)
            if k == 0:                                   # rows no lookup hit still hold their first values, bit for bit
                rest = np.ones(n_hot[z], dtype=bool)
                rest[uniq[z]] = False
                assert got[rest].tobytes() == before[z][rest].tobytes(), f"untouched rows of table {z} changed"
    dbg = hp.backward_sgd(hb, gouts[0], lr, debug=True)
    hp.sync()
    uniq, runlen, _ = O.embbag_bwd_sgd(Wref, S_, slots, offs, g_np[0], lr)
    for z in range(nt):
        assert np.array_equal(dbg[0][z].cpu().numpy(), uniq[z]), f"distinct slots of table {z} differ"
        assert np.array_equal(dbg[1][z].cpu().numpy(), runlen[z]), f"multiplicities of table {z} differ"


@pytest.mark.parametrize("case", range(16))
def test_random_pipeline(dev, case):
    """A random workload (table sizes, bag shapes, skew, hot rule) through every stage: histogram,
    cutoff, remap and hot tables, partition of an unconditioned chunk, forward and backward of its
    hot part."""
    rng = np.random.default_rng(52000 + case)
    nt = int(rng.choice([1, 2, 3, 7, 8, 26, 33, 64]))
    dim = int(rng.choice([1, 3, 4, 8, 16, 24, 64, 128, 132]))
    rows = tuple(int(x) for x in np.exp(rng.uniform(np.log(2), np.log(int(rng.choice([2000, 60000, 500000]))), nt)).astype(np.int64))
    kinds = []
    for _ in range(nt):
        k = str(rng.choice(["one", "uniform", "poisson"], p=[0.5, 0.3, 0.2]))
        if k == "one":
            kinds.append("one")
        elif k == "uniform":
            kinds.append(f"uniform:{int(rng.integers(0, 2))}:{int(rng.integers(2, 40))}")
        else:
            kinds.append(f"poisson:{int(rng.integers(1, 12))}:1:{int(rng.integers(12, 40))}")
    batch = int(rng.choice([1, 7, 64, 300, 1024, 2500]))
    prof = int(rng.choice([1000, 20000, 100000]))
    zipf = float(rng.choice([0.6, 1.0, 1.3]))
    if rng.random() < 0.5:
        rule = dict(hot_rule="cutoff", cutoff=int(rng.choice([0, 0, 1, 1, 2])))
    else:
        rule = dict(hot_rule="budget", budget_bytes=int(sum(rows) * dim * 4 * float(rng.choice([0.05, 0.5, 0.9, 1.5, 3.0]))) + 64,
                    small_table_bytes=int(rng.choice([1, 4096, 1 << 20])))
    w = S.Workload(f"random{case}", 90 + case % 7, rows, dim, tuple(kinds), zipf, batch, prof, lr=0.02,
                   seed=int(rng.integers(1, 1 << 40)), **rule)
    mat = bool(rng.random() < 0.4) and sum(rows) * dim < 30_000_000
    print(f"case {case}: tables={nt} dim={dim} rows={min(rows)}..{max(rows)} batch={batch} profile={prof} zipf={zipf} {rule} "
          f"materialise={mat}", flush=True)
    p = T.Pipeline(w, dev, profile_chunks=int(rng.integers(1, 4)), materialise=mat)
    p.check_profile()
    try:
        p.check_cutoff()
    except O.OracleError:
        pytest.skip("no threshold fits this budget (the oracle says so before the library is asked)")
    p.check_build()
    hb = p.check_partition(S.make_chunk(w, 5, 0, 3 * batch + 37))
    if hb.n_samples == 0 or sum(p.n_hot) == 0:
        return
    p.check_forward(hb)
    p.check_backward(hb, stream=20)
    p.check_forward(hb, exact_gather=False)
    p.check_backward(hb, stream=21, presort=hb)
    if all(k == "one" for k in kinds) and hb.n_samples <= 16384:
        p.check_forward(hb, exact_gather=False, fused=True)
        p.check_backward(hb, stream=23)
