"""GPU parity of the steps around the hot path: embedding synchronisation between the hot
tables and the full tables (Sec. 3 (4); Sec. 6.2), and the sampled estimate of the hot size
with its confidence interval and threshold search (Sec. 4.1.2, Eq. 2-4).  Row copies and
chunk counts are compared bit for bit; the fp64 statistics to 1e-12 relative (the summation
order of at most a few dozen terms may differ), the interval's half-width to 1e-8 relative
(the library computes the Student-t quantile itself, to that accuracy)."""
import numpy as np
import pytest
import torch

from oracle import fae_oracle as O
from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd import synth as S
from paper_2103_00686_amd.hotpath import HotPath

import fae_testlib as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return torch.device("cuda", 0)


def _manual_hotpath(rows, dim, hot_ids, hotW, dev):
    hp = HotPath(rows, dim, 0)
    hp.n_hot = [int(h.size) for h in hot_ids]
    hp.hot_ids = [torch.from_numpy(np.ascontiguousarray(h if h.size else np.zeros(1, np.int32))).to(dev) for h in hot_ids]
    hp.hotW = [torch.from_numpy(np.ascontiguousarray(w if w.shape[0] else np.zeros((1, dim), np.float32))).to(dev)
               for w in hotW]
    return hp


@pytest.mark.parametrize("dim", [64, 16, 6, 1, 132])
def test_sync_rows_both_directions_bit_exact(dev, dim):
    """Several tables in one launch: one with every row hot, one with none, ragged sizes that
    leave partial workgroups, vector and scalar row widths."""
    rng = np.random.default_rng(100 + dim)
    rows = [10_007, 513, 4_096, 77]
    n_hot = [3_001, 513, 0, 5]
    hot_ids = [np.sort(rng.choice(r, n, replace=False)).astype(np.int32) for r, n in zip(rows, n_hot)]
    W = [rng.standard_normal((r, dim)).astype(np.float32) for r in rows]
    hotW = [rng.standard_normal((n, dim)).astype(np.float32) for n in n_hot]
    hp = _manual_hotpath(rows, dim, hot_ids, hotW, dev)
    Wd = [torch.from_numpy(w).to(dev) for w in W]
    hp.sync_to_full(Wd)
    hp.sync()
    for z in range(len(rows)):
        ref = O.scatter_rows(W[z], hot_ids[z], hotW[z])
        assert Wd[z].cpu().numpy().tobytes() == ref.tobytes(), f"hot -> full, table {z}"
    # the other direction, from fresh full tables
    W2 = [rng.standard_normal((r, dim)).astype(np.float32) for r in rows]
    W2d = [torch.from_numpy(w).to(dev) for w in W2]
    hp.sync_from_full(W2d)
    hp.sync()
    for z in range(len(rows)):
        ref = O.gather_rows(W2[z], hot_ids[z])
        assert hp.hotW[z][:n_hot[z]].cpu().numpy().tobytes() == ref.tobytes(), f"full -> hot, table {z}"
        assert W2d[z].cpu().numpy().tobytes() == W2[z].tobytes()           # the source is not written


@pytest.mark.parametrize("dim", [64, 63])  # 16-byte and scalar columns
@pytest.mark.parametrize("extra", [-1, 0])  # rows of 144 MiB are streamed past the caches, fewer are not
def test_sync_rows_of_either_kind_of_access(dev, dim, extra):
    n = -(-(144 << 20) // (4 * dim)) + extra
    n_hot = [n // 3, 0, n - n // 3]
    rows = [2 * r + 5 for r in n_hot]
    gen = torch.Generator(device=dev).manual_seed(dim)
    hp = HotPath(rows, dim, 0)
    hp.n_hot = n_hot
    hp.hot_ids = [torch.randperm(r, device=dev, generator=gen)[:h].sort().values.int() for r, h in zip(rows, n_hot)]
    hp.hotW = [torch.randn((max(h, 1), dim), device=dev, generator=gen) for h in n_hot]
    W = [torch.randn((r, dim), device=dev, generator=gen) for r in rows]
    want = [w.clone() for w in W]
    for z, h in enumerate(n_hot):
        want[z][hp.hot_ids[z].long()] = hp.hotW[z][:h]
    hp.sync_to_full(W)
    hp.sync()
    assert all(torch.equal(a, b) for a, b in zip(W, want))
    for w in W:
        w.mul_(-2.0)
    hp.sync_from_full(W)
    hp.sync()
    for z, h in enumerate(n_hot):
        assert torch.equal(hp.hotW[z][:h], W[z][hp.hot_ids[z].long()])


def test_sync_rows_reports_bad_ids_and_arguments(dev):
    rows, dim = [100], 8
    ids = np.array([3, 250, 7], dtype=np.int32)                           # 250 is outside the table
    hp = _manual_hotpath(rows, dim, [ids], [np.ones((3, dim), np.float32)], dev)
    Wd = [torch.zeros((100, dim), dtype=torch.float32, device=dev)]
    hp.sync_to_full(Wd)
    with pytest.raises(B.FaeError) as e:
        hp.sync()
    assert e.value.code == B.FAE_ERANGE
    got = Wd[0].cpu().numpy()
    assert got[3].min() == 1.0 and got[7].min() == 1.0 and got.sum() == 2 * dim   # valid rows copied, nothing else
    with pytest.raises(B.FaeError):
        B.fae_sync_hot_rows(hp.ctx, hp.tables, [3], hp.hot_ids, hp.hotW, Wd, 7)
    with pytest.raises(B.FaeError):
        B.fae_sync_hot_rows(hp.ctx, hp.tables, [101], hp.hot_ids, hp.hotW, Wd, B.FAE_SYNC_HOT_TO_FULL)


@pytest.mark.parametrize("cfg_id", [1, 2, 4])
def test_swap_after_training_steps(dev, cfg_id):
    """Hot mini-batches train the hot tables, then the swap writes them back: the full
    tables of the two sides agree within the tolerance the updates carry, cold rows are
    bit-identical, and fetching the rows again gives back the hot tables bit for bit."""
    w = S.workload(cfg_id, "test")
    p = T.Pipeline(w, dev, profile_chunks=2, materialise=True)
    p.check_profile()
    p.check_cutoff()
    p.check_build()
    batches = T.hot_batches(p, 2)
    for i, hb in enumerate(batches):
        p.check_backward(hb, stream=40 + i)
    full_ref = [S.full_table(w, z).numpy() for z in range(w.n_tables)]
    full_dev = [torch.from_numpy(f).to(dev) for f in full_ref]
    p.hp.sync_to_full(full_dev)
    p.hp.sync()
    for z in range(w.n_tables):
        n = p.n_hot[z]
        ref = O.scatter_rows(full_ref[z], p.hot_ids[z], p.hotW[z])
        got = full_dev[z].cpu().numpy()
        cold = np.ones(w.rows[z], bool)
        cold[p.hot_ids[z]] = False
        assert got[cold].tobytes() == full_ref[z][cold].tobytes(), f"cold rows of table {z} changed"
        err = np.abs(got[p.hot_ids[z]].astype(np.float64) - ref[p.hot_ids[z]].astype(np.float64))
        assert (err <= p.wtol[z].astype(np.float64) + 1e-30).all(), f"hot rows of table {z} outside the carried tolerance"
        assert got[p.hot_ids[z]].tobytes() == p.hp.hotW[z][:n].cpu().numpy().tobytes()   # a copy, not arithmetic
    before = [x.clone() for x in p.hp.hotW]
    for x in p.hp.hotW:
        x.zero_()
    p.hp.sync_from_full(full_dev)
    p.hp.sync()
    for z in range(w.n_tables):
        assert torch.equal(p.hp.hotW[z][:p.n_hot[z]], before[z][:p.n_hot[z]])


@pytest.mark.parametrize("cfg_id,m,n", [(3, 1024, 35), (2, 256, 35), (5, 1000, 12)])
def test_chunk_counts_and_interval(dev, cfg_id, m, n):
    """Eq. 2 bit-exact per chunk, Eq. 3 and Eq. 4 in fp64, for several cutoffs; includes tables
    smaller than n chunks (a census) and short last chunks (m does not divide the rows)."""
    w = S.workload(cfg_id, "test")
    p = T.Pipeline(w, dev, profile_chunks=2)
    p.check_profile()
    chunks = [S.sample_chunks(w, z, m, n) for z in range(w.n_tables)]
    for z in range(w.n_tables):                     # make sure the short last chunk is among them
        N = -(-w.rows[z] // m)
        if N - 1 not in chunks[z]:
            chunks[z][0] = N - 1
    for H in (0, 1, 2, 5, 1 << 31):
        est, Cs = p.hp.estimate_hot([H] * w.n_tables, chunks, m, 0.999)
        for z in range(w.n_tables):
            ref_C = O.chunk_counts(p.cnts[z], m, chunks[z], H)
            assert Cs[z] == ref_C.tolist(), f"chunk counts of table {z} at H={H}"
            if len(chunks[z]) < 2:
                continue
            rows, half, ybar, s = O.estimate_hot_rows(p.cnts[z], m, chunks[z], H, 0.999)
            e = est[z]
            assert e["N"] == -(-w.rows[z] // m) and e["n"] == len(chunks[z])
            for got, ref in ((e["rows"], rows), (e["ybar"], ybar), (e["s"], s)):
                assert abs(got - ref) <= 1e-12 * max(abs(ref), 1.0)
            assert abs(e["half_rows"] - half) <= 1e-8 * max(half, 1.0)   # carries the t quantile (1e-8, see host tests)
            if e["n"] == e["N"]:                     # census: exact count, no width
                assert e["half_rows"] == 0.0 and abs(e["rows"] - O.count_hot(p.cnts[z], H)) < 1e-6


def test_estimate_rejects_bad_chunks(dev):
    w = S.workload(1, "test")
    p = T.Pipeline(w, dev, profile_chunks=1)
    p.check_profile()
    good = [S.sample_chunks(w, z, 64, 4) for z in range(w.n_tables)]
    for bad in ([good[0][0], good[0][0]], [-1], [10 ** 9]):
        chunks = [list(bad)] + good[1:]
        with pytest.raises(B.FaeError) as e:
            p.hp.estimate_hot([1] * w.n_tables, chunks, 64, 0.999)
        assert e.value.code == B.FAE_EINVAL
    with pytest.raises(B.FaeError):
        p.hp.estimate_hot([1] * w.n_tables, good, 64, 1.5)


@pytest.mark.parametrize("cfg_id,frac", [(2, 0.10), (2, 0.005), (3, 0.05), (3, 2.0), (3, 0.002), (5, 0.001)])
def test_sampled_threshold_search(dev, cfg_id, frac):
    """Statistical Optimizer on the sampled logger: same c and cutoffs as the oracle's scan,
    for budgets that make the answer c = 0, a small c, and a c past the first doublings."""
    w = S.workload(cfg_id, "test")
    p = T.Pipeline(w, dev, profile_chunks=2)
    p.check_profile()
    m, n = 256, 35
    chunks = [S.sample_chunks(w, z, m, n, draw=1) for z in range(w.n_tables)]
    T_ = [sum(ch.n_lookups[z] for ch in p.prof) for z in range(w.n_tables)]
    t_denom = max(max(T_), 1)
    budget = int(frac * sum(w.rows) * w.dim * 4)
    small = 1 << 14
    c_ref, H_ref = O.sampled_budget_cutoff(w.dim, p.cnts, T_, t_denom, budget, small, m, chunks)
    c, H, est = p.hp.choose_cutoff_sampled(budget, chunks, m, 0.999, small)
    assert (c, H) == (c_ref, H_ref), f"gpu {(c, H)} vs oracle {(c_ref, H_ref)}"
    total = 0.0
    for z in range(w.n_tables):
        if w.rows[z] * w.dim * 4 < small:
            assert est[z]["rows"] == w.rows[z] and est[z]["half_rows"] == 0.0
        else:
            rows, half, _, _ = O.estimate_hot_rows(p.cnts[z], m, chunks[z], H[z], 0.999)
            assert abs(est[z]["rows"] - rows) <= 1e-9 * max(rows, 1.0)
            if len(chunks[z]) >= 2:          # one chunk has no standard deviation: reported as 0
                assert abs(est[z]["half_rows"] - half) <= 1e-8 * max(half, 1.0)
            else:
                assert est[z]["half_rows"] == 0.0
        total += est[z]["rows"] * w.dim * 4
    assert total <= budget * (1 + 1e-12)
