"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is a dict of plain values:
  path      which call sequence (see ``prepare`` and ``run``)
  rows      rows of every table, comma-separated (the hot tables' rows for forward and train)
  bags      bag kind of every table, comma-separated (``one``, ``uniform:a:b``, ``poisson:lam:a:b``)
  dim       row dimension, fp32
  zipf      skew of the accesses
  samples   samples in the batch (forward, train) or in the chunk (profile, partition)
and, where the path has them, ``cycle`` (train: hot batches taken in turn in one pass),
``optimizer`` / ``pooling``, ``index_bits``, ``profiled`` (samples behind the access counters),
``budget`` (bytes for the hot rows) and ``source`` (where hot rows come from).

Popularity follows a bounded Zipf law over a seeded permutation of the rows, as in the
package's own workloads; another seed is another permutation, other draws and other gradients.
"""
import math

import numpy as np
import torch

from paper_2103_00686_amd import binding as B
from paper_2103_00686_amd import synth
from paper_2103_00686_amd.hotpath import HotBatch, HotPath

SMALL_TABLE = 1 << 20  # tables below this many bytes are hot as a whole (HotPath's default)
LR = 0.01


def _text(values):
    return ",".join(str(v) for v in values)


def _rows(case):
    return tuple(int(v) for v in case["rows"].split(","))


def _bags(case):
    return tuple(case["bags"].split(","))


def listed():
    law = synth.loguniform_rows
    kaggle = law(26, 10, 200_000, synth.SEED, 2, 9001)      # hot rows of a 26-table set, 16 wide
    terabyte = law(26, 10, 400_000, synth.SEED, 3, 9002)    # about one million hot rows, 64 wide
    full = law(26, 10, 40_000_000, synth.SEED, 3, 9002)     # the same set's full tables: 72 M rows
    one26 = _text(["one"] * 26)
    return [
        # serving a behaviour history: long uneven bags, a row width that fills no power of two
        dict(name="forward_4x6007_d100_bags", path="forward", rows="1000000,300000,50000,900", dim=100, zipf=1.0,
             bags="uniform:1:100,uniform:1:30,poisson:20:1:64,one", samples=6007),
        # the smallest training step: one table, a thousand samples
        dict(name="train_1x1024_d16", path="train", rows="100000", bags="one", dim=16, zipf=1.05, samples=1024, cycle=1),
        # Kaggle-like: 26 one-hot tables, 4096 samples
        dict(name="train_26x4096_d16", path="train", rows=_text(kaggle), bags=one26, dim=16, zipf=1.1, samples=4096, cycle=1),
        # Terabyte-like, the headline workload of bench.py
        dict(name="train_26x16384_d64", path="train", rows=_text(terabyte), bags=one26, dim=64, zipf=1.2, samples=16384, cycle=1),
        # the same tables with the large batches that data-parallel training takes; ragged
        dict(name="train_26x50001_d64", path="train", rows=_text(terabyte), bags=one26, dim=64, zipf=1.2, samples=50001, cycle=1),
        # Taobao-like: user / item / category with behaviour histories; four batches in turn, so
        # the call sequence that sorts the next batch ahead is the one that runs
        dict(name="train_3x2048_d32_bags", path="train", rows="1000000,4000000,10000", bags="one,uniform:1:100,uniform:1:100",
             dim=32, zipf=1.0, samples=2048, cycle=4),
        # weak skew, wide rows, ten million lookups: the largest step
        dict(name="train_8x65536_d128_bags", path="train", rows=_text([1_000_000] * 8), bags=_text(["poisson:20:1:64"] * 8),
             dim=128, zipf=0.9, samples=65536, cycle=1),
        # mean pooling and row-wise Adagrad on a ragged batch of short bags
        dict(name="train_5x3001_d20_adagrad", path="train_opts", rows="250000,40000,3000,77,120000", dim=20, zipf=1.05,
             bags="uniform:1:10,one,uniform:1:30,one,poisson:20:1:64", samples=3001, pooling="mean", optimizer="adagrad"),
        # pre-processing of a Terabyte-like set: count accesses of a chunk of the sampled stream
        dict(name="profile_26x262144", path="profile", rows=_text(full), bags=one26, dim=64, zipf=1.2, samples=262144, index_bits=32),
        # threshold under the memory budget, classification, hot tables copied out of the full ones
        dict(name="build_16_tables_d64", path="build", rows=_text(law(16, 10, 40_000_000, synth.SEED, 3, 9002)), bags=_text(["one"] * 16),
             dim=64, zipf=1.2, profiled=1 << 20, budget=1 << 29, source="device"),
        # hot / cold split of a chunk of raw inputs
        dict(name="partition_26x262144", path="partition", rows=_text(full), bags=one26, dim=64, zipf=1.2, samples=262144, profiled=1 << 18,
             budget=1 << 29, index_bits=32),
        # a swap between hot and cold batches: 0.2 GiB of hot rows into the full tables and back
        dict(name="sync_26_tables_d64", path="sync", rows=_text(law(26, 10, 10_000_000, synth.SEED, 2, 9001)), bags=one26, dim=64,
             zipf=1.1, profiled=1 << 19, budget=1 << 29),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges.  Sizes follow their logarithm; a case that would cost
    more than the largest listed step is made smaller until it does not."""
    path = rng.choice(["train", "train", "train", "train_opts", "forward", "profile", "build", "partition", "sync"])
    dim = rng.choice([8, 16, 20, 32, 50, 64, 100, 128])
    zipf = rng.choice([0.9, 1.0, 1.05, 1.1, 1.2])
    if path in ("forward", "train", "train_opts"):
        multi = path == "train_opts" or rng.random() < 0.4
        nt = rng.choice([1, 3, 5, 8]) if multi else rng.choice([1, 4, 8, 13, 26])
        hi = _log(rng, 20_000, 1_000_000)
        rows = [_log(rng, 10, hi) for _ in range(nt - 1)] + [hi]
        kinds = ["uniform:1:10", "uniform:1:30", "uniform:1:100", "poisson:20:1:64", "one"] if multi else ["one"]
        bags = [rng.choice(kinds) for _ in range(nt)]
        samples = _log(rng, 64 if path == "forward" else 512, 65536)
        per_sample = sum(_mean_length(b) for b in bags)
        while samples * per_sample * dim > 6e8 or samples * nt * dim > 1.2e8 or samples * per_sample > 1e7:
            samples = samples * 2 // 3
        case = dict(path=path, rows=_text(rows), bags=_text(bags), dim=dim, zipf=zipf, samples=samples)
        if path == "train":
            case["cycle"] = rng.choice([1, 1, 2]) if samples * per_sample < 1e6 else 1
        if path == "train_opts":
            case["pooling"] = rng.choice(["sum", "mean"])
            case["optimizer"] = rng.choice(["sgd", "adagrad", "adagrad"])
        return case
    nt = rng.choice([1, 3, 8, 16])
    hi = _log(rng, 100_000, 40_000_000)
    rows = [_log(rng, 10, hi) for _ in range(nt - 1)] + [hi]
    while sum(rows) > 80_000_000 or (path == "sync" and sum(rows) * dim > 1_500_000_000):
        rows = [max(10, r // 2) for r in rows]
    bags = [rng.choice(["one", "one", "uniform:1:30", "poisson:20:1:64"]) if path in ("profile", "partition") and nt <= 8 else "one"
            for _ in range(nt)]
    per_sample = sum(_mean_length(b) for b in bags)
    case = dict(path=path, rows=_text(rows), bags=_text(bags), dim=dim, zipf=zipf)
    if path in ("profile", "partition"):
        samples = _log(rng, 2048, 1 << 19)
        while samples * per_sample > 1.2e7:
            samples = samples * 2 // 3
        case["samples"] = samples
        case["index_bits"] = rng.choice([32, 32, 64])
    if path != "profile":
        case["profiled"] = _log(rng, 1 << 15, 1 << 20)
        while case["profiled"] * per_sample > 1.7e7:
            case["profiled"] //= 2
        case["budget"] = 1 << rng.randint(26, 29)
        while case["budget"] < 2 * SMALL_TABLE * nt:
            case["budget"] *= 2
    if path == "build":
        case["source"] = rng.choice(["device", "procedural"]) if sum(rows) * dim < 5_000_000_000 else "procedural"
    return case


# --------------------------------------------------------------------------------------
def _workload(case, seed):
    return synth.Workload(case["path"], 50, _rows(case), case["dim"], _bags(case), case["zipf"], case.get("samples", 0),
                          case.get("profiled", 0), "cutoff", lr=LR, seed=seed)


def _chunk(w, stream, samples, bits=32):
    ch = synth.make_chunk(w, stream, 0, samples, "cuda")
    idx = [i.to(torch.int64) for i in ch.indices] if bits == 64 else ch.indices
    return B.Batch(ch.n_samples, idx, ch.offsets, ch.n_lookups, bits)


def _profiled(case, w):
    """A HotPath whose counters hold `profiled` samples of the stream."""
    hp = HotPath(w.rows, w.dim)
    done, most = 0, max(1, int(4e6 / sum(_mean_length(b) for b in w.bag_kinds)))
    stream = 100
    while done < case["profiled"]:
        n = min(most, case["profiled"] - done)
        hp.profile(_chunk(w, stream, n))
        done += n
        stream += 1
    return hp


def prepare(case, seed):
    path = case["path"]
    w = _workload(case, seed)
    nt = len(w.rows)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    st = {"path": path}
    if path in ("forward", "train", "train_opts"):
        hp = st["hp"] = HotPath(w.rows, w.dim)
        hp.alloc_counts()
        hp.build([0] * nt, w.rows, seed=seed)  # every row is hot: slot = row
        hbs, gouts, outs = [], [], []
        for k in range(case.get("cycle", 1)):
            ch = synth.make_chunk(w, k, 0, case["samples"], "cuda")
            hbs.append(HotBatch(ch.n_samples, ch.indices, ch.offsets, list(ch.n_lookups)))
            outs.append(torch.empty((ch.n_samples, nt, w.dim), dtype=torch.float32, device="cuda"))
            if path != "forward":
                gouts.append(torch.randn((ch.n_samples, nt, w.dim), dtype=torch.float32, device="cuda", generator=gen))
        st.update(hbs=hbs, gouts=gouts, outs=outs)
        if path == "train":
            # one batch: forward and backward of that batch, nothing of another one beside it
            st["steps"], _ = hp.prepare_steps(hbs, gouts, outs, LR, single_stream=len(hbs) == 1)
        if path == "train_opts":
            st["ws"] = hp.bwd_workspace(hbs[0])
            st["pooling"] = B.FAE_POOL_MEAN if case["pooling"] == "mean" else B.FAE_POOL_SUM
            st["optimizer"] = B.FAE_OPT_ROWWISE_ADAGRAD if case["optimizer"] == "adagrad" else B.FAE_OPT_SGD
            st["state"] = [torch.zeros(max(r, 1), dtype=torch.float32, device="cuda") for r in w.rows]
    elif path == "profile":
        st["hp"] = HotPath(w.rows, w.dim)
        st["hp"].alloc_counts()
        st["chunk"] = _chunk(w, 0, case["samples"], case["index_bits"])
    else:
        hp = st["hp"] = _profiled(case, w)
        st.update(budget=case["budget"], seed=seed, hot=_hot_buffers(hp, case["budget"]), W=None)
        if case.get("source") == "device" or path == "sync":
            st["W"] = [torch.empty((r, w.dim), dtype=torch.float32, device="cuda").uniform_(-0.05, 0.05, generator=gen) for r in w.rows]
        if path != "build":
            _, _, st["n_hot"] = _build(st, None)
        if path == "sync":
            for t in st["hot"]["rows"]:
                t.add_(0.5)  # trained since: the two copies differ
        if path == "partition":
            ch = st["chunk"] = _chunk(w, 0, case["samples"], case["index_bits"])
            S = ch.n_samples
            # what a loader keeps from chunk to chunk: sized for the longest bags
            st["lists"] = [torch.zeros(S, dtype=torch.int32, device="cuda") for _ in range(2)]
            st["slots"] = [torch.zeros(S * _longest(b), dtype=torch.int32, device="cuda") for b in w.bag_kinds]
            st["offsets"] = [torch.zeros(S + 1, dtype=torch.int32, device="cuda") for _ in w.rows]
            st["ws"] = torch.empty(B.fae_partition_workspace_bytes(hp.tables, S), dtype=torch.uint8, device="cuda")
    return st


def _hot_buffers(hp, budget):
    """Hot tables as a trainer holds them: room for what the budget allows, filled as far as needed."""
    caps = [min(r, budget // (4 * hp.dim)) for r in hp.tables.rows]
    new = lambda shape, t: torch.zeros(shape, dtype=t, device="cuda")  # noqa: E731
    return {"caps": caps, "remap": [new(r, torch.int32) for r in hp.tables.rows], "ids": [new(c, torch.int32) for c in caps],
            "rows": [new((c, hp.dim), torch.float32) for c in caps],
            "ws": torch.empty(B.fae_build_workspace_bytes(hp.tables), dtype=torch.uint8, device="cuda")}


def _build(st, W):
    hp, hot = st["hp"], st["hot"]
    c, cutoff, _ = hp.choose_cutoff(st["budget"])
    kind = B.FAE_SRC_PROCEDURAL if W is None else B.FAE_SRC_DEVICE
    n_hot = B.fae_build_hot_tables(hp.ctx, hp.tables, hp.counts, cutoff, kind, W, st["seed"], hot["remap"], hot["ids"], hot["rows"],
                                   hot["caps"], hot["ws"])
    return c, cutoff, n_hot


def run(st):
    path, hp = st["path"], st["hp"]
    if path == "forward":
        return hp.forward(st["hbs"][0], st["outs"][0])
    if path == "train":
        for step in st["steps"]:
            step()
        return {"out": st["outs"], "weights": hp.hotW}
    if path == "train_opts":
        hb, out, gout = st["hbs"][0], st["outs"][0], st["gouts"][0]
        stride = hp.nt * hp.dim
        B.fae_embbag_fwd_opts(hp.ctx, hp.hot_tables, hp.hotW, hb.batch(), out, stride, st["pooling"])
        B.fae_embbag_bwd_opts(hp.ctx, hp.hot_tables, hp.hotW, hb.batch(), gout, stride, LR, st["ws"], st["pooling"],
                              st["optimizer"], 1e-8, st["state"])
        return {"out": out, "weights": hp.hotW, "state": st["state"]}
    if path == "profile":
        hp.profile(st["chunk"])
        return hp.counts
    hot = st["hot"]
    if path == "build":
        c, cutoff, n_hot = _build(st, st["W"])
        return {"cutoff": np.array([c] + list(cutoff), dtype=np.int64), "n_hot": np.array(n_hot, dtype=np.int64),
                "remap": hot["remap"], "ids": hot["ids"], "rows": hot["rows"]}
    if path == "partition":
        n_hot, n_lookups = B.fae_partition_batch(hp.ctx, hp.tables, st["chunk"], hot["remap"], st["lists"][0], st["lists"][1], st["slots"],
                                                 st["offsets"], st["ws"])
        return {"counts": np.array([n_hot] + list(n_lookups), dtype=np.int64), "lists": st["lists"], "slots": st["slots"],
                "offsets": st["offsets"]}
    # training switches to cold batches and back: the full tables take the hot rows, then give them back
    for direction in (B.FAE_SYNC_HOT_TO_FULL, B.FAE_SYNC_FULL_TO_HOT):
        B.fae_sync_hot_rows(hp.ctx, hp.tables, st["n_hot"], hot["ids"], hot["rows"], st["W"], direction)
    return {"full": st["W"], "hot": hot["rows"]}


# --------------------------------------------------------------------------------------
def _mean_length(kind):
    parts = kind.split(":")
    if parts[0] == "one":
        return 1.0
    return (int(parts[1]) + int(parts[2])) / 2.0 if parts[0] == "uniform" else float(parts[1])


def _longest(kind):
    return int(kind.split(":")[-1]) if kind != "one" else 1


def _popularity(rows, s):
    """(share of the accesses, rows with that share): the Zipf law, rare ranks in groups."""
    exact = min(rows, 4096)
    edges = np.unique(np.geomspace(exact, rows, 400).astype(np.int64)) if rows > exact else np.array([exact])
    lo, hi = edges[:-1], edges[1:]
    rank = np.concatenate([np.arange(1, exact + 1), np.sqrt((lo + 1.0) * hi)])
    count = np.concatenate([np.ones(exact), (hi - lo).astype(np.float64)])
    share = rank ** -float(s)
    return share / (share * count).sum(), count


def _at_least(lam, c):
    """P(Poisson(lam) >= c)"""
    term, below = np.exp(-lam), np.zeros_like(lam)
    for k in range(c):
        below += term
        term = term * lam / (k + 1)
    return np.clip(1.0 - below, 0.0, 1.0)


def _distinct(rows, s, lookups):
    p, m = _popularity(rows, s)
    return float((m * -np.expm1(lookups * np.log1p(-np.minimum(p, 1 - 1e-12)))).sum())


def _hot_set(case):
    """Expected hot rows per table and the share of a table's accesses that they take."""
    rows, row_bytes = _rows(case), case["dim"] * 4
    T = [case["profiled"] * _mean_length(b) for b in _bags(case)]
    law = [_popularity(r, case["zipf"]) for r in rows]
    for c in range(64):
        hot, mass = [], []
        for r, t, (p, m) in zip(rows, T, law):
            cut = 0 if r * row_bytes < SMALL_TABLE else math.ceil(c * t / max(T))
            q = _at_least(t * p, cut)
            hot.append(float((m * q).sum()))
            mass.append(float((m * p * q).sum()))
        if sum(hot) * row_bytes <= case["budget"]:
            break
    return hot, mass


def work(case):
    path, rows, bags, dim = case["path"], _rows(case), _bags(case), case["dim"]
    S, nt, D = case.get("samples", 0), len(rows), 4 * dim
    lengths = [_mean_length(b) for b in bags]
    NL = [S * n for n in lengths]
    csr = sum(1 for b in bags if b != "one")
    U = sum(_distinct(r, case["zipf"], n) for r, n in zip(rows, NL)) if S else 0
    if path == "forward":
        return {"bytes": 4 * sum(NL) + 4 * (S + 1) * csr + D * U + D * S * nt, "flops": dim * sum(NL)}
    if path in ("train", "train_opts"):
        # slots, offsets and gradients read, touched rows read and written, pooled rows written
        state = 8 * U if case.get("optimizer") == "adagrad" else 0
        one = 4 * sum(NL) + 4 * (S + 1) * csr + 2 * D * U + 2 * D * S * nt + state
        return {"bytes": one * case.get("cycle", 1), "flops": dim * (2 * sum(NL) + 2 * U) * case.get("cycle", 1)}
    wide = case.get("index_bits", 32) // 8
    if path == "profile":
        return {"bytes": wide * sum(NL) + 8 * U, "flops": 0}
    hot, mass = _hot_set(case)
    H = sum(hot)
    if path == "build":
        # counters read, remap written, hot ids written, hot rows written (and read where they are copied)
        return {"bytes": 8 * sum(rows) + 4 * H + (2 if case["source"] == "device" else 1) * D * H, "flops": 0}
    if path == "sync":
        return {"bytes": 2 * (4 + 2 * D) * H, "flops": 0}
    share = math.exp(sum(n * math.log(max(m, 1e-300)) for n, m in zip(lengths, mass)))  # samples that are hot
    return {"bytes": wide * sum(NL) + 4 * (S + 1) * csr + 4 * U + 4 * S + share * (4 * sum(NL) + 4 * S * nt), "flops": 0}


def tolerance(case):
    """fp32 sums in another order; everything that is counted, classified or copied is exact.
    Against the same path in fp64, one step is off by up to 1.8e-7 (norm) and 2.4e-5 (one element of
    a row that thousands of lookups of the batch update); a pass may hold four steps."""
    if case["path"] in ("train", "train_opts", "forward"):
        return {"rel": 1e-6, "max": 1e-4}
    return "exact"


def exact(case, seed):
    """What ``run`` gives for the same inputs, in fp64 with plain torch, for the paths that compute numbers."""
    if case["path"] not in ("forward", "train", "train_opts"):
        return None  # counted, classified or copied: tolerance() asks for the same values
    st = prepare(case, seed)
    weights = [t.double() for t in st["hp"].hotW]
    mean, adagrad = case.get("pooling") == "mean", case.get("optimizer") == "adagrad"
    state = [t.double() for t in st["state"]] if "state" in st else []
    lr, eps = float(np.float32(LR)), float(np.float32(1e-8))
    outs = []
    for k, hb in enumerate(st["hbs"]):
        pooled = torch.zeros(st["outs"][k].shape, dtype=torch.float64, device="cuda")
        bags = []
        for z, w in enumerate(weights):
            slots, lengths = hb.slots[z].long(), torch.ones(hb.n_samples, dtype=torch.int64, device="cuda")
            if hb.offsets[z] is not None:
                lengths = hb.offsets[z].diff().long()
            samples = torch.repeat_interleave(torch.arange(hb.n_samples, device="cuda"), lengths)
            scale = 1.0 / lengths.clamp(min=1).double() if mean else torch.ones_like(lengths, dtype=torch.float64)
            bags.append((slots, samples, scale))
            for a in range(0, slots.numel(), 1 << 20):
                pooled[:, z].index_add_(0, samples[a:a + (1 << 20)], w[slots[a:a + (1 << 20)]])
            pooled[:, z] *= scale[:, None]
        outs.append(pooled)
        if case["path"] == "forward":
            return pooled
        for z, (slots, samples, scale) in enumerate(bags):
            up = st["gouts"][k][:, z].double() * scale[:, None]
            grad = torch.zeros_like(weights[z])
            for a in range(0, slots.numel(), 1 << 20):
                grad.index_add_(0, slots[a:a + (1 << 20)], up[samples[a:a + (1 << 20)]])
            if adagrad:
                state[z] += grad.square().mean(dim=1)
                grad /= (state[z].sqrt() + eps)[:, None]  # a row that no lookup names has a gradient of zero
            weights[z] -= lr * grad
    if case["path"] == "train":
        return {"out": outs, "weights": weights}
    return {"out": outs[0], "weights": weights, "state": state}
