"""The framework's work, case by case: planning a trace of lookups, and training embedding tables over a planned trace.

A case is one of three kinds of call a training program makes:

  plan    bp_oracle_plan over a whole trace of lookup ids that lies on the GPU
  stream  bp_oracle_plan_chunk over a trace that arrives chunk by chunk, state carried from chunk to chunk
  train   CachedEmbeddingTrainer over a planned trace: for every batch cache maintenance, forward, backward + update
          (or the overlapped schedule), and the last write-backs

Sizes are those of the benchmark configurations (table counts and cardinalities, embedding dimensions, batch sizes,
lookaheads, optimizers), shortened in the number of batches, plus ragged and odd ones.  Ids are Zipf-distributed over a
seeded permutation of every table's rows, one id per (sample, table) or a bag of several, sample-major.
"""
import math

import numpy as np
import torch

import paper_2202_12429_amd as bp
from paper_2202_12429_amd.runner import CachedEmbeddingTrainer

DEV = "cuda:0"


def _case(name, kind, tables, rows, small, batch, iters, lookahead, capacity, zipf, dim=16, dtype="f32", optimizer="sgd",
          bag_min=1, bag_max=1, grouping=True, slot_map=True, host_table=False, overlap=False, reserve=0, emit=0, bend=1.0):
    """rows: rows of the largest table; small: rows of the smallest; the others lie between them, log-spaced (bend < 1:
    more of them near the largest)."""
    return dict(name=name, kind=kind, tables=tables, rows=rows, small=small, bend=bend, batch=batch, iters=iters,
                lookahead=lookahead, capacity=capacity, zipf=zipf, dim=dim, dtype=dtype, optimizer=optimizer,
                bag_min=bag_min, bag_max=bag_max, grouping=grouping, slot_map=slot_map, host_table=host_table,
                overlap=overlap, reserve=reserve, emit=emit)


def listed():
    return [
        # ---- planning
        # the smallest job anybody plans: 8 tables, batch 256, 50 batches; launches and round trips to the host count
        _case("plan_tiny", "plan", 8, 10_000, 10_000, 256, 50, 20, 4_096, 1.2),
        # a Criteo-shaped epoch: 26 tables, 200 batches of 16,384, both passes walk the row records (no slot map)
        _case("plan_d48", "plan", 26, 10_000_000, 3, 16_384, 200, 400, 676_000, 1.0994, 48, optimizer="adagrad",
              slot_map=False, bend=0.55),
        # bags of up to 50 ids; the pooled forward pass needs the slot of every lookup
        _case("plan_bags", "plan", 20, 5_000_000, 5_000_000, 8_192, 12, 300, 4_000_000, 1.1, 64, bag_max=50),
        # ids arriving while training runs: 4 chunks of 8 batches, each with its lookahead window behind it
        _case("plan_stream", "stream", 26, 1_000_000, 10, 16_384, 32, 16, 400_000, 1.147, emit=8),
        # ---- training
        # launch-bound steps of 2,048 lookups
        _case("train_tiny", "train", 8, 10_000, 10_000, 256, 20, 20, 4_096, 1.2),
        # odd everything: 7 tables, 613 samples, bags of 0 to 9 ids, 80-byte rows; the backward pass sorts the slots itself
        _case("train_odd", "train", 7, 3_001, 57, 613, 10, 6, 15_000, 1.1, 20, optimizer="adagrad", bag_min=0, bag_max=9,
              grouping=False),
        # 64-byte rows, small tables, SGD
        _case("train_d16", "train", 26, 1_000_000, 10, 16_384, 12, 200, 84_271, 1.147, 16, slot_map=False),
        # the benchmark's step: 192-byte rows, element-wise Adagrad, table in HBM
        _case("train_d48", "train", 26, 10_000_000, 3, 16_384, 12, 400, 676_000, 1.0994, 48, optimizer="adagrad",
              slot_map=False, bend=0.55),
        # the same step with a (smaller) table in pinned host memory and maintenance overlapped with training
        _case("train_d48_host", "train", 26, 600_000, 3, 16_384, 8, 400, 240_000, 1.0994, 48, optimizer="adagrad",
              slot_map=False, host_table=True, overlap=True, reserve=40_960),
        # bags of up to 50 ids, 256-byte rows: pooled forward, about 4.2 M lookups a batch
        _case("train_bags_d64", "train", 20, 1_000_000, 1_000_000, 8_192, 6, 300, 4_000_000, 1.1, 64, bag_max=50),
        # bf16 storage, 256-byte rows, row-wise Adagrad, 1.3 M lookups a batch
        _case("train_bf16_d128", "train", 40, 500_000, 500_000, 32_768, 6, 500, 3_000_000, 1.05, 128, "bf16",
              "adagrad_rowwise"),
        # the widest fp32 rows (1 KiB) at an ordinary batch size
        _case("train_d256", "train", 13, 50_000, 200, 1_024, 10, 40, 60_000, 1.05, 256, optimizer="adagrad"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plan", "plan", "stream", "train", "train", "train"])
    tables = rng.randint(1, 40)
    dtype = "f32" if rng.random() < 0.7 else "bf16"
    dim = rng.choice([4, 8, 12, 16, 20, 32, 36, 48, 64, 96, 100, 128, 192, 256] if dtype == "f32"
                     else [8, 16, 24, 40, 64, 96, 128, 256, 512])
    optimizer = rng.choice(["sgd", "adagrad", "adagrad_rowwise"])
    # the table (weights and state) fits 12 GB
    record = dim * (4 if dtype == "f32" else 2) + (4 * dim if optimizer == "adagrad" else 4)
    rows = _log_int(rng, 50, min(1_000_000, int(12e9 / (record * tables))))
    small = rows if rng.random() < 0.4 else _log_int(rng, 3, rows)
    bag_max = 1 if rng.random() < 0.6 else rng.randint(2, 50)
    bag_min = 1 if bag_max == 1 else rng.choice([0, 1])
    mean_bag = (bag_min + bag_max) / 2
    # lookups of a batch, and batches
    n = _log_int(rng, 60, 1_300_000 if bag_max == 1 else 4_000_000)
    if kind == "train":
        n = min(n, 250_000_000 / dim)
    batch = max(1, min(32_768, int(n / (tables * mean_bag))))
    n = batch * tables * mean_bag
    if kind == "train":
        iters = rng.randint(2, max(2, min(24, int(600_000_000 / (n * dim)))))
    else:
        iters = max(2, min(400, int(_log_int(rng, 50_000, 60_000_000) / n)))
    lookahead = _log_int(rng, 1, 500)
    grouping = rng.random() < 0.85
    slot_map = not grouping or bag_max > 1 or rng.random() < 0.6
    emit, host, reserve = 0, False, 0
    most = int(batch * tables * bag_max) + 1024          # no batch has more distinct rows
    capacity = max(most, min(3_000_000, int(most * rng.uniform(1.0, 4.0))))
    if kind == "stream":
        lookahead = rng.randint(2, 24)
        iters = max(2, min(iters, 64, int(20_000_000 / n)))
        emit = rng.randint(1, iters)
        slot_map = True
    if kind == "train" and n < 200_000 and rng.random() < 0.15:
        host, reserve, capacity = True, most, 3 * most
    c = _case("", kind, tables, rows, small, batch, iters, lookahead, capacity, round(rng.uniform(1.02, 1.25), 4), dim,
              dtype, optimizer, bag_min, bag_max, grouping, slot_map, host, host, reserve, emit)
    del c["name"]
    return c


# ---- inputs --------------------------------------------------------------------------------------------------------
def _table_rows(c):
    """Rows of every table, from the smallest to the largest, log-spaced."""
    nt, lo, hi = c["tables"], c["small"], c["rows"]
    if nt == 1 or lo == hi:
        return [hi] * nt
    return [max(1, int(round(lo * (hi / lo) ** ((k / (nt - 1)) ** c["bend"])))) for k in range(nt)]


def _weights(n, s, device=DEV):
    """Running sums of r ** -s over the ranks r = 1..n, in whole numbers: the same from run to run, in whatever order
    the GPU adds them."""
    p = torch.arange(1, n + 1, dtype=torch.float64, device=device).pow_(-s)
    return (p * 2.0 ** 44).to(torch.int64).clamp_(min=1).cumsum_(0)


def _lookups(c, seed):
    """(ids on the GPU, iter_offsets on the host, per-batch bag offsets on the GPU or None for one id per bag).

    How popular a row every lookup asks for is the case's own; which row of its table that is comes from the seed.  The
    lists of a plan so have the same lengths for every seed, and other contents."""
    gen = torch.Generator(device=DEV).manual_seed(1_000_003 * seed + 17)
    popularity = torch.Generator(device=DEV).manual_seed(4_242)
    T, B, nt = c["iters"], c["batch"], c["tables"]
    rows = _table_rows(c)
    one = c["bag_min"] == 1 and c["bag_max"] == 1
    if one:
        lens = None
        offsets = np.arange(T + 1, dtype=np.int64) * (B * nt)
        bag_off = None
    else:
        lens = torch.randint(c["bag_min"], c["bag_max"] + 1, (T, B * nt), generator=popularity, device=DEV)
        per_bag = torch.zeros((T, B * nt + 1), dtype=torch.int64, device=DEV)
        torch.cumsum(lens, 1, out=per_bag[:, 1:])
        offsets = np.concatenate([[0], np.cumsum(per_bag[:, -1].cpu().numpy())]).astype(np.int64)
        bag_off = [per_bag[i] for i in range(T)]
    N = int(offsets[-1])
    ids = torch.empty(N, dtype=torch.int64, device=DEV)
    table_of = None if one else (torch.arange(B * nt, device=DEV) % nt).repeat(T).repeat_interleave(lens.reshape(-1))
    base = 0
    for t, n in enumerate(rows):
        perm = torch.randperm(n, generator=gen, device=DEV)
        where = ids.view(T * B, nt)[:, t] if one else torch.nonzero(table_of == t).reshape(-1)
        u = torch.rand(where.shape[0], dtype=torch.float64, generator=popularity, device=DEV)
        upto = _weights(n, c["zipf"])
        rank = torch.searchsorted(upto, (u * upto[-1]).to(torch.int64), right=True).clamp_(max=n - 1)
        got = perm[rank] + base
        if one:
            where.copy_(got)
        else:
            ids[where] = got
        base += n
    return ids, offsets, bag_off


def _config(c):
    return bp.make_config(sum(_table_rows(c)), c["capacity"], c["dim"], c["dtype"], c["optimizer"], c["lookahead"],
                          reserve=c["reserve"])


def prepare(case, seed):
    c = dict(case)
    cfg = _config(c)
    ids, offsets, bag_off = _lookups(c, seed)
    st = dict(case=c, cfg=cfg, ids=ids, offsets=offsets)
    if c["kind"] == "plan":
        need = bp.bp_oracle_plan_workspace_bytes(cfg, int(offsets[-1]), c["iters"], c["grouping"])
        st["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        return st
    if c["kind"] == "stream":
        chunks, T, emit = [], c["iters"], c["emit"]
        for a in range(0, T, emit):      # the batches of the chunk and the window its decisions look into
            b = min(T, a + emit)
            e = min(T, b + c["lookahead"] - 1)
            chunks.append((ids[int(offsets[a]):int(offsets[e])], offsets[a:e + 1] - offsets[a], b - a))
        st["chunks"] = chunks
        return st
    gen = torch.Generator(device=DEV).manual_seed(1_000_003 * seed + 29)
    R, D, bags = int(cfg.total_rows), c["dim"], c["batch"] * c["tables"]
    wdt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    w = torch.empty((R, D), dtype=wdt, device=DEV).uniform_(-0.05, 0.05, generator=gen)
    s = {"sgd": None, "adagrad": torch.zeros((R, D), dtype=torch.float32, device=DEV) if c["optimizer"] == "adagrad" else None,
         "adagrad_rowwise": torch.zeros(R, dtype=torch.float32, device=DEV) if c["optimizer"] == "adagrad_rowwise" else None}[c["optimizer"]]
    if c["host_table"]:
        w = torch.empty((R, D), dtype=wdt, pin_memory=True).copy_(w)
        s = None if s is None else torch.empty(s.shape, dtype=torch.float32, pin_memory=True).copy_(s)
    most = int(np.diff(offsets).max())
    tr = CachedEmbeddingTrainer(cfg, w, s, device=DEV, max_lookups=most, max_bags=bags, grouping=c["grouping"],
                                slot_map=c["slot_map"])
    tr.plan(ids, offsets)
    # a few upstream gradients in turn: what the dense model hands back batch after batch
    grads = [torch.randn((bags, D), dtype=torch.float32, device=DEV, generator=gen) for _ in range(3)]
    st.update(trainer=tr, table=w, state=s, grads=grads, bag_off=bag_off, bags=bags,
              outs=[torch.empty((bags, D), dtype=torch.float32, device=DEV) for _ in range(c["iters"])])
    return st


# ---- one pass ------------------------------------------------------------------------------------------------------
def _plan_outputs(p, n, first, last):
    """What a plan of batches [0, last) says, n lookups of them; `first`: list entries before them are not theirs."""
    out = {"L_eff": p.L_eff, "peak": p.peak_occupancy, "min_capacity": p.min_capacity, "pairs": p.n_unique_pairs,
           "prefetch_offsets": p.prefetch_offsets, "evict_offsets": p.evict_offsets, "keep_offsets": p.keep_offsets,
           "occupancy": p.occupancy}
    for which in ("prefetch", "evict", "keep"):
        off = getattr(p, which + "_offsets")
        a, b = int(off[0]) if first else 0, int(off[last])
        out[which + "_ids"] = getattr(p, which + "_ids")[a:b]
        second = "keep_ttl" if which == "keep" else which + "_slots"
        out[second] = getattr(p, second)[a:b]
    if p.lookup_slots is not None:
        out["lookup_slots"] = p.lookup_slots[:n]
    if p.grouped_lookups is not None:
        a, b = int(p.keep_offsets[0]) if first else 0, int(p.keep_offsets[last])
        out.update(grouped_lookups=p.grouped_lookups[:n], row_recs=p.row_recs[a:b],
                   piece_recs=p.piece_recs[:int(p.piece_offsets[last])], piece_offsets=p.piece_offsets)
    return out


def run(state):
    c, cfg = state["case"], state["cfg"]
    if c["kind"] == "plan":
        p = bp.bp_oracle_plan(cfg, state["ids"], state["offsets"], workspace=state["workspace"], grouping=c["grouping"],
                              slot_map=c["slot_map"])
        return _plan_outputs(p, int(state["offsets"][-1]), False, c["iters"])
    if c["kind"] == "stream":
        # the last chunk's plan and the state it leaves depend on every chunk before it
        carried, p = None, None
        for ids, offsets, emit in state["chunks"]:
            p, carried = bp.bp_oracle_plan_chunk(cfg, ids, offsets, emit, carried, grouping=c["grouping"])
        out = _plan_outputs(p, int(offsets[emit]), True, emit)
        out.update(resident_ids=carried.resident_ids[:carried.n_resident], ring=carried.ring)
        return out
    tr, grads, bag_off, bags, outs = (state[k] for k in ("trainer", "grads", "bag_off", "bags", "outs"))
    if c["overlap"]:
        tr.begin()
        for i in range(c["iters"]):
            tr.acquire(i)
            b = None if bag_off is None else bag_off[i]
            tr.forward(i, b, bags, out=outs[i])
            tr.backward_update(i, b, bags, grads[i % len(grads)])
            tr.release(i)
        tr.end()
    else:
        for i in range(c["iters"]):
            tr.maintain(i)
            b = None if bag_off is None else bag_off[i]
            tr.forward(i, b, bags, out=outs[i])
            tr.backward_update(i, b, bags, grads[i % len(grads)])
        tr.flush()
    return {"pooled": outs, "table": state["table"], "state": state["state"]}


# ---- what a pass cannot do without ---------------------------------------------------------------------------------
def _distinct(c, samples):
    """Expected number of distinct rows among the lookups of `samples` samples."""
    total = 0.0
    draws = samples * (c["bag_min"] + c["bag_max"]) / 2
    for n in _table_rows(c):
        edges = np.unique(np.concatenate([np.arange(1, min(n, 512) + 1),
                                          np.geomspace(1, n, 400).astype(np.int64), [n]]))
        p_edge = edges.astype(np.float64) ** -c["zipf"]
        width = np.diff(edges)
        mass = p_edge[0] + float(np.sum(0.5 * (p_edge[:-1] + p_edge[1:]) * width))
        seen = 1.0 - np.exp(-draws * p_edge / mass)
        total += seen[0] + float(np.sum(0.5 * (seen[:-1] + seen[1:]) * width))
    return total


def work(case):
    c = dict(case)
    T, bags = c["iters"], c["batch"] * c["tables"]
    n = bags * (c["bag_min"] + c["bag_max"]) / 2
    u = min(_distinct(c, c["batch"]), n)
    ever = min(_distinct(c, c["batch"] * T), n * T)
    if c["kind"] in ("plan", "stream"):
        # ids in; keep list, prefetch and evict lists, and what was asked for out
        per = 8 * n + 12 * u + (4 * n if c["slot_map"] else 0) + (4 * n + 16 * u if c["grouping"] else 0)
        return {"bytes": T * per + 24 * ever, "flops": 0}
    row = c["dim"] * (4 if c["dtype"] == "f32" else 2)
    st = {"sgd": 0, "adagrad": 4 * c["dim"], "adagrad_rowwise": 4}[c["optimizer"]]
    multi = 8 * (bags + 1) if c["bag_max"] > 1 else 0
    fwd = 4 * n + multi + u * row + bags * c["dim"] * 4
    bwd = 4 * n + multi + min(n, bags) * c["dim"] * 4 + 2 * u * (row + st)
    moved = 4 * ever * (row + st) + 24 * ever             # into the cache once and back once, read and written
    return {"bytes": T * (fwd + bwd) + moved, "flops": 2.0 * T * n * c["dim"]}


def tolerance(case):
    if case["kind"] in ("plan", "stream"):
        return "exact"
    # A row's gradient is an fp64 sum rounded once, so another order of addition changes it by at most one fp32
    # rounding, and the pooled sums of up to 50 fp32 terms by a few; with bf16 storage one such rounding may move a
    # stored value to its neighbour (2^-8 of it) here and there.
    return {"rel": 1e-6, "max": 4e-6} if case["dtype"] == "f32" else {"rel": 4e-5, "max": 1.6e-2}
