"""The work a program has this library do, as cases that can be timed.

A case is a dict of plain values.  `listed()` names twelve of them, `draw(rng)` makes more over the same ranges,
`prepare` builds what a program holds before the call (tables, batches, the context, the kept output buffers), `run`
is one pass through the public entry points and returns what the pass computed, `work` counts the bytes and
operations of a pass that no implementation can avoid, `tolerance` says how far another correct implementation at
the same precision may be off.

Kinds of passes
  step      fs_prioritized_step: one self-contained iteration (dedup, split, both update passes, lookup)
  loop      StepLoop: ten iterations of the pipelined schedule of one shard's tables, then a join on the stream
  ops       the five plain operations called one after the other
  lookup    fs_gather_jagged alone
  parts     the start of Backward as a job with several ranks runs it: gradients split into the collision part and
            the exclusive part, class order rewritten for them, both update passes on the packed parts
  balance   the load balancer: partition the samples by length, then permute the gathered IDs
  shuffle   ranged dispatch, ranged combine and keyed transpose of one keyed jagged tensor

Sequence lengths are the quantiles of their distribution at evenly spaced points, shuffled by the seed: the batches of
a case differ a little in size, but a batch has the same size whatever the seed.  Row IDs are bounded Zipf ranks
(P(k) ~ k^-alpha) scattered over the table by a fixed affine bijection, gradients are N(0, 1), tables hold the
integer-hash initial values.  Output buffers are sized for the batch, as a program that cannot know the number of
distinct rows beforehand sizes them, and start zeroed.
"""
import functools
import math

import numpy as np
import torch

import paper_2604_24073_amd as fs
from paper_2604_24073_amd.schedule import StepLoop, TableBuffers

LR, EPS = 0.01, 1e-8
LOOP_STEPS = 10                 # iterations of one pass of a loop
MAX_IDS = 1 << 21               # what the one context of the plain calls is sized for
ZIPF_HEAD = 1 << 16             # ranks whose probabilities are summed one by one; the tail is integrated
LONG_HISTORY = 16_384           # the 5 % long histories of the skewed batches


# ---- the cases -------------------------------------------------------------------------------------------------
def _batch(users, rule, lo, hi, alpha):
    return {"users": users, "lengths": rule, "lo": lo, "hi": hi, "alpha": alpha}


def listed():
    return [
        # the smallest iteration there is: a new model's first table, or one shard of very many; all latency
        {"name": "step_tiny", "kind": "step", "rows": 10_000, "dim": 64, "dtype": "f32",
         **_batch(32, "uniform", 1, 64, "1.1")},
        # the same call on a whole batch of one shard: an iteration that cannot be pipelined (the last one before an
        # evaluation, a program that looks at its table after every step)
        {"name": "step_shard", "kind": "step", "rows": 4_000_000, "dim": 128, "dtype": "f32",
         **_batch(1024, "powerlaw", 16, 4096, "1.05")},
        # steady-state training of one table shard
        {"name": "loop_shard", "kind": "loop", "rows": "4000000", "dim": "128", "dtype": "f32", "batches": 2,
         "two_part": False, "drift": False, **_batch(1024, "powerlaw", 16, 4096, "1.05")},
        # steady-state training of a shard that holds eight tables of different widths: the largest pass
        {"name": "loop_eight_tables", "kind": "loop",
         "rows": "1000000,2000000,4000000,4000000,8000000,8000000,16000000,16000000",
         "dim": "64,128,256,64,128,256,64,128", "dtype": "f32", "batches": 2, "two_part": False, "drift": False,
         **_batch(2048, "powerlaw", 1, 8192, "1.0,1.05,1.1,1.1,1.15,1.2,1.15,1.2")},
        # bf16 weights, a few users with very long histories, one row that takes a fifth of all occurrences
        {"name": "loop_long_bf16", "kind": "loop", "rows": "32000000", "dim": "128", "dtype": "bf16", "batches": 2,
         "two_part": False, "drift": False, **_batch(512, "skew", 8, 256, "1.2")},
        # streaming training on a table of 33 GB whose popular rows change from batch to batch
        {"name": "loop_stream", "kind": "loop", "rows": "64000000", "dim": "128", "dtype": "f32", "batches": 10,
         "two_part": False, "drift": True, **_batch(4096, "powerlaw", 1, 4096, "1.05")},
        # three small tables of uneven widths, the lookup taken in its two parts
        {"name": "loop_two_part", "kind": "loop", "rows": "300007,77777,1500000", "dim": "96,32,200", "dtype": "f32",
         "batches": 2, "two_part": True, "drift": False, **_batch(301, "powerlaw", 3, 777, "1.05,1.1,1.2")},
        # the plain operations, for a program that schedules them itself; nothing a power of two
        {"name": "ops_ragged", "kind": "ops", "rows": 1_234_567, "dim": 100, "dtype": "f32",
         **_batch(777, "powerlaw", 1, 1999, "1.1")},
        # serving: only the lookup, bf16 rows of 128 bytes
        {"name": "lookup_serving", "kind": "lookup", "rows": 16_000_000, "dim": 64, "dtype": "bf16",
         **_batch(256, "powerlaw", 1, 1024, "1.05")},
        # Backward on one of several ranks: gradients packed for the two exchanges, updates from the packed parts
        {"name": "parts_wide", "kind": "parts", "rows": 2_000_000, "dim": 256, "dtype": "f32",
         **_batch(512, "powerlaw", 16, 4096, "1.1")},
        # balancing the batch of a job of 64 ranks: samples dealt by length, IDs permuted
        {"name": "balance_ids", "kind": "balance", "ranks": 64, "rule": "fbs", "rows": 4_000_000,
         **_batch(65_536, "powerlaw", 16, 4096, "1.05")},
        # what stages the exchanges of a batch of gathered rows (512 bytes each): dispatch, combine, transpose
        {"name": "shuffle_rows", "kind": "shuffle", "ranks": 8, "keys": 4, "words": 128, "rows": 4_000_000,
         **_batch(256, "powerlaw", 16, 4096, "1.05")},
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_lengths(rng, users_lo, users_hi, most):
    """A batch of at most about `most` IDs: users over the logarithm of the range, then a length rule that fits."""
    users = _log_between(rng, users_lo, users_hi)
    rule = rng.choice(["uniform", "powerlaw", "powerlaw", "skew"])
    lo = _log_between(rng, 1, 16)
    hi = _log_between(rng, 64, 8192)
    case = _batch(users, rule, lo, hi, "1.1")
    if rule == "skew":
        case["hi"] = hi = min(hi, 512)
    while int(_lengths(case).sum()) > most and (case["hi"] > 2 * lo + 1 or case["users"] > users_lo):
        if case["hi"] > 2 * lo + 1:
            case["hi"] = max(2 * lo + 1, case["hi"] * 3 // 4)
        else:
            case["users"] = max(users_lo, case["users"] * 3 // 4)
        if rule == "skew":
            case["users"] = max(users_lo, case["users"] * 3 // 4)
    return case


def _draw_dim(rng, dtype):
    """The widths the configurations use, and any other the library takes."""
    unit = 4 if dtype == "f32" else 8
    return rng.choice([64, 128, 256]) if rng.random() < 0.5 else unit * rng.randint(16 // unit, 256 // unit)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "loop", "loop", "loop", "ops", "lookup", "parts", "balance", "shuffle"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    alpha = lambda: "%.3g" % rng.uniform(1.0, 1.2)  # noqa: E731
    if kind == "loop":
        n_tab = rng.choice([1, 1, 2, 3, 5])
        case = {"kind": "loop", "rows": ",".join(str(_log_between(rng, 10_000, 16_000_000)) for _ in range(n_tab)),
                "dim": ",".join(str(_draw_dim(rng, dtype)) for _ in range(n_tab)), "dtype": dtype,
                "batches": rng.choice([2, 4]), "two_part": rng.random() < 0.25, "drift": rng.random() < 0.25}
        case.update(_draw_lengths(rng, 32, 4096, 1_000_000 // n_tab))
        case["alpha"] = ",".join(alpha() for _ in range(n_tab))
        return case
    if kind == "balance":
        case = {"kind": "balance", "ranks": rng.choice([2, 7, 8, 64, 256]), "rule": rng.choice(["fbs", "vbs"]),
                "rows": _log_between(rng, 10_000, 16_000_000)}
        case.update(_draw_lengths(rng, 512, 131_072, 16_000_000))
    elif kind == "shuffle":
        case = {"kind": "shuffle", "ranks": rng.choice([2, 7, 8, 64]), "keys": rng.randint(1, 8),
                "words": rng.choice([1, 2, 2, 32, 64, 100, 128]), "rows": _log_between(rng, 10_000, 16_000_000)}
        # at least a sample per rank; at most about 150 MB of values
        most = 40_000_000 // case["words"] // case["keys"]
        case.update(_draw_lengths(rng, 128, 8192, min(2_000_000, most)))
    else:
        case = {"kind": kind, "rows": _log_between(rng, 10_000, 16_000_000), "dim": _draw_dim(rng, dtype), "dtype": dtype}
        case.update(_draw_lengths(rng, 32, 4096, 1_000_000))
    case["alpha"] = alpha()
    return case


# ---- inputs ----------------------------------------------------------------------------------------------------
def _lengths(case, number=0):
    """int64 [users]: lengths of batch `number` of the case, ascending: quantiles of the length rule."""
    n, lo, hi = case["users"], case["lo"], case["hi"]
    q = (np.arange(n) + (0.5 + 0.382 * number) % 1.0) / n
    if case["lengths"] == "powerlaw":               # density x^-1.5 on [lo, hi + 1)
        a, b = lo ** -0.5, (hi + 1) ** -0.5
        x = (a + q * (b - a)) ** -2.0
    else:
        x = lo + q * (hi + 1 - lo)
    lens = np.clip(np.floor(x).astype(np.int64), lo, hi)
    if case["lengths"] == "skew":                   # 5 % of the users have a very long history
        long = max(1, round(0.05 * n))
        lens = np.concatenate([lens[:n - long], np.full(long, LONG_HISTORY, np.int64)])
    return lens


def _zipf_parts(alpha, rows):
    """(cumulative weights of the head ranks, rank the tail starts at, weight of the tail)."""
    head = min(rows, ZIPF_HEAD)
    cum = np.cumsum(np.arange(1, head + 1, dtype=np.float64) ** -alpha)
    tail = _power_integral(head + 0.5, rows + 0.5, alpha) if rows > head else 0.0
    return cum, head, tail


def _power_integral(a, b, alpha):
    e = 1.0 - alpha
    return math.log(b / a) if abs(e) < 1e-9 else (b ** e - a ** e) / e


def _zipf_rows(gen, n, alpha, rows, iteration, drift):
    """n row IDs on the GPU: Zipf ranks, scattered over the table by an affine bijection; with `drift` the hottest
    1 % of the ranks turn by a tenth of their number per iteration."""
    cum, head, tail = _zipf_parts(alpha, rows)
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen) * (cum[-1] + tail)
    pos = torch.searchsorted(torch.from_numpy(cum).cuda(), u).clamp_(max=head - 1)
    if rows > head:
        e, v = 1.0 - alpha, (u - cum[-1]).clamp_(min=0.0)
        x = torch.exp(v) * (head + 0.5) if abs(e) < 1e-9 else ((head + 0.5) ** e + e * v) ** (1.0 / e)
        pos = torch.where(u < cum[-1], pos, (x + 0.5).floor().to(torch.int64).clamp_(head + 1, rows) - 1)
    if drift:
        hot = max(rows // 100, 1)
        pos = torch.where(pos < hot, (pos + iteration * ((hot + 9) // 10)) % hot, pos)
    a = int(0.6180339887498949 * rows) | 1
    while math.gcd(a, rows) != 1:
        a += 2
    return (a * pos + rows // 3) % rows


def _jagged(case, rng, number=0):
    """(lengths in batch order, offsets) of batch `number`, on the host."""
    lens = rng.permutation(_lengths(case, number))
    return lens, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


def _batches(case, alpha, rows, count, rng, gen, drift=False):
    """`count` consecutive batches of one table: [(values, offsets)] on the GPU."""
    out = []
    for t in range(count):
        _, offs = _jagged(case, rng, t)
        out.append((_zipf_rows(gen, int(offs[-1]), alpha, rows, t, drift), torch.from_numpy(offs).cuda()))
    return out


SPLIT = ("co", "co_slot", "ex", "ex_slot", "ex_next", "ex_next_slot", "counts")


def _zeroed(buffers):
    for t in buffers.values():
        if isinstance(t, torch.Tensor):
            t.zero_()
    return buffers


def _kept(buffers, *names):
    return {k: buffers[k] for k in names}


def _normal(gen, n, dim):
    return torch.randn((n, dim), dtype=torch.float32, device="cuda", generator=gen)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _table(ctx, rows, dim, dtype):
    table = torch.empty((rows, dim), dtype=dtype, device="cuda")
    fs.fs_init_table_hash(ctx, table)
    return table, torch.zeros(rows, dtype=torch.float32, device="cuda")


@functools.lru_cache(maxsize=None)
def _context():
    """One context per process and GPU, sized for the largest batch: what a program keeps for the plain calls."""
    return fs.Context(max_ids=MAX_IDS, max_dim=fs.FS_MAX_DIM)


def _numbers(text, cast):
    return [cast(x) for x in str(text).split(",")]


# ---- step: one self-contained iteration ------------------------------------------------------------------------
def _prepare_step(case, rng, gen):
    ctx, dim = _context(), case["dim"]
    table, state = _table(ctx, case["rows"], dim, _dtype(case))
    bat = _batches(case, float(case["alpha"]), case["rows"], 2, rng, gen)
    lays = [_zeroed(fs.alloc_layout(v.numel(), "cuda", sorted_ids=True)) for v, _ in bat]
    fs.fs_unique_ids(ctx, bat[0][0], case["rows"], out=lays[0])
    turns = []
    for b in (0, 1):                                 # batch b is updated, the other one looked up, in turn
        v, offs = bat[1 - b]
        n = bat[b][0].numel()
        split = _zeroed(fs.alloc_split(n, v.numel(), "cuda"))
        emb = torch.zeros((v.numel(), dim), dtype=table.dtype, device="cuda")
        grads = _normal(gen, n, dim)
        args = fs.make_step_args(table, state, LR, EPS, lays[b], grads, v, offs, lays[1 - b], split, None, emb)
        out = {"table": table, "state": state, "emb": emb, **_kept(lays[1 - b], "unique", "seg_offsets", "perm", "n_unique"),
               **_kept(split, *SPLIT)}
        turns.append((args, out, (grads, split)))
    return {"ctx": ctx, "turns": turns, "turn": 0, "keep": (bat, lays)}


def _run_step(s):
    args, out, _ = s["turns"][s["turn"]]
    s["turn"] ^= 1
    fs.fs_prioritized_step(s["ctx"], args)
    return out


# ---- loop: the pipelined schedule ------------------------------------------------------------------------------
def _prepare_loop(case, rng, gen):
    bufs = []
    for rows, dim, alpha in zip(_numbers(case["rows"], int), _numbers(case["dim"], int), _numbers(case["alpha"], float)):
        bat = _batches(case, alpha, rows, case["batches"], rng, gen, case["drift"])
        table = torch.empty((rows, dim), dtype=_dtype(case), device="cuda")
        bufs.append(TableBuffers(table, torch.zeros(rows, dtype=torch.float32, device="cuda"), [v for v, _ in bat],
                                 [o for _, o in bat], [_normal(gen, v.numel(), dim) for v, _ in bat], LR, EPS))
    loop = StepLoop(bufs, two_part=case["two_part"], emb_rotation=3 if case["two_part"] else None)
    for b in bufs:
        fs.fs_init_table_hash(loop.ctxs[0], b.table)
    loop.prime()
    return {"loop": loop, "bufs": bufs, "step": 0}


def _run_loop(s):
    loop = s["loop"]
    loop.run(s["step"], LOOP_STEPS)
    s["step"] += LOOP_STEPS
    for ctx, stream in zip(loop.ctxs, loop.streams):
        fs.fs_step_join(ctx, stream)
    last = s["step"] - 1
    return {"tables": [b.table for b in s["bufs"]], "states": [b.state for b in s["bufs"]],
            "embs": [b.emb_of_step(last)[:b.n[(last + 1) % b.T]] for b in s["bufs"]]}


# ---- ops: the plain operations one after the other ---------------------------------------------------------------
def _prepare_ops(case, rng, gen):
    ctx, dim = _context(), case["dim"]
    table, state = _table(ctx, case["rows"], dim, _dtype(case))
    (v0, _), (v1, o1) = _batches(case, float(case["alpha"]), case["rows"], 2, rng, gen)
    lay0 = fs.fs_unique_ids(ctx, v0, case["rows"])
    lay1 = _zeroed(fs.alloc_layout(v1.numel(), "cuda"))
    split = _zeroed(fs.alloc_split(v0.numel(), v1.numel(), "cuda"))
    grads = _normal(gen, v0.numel(), dim)
    reduced = torch.zeros((v0.numel(), dim), dtype=torch.float32, device="cuda")
    emb = torch.zeros((v1.numel(), dim), dtype=table.dtype, device="cuda")
    out = {"table": table, "state": state, "emb": emb, "reduced": reduced,
           **_kept(lay1, "unique", "seg_offsets", "perm", "inverse", "n_unique"), **_kept(split, *SPLIT)}
    return {"ctx": ctx, "table": table, "state": state, "rows": case["rows"], "v0": v0, "v1": v1, "o1": o1, "lay0": lay0,
            "lay1": lay1, "split": split, "grads": grads, "reduced": reduced, "emb": emb, "out": out}


def _run_ops(s):
    ctx, lay0, lay1, sp, cap = s["ctx"], s["lay0"], s["lay1"], s["split"], s["v0"].numel()
    fs.fs_unique_ids(ctx, s["v1"], s["rows"], out=lay1)
    fs.fs_collision_split(ctx, lay0["unique"], lay0["n_unique"], lay1["unique"], lay1["n_unique"], cap, s["v1"].numel(), out=sp)
    fs.fs_segment_reduce_grads(ctx, s["grads"], lay0["perm"], lay0["seg_offsets"], lay0["n_unique"], out=s["reduced"],
                               inverse=lay0["inverse"])
    fs.fs_rowwise_adagrad_update(ctx, s["table"], s["state"], sp["co"], sp["co_slot"], sp["counts"][0:1], cap, s["reduced"],
                                 LR, EPS)
    fs.fs_gather_jagged(ctx, s["table"], s["v1"], s["o1"], out=s["emb"])
    fs.fs_rowwise_adagrad_update(ctx, s["table"], s["state"], sp["ex"], sp["ex_slot"], sp["counts"][1:2], cap, s["reduced"],
                                 LR, EPS)
    return s["out"]


# ---- lookup ------------------------------------------------------------------------------------------------------
def _prepare_lookup(case, rng, gen):
    ctx = _context()
    table, _ = _table(ctx, case["rows"], case["dim"], _dtype(case))
    (values, offsets), = _batches(case, float(case["alpha"]), case["rows"], 1, rng, gen)
    out = torch.empty((values.numel(), case["dim"]), dtype=table.dtype, device="cuda")
    return {"ctx": ctx, "table": table, "values": values, "offsets": offsets, "out": out}


def _run_lookup(s):
    return fs.fs_gather_jagged(s["ctx"], s["table"], s["values"], s["offsets"], out=s["out"])


# ---- parts: the gradients packed for two exchanges, updates from the packed parts ----------------------------------
def _prepare_parts(case, rng, gen):
    ctx, dim = _context(), case["dim"]
    table, state = _table(ctx, case["rows"], dim, _dtype(case))
    (v0, _), (v1, _) = _batches(case, float(case["alpha"]), case["rows"], 2, rng, gen)
    lay0, lay1 = fs.fs_unique_ids(ctx, v0, case["rows"]), fs.fs_unique_ids(ctx, v1, case["rows"])
    split = fs.fs_collision_split_classes(ctx, lay0, lay1["unique"], lay1["n_unique"], v1.numel())
    n = v0.numel()
    grads = _normal(gen, n, dim)
    ints = lambda: torch.zeros(n, dtype=torch.int32, device="cuda")  # noqa: E731
    parts = {"co_index": ints(), "g_co": torch.zeros_like(grads), "ex_index": ints(), "g_ex": torch.zeros_like(grads),
             "part_pos": ints(), "counts": torch.zeros(2, dtype=torch.int64, device="cuda")}
    return {"ctx": ctx, "table": table, "state": state, "lay": lay0, "split": split, "grads": grads, "parts": parts,
            "out": {"table": table, "state": state, **parts}}


def _run_parts(s):
    ctx, lay, parts = s["ctx"], s["lay"], s["parts"]
    fs.fs_split_grads(ctx, s["grads"], lay, s["split"], out=parts)
    order = fs.fs_class_order_for_parts(ctx, parts, lay["n"], s["split"])
    fs.fs_reduce_update_class(ctx, 0, s["table"], s["state"], LR, EPS, parts["g_co"], lay, order)
    fs.fs_reduce_update_class(ctx, 1, s["table"], s["state"], LR, EPS, parts["g_ex"], lay, order)
    return s["out"]


# ---- balance: samples dealt to ranks by length, IDs permuted ---------------------------------------------------------
def _prepare_balance(case, rng, gen):
    lens, offs = _jagged(case, rng)
    values = _zipf_rows(gen, int(offs[-1]), float(case["alpha"]), case["rows"], 0, False)
    lengths = torch.from_numpy(lens).cuda()
    top = LONG_HISTORY if case["lengths"] == "skew" else case["hi"]
    # work grows a little faster than the length: weights L^1.2, scaled to integers
    weights = torch.from_numpy((np.arange(top + 1, dtype=np.float64) ** 1.2 * 16).astype(np.int64)).cuda()
    pair = (torch.empty(lens.size, dtype=torch.int32, device="cuda"), torch.empty(case["ranks"] + 1, dtype=torch.int64, device="cuda"))
    offsets = torch.from_numpy(offs).cuda()
    return {"ctx": _context(), "values": values, "offsets": offsets, "lengths": lengths, "top": top, "weights": weights,
            "ranks": case["ranks"], "rule": case["rule"], "pair": pair, "out": (torch.empty_like(values), torch.empty_like(offsets))}


def _run_balance(s):
    if s["rule"] == "fbs":
        sample_of, rank_offsets = fs.fs_partition_fbs(s["ctx"], s["lengths"], s["top"], s["ranks"], out=s["pair"])
    else:
        sample_of, rank_offsets = fs.fs_partition_vbs(s["ctx"], s["lengths"], s["weights"], s["ranks"])
    values, offsets = fs.fs_jagged_indexed_permute(s["ctx"], s["values"], s["offsets"], sample_of, s["values"].numel(), out=s["out"])
    return {"sample_of": sample_of, "rank_offsets": rank_offsets, "values": values, "offsets": offsets}


# ---- shuffle: the staging of the exchanges ---------------------------------------------------------------------------
def _prepare_shuffle(case, rng, gen):
    keys, users, words = case["keys"], case["users"], case["words"]
    lens = np.concatenate([_jagged(case, rng, k)[0] for k in range(keys)])          # feature-major segments
    offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)).cuda()
    n = int(lens.sum())
    if words == 2:                                                               # IDs
        values = _zipf_rows(gen, n, float(case["alpha"]), case["rows"], 0, False)
    else:                                                                        # gathered rows
        values = _normal(gen, n, words)
    ranks = np.linspace(0, users, case["ranks"] + 1).astype(np.int64)
    ranks[1:-1] += rng.integers(-(users // case["ranks"] // 4), users // case["ranks"] // 4 + 1, case["ranks"] - 1)
    new = lambda: (torch.empty_like(values), torch.empty_like(offsets))  # noqa: E731
    return {"ctx": _context(), "values": values, "offsets": offsets, "keys": keys, "users": users,
            "ranks": torch.from_numpy(ranks).cuda(),
            "sent": new() + (torch.empty(case["ranks"], dtype=torch.int64, device="cuda"),), "back": new(), "turned": new()}


def _run_shuffle(s):
    ctx, keys, users = s["ctx"], s["keys"], s["users"]
    sent = fs.fs_jagged_ranged_dispatch(ctx, s["values"], s["offsets"], keys, users, s["ranks"], out=s["sent"])
    back = fs.fs_jagged_ranged_combine(ctx, sent[0], sent[1], keys, users, s["ranks"], out=s["back"])
    turned = fs.fs_jagged_keyed_transpose(ctx, s["values"], s["offsets"], keys, users, out=s["turned"])
    return {"sent": sent, "back": back, "turned": turned}


_PREPARE = {"step": _prepare_step, "loop": _prepare_loop, "ops": _prepare_ops, "lookup": _prepare_lookup,
            "parts": _prepare_parts, "balance": _prepare_balance, "shuffle": _prepare_shuffle}
_RUN = {"step": _run_step, "loop": _run_loop, "ops": _run_ops, "lookup": _run_lookup, "parts": _run_parts,
        "balance": _run_balance, "shuffle": _run_shuffle}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    state = _PREPARE[case["kind"]](case, np.random.default_rng(seed), gen)
    state["run"] = _RUN[case["kind"]]
    return state


def run(state):
    return state["run"](state)


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def _expected_rows(n, alpha, rows):
    """(distinct rows, rows shared with the next batch, occurrences of shared rows) expected of a batch of n IDs."""
    cum, head, tail = _zipf_parts(alpha, rows)
    weight, count = np.diff(cum, prepend=0.0), np.ones(head)
    if rows > head:
        edges = np.geomspace(head + 0.5, rows + 0.5, 2049)
        mass = np.array([_power_integral(a, b, alpha) for a, b in zip(edges, edges[1:])])
        weight, count = np.concatenate([weight, mass / np.diff(edges)]), np.concatenate([count, np.diff(edges)])
    mean = n * weight / (cum[-1] + tail)
    seen = -np.expm1(-mean)
    return float((count * seen).sum()), float((count * seen * seen).sum()), float((count * mean * seen).sum())


def _unique_bytes(n, u, inverse):
    return 8 * n + 8 * u + 4 * u + 4 * n + (4 * n if inverse else 0)     # IDs in; rows, boundaries, order (and inverse) out


def _split_bytes(u, co):
    return 8 * 2 * u + 12 * (2 * u - co)                                   # both lists in; three lists with their slots out


def _update_bytes(n, u, dim, w):
    return 4 * n * dim + 4 * n + u * (2 * dim * w + 8 + 8)                 # gradients, order; rows and state both ways, row IDs


def _lookup_bytes(n, u, dim, w):
    return 8 * n + u * dim * w + n * dim * w


def work(case):
    kind, n = case["kind"], int(_lengths(case).sum())
    if kind == "balance":
        b = case["users"]
        return {"bytes": 16 * n + 8 * b + 4 * b + 8 * b + 8 * b, "flops": 0}
    if kind == "shuffle":
        # each of the three reads the values and the offsets and writes them
        segs, total = case["keys"] * case["users"], case["keys"] * n
        return {"bytes": 3 * (2 * total * 4 * case["words"] + 16 * segs), "flops": 0}
    w = 4 if case["dtype"] == "f32" else 2
    if kind == "loop":
        total = {"bytes": 0.0, "flops": 0.0}
        for rows, dim, alpha in zip(_numbers(case["rows"], int), _numbers(case["dim"], int), _numbers(case["alpha"], float)):
            u, co, _ = _expected_rows(n, alpha, rows)
            step = _unique_bytes(n, u, False) + _split_bytes(u, co) + _update_bytes(n, u, dim, w) + _lookup_bytes(n, u, dim, w)
            total["bytes"] += LOOP_STEPS * step
            total["flops"] += LOOP_STEPS * (n * dim + 4 * u * dim)
        return total
    rows, dim, alpha = case["rows"], case["dim"], float(case["alpha"])
    u, co, co_occ = _expected_rows(n, alpha, rows)
    if kind == "lookup":
        return {"bytes": _lookup_bytes(n, u, dim, w), "flops": 0}
    update = {"bytes": _update_bytes(n, u, dim, w), "flops": n * dim + 4 * u * dim}
    if kind == "parts":
        # the packed gradients are written (they are what is sent) and the row order of the batch comes and goes
        return {"bytes": update["bytes"] + 4 * n * dim + 4 * n + 8 * n, "flops": update["flops"]}
    index = _unique_bytes(n, u, kind == "ops") + _split_bytes(u, co)
    reduced = 4 * u * dim if kind == "ops" else 0                         # the summed gradients are one of the results
    return {"bytes": index + update["bytes"] + reduced + _lookup_bytes(n, u, dim, w), "flops": update["flops"]}


def tolerance(case):
    """Lookups and shuffles move bits.  Updates add in fp64 and round to fp32 in few places; a bf16 weight may round
    the other way."""
    if case["kind"] in ("lookup", "balance", "shuffle"):
        return "exact"
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
