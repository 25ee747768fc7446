"""What one parameter-server shard does all day, as measurable cases.

Each case is one call (or the few calls of one operation) through the public
entry points of ``paper_2205_11048_amd``, at sizes of the five workloads of
``synth/configs.py``, of the tests and of ``bench.py``:

* ``step``    -- one whole push-step of ``GBAStep.run`` (token weights, dense
                 sum + optimiser, sparse aggregation + row apply);
* ``sparse``  -- the sparse half of a step on its own (aggregate and apply);
* ``means``   -- ``gba_aggregate_sparse`` alone, for a program that applies the
                 per-ID means itself or sends them on;
* ``dense``   -- the dense half of a step on its own;
* ``early``   -- gradients folded into the running sum as they arrive, then the
                 finishing call of the step;
* ``pull``    -- a worker's request for embedding rows;
* ``lookup``  -- a batch of 64-bit IDs mapped to rows, every ID known;
* ``build``   -- the first batch on an empty 64-bit index.

Inputs are made on the GPU from the seed: Zipf-skewed IDs spread over the
table, normal gradients, staleness drawn per contribution.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2205_11048_amd as gba
from paper_2205_11048_amd.step import GBAStep

STEP = 1000          # the global step being applied
SIGMA = 1e-2         # standard deviation of the gradients
LR = {"adagrad": 0.01, "adam": 1e-3}
EPS = 1e-8
BETA1, BETA2 = 0.9, 0.999
ADAM_T = STEP + 1


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest whole step: a toy shard, or one of hundreds of shards
        dict(name="step_small", op="step", K=4, N=20_480, fields=0, zipf=1.1, R=100_000, D=16, P=65_536,
             stale="uniform", stale_par=3.0, iota=2, opt="adagrad"),
        # one-hot click-through data: 26 fields of 32 local batches of 1024 samples, wide rows
        dict(name="step_one_hot", op="step", K=32, N=851_968, fields=26, zipf=1.05, R=10_000_000, D=64, P=2_000_000,
             stale="geometric", stale_par=0.5, iota=3, opt="adagrad"),
        # multi-hot histories of 200 IDs, 100 workers, Adam, narrow rows
        dict(name="step_multi_hot_adam", op="step", K=100, N=10_240_000, fields=0, zipf=1.2, R=100_000_000, D=16,
             P=8_000_000, stale="geometric", stale_par=0.4, iota=4, opt="adam"),
        # the sparse half of the largest workload: 256 contributions of 256,000
        # IDs (the table of 100 M rows lets a state fit the card three times)
        dict(name="sparse_largest", op="sparse", K=256, N=65_536_000, fields=0, zipf=1.1, R=100_000_000, D=32,
             stale="geometric", stale_par=0.3, iota=8, opt="adagrad", decay="token", norm="per_id", ragged=0),
        # per-ID staleness (the tags of the rows decide), Adam, 64 contributions of uneven sizes
        dict(name="sparse_id_tag_adam", op="sparse", K=64, N=6_553_613, fields=0, zipf=1.05, R=20_000_000, D=32,
             stale="uniform", stale_par=5.0, iota=4, opt="adam", decay="id_tag", norm="per_id", ragged=1),
        # the means alone: fractional weights (another decay policy), divided by K, wide rows, uneven sizes
        dict(name="means_ragged_wide", op="means", K=50, N=300_007, fields=0, zipf=1.1, R=1_234_567, D=128,
             stale="uniform", stale_par=4.0, iota=3, decay="token", norm="by_k", ragged=1, fraction=1),
        # the dense half of the workload with the most dense parameters (half of them, so three states fit)
        dict(name="dense_adam_large", op="dense", K=64, P=100_000_000, stale="uniform", stale_par=5.0, iota=4,
             opt="adam"),
        # a dense shard of an odd size
        dict(name="dense_adagrad_odd", op="dense", K=37, P=1_000_003, stale="geometric", stale_par=0.5, iota=3,
             opt="adagrad"),
        # a step's dense gradients summed as they arrive, sixteen at a time, then applied
        dict(name="early_sum", op="early", K=64, J=16, P=16_000_000, stale="geometric", stale_par=0.3, iota=8,
             opt="adagrad"),
        # a worker's request for one local batch: 1024 samples of 26 one-hot fields, and 256,000 multi-hot IDs
        dict(name="pull_one_hot", op="pull", N=26_624, fields=26, zipf=1.05, R=10_000_000, D=64),
        dict(name="pull_multi_hot", op="pull", N=256_000, fields=0, zipf=1.1, R=100_000_000, D=32),
        # a global batch of 64-bit IDs on an index that knows them
        dict(name="lookup_known", op="lookup", N=6_553_600, fields=0, zipf=1.05, R=20_000_000, capacity_log2=22),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges (the largest sizes stay below
    the largest listed case's)."""
    op = rng.choice(["step", "step", "sparse", "sparse", "means", "dense", "early", "pull", "pull", "lookup",
                     "build"])
    stale = rng.choice([("uniform", float(rng.randint(1, 6))), ("geometric", rng.choice([0.3, 0.4, 0.5]))])
    stale = dict(stale=stale[0], stale_par=stale[1], iota=rng.randint(1, 8))
    ids = dict(fields=rng.choice([0, 0, 0, 13, 26]), zipf=rng.choice([1.05, 1.1, 1.2]))
    D = rng.choice([8, 16, 16, 20, 32, 32, 32, 48, 64, 64, 100, 128])
    N = _log_int(rng, 2_000, 20_000_000)
    while N * D > 1_000_000_000:
        N //= 2
    R = min(_log_int(rng, 20_000, 100_000_000), 3_000_000_000 // D)
    opt = rng.choice(["adagrad", "adam"])
    if op == "step":
        K = rng.randint(1, 128)
        P = min(_log_int(rng, 10_000, 20_000_000), 2_000_000_000 // K)
        return dict(op=op, K=K, N=N, R=R, D=D, P=P, opt=opt, **ids, **stale)
    if op in ("sparse", "means"):
        c = dict(op=op, K=_log_int(rng, 1, 300), N=N, R=R, D=D, decay=rng.choice(["token", "token", "id_tag"]),
                 norm=rng.choice(["per_id", "per_id", "by_k"]), ragged=rng.randint(0, 1), **ids, **stale)
        if op == "sparse":
            c["opt"] = opt
        elif c["decay"] == "token":
            c["fraction"] = rng.randint(0, 1)
        return c
    if op == "dense":
        K = _log_int(rng, 2, 256)
        return dict(op=op, K=K, P=_log_int(rng, 20_000, min(100_000_000, 6_000_000_000 // K)), opt=opt, **stale)
    if op == "early":
        J = rng.choice([1, 4, 16, 32])
        return dict(op=op, K=J * rng.randint(2, 6), J=J, P=_log_int(rng, 100_000, 16_000_000), opt=opt, **stale)
    if op == "pull":
        return dict(op=op, N=_log_int(rng, 1_000, 1_500_000), R=R, D=D, **ids)
    n = _log_int(rng, 10_000, 10_000_000)
    if op == "lookup":
        return dict(op=op, N=n, R=_log_int(rng, 100_000, 50_000_000), capacity_log2=rng.randint(20, 24), **ids)
    return dict(op=op, N=n, R=_log_int(rng, 100_000, 50_000_000), capacity_log2=(2 * n).bit_length(), **ids)


# ------------------------------------------------------------------ inputs
def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 64 + stream) & ((1 << 62) - 1))
    return g


def _normal(seed, stream, *shape, sigma=SIGMA):
    return torch.empty(shape, device="cuda").normal_(0.0, sigma, generator=_generator(seed, stream))


def _uniform(seed, stream, lo, hi, *shape):
    return torch.empty(shape, device="cuda").uniform_(lo, hi, generator=_generator(seed, stream))


def _state(seed, stream, opt, *shape):
    """Optimiser slots as training leaves them."""
    if opt == "adagrad":
        return [_uniform(seed, stream, 1.0 / 16, 5.0 / 16, *shape)]
    return [_normal(seed, stream, *shape, sigma=1e-3), _uniform(seed, stream + 1, 1e-6, 1e-4, *shape)]


def _spread(rank0, n):
    """Ranks spread over n rows: r -> (a r + b) mod n, a coprime to n."""
    a = 2654435761 % n if n > 1 else 1
    a = a or 1
    while math.gcd(a, n) != 1:
        a += 1
    return (rank0 * a + 1442695040888963407 % n) % n


def _zipf_ids(case, seed):
    """N IDs whose ranks follow (to a few percent) a Zipf law over the rows, or
    over each of the equal fields of the rows in turn."""
    N, R, s = case["N"], case["R"], case["zipf"]
    fields = case["fields"]
    n = max(R // fields, 1) if fields else R
    u = torch.rand(N, device="cuda", dtype=torch.float64, generator=_generator(seed, 1))
    lo, hi = 0.5 ** (1.0 - s), (n + 0.5) ** (1.0 - s)
    x = u.mul_(hi - lo).add_(lo).pow_(1.0 / (1.0 - s))
    rank0 = x.add_(0.5).floor_().to(torch.int64).clamp_(1, n).sub_(1)
    row = _spread(rank0, n)
    if fields:
        row += torch.arange(N, device="cuda", dtype=torch.int64) % fields * n
    return row


def _expected_distinct(case):
    """Expected number of distinct IDs among the N draws."""
    N, R, s = case["N"], case["R"], case["zipf"]
    fields = case["fields"]
    n, draws = (max(R // fields, 1), N / fields) if fields else (R, N)
    edge = np.unique(np.concatenate([np.arange(1, min(n, 4000) + 1),
                                     np.geomspace(1, n, 4000).astype(np.int64)])).astype(np.float64)
    lo = np.append(edge, n + 1.0) - 0.5
    mass = np.abs(np.diff(lo ** (1.0 - s))) / abs((n + 0.5) ** (1.0 - s) - 0.5 ** (1.0 - s))
    width = np.diff(lo)
    return float(np.sum(width * -np.expm1(-draws * mass / width))) * (fields or 1)


def _tokens(case, seed):
    g = _generator(seed, 2)
    u = torch.rand(case["K"], device="cuda", dtype=torch.float64, generator=g)
    if case["stale"] == "uniform":
        s = torch.floor(u * (case["stale_par"] + 1.0))
    else:
        s = torch.floor(torch.log1p(-u) / math.log1p(-case["stale_par"]))
    return STEP - s.to(torch.int64)


def _kept(case):
    """Expected share of the contributions within the tolerance (by ID, for rows that the step before updated)."""
    most = case["iota"] - (1 if case.get("decay") == "id_tag" else 0)
    if case["stale"] == "uniform":
        return min(1.0, (most + 1.0) / (case["stale_par"] + 1.0))
    return 1.0 - (1.0 - case["stale_par"]) ** (most + 1)


def _offsets(case, seed):
    K, N = case["K"], case["N"]
    if case.get("ragged"):
        cut = torch.randint(0, N + 1, (K - 1,), device="cuda", generator=_generator(seed, 3)).sort().values
        zero = torch.zeros(1, dtype=torch.int64, device="cuda")
        return torch.cat([zero, cut.to(torch.int64), zero + N])
    return torch.tensor([N * m // K for m in range(K + 1)], dtype=torch.int64, device="cuda")


def _inputs(case, seed):
    """The tensors of a case that no entry point has touched yet."""
    op, x = case["op"], {}
    if op in ("step", "sparse", "means", "dense", "early"):
        x["tokens"] = _tokens(case, seed)
    if op in ("step", "dense", "early"):
        P, K = case["P"], case["K"]
        x["grads"] = [_normal(seed, 8, P) if m == 0 else _normal(seed * 4099 + m, 9, P) for m in range(K)]
        x["param"] = _uniform(seed, 10, -1.0 / 16, 1.0 / 16, P)
        x["dense_slots"] = _state(seed, 11, case["opt"], P)
    if op in ("step", "sparse", "means"):
        N, R, D = case["N"], case["R"], case["D"]
        x["ids"] = _zipf_ids(case, seed)
        x["rows"] = _normal(seed, 13, N, D)
        x["offsets"] = _offsets(case, seed)
        if op != "means":
            x["table"] = _uniform(seed, 14, -1.0 / 16, 1.0 / 16, R, D)
            x["table_slots"] = _state(seed, 15, case["opt"], R, D)
        if case.get("decay") == "id_tag":
            age = torch.randint(-1, 8, (R,), device="cuda", generator=_generator(seed, 17))
            x["tag"] = torch.where(age < 0, -1, STEP - 1 - age).to(torch.int32)
        if case.get("fraction"):   # another decay policy: halves per step of staleness, nothing past the tolerance
            s = STEP - x["tokens"]
            x["w"] = torch.where(s <= case["iota"], 0.5 ** s.to(torch.float32), 0.0).to(torch.float32)
    if op == "pull":
        x["ids"] = _zipf_ids(case, seed)
        x["table"] = _uniform(seed, 14, -1.0 / 16, 1.0 / 16, case["R"], case["D"])
    if op in ("lookup", "build"):
        x["ids"] = _scramble(_zipf_ids(case, seed))
    return x


def _scramble(ids):
    """Table rows as 64-bit feature IDs (an odd multiplier modulo 2^64 is one-to-one)."""
    return ids * -7046029254386353131 + 1


def _zeros(n, dtype):
    return torch.zeros(n, dtype=dtype, device="cuda")


def prepare(case, seed):
    op = case["op"]
    x = _inputs(case, seed)
    st = dict(case=case, **x)
    st["err"] = _zeros(1, torch.int32)
    if op == "step":
        step = GBAStep(case["K"], case["N"], case["D"], case["R"], case["P"])
        for t in (step.unique_ids, step.seg_offsets, step.contrib_count, step.active_count):
            t.zero_()   # only the first U entries are written: what lies past them compares as zero
        st["step"] = step
        step.grad_table(x["grads"])
    if op in ("dense", "early"):
        st["w"] = _zeros(case["K"], torch.float32)
        st["grad_table"] = gba.pointer_table(x["grads"])
    if op == "early":
        st["run"] = _zeros(case["P"], torch.float64)
    if op in ("sparse", "means"):
        K, N, R, D = case["K"], case["N"], case["R"], case["D"]
        st["unique_ids"] = _zeros(N, torch.int64)
        st["seg_offsets"] = _zeros(N + 1, torch.int64)
        st["contrib_count"] = _zeros(N, torch.int32)
        st["active_count"] = _zeros(N, torch.int32)
        st["num_unique"] = _zeros(1, torch.int64)
        if "w" not in st:
            st["w"] = _zeros(K, torch.float32)
        if op == "sparse":
            size = gba.gba_aggregate_apply_sparse_workspace_size(N, K, D, R, case["opt"])
        else:
            size = gba.gba_aggregate_sparse_workspace_size(N, K, D, R)
            st["agg"] = torch.zeros((N, D), device="cuda")
        st["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    if op == "pull":
        N, R, D = case["N"], case["R"], case["D"]
        st["unique_ids"] = _zeros(N, torch.int64)
        st["inverse"] = _zeros(N, torch.int32)
        st["rows"] = torch.zeros((N, D), device="cuda")
        st["num_unique"] = _zeros(1, torch.int64)
        st["workspace"] = torch.empty(gba.gba_pull_workspace_size(N, R), dtype=torch.uint8, device="cuda")
    if op in ("lookup", "build"):
        N, cap = case["N"], 1 << case["capacity_log2"]
        st["slot_ids"] = _zeros(cap, torch.int64)
        st["slot_rows"] = _zeros(cap, torch.int32)
        st["num_rows"] = _zeros(1, torch.int64)
        st["num_new"] = _zeros(1, torch.int64)
        st["max_rows"] = cap // 2
        st["row_ids"] = _zeros(st["max_rows"], torch.int64)
        st["rows_out"] = _zeros(N, torch.int64)
        st["workspace"] = torch.empty(gba.gba_hash_workspace_size(N), dtype=torch.uint8, device="cuda")
        if op == "lookup":
            # the index as earlier steps left it (half of its slots at most):
            # IDs that arrived one by one, so that their rows are in order
            known = torch.unique(x["ids"])
            most = cap // 2
            if known.numel() > most:
                keep = known[torch.randperm(known.numel(), device="cuda", generator=_generator(seed, 4))[:most]]
                at = torch.randint(0, most, (N,), device="cuda", generator=_generator(seed, 5))
                known_set = keep.sort().values
                pos = torch.searchsorted(known_set, x["ids"]).clamp_(max=most - 1)
                x["ids"] = torch.where(known_set[pos] == x["ids"], x["ids"], known_set[at])
                known = torch.unique(x["ids"])
                st["ids"] = x["ids"]
            gba.gba_hash_clear(st["slot_ids"], st["slot_rows"])
            ws = torch.empty(gba.gba_hash_workspace_size(known.numel()), dtype=torch.uint8, device="cuda")
            gba.gba_hash_find_or_insert(st["slot_ids"], st["slot_rows"], known, torch.empty_like(known),
                                        st["num_rows"], st["max_rows"], ws, st["row_ids"])
            torch.cuda.synchronize()
    return st


# ------------------------------------------------------------------ the calls
def _push(st):
    case = st["case"]
    decay = gba.DECAY_ID_TAG if case.get("decay") == "id_tag" else gba.DECAY_TOKEN
    norm = gba.NORM_BY_K if case["norm"] == "by_k" else gba.NORM_PER_ID_COUNT
    if not case.get("fraction"):
        gba.gba_token_weights(st["tokens"], STEP, case["iota"], st["w"], err=st["err"])
    head = (st["ids"], st["rows"], st["offsets"], case["R"], st["w"], st["tokens"], STEP, case["iota"],
            st.get("tag"), decay, norm, st["unique_ids"], st["seg_offsets"], st["contrib_count"],
            st["active_count"])
    out = {k: st[k] for k in ("unique_ids", "seg_offsets", "contrib_count", "active_count", "num_unique")}
    if "tag" in st:
        out["tag"] = st["tag"]
    if case["op"] == "means":
        gba.gba_aggregate_sparse(*head, st["agg"], st["num_unique"], st["workspace"], st["err"])
        out["agg"] = st["agg"]
        return out
    if case["opt"] == "adagrad":
        gba.gba_aggregate_apply_sparse_adagrad(*head, None, st["num_unique"], st["table"], st["table_slots"][0],
                                               LR["adagrad"], EPS, st["workspace"], st["err"])
    else:
        gba.gba_aggregate_apply_sparse_adam(*head, None, st["num_unique"], st["table"], st["table_slots"][0],
                                            st["table_slots"][1], LR["adam"], BETA1, BETA2, EPS, ADAM_T,
                                            st["workspace"], st["err"])
    out["table"] = st["table"]
    out["table_slots"] = list(st["table_slots"])
    return out


def _dense(st):
    case = st["case"]
    gba.gba_token_weights(st["tokens"], STEP, case["iota"], st["w"], err=st["err"])
    if case["op"] == "early":
        J = case["J"]
        for m in range(0, case["K"], J):
            gba.gba_accumulate_dense(st["grad_table"][m:m + J], st["w"][m:m + J], case["P"], st["run"])
        if case["opt"] == "adagrad":
            gba.gba_finalize_apply_dense_adagrad(st["run"], case["K"], case["P"], st["param"], st["dense_slots"][0],
                                                 LR["adagrad"], EPS)
        else:
            gba.gba_finalize_apply_dense_adam(st["run"], case["K"], case["P"], st["param"], *st["dense_slots"],
                                              LR["adam"], BETA1, BETA2, EPS, ADAM_T)
    elif case["opt"] == "adagrad":
        gba.gba_aggregate_apply_dense_adagrad(st["grad_table"], st["w"], case["P"], st["param"],
                                              st["dense_slots"][0], LR["adagrad"], EPS)
    else:
        gba.gba_aggregate_apply_dense_adam(st["grad_table"], st["w"], case["P"], st["param"], *st["dense_slots"],
                                           LR["adam"], BETA1, BETA2, EPS, ADAM_T)
    return {"param": st["param"], "dense_slots": list(st["dense_slots"])}


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "step":
        step = st["step"]
        step.run(tokens=st["tokens"], step=STEP, iota=case["iota"], grads=st["grads"], ids=st["ids"],
                 rows=st["rows"], offsets=st["offsets"], param=st["param"], dense_slots=st["dense_slots"],
                 table=st["table"], table_slots=st["table_slots"], optimizer=case["opt"], lr=LR[case["opt"]],
                 eps=EPS, beta1=BETA1, beta2=BETA2, t=ADAM_T)
        return {"g_bar": step.g_bar, "param": st["param"], "dense_slots": list(st["dense_slots"]),
                "table": st["table"], "table_slots": list(st["table_slots"]), "unique_ids": step.unique_ids,
                "seg_offsets": step.seg_offsets, "contrib_count": step.contrib_count,
                "active_count": step.active_count, "num_unique": step.num_unique}
    if op in ("sparse", "means"):
        return _push(st)
    if op in ("dense", "early"):
        return _dense(st)
    if op == "pull":
        gba.gba_pull_rows(st["ids"], st["table"], st["unique_ids"], st["inverse"], st["rows"], st["num_unique"],
                          st["workspace"], st["err"])
        return {"unique_ids": st["unique_ids"], "inverse": st["inverse"], "rows": st["rows"],
                "num_unique": st["num_unique"]}
    if op == "lookup":
        gba.gba_hash_find_or_insert(st["slot_ids"], st["slot_rows"], st["ids"], st["rows_out"], st["num_rows"],
                                    st["max_rows"], st["workspace"], st["row_ids"], st["num_new"], st["err"])
        return {"rows": st["rows_out"], "num_rows": st["num_rows"], "num_new": st["num_new"]}
    # build: which row an ID gets is not fixed, so the rows come back as the IDs they now stand for
    gba.gba_hash_clear(st["slot_ids"], st["slot_rows"])
    st["num_rows"].zero_()
    gba.gba_hash_find_or_insert(st["slot_ids"], st["slot_rows"], st["ids"], st["rows_out"], st["num_rows"],
                                st["max_rows"], st["workspace"], st["row_ids"], st["num_new"], st["err"])
    return {"ids_of_rows": st["row_ids"][st["rows_out"]], "num_rows": st["num_rows"], "num_new": st["num_new"]}


# ------------------------------------------------------------------ accounts
def work(case):
    """What a pass cannot do without: the kept dense gradients and rows read
    once, parameters and state read and written, IDs and outputs once."""
    op, nbytes, flops = case["op"], 0.0, 0.0
    slots = 2 if case.get("opt") == "adam" else 1
    if op in ("step", "dense", "early"):
        P, kept = case["P"], case["K"] * _kept(case)
        nbytes += kept * P * 4 + (2 + 2 * slots) * P * 4 + (P * 4 if op == "step" else 0)
        flops += 2 * kept * P + 10 * P
    if op in ("step", "sparse", "means"):
        N, D, U = case["N"], case["D"], _expected_distinct(case)
        kept = N * _kept(case)
        nbytes += N * 8 + kept * D * 4 + U * 24
        nbytes += U * D * 4 if op == "means" else U * (2 + 2 * slots) * D * 4
        if case.get("decay") == "id_tag":
            nbytes += 8 * U
        flops += 2 * kept * D + 10 * U * D
    if op == "pull":
        U = _expected_distinct(case)
        nbytes += case["N"] * (8 + 4) + U * (8 + 2 * 4 * case["D"])
    if op in ("lookup", "build"):
        U = min(_expected_distinct(case), 1 << (case["capacity_log2"] - 1))
        nbytes += case["N"] * 16 + U * 12
        if op == "build":
            nbytes += (1 << case["capacity_log2"]) * 12 + U * 20 + case["N"] * 24
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Sums are float64 and rounded to float32 once, the optimiser is float32:
    a few float32 roundings of the stored values, at any order of the sums
    (against float64 every output is 0.1 to 4.5e-8 off)."""
    op = case["op"]
    if op in ("pull", "lookup", "build"):
        return "exact"
    return {"rel": 2e-7, "max": 5e-6}


# ------------------------------------------------------------------ in 64 bits
def _exact_update(opt, p, slots, g):
    """One optimiser update in float64 (p, slots, g float64)."""
    lr = LR[opt]
    if opt == "adagrad":
        a = slots[0] + g * g
        return p - lr * g / (a.sqrt() + EPS), [a]
    m = BETA1 * slots[0] + (1.0 - BETA1) * g
    v = BETA2 * slots[1] + (1.0 - BETA2) * g * g
    mh, vh = m / (1.0 - BETA1 ** ADAM_T), v / (1.0 - BETA2 ** ADAM_T)
    return p - lr * mh / (vh.sqrt() + EPS), [m, v]


def _exact_weights(case, x):
    if "w" in x:
        return x["w"].double()
    return (STEP - x["tokens"] <= case["iota"]).double()


def _exact_dense(case, x, out):
    w = _exact_weights(case, x)
    g = torch.zeros(case["P"], dtype=torch.float64, device="cuda")
    for m, grad in enumerate(x["grads"]):
        if float(w[m]) != 0.0:
            g += float(w[m]) * grad.double()
    x["grads"].clear()
    g /= case["K"]
    out["param"], out["dense_slots"] = _exact_update(case["opt"], x["param"].double(),
                                                     [s.double() for s in x["dense_slots"]], g)
    return g


def _exact_sparse(case, x, out):
    N, D, K, R = case["N"], case["D"], case["K"], case["R"]
    unique, inverse = torch.unique(x["ids"], return_inverse=True)
    U = unique.numel()
    j = torch.arange(N, device="cuda")
    m = torch.searchsorted(x["offsets"][1:].contiguous(), j, right=True)
    if case.get("decay") == "id_tag":
        s = (x["tag"][x["ids"]].to(torch.int64) - x["tokens"][m] + 1).clamp_(min=0)
        weight = (s <= case["iota"]).double()
    else:
        weight = _exact_weights(case, x)[m]
    pairs = torch.unique(inverse * K + m)
    count = torch.bincount(pairs // K, minlength=U)
    seen = torch.unique((inverse * K + m)[weight != 0])
    active = torch.bincount(seen // K, minlength=U)
    mean = torch.zeros((U, D), dtype=torch.float64, device="cuda")
    for a in range(0, N, 1 << 22):
        b = min(N, a + (1 << 22))
        mean.index_add_(0, inverse[a:b], x["rows"][a:b].double() * weight[a:b, None])
    mean /= K if case.get("norm") == "by_k" else count[:, None].double()
    if case["op"] == "means":
        out["agg"] = torch.zeros((N, D), dtype=torch.float64, device="cuda")
        out["agg"][:U] = mean
        return
    on = active > 0
    rows, g = unique[on], mean[on]
    table, slots = x["table"].double(), [s.double() for s in x["table_slots"]]
    p, new = _exact_update(case["opt"], table[rows], [s[rows] for s in slots], g)
    table[rows] = p
    for s, v in zip(slots, new):
        s[rows] = v
    out["table"], out["table_slots"] = table, slots


def exact(case, seed):
    """The floating outputs of ``run`` in float64; whole values have none."""
    op = case["op"]
    if op in ("lookup", "build"):
        return None
    x, out = _inputs(case, seed), {}
    if op == "pull":
        unique = torch.unique(x["ids"])
        rows = torch.zeros((case["N"], case["D"]), dtype=torch.float64, device="cuda")
        rows[:unique.numel()] = x["table"][unique].double()
        return {"rows": rows}
    if op in ("step", "dense", "early"):
        g = _exact_dense(case, x, out)
        if op == "step":
            out["g_bar"] = g
    if op in ("step", "sparse", "means"):
        _exact_sparse(case, x, out)
    return out
