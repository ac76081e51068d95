"""The work whose speed counts: what a planner has this library do, through its public entry points.

Every case is one call chain of a planner, from the tables it has in hand to the plans it reads:

  plan        fill the tables of a batch of stage searches, read plans back (the best one of every instance, or
              those of a window of budgets below the device's)
  curve       the same, and the whole curve best(e) with its last strategies
  budget      the same fill, then the largest forward budget whose plan fits the overall memory (Algorithm 3)
  partition   the pipeline-partition search (Algorithm 2) of many (batch size, PP degree) pairs
  model       layer shapes through the analytic cost model on the device into the fill, then the plans

Everything is decided by integers and by fp32 / fp64 operations in a stated order, so the results of two correct
implementations are the same bit by bit.
"""
import numpy as np
import torch

import gbmw_inputs as gi
import paper_2307_02031_amd as g

HW = gi.default_hardware(unit_mb=1.0)


def listed():
    solve = dict(data="uniform", B=1, L_lo=4, L_hi=4, S=4, E=256, values_only=False, host=False, window=1)
    return [
        # The smallest search (benchmark workload 1): a call's latency.
        dict(solve, name="plan_tiny", task="plan"),
        # One stage of a 24-layer model with the 22 strategies of 8 devices without checkpointing (workload 2),
        # inputs straight from host arrays, and the whole budget curve.
        dict(solve, name="curve_22", task="curve", L_lo=24, L_hi=24, S=22, E=8192, host=True),
        # One stage with the 44 strategies with checkpointing (workload 3), one plan.
        dict(solve, name="plan_44", task="plan", data="structured", L_lo=32, L_hi=32, S=44, E=16384),
        # Small ragged stages, sizes off every tile edge.
        dict(solve, name="plan_ragged", task="plan", B=37, L_lo=2, L_hi=19, S=21, E=4999, window=7),
        # The batched workload (4): 64 stages of 6 to 24 layers, the plans of a window of budgets below E.
        dict(solve, name="plan_batch_44", task="plan", data="structured", B=64, L_lo=6, L_hi=24, S=44, E=32768,
             window=256),
        # The same size without argmin records and with Algorithm 3's overall-memory check.
        dict(solve, name="budget_batch_44", task="budget", data="structured", B=64, L_lo=6, L_hi=24, S=44, E=32768,
             values_only=True),
        # The large batched workload (5): deep stages, 64 strategies, the finest budget axis.
        dict(solve, name="plan_batch_64", task="plan", B=16, L_lo=96, L_hi=96, S=64, E=65536, window=64),
        # 128 strategies, the upper end of the register-blocked kernel (as in the benchmark).
        dict(solve, name="plan_batch_128", task="plan", B=16, L_lo=8, L_hi=8, S=128, E=32768, window=256),
        # The whole decision-tree set of 64 devices with checkpointing, cost-model tables, with the budget curve.
        dict(solve, name="curve_186", task="curve", data="model", B=4, L_lo=24, L_hi=24, S=186, E=16384),
        # Algorithm 2 on the benchmark's 16 pairs: 48 layers, 44 strategies, PP degrees 2 to 16.
        dict(name="partition_44", task="partition", data="structured", pairs=16, Lm=48, S=44, E=32768, overall=False),
        # The planner's own search: cost-model tables of a 48-layer model on 8 devices, PP degrees 1 to 8, every
        # stage search with the overall-memory check.
        dict(name="partition_model", task="partition", data="model", pairs=32, Lm=48, S=22, E=16384, overall=True),
        # Layer shapes to plans on the device, a model of 48 layers in two stages, two batch sizes.
        dict(solve, name="model_22", task="model", data="model", B=4, L_lo=24, L_hi=24, S=22, E=16384),
    ]


MODEL_SETS = {22: (8, True), 46: (64, True), 78: (16, False), 186: (64, False)}   # strategies: (devices, Takeaway #3)
MOST_UPDATES = 6.0e10
MOST_CELLS = 1.0e9


def draw(rng):
    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    while True:
        if rng.random() < 0.2:
            data = rng.choice(["structured", "model"])
            c = dict(task="partition", data=data, pairs=4 * rng.randint(1, 8), Lm=rng.randint(16, 48),
                     S=rng.choice([22, 44]) if data == "structured" else 22, overall=rng.random() < 0.5,
                     E=log(16384 if data == "structured" else 4096, 32768))
            if c["pairs"] * 8.0 * c["Lm"] * c["E"] * c["S"] ** 2 <= 10 * MOST_UPDATES:
                return c
            continue
        data = rng.choice(["structured", "uniform", "uniform", "model"])
        task = rng.choice(["plan", "curve", "budget"] + (["model"] if data == "model" else ["plan"]))
        S = log(3, 200) if data == "uniform" else rng.choice([22, 44] if data == "structured" else list(MODEL_SETS))
        lo = log(2, 24 if data == "structured" else 48)
        floor = {"uniform": 256, "structured": 320 * (lo + 16), "model": 4096}[data]   # budgets that some plan fits
        c = dict(task=task, data=data, B=2 * log(1, 8) if data == "model" else log(1, 64), L_lo=lo,
                 L_hi=lo if data == "model" else lo + rng.randint(0, 16), S=S, E=log(floor, 65536),
                 values_only=task == "budget" or rng.random() < 0.2, host=task != "model" and rng.random() < 0.3,
                 window=rng.choice([1, 1, 64, 256]))
        c["window"] = min(c["window"], c["E"] + 1)
        rows = c["B"] * (c["L_lo"] + c["L_hi"]) / 2.0
        if rows * c["E"] * S * S <= MOST_UPDATES and rows * c["E"] * S <= MOST_CELLS:
            return c


def shapes(L, rs):
    """Layers of a 48-layer transformer (a row of the paper's model table), each a little different."""
    base = gi.table1_layers("BERT-Huge-48", layers=L)
    return base * rs.uniform(0.75, 1.25, (L, 1))


def model_set(S):
    devices, takeaway3 = MODEL_SETS[S]
    sets = g.gbmw_enumerate_strategies(devices, True, takeaway3)
    assert len(sets) == S
    return sets


def model_tables(state):
    """The cost model for B / 2 batch sizes of a two-stage pipeline -> c, M, R of B stage searches, on the device."""
    L, cs, Ms, Rs = state["L"][0], [], [], []
    for Bm in state["batches"]:
        t = g.gbmw_cost_model(state["layers"], state["set"], HW, Bm, 2, device=True)
        for i in range(2):
            rows = slice(i * L, (i + 1) * L)
            cs.append(t["c"][rows]), Ms.append(t["M"][i, rows]), Rs.append(t["R"][rows])
    return torch.cat(cs), torch.cat(Ms), torch.cat(Rs)


def prepare(case, seed):
    rs = np.random.RandomState(seed % (1 << 31))
    if case["task"] == "partition":
        return prepare_partition(case, seed, rs)
    B, S, E = case["B"], case["S"], case["E"]
    # every depth of the range in turn, in a scrambled order; the deepest is there whatever the batch size
    L = (case["L_hi"] - (7 * np.arange(B)) % (case["L_hi"] - case["L_lo"] + 1)).astype(np.int32)
    st = dict(case=case, L=L, ctx=None)
    if case["data"] == "model":
        n = int(L[0])
        st.update(layers=shapes(2 * n, rs), set=model_set(S), batches=list(np.sort(rs.uniform(0.5, 4.0, B // 2))))
        if case["task"] != "model":
            st["c"], st["M"], st["R"] = model_tables(st)
    else:
        parts = []
        for b in range(B):
            n = int(L[b])
            if case["data"] == "structured":              # the batched workload's recipe: batch sizes scale both
                scale = 2.0 ** ((b // 4) % 4) / 4.0 if B > 1 else 1.0
                parts.append(gi._structured_instance(gi.Stream(seed, lane=b), n, S, act_scale=scale, cost_scale=scale))
            else:                                         # memory such that the budget binds
                hi = max(2, min(3 * E // n, E // 8))
                p = gi.random_instance(1000 * seed + b, n, S, E, c_rng=(1.0, 100.0), M_rng=(max(1, hi // 16), hi),
                                       R_rng=(0.0, 10.0))
                parts.append((p.c, p.M, p.R))
        c, M, R = (np.concatenate([p[k] for p in parts]) for k in range(3))
        st["c"], st["M"], st["R"] = c.astype(np.float32), M.astype(np.int32), R.astype(np.float32)
    if case["host"]:
        for k in "cMR":
            st[k] = st[k].cpu().numpy() if isinstance(st[k], torch.Tensor) else st[k]
    elif "c" in st:
        for k in "cMR":
            st[k] = st[k] if isinstance(st[k], torch.Tensor) else torch.from_numpy(st[k]).cuda()
    if case["task"] == "budget":
        M = st["M"].cpu().numpy() if isinstance(st["M"], torch.Tensor) else st["M"]
        Oms = np.floor(M * rs.random_sample(M.shape)).astype(np.int32)
        top = max(1, int(np.minimum(M, E // 8).max()))
        st["O"] = (M - Oms, rs.randint(0, top + 1, M.shape).astype(np.int32), Oms)
    w = case["window"]
    st["qi"] = np.repeat(np.arange(B, dtype=np.int32), w)
    st["qe"] = np.tile(np.arange(E - w + 1, E + 1, dtype=np.int32), B)
    return st


def prepare_partition(case, seed, rs):
    S, E, Lm, n = case["S"], case["E"], case["Lm"], case["pairs"]
    degrees = [2, 4, 8, 16] if case["data"] == "structured" else [1, 2, 4, 8]
    sets = {P: g.gbmw_enumerate_strategies(8 // P) for P in degrees} if case["data"] == "model" else None
    layers = shapes(Lm, rs)
    a = {k: [] for k in ("P", "c", "cns", "R", "M", "p0", "p_t", "O_b", "O_ms", "batch", "group")}
    for k in range(n):
        P, q = degrees[k % 4], k // 4
        if sets is None:
            m = gi.structured_pipeline_model(seed + q, Lm, P, E, m=8, S=S, act_scale=0.5 * 2.0 ** (q % 4))
            m = gi.with_memory_split(m, seed + k, max(1, E // 8))
            c, cns, R, M, Ob, Oms = m.c, m.c_ns, m.R, m.M, m.Ob, m.Oms
        else:                                             # smaller strategy sets are padded with forbidden ones
            t = g.gbmw_cost_model(layers, sets[P], HW, 1.0 + q, P)
            ns = len(sets[P])
            c, cns = np.full((Lm, S), np.inf, np.float32), np.full((Lm, S), np.inf, np.float32)
            R = np.zeros((Lm, S, S), np.float32)
            M, Ob, Oms = (np.zeros((P, Lm, S), np.int32) for _ in range(3))
            c[:, :ns], cns[:, :ns], R[:, :ns, :ns] = t["c"], t["c_nosync"], t["R"]
            M[:, :, :ns], Ob[:, :, :ns], Oms[:, :, :ns] = t["M"], t["O_b"], t["O_ms"]
        for key, v in (("P", [P]), ("c", c), ("cns", cns), ("R", R), ("M", M.reshape(P * Lm, S)),
                       ("p0", gi.proportional_partition(Lm, 1.0 / np.arange(P, 0, -1))),
                       ("p_t", gi.proportional_partition(Lm, np.ones(P))), ("O_b", Ob.reshape(P * Lm, S)),
                       ("O_ms", Oms.reshape(P * Lm, S)), ("batch", [8.0 * (q + 1)]), ("group", [q])):
            a[key].append(np.asarray(v))
    return dict(case=case, ctx=None, a={k: np.concatenate(v) for k, v in a.items()}, Lm=[Lm] * n, m=[8] * n)


def run(state):
    case = state["case"]
    if case["task"] == "partition":
        a, over = state["a"], case["overall"]
        res, state["ctx"] = g.gbmw_partition_search(
            a["P"], state["Lm"], state["m"], a["c"], a["cns"], a["R"], a["M"], a["p0"], a["p_t"], case["S"],
            case["E"], max_iter=32, ctx=state["ctx"], batch_size=a["batch"], batch_group=a["group"],
            O_b=a["O_b"] if over else None, O_ms=a["O_ms"] if over else None)
        return {k: v for k, v in res.items() if k != "device_ms"}
    if case["task"] == "model":
        c, M, R = model_tables(state)
    else:
        c, M, R = state["c"], state["M"], state["R"]
    flags = g.GBMW_FLAG_LAZY_ARGMIN if case["values_only"] else 0
    ctx = g.gbmw_dp_solve_batched(state["L"], c, M, R, case["S"], case["E"], flags=flags, ctx=state["ctx"])
    state["ctx"] = ctx
    out = {}
    if case["task"] == "budget":
        out["budget"] = g.gbmw_select_forward_budget(ctx, *state["O"])
    else:
        out["plans"] = g.gbmw_backtrack(ctx, state["qi"], state["qe"])
    if case["task"] == "curve":
        out["best"] = g.gbmw_get_best(ctx)
    if case["task"] == "model":
        out["tables"] = (c, M, R)
    return out


def work(case):
    """Every input read once and every output written once; an entry of R enters at least one addition and one
    comparison.  (How many of the E + 1 budgets have to be looked at depends on the values.)"""
    S = case["S"]
    if case["task"] == "partition":
        n, Lm = case["pairs"], case["Lm"]
        mean_P = 7.5 if case["data"] == "structured" else 3.75
        rows, stage_rows = n * Lm, n * Lm * mean_P
        trace = 32 * n * (4 * 16 + 12)
        return {"bytes": 4.0 * (rows * (S * S + 2 * S) + stage_rows * S * (3 if case["overall"] else 1) + trace),
                "flops": 2.0 * rows * S * S}
    B, rows = case["B"], case["B"] * (case["L_lo"] + case["L_hi"]) / 2.0
    nq = B * case["window"]
    bytes_ = 4.0 * rows * (S * S + 2 * S) + nq * (case["L_hi"] + 16.0)
    if case["task"] == "curve":
        bytes_ += 5.0 * B * (case["E"] + 1)
    if case["task"] == "budget":
        bytes_ += 12.0 * rows * S
    return {"bytes": bytes_, "flops": 2.0 * rows * S * S}


def tolerance(case):
    """Bit-exact by contract: stated order of the additions, the lowest index among equals."""
    return "exact"
