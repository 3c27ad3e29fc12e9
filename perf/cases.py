"""The work that users of this framework have it do, as cases whose time can be measured.

Every case goes through the package's public entry points (paper_2211_13878_amd.binding and
.alg1).  A case is a dict of plain values:

    kind     "search"   one batch of plan searches: Solver.solve and Solver.backtrack
             "static"   the same for a caller that cannot allocate: galv_dp_solve_static
             "budgets"  one solve, then the optimum of every memory limit and the plans of a few
             "coarse"   coarsened search: galv_dp_coarsen, solve, backtrack, galv_dp_expand_plan
             "alg1"     Algorithm 1 as a whole: the outer loop over batch sizes and pipeline degrees
    family   how the tables' values are drawn (below); the ranges of the repository's five
             configurations, with the memory range scaled by (budget / layers)
    B, L, S, E      searches in the batch, layers, strategies, memory budget in units
    spread   budgets spread evenly from E / 4 to E instead of E for all
    c_scale  unit of time of all costs: 1 as configured; 10 makes plan costs outgrow 32 bits;
             1000 stands for costs in nanoseconds where the configurations hold microseconds
    r_scale  transition costs times this (a slow interconnect: changing layout costs as much as a layer)

All results are whole numbers, so every comparison is exact.
"""
import math

import numpy as np
import torch

from paper_2211_13878_amd import alg1, binding, workloads

# family: (smallest and largest m in units of E / L, c range, largest R, share of unusable (layer, strategy))
FAMILIES = {
    "tiny":   ((1 / 64, 1 / 2), (1_000, 100_000), 20_000, 0.0),       # independent layers, few strategies
    "layers": ((1 / 8, 2), (10_000, 1_000_000), 50_000, 0.10),        # layers of one shape, +-5 %
    "encdec": ((1 / 8, 2), (10_000, 1_000_000), 50_000, 0.10),        # two layer types, the second 1.5 times the first
    "depth":  ((3 / 32, 6), (10_000, 1_000_000), 100_000, 0.05),      # deep stacks of one shape, wider memory range
    "stress": ((1 / 32, 8), (1_000, 10_000_000), 1_000_000, 0.0),     # independent layers, 1 % of cells tied
}
BASE = {"spread": False, "c_scale": 1, "r_scale": 1}


def listed():
    def case(name, kind, family, B, L, S, E, **more):
        return {"name": name, "kind": kind, "family": family, "B": B, "L": L, "S": S, "E": E, **BASE, **more}

    return [
        # the smallest call: one small model, planned while somebody waits; launches and latency
        case("tiny", "search", "tiny", 1, 4, 6, 256),
        # a planner inside a serving loop or a graph capture, which may not allocate
        case("static", "static", "layers", 3, 6, 22, 1500),
        # one model, odd sizes throughout: a user's single search
        case("single", "search", "depth", 1, 37, 29, 9973),
        # a 32-layer encoder on 8 GPUs (22 strategies): 16 GB in units of 1 MB, eight batch sizes
        case("encoder", "search", "layers", 8, 32, 22, 16384),
        # a 24 + 24 layer encoder-decoder, 24 GB, transition costs that depend on the layer type
        case("encdec", "search", "encdec", 32, 48, 22, 24576),
        # a 96-layer decoder, 44 strategies, 64 budgets from 8 to 32 GB
        case("decoder", "search", "depth", 64, 96, 44, 32768, spread=True),
        # the largest search one GPU holds: 128 layers x 128 strategies x 65536 units, 16 searches
        case("stress", "search", "stress", 16, 128, 128, 65536),
        # costs measured in nanoseconds: 64-bit sums and large transition costs
        case("nanoseconds", "search", "depth", 16, 48, 44, 16384, c_scale=1000),
        # changing layout is as dear as a layer: few strategies can be ruled out
        case("slow_links", "search", "depth", 12, 48, 44, 16384, r_scale=10),
        # one solve, every memory limit: the trade-off curve and the plans of four limits per search
        case("budgets", "budgets", "layers", 8, 24, 22, 20001),
        # exploration at a quarter of the layers' and a sixteenth of the budget's resolution
        case("coarse", "coarse", "depth", 16, 96, 44, 32768, fuse=2, gran=16),
        # Algorithm 1 on 8 GPUs for a 48-layer model: batch sizes 1, 2, ... until nothing fits
        {"name": "optimize", "kind": "alg1", "L": 48, "N": 8, "E": 6000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the listed kinds, sizes log-uniform over the listed ranges."""
    kind = rng.choice(["search"] * 6 + ["static", "budgets", "coarse", "alg1"])
    if kind == "alg1":
        return {"kind": kind, "L": rng.randint(16, 96), "N": rng.choice([4, 8, 16]), "E": _log(rng, 2000, 16000)}
    family = rng.choice(["tiny", "layers", "encdec", "depth", "stress"])
    S = _log(rng, 6, 128)
    while True:
        if kind == "static":
            B, L, E = rng.randint(1, 4), rng.randint(3, 12), _log(rng, 256, 2048)
            if binding.galv_dp_workspace_bytes(binding.make_desc(B, L, S, E, 2)) > binding.GALV_DP_STATIC_BYTES:
                S = _log(rng, 6, 44)
                continue
        else:
            B, L, E = _log(rng, 1, 64), _log(rng, 4, 128), _log(rng, 256, 65536)
            if B * L * E * S > 16 * 96 * 65536 * 96:     # no larger than the largest listed case
                continue
        break
    case = {"kind": kind, "family": family, "B": B, "L": L, "S": S, "E": E, **BASE,
            "spread": rng.random() < 0.3,
            "c_scale": rng.choice([1, 1, 1, 10, 1000]),
            # (nearly all candidates count with large transition costs: kept to sizes of the listed such case)
            "r_scale": rng.choice([1, 1, 3, 10]) if B * L * E * S * S <= 12 * 48 * 16384 * 44 * 44 else 1}
    if kind == "coarse":
        case.update(fuse=rng.choice([1, 2, 4]), gran=rng.choice([1, 4, 16, 64]))
    return case


def _tables(case, seed):
    """numpy arrays c, m, R, r_idx, budget of one case (the array contract of workloads.py)."""
    B, L, S, E = case["B"], case["L"], case["S"], case["E"]
    (m_lo, m_hi), (c_lo, c_hi), r_hi, unusable = FAMILIES[case["family"]]
    m_lo, m_hi = max(1, round(m_lo * E / L)), max(2, round(m_hi * E / L))
    rng = np.random.default_rng(seed)
    types = 2 if case["family"] == "encdec" else 1
    R = rng.integers(0, r_hi + 1, size=(B, 1, S, S), dtype=np.int64)
    R[:, :, np.arange(S), np.arange(S)] = 0
    if case["family"] in ("tiny", "stress"):
        m = rng.integers(m_lo, m_hi + 1, size=(B, L, S))
        c = rng.integers(c_lo, c_hi + 1, size=(B, L, S))
        if case["family"] == "stress":               # two strategies per search that copy another one
            for b in range(B):
                for a, d in (sorted(p) for p in rng.choice(S, size=(2, 2), replace=False)):
                    R[b, 0, d, :] = R[b, 0, a, :]
                    R[b, 0, :, d] = R[b, 0, :, a]
                    R[b, 0, [a, d, a, d], [d, a, a, d]] = 0
                    rows = rng.random(size=L) < 0.64
                    c[b, rows, d], m[b, rows, d] = c[b, rows, a], m[b, rows, a]
    else:
        scale = np.where(np.arange(L) >= L // 2, 1.5, 1.0) if types == 2 else np.ones(L)
        jitter = lambda base: np.rint(base[:, None, :] * scale[None, :, None] *
                                      (1.0 + rng.uniform(-0.05, 0.05, size=(B, L, S))))
        m = jitter(rng.integers(m_lo, m_hi + 1, size=(B, S)).astype(np.float64))
        c = jitter(rng.integers(c_lo, c_hi + 1, size=(B, S)).astype(np.float64))
    m[rng.random(size=(B, L, S)) < unusable] = E + 1
    r_idx = np.zeros((B, L), np.int32)
    if types == 2:
        R = np.concatenate([R, 2 * R], axis=1)
        r_idx[:, L // 2] = 1                         # the boundary between the two layer types
    budget = np.rint(np.linspace(E / 4, E, B)) if case["spread"] and B > 1 else np.full(B, E)
    k = case["c_scale"]
    return (np.ascontiguousarray(c.astype(np.int64) * k), np.ascontiguousarray(m.astype(np.int32)),
            np.ascontiguousarray(R * (k * case["r_scale"])), r_idx, budget.astype(np.int32))


def _sizes(case):
    """Batch sizes that Algorithm 1 can look at: every layer takes at least 20 + 4 * batch units of memory
    (workloads.Alg1Model), and the first size that does not fit ends the search."""
    return case["E"] // (4 * case["L"]) + 2


def prepare(case, seed):
    if case["kind"] == "alg1":
        # (the cost model is host code of the user's: Algorithm 1 asks it for tables)
        return {"case": case, "model": workloads.Alg1Model(seed, case["L"], case["N"], alg1.strategy_counts(case["N"]))}
    tables = tuple(torch.from_numpy(a).cuda() for a in _tables(case, seed))
    B, L, S, E, nR = case["B"], case["L"], case["S"], case["E"], tables[2].shape[1]
    state = {"case": case, "tables": tables}
    if case["kind"] == "static":
        state["desc"] = binding.make_desc(B, L, S, E, nR)
        state["out"] = (torch.empty(B, dtype=torch.int64, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda"),
                        torch.empty((B, L), dtype=torch.int32, device="cuda"))
    elif case["kind"] == "coarse":
        Lc = (L + case["fuse"] - 1) // case["fuse"]
        state["solver"] = binding.Solver(B, Lc, S, E // case["gran"], nR)
    else:
        state["solver"] = binding.Solver(B, L, S, E, nR)
        if case["kind"] == "budgets":                # 40, 60, 80 and 100 % of the device's memory
            limits = (tables[4][:, None] * torch.tensor([2, 3, 4, 5], device="cuda") // 5).to(torch.int32)
            state["limits"] = limits.reshape(-1).contiguous()
            state["who"] = torch.arange(B, dtype=torch.int32, device="cuda").repeat_interleave(4).contiguous()
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "alg1":
        r = alg1.optimize(state["model"], case["N"], case["E"], range(1, 100000))
        # (how many batch sizes fit depends on the model: the results fill arrays of the largest size there can be)
        c_p = np.full((_sizes(case), r.c_p.shape[1]), -1, np.int64)
        c_p[:len(r.c_p)] = r.c_p
        plan = np.full(case["L"], -1, np.int64)
        for i, s in enumerate(s for stage in r.plans or [] for s in stage):
            plan[i] = s
        return {"batch": r.batch or 0, "pp": r.pp or 0, "cost": r.cost or 0, "n_explored": r.n_explored, "c_p": c_p, "plan": plan}
    if kind == "static":
        binding.galv_dp_solve_static(state["desc"], *state["tables"], *state["out"])
        return state["out"]
    solver = state["solver"]
    if kind == "coarse":
        c, m, R, r_idx, budget = state["tables"]
        c2, m2, r2, e2 = binding.galv_dp_coarsen(case["fuse"], case["gran"], c, m, R, r_idx, budget)
        cost, last = solver.solve(c2, m2, R, r2, e2)
        return cost, last, binding.galv_dp_expand_plan(solver.backtrack(), case["L"], case["fuse"])
    cost, last = solver.solve(*state["tables"])
    if kind == "budgets":
        return (cost, last) + solver.best_per_budget() + solver.backtrack_queries(state["who"], state["limits"])
    return cost, last, solver.backtrack()


def work(case):
    """Bytes: the tables read once, the results written once.  Operations: one addition and one
    comparison for the best cost of every budget column at every layer."""
    L, E = case["L"], case["E"]
    if case["kind"] == "alg1":
        degrees = {1 << k: n for k, n in ((k, len(alg1.group_strategies(case["N"] >> k)))
                                          for k in range(case["N"].bit_length())) if (1 << k) <= L}
        sizes = max(1, _sizes(case) // 2)            # about as many batch sizes fit
        per = sum(P * (math.ceil(L / P) * n * 12 + n * n * 8) for P, n in degrees.items())
        return {"bytes": sizes * per, "flops": sizes * 2 * L * (E + 1) * len(degrees)}
    B, S = case["B"], case["S"]
    columns = sum(int(e) + 1 for e in (np.linspace(E / 4, E, B) if case["spread"] and B > 1 else np.full(B, E)))
    matrices = 2 if case["family"] == "encdec" else 1
    inputs = B * (L * S * 12 + matrices * S * S * 8 + L * 4 + 4)
    outputs = B * (12 + 4 * L)
    layers = L
    if case["kind"] == "budgets":
        outputs = B * 12 + B * (E + 1) * 12 + 4 * B * (8 + 4 * L)
    if case["kind"] == "coarse":
        layers, columns = math.ceil(L / case["fuse"]), columns // case["gran"] + B
    return {"bytes": inputs + outputs, "flops": 2 * layers * columns}


def tolerance(case):
    return "exact"
