"""The work that a planner built on this library has it do, as cases that can be timed and compared.

A case is a dict of sizes and options. Five kinds:

  plan    one planning step: the caller's selection (or Eq. (1) over relevance scores) becomes a plan,
          the selected groups are gathered and re-positioned, the new prompt tokens attend over them and
          the per-segment masses come out
  cluster a prefill-only clustering pass: the same with the values left in the pool, then the scores of
          the new objects against every group and the join / new-group decision
  tier    consecutive planning steps over the residency tier: Eq. (1) over slowly drifting scores, the
          missing groups loaded from the host store, the next selection prefetched beside the attention
  decode  tokens decoded one at a time over a context that was gathered once
  append  new objects' keys and values saved at the end of their groups

Group lengths, selections and values are drawn from the seed, with the distributions of the package's
own workload generator; sizes follow its configurations and the tests.
"""
import math

import numpy as np
import torch

from paper_2510_18546_amd import binding as B

DEV = "cuda:0"
_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "i8": torch.int8}


def _case(**kw):
    """A whole case: the fields that every kind has, and what the caller says."""
    c = {"kind": "plan", "dtype": "bf16", "agents": 1, "q_heads": 32, "kv_heads": 8, "head_dim": 128, "groups": 64,
         "capacity": 128, "len_lo": 64, "len_hi": 128, "selected": 16, "new": 256, "scored": False, "mass": "reduced",
         "objects": 0, "steps": 1}
    assert set(kw) - {"name"} <= set(c)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest planning step: a tiny fp32 layer, four groups of 32 tokens, masses of every row
        _case(name="plan tiny fp32", dtype="f32", q_heads=4, kv_heads=1, head_dim=64, groups=8, capacity=32, len_lo=32,
              len_hi=32, selected=4, new=64, mass="rows"),
        # an ordinary planning step of one agent on a Llama-3.2-11B-shaped layer: ragged groups, about 1.5 K tokens
        _case(name="plan ragged map"),
        # a large map: 8 K cached tokens, 512 new ones (the default workload of the benchmark)
        _case(name="plan large map", groups=256, capacity=256, len_lo=256, len_hi=256, selected=32, new=512),
        # the same map, ragged, on a layer of 56 query heads, the groups retrieved by Eq. (1) under a token budget
        _case(name="retrieve and plan, 56 heads", q_heads=56, groups=256, capacity=256, len_lo=192, len_hi=256,
              selected=32, new=512, scored=True),
        # sixteen agents planning over one shared map
        _case(name="plan 16 agents", agents=16, groups=512, len_lo=32, selected=24, new=128),
        # decoding agents fetch their whole context anew for one token: 64 agents, 16 K tokens each
        _case(name="gather for 64 agents", agents=64, groups=1024, capacity=256, len_lo=256, len_hi=256, selected=64,
              new=1, mass="none"),
        # a map kept in 8 bits: four agents, ragged groups, masses of every row
        _case(name="plan int8 map", dtype="i8", agents=4, groups=256, selected=32, new=129, mass="rows"),
        # clustering of 16 new objects against 24 groups, four agents
        _case(name="cluster 16 objects", kind="cluster", agents=4, groups=128, len_lo=32, selected=24, new=256,
              objects=16),
        # an episode's consecutive planning steps when device memory holds a part of the map
        _case(name="plan over the tier", kind="tier", groups=256, len_lo=96, selected=16, new=128, steps=8, scored=True),
        # the decode phase after a plan on the large map: 40 tokens, one at a time
        _case(name="decode after a plan", kind="decode", groups=64, capacity=256, len_lo=256, len_hi=256, selected=32,
              new=40, mass="none"),
        # one decoded token of 64 agents, 16 K tokens of context each, with the masses of its rows
        _case(name="decode 64 agents", kind="decode", agents=64, groups=1024, capacity=256, len_lo=256, len_hi=256,
              selected=64, new=1, mass="rows"),
        # eight new objects of about 20 tokens join their groups
        _case(name="append 8 objects", kind="append", capacity=128, len_hi=96, new=160, objects=8, mass="none"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / 5e14


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        case = _draw(rng)
        if _cost(case) <= limit:
            return case


def _draw(rng):
    kind = rng.choice(["plan", "plan", "plan", "cluster", "tier", "decode", "decode", "append"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "bf16", "i8", "f32"])
    if kind == "tier" and dtype == "i8" or kind == "cluster":
        dtype = "bf16"
    d = rng.choice([64, 128, 128])
    kv = rng.choice([1, 2, 4, 8, 8])
    ratio = rng.choice([1, 2, 3, 4, 4, 7])
    if dtype == "f32":
        # small layers: single precision is for small configurations and for checks
        kv, ratio = rng.choice([1, 2]), rng.choice([1, 2, 4])
    cap = rng.choice([32, 64, 96, 128, 130, 200, 256])
    hi = rng.randint(max(1, 3 * cap // 4), cap)
    lo = rng.randint(hi // 4, hi)
    selected = _log(rng, 2, 8 if dtype == "f32" else 64)
    agents = rng.choice([1, 1, 1, 2, 3, 4, 16])
    new = _log(rng, 16, 512)
    steps, objects, scored, mass = 1, 0, False, rng.choice(["reduced", "reduced", "rows", "none"])
    if dtype == "f32":
        agents, new = min(agents, 2), _log(rng, 4, 129)
    if kind == "plan":
        scored = agents == 1 and rng.random() < 0.4
        if rng.random() < 0.15:
            new = 1
    elif kind == "cluster":
        objects, new, mass = _log(rng, 2, 32), _log(rng, 64, 512), "none"
    elif kind == "tier":
        agents, steps, scored, mass = 1, rng.randint(2, 8), True, "reduced"
        selected = min(selected, 32)
        new = max(new, 48)
    elif kind == "decode":
        agents, new, mass = rng.choice([1, 1, 2, 4, 16, 64]), _log(rng, 1, 40), rng.choice(["none", "none", "rows"])
        if dtype == "f32":
            agents, new = min(agents, 2), min(new, 8)
    elif kind == "append":
        objects = _log(rng, 1, 16)
        new, selected, agents, mass = objects * rng.randint(1, 24), 1, 1, "none"
        cap = max(cap, 64)
        hi = cap - 24
        lo = hi // 2
    groups = max(2 * selected, 2 * objects, _log(rng, 8, 256))
    return _case(kind=kind, dtype=dtype, agents=agents, q_heads=kv * ratio, kv_heads=kv, head_dim=d, groups=groups,
                 capacity=cap, len_lo=lo, len_hi=hi, selected=selected, new=new, scored=scored, mass=mass,
                 objects=objects, steps=steps)


# ---------------------------------------------------------------------------
# what a user's program has in hand
# ---------------------------------------------------------------------------
def _randn(gen, shape, dtype, scale=1.0):
    x = torch.empty(shape, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=DEV)
    x.normal_(generator=gen)
    return x if scale == 1.0 else x.mul_(scale)


def _budget(case):
    """Token budget of Eq. (1) that `selected` groups of average length fill."""
    return case["selected"] * (case["len_lo"] + case["len_hi"]) // 2


def _max_selected(case):
    """The most groups that the budget of Eq. (1) can hold."""
    return min(case["groups"], _budget(case) // max(case["len_lo"], 1) + 1)


def _scores(x):
    """Relevance scores in which at least one group stands above the threshold 0."""
    x = x.astype(np.float32)
    x[0] = abs(x[0]) + 0.125
    return x


def _buffer(case, n_most):
    """Zeros for the gathered keys, or values, of plans of up to `n_most` groups an agent."""
    rows = -(-(n_most * case["capacity"] + case["new"]) // 64) * 64
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    return torch.zeros(case["agents"] * case["kv_heads"] * rows * case["head_dim"], dtype=dt, device=DEV)


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    G, Hkv, C, D, Hq = case["groups"], case["kv_heads"], case["capacity"], case["head_dim"], case["q_heads"]
    Bn, Nq, dt, kind = case["agents"], case["new"], case["dtype"], case["kind"]
    s.lens = rng.integers(case["len_lo"], case["len_hi"] + 1, size=G).astype(np.int32)
    s.base = 10000.0 if dt == "f32" else 500000.0
    s.prepared = dt != "f32" and (Hq // Hkv) * Nq > 32
    if kind == "tier":
        return _prepare_tier(s, gen, rng)

    # ---- the pool ----
    s.scales = None
    if dt == "i8":
        k, v = (torch.randint(-127, 128, (G, Hkv, C, D), dtype=torch.int8, device=DEV, generator=gen) for _ in range(2))
        # codes are uniform: a scale of sqrt(3) / 127 gives values of unit variance
        s.scales = [(torch.rand((G, Hkv, C), device=DEV, generator=gen) * 0.5 + 0.75) * (3.0 ** 0.5 / 127.0)
                    for _ in range(2)]
    else:
        k, v = _randn(gen, (G, Hkv, C, D), dt), _randn(gen, (G, Hkv, C, D), dt)
    act = "f32" if dt == "f32" else "bf16"
    s.q = _randn(gen, (Bn, Nq, Hq, D), act)
    s.k_new, s.v_new = _randn(gen, (Bn, Nq, Hkv, D), act), _randn(gen, (Bn, Nq, Hkv, D), act)
    lists = [rng.choice(G, size=case["selected"], replace=False).astype(np.int32) for _ in range(Bn)]
    if kind == "cluster":
        _plant_objects(s, k, lists, rng)
    s.sel = np.concatenate(lists)
    s.sel_ptr = np.arange(Bn + 1, dtype=np.int32) * case["selected"]
    s.scores = _scores(rng.standard_normal(G))
    n_most = _max_selected(case) if case["scored"] else case["selected"]
    s.pool = B.kv_pool_create(k, v, s.lens, Hq, s.base, n_most * C + Nq)
    if s.scales is not None:
        B.kv_pool_set_scales(s.pool, *s.scales)
    if kind == "append":
        return _prepare_append(s, rng)

    # ---- buffers for the largest selection; a smaller one uses their front ----
    plan = _select(s)
    if kind == "cluster":
        plan.values_from_pool(True)
    s.kc, s.vt = _buffer(case, n_most), _buffer(case, n_most)
    s.q_prep = torch.empty_like(s.q) if s.prepared else None
    s.out = torch.empty_like(s.q)
    s.mass = None
    if case["mass"] == "rows":
        s.mass = torch.zeros((Bn, Nq, Hq, n_most + 1), dtype=torch.float32, device=DEV)
    elif case["mass"] == "reduced":
        s.mass = torch.zeros((Bn, n_most + 1), dtype=torch.float32, device=DEV)
    if kind == "decode":
        # the context is gathered once; the new tokens' rows are filled by the steps
        B.gather_rope(s.pool, plan, torch.zeros_like(s.k_new), torch.zeros_like(s.v_new), s.kc, s.vt)
        s.plan = plan
        s.ws = torch.zeros(max(B.decode_workspace_bytes(s.pool, plan, 1), 256), dtype=torch.uint8, device=DEV)
        s.rows = [[t[:, i:i + 1].contiguous() for t in (s.q, s.k_new, s.v_new)] for i in range(Nq)]
        s.out = torch.zeros((Nq,) + tuple(s.rows[0][0].shape), dtype=s.q.dtype, device=DEV)
        s.outs, s.masses = s.out.unbind(0), [None] * Nq
        if s.mass is not None:
            s.mass = torch.zeros((Nq, Bn, 1, Hq, n_most + 1), dtype=torch.float32, device=DEV)
            s.masses = s.mass.unbind(0)
        return s
    s.ws = B.alloc_workspace(s.pool, plan)
    if kind == "cluster":
        s.spans = np.linspace(0, Nq, case["objects"] + 1).astype(np.int32)
        s.score = torch.zeros((Bn, case["objects"], n_most + 1), dtype=torch.float32, device=DEV)
        s.assign = torch.zeros((Bn, case["objects"]), dtype=torch.int32, device=DEV)
    plan.close()
    return s


def _plant_objects(s, k, lists, rng):
    """Every group has a direction of its own in the slowly rotating coordinates, which its keys lean to; the
    tokens of a new object lean to the direction of one of the agent's groups, the one it belongs to."""
    case = s.case
    D, n_obj = case["head_dim"], case["objects"]
    slow = np.r_[3 * D // 8:D // 2, 7 * D // 8:D]
    u = np.zeros((case["groups"], D), np.float32)
    u[:, slow] = rng.choice([-1.0, 1.0], size=(case["groups"], len(slow))) / np.sqrt(len(slow))
    u = torch.from_numpy(u).to(DEV)
    lean = (6.0 * D ** 0.5) ** 0.5
    k += (lean * u).to(k.dtype)[:, None, None, :]
    spans = np.linspace(0, case["new"], n_obj + 1).astype(np.int32)
    for b in range(case["agents"]):
        of = rng.choice(lists[b], size=n_obj)
        for o in range(n_obj):
            s.q[b, spans[o]:spans[o + 1]] += (lean * u[of[o]]).to(s.q.dtype)


def _prepare_append(s, rng):
    case = s.case
    s.groups = rng.choice(case["groups"], size=case["objects"], replace=False).astype(np.int64)
    n = case["new"] // case["objects"]
    s.parts = [(int(g), s.k_new[0, i * n:(i + 1) * n].contiguous(), s.v_new[0, i * n:(i + 1) * n].contiguous())
               for i, g in enumerate(s.groups)]
    return s


def _prepare_tier(s, gen, rng):
    case = s.case
    G, Hkv, C, D, Hq, Nq = (case[f] for f in ("groups", "kv_heads", "capacity", "head_dim", "q_heads", "new"))
    dt = _DTYPES[case["dtype"]]
    # slots for a quarter more than the largest selection
    n_slots = min(G, _max_selected(case) * 5 // 4 + 1)
    k, v = (torch.zeros((n_slots, Hkv, C, D), dtype=dt, device=DEV) for _ in range(2))
    s.tier = B.kv_tier_create(k, v, G, Hq, s.base, _max_selected(case) * C + Nq)
    ks, vs = (_randn(gen, (G, Hkv, C, D), case["dtype"]).cpu() for _ in range(2))
    for g in range(G):
        n = int(s.lens[g])
        B.kv_tier_put(s.tier, g, ks[g, :, :n].contiguous(), vs[g, :, :n].contiguous())
    s.q = _randn(gen, (1, Nq, Hq, D), case["dtype"])
    s.k_new, s.v_new = _randn(gen, (1, Nq, Hkv, D), case["dtype"]), _randn(gen, (1, Nq, Hkv, D), case["dtype"])
    # relevance scores that change little between adjacent steps
    rho = 0.98
    s.scores = [rng.standard_normal(G)]
    for _ in range(case["steps"] - 1):
        s.scores.append(rho * s.scores[-1] + math.sqrt(1.0 - rho * rho) * rng.standard_normal(G))
    s.scores = [_scores(x) for x in s.scores]
    s.kc, s.vt = _buffer(case, _max_selected(case)), _buffer(case, _max_selected(case))
    s.q_prep = torch.empty_like(s.q) if s.prepared else None
    s.out = torch.zeros((case["steps"],) + tuple(s.q.shape), dtype=s.q.dtype, device=DEV)
    s.mass = torch.zeros((case["steps"], _max_selected(case) + 1), dtype=torch.float32, device=DEV)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _select(s):
    case = s.case
    if case["scored"]:
        return B.segment_select_scored(s.pool, s.scores, 0.0, _budget(case), case["new"])[1]
    return B.segment_select(s.pool, s.sel, s.sel_ptr, case["new"])


def run(s):
    return {"plan": _run_plan, "cluster": _run_cluster, "tier": _run_tier, "decode": _run_decode,
            "append": _run_append}[s.case["kind"]](s)


def _attend(s, pool, plan, ws, out, mode, mass):
    if s.prepared:
        B.segmented_prefill_attention_prepared(pool, plan, s.q_prep, s.kc, s.vt, out, ws,
                                               mass if mode == "reduced" else None)
    else:
        B.segmented_prefill_attention(pool, plan, s.q, s.kc, s.vt, out, ws)
        if mode == "reduced":
            B.segment_attention_mass(pool, plan, ws, 1, mass)
    if mode == "rows":
        B.segment_attention_mass(pool, plan, ws, 0, mass)


def _gather(s, pool, plan):
    if s.prepared:
        B.gather_rope_queries(pool, plan, s.k_new, s.v_new, s.q, s.kc, s.vt, s.q_prep)
    else:
        B.gather_rope(pool, plan, s.k_new, s.v_new, s.kc, s.vt)


def _run_plan(s):
    plan = _select(s)
    _gather(s, s.pool, plan)
    _attend(s, s.pool, plan, s.ws, s.out, s.case["mass"], s.mass)
    plan.close()
    return {"out": s.out, "mass": s.mass, "context": (s.kc, s.vt)}


def _run_cluster(s):
    plan = _select(s)
    plan.values_from_pool(True)
    _gather(s, s.pool, plan)
    _attend(s, s.pool, plan, s.ws, s.out, "none", None)
    B.segment_cluster_assign(s.pool, plan, s.ws, s.spans, s.score, s.assign, threshold=0.02)
    plan.close()
    return {"out": s.out, "score": s.score, "assign": s.assign}


def _run_tier(s):
    case = s.case
    groups = B.kv_tier_select_scored(s.tier, s.scores[0], 0.0, _budget(case))
    for t in range(case["steps"]):
        slots = B.kv_tier_fetch(s.tier, groups)
        plan = B.segment_select(s.tier.pool, slots, [0, len(slots)], case["new"])
        ws = B.alloc_workspace(s.tier.pool, plan)
        _gather(s, s.tier.pool, plan)
        B.kv_tier_fence(s.tier)
        if t + 1 < case["steps"]:
            groups = B.kv_tier_select_scored(s.tier, s.scores[t + 1], 0.0, _budget(case))
            B.kv_tier_prefetch(s.tier, groups)
        _attend(s, s.tier.pool, plan, ws, s.out[t], "reduced", s.mass[t])
        plan.close()
    return {"out": s.out, "mass": s.mass, "context": (s.kc, s.vt)}


def _run_decode(s):
    for i, (q, k, v) in enumerate(s.rows):
        B.segmented_decode_step(s.pool, s.plan, i, q, k, v, s.kc, s.vt, s.outs[i], s.ws, mass_out=s.masses[i])
    return {"out": s.out, "mass": s.mass, "context": (s.kc, s.vt)}


def _run_append(s):
    for g, k, v in s.parts:
        B.kv_pool_append(s.pool, g, k, v)
    for g, _, _ in s.parts:              # the groups as they were, for the next pass
        B.kv_pool_set_len(s.pool, g, int(s.lens[g]))
    return {"k": s.pool.k, "v": s.pool.v, "scales": s.scales}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Expected bytes and operations (lengths at their mean): pool rows of the distinct selected groups, the new
    tokens and the queries read once, outputs, masses and (where a decode phase reads it afterwards) the context
    written once; 4 Hq D operations per visible (query, key) pair."""
    L = (case["len_lo"] + case["len_hi"]) / 2
    Bn, Nq, Hq, Hkv, D, S = (case[f] for f in ("agents", "new", "q_heads", "kv_heads", "head_dim", "selected"))
    es = 4 if case["dtype"] == "f32" else 2
    row_pool = 2 * Hkv * (D * (1 if case["dtype"] == "i8" else es) + (4 if case["dtype"] == "i8" else 0))
    row_ctx = 2 * Hkv * D * es
    if case["kind"] == "append":
        n = case["new"] // case["objects"] * case["objects"]
        return {"bytes": n * (row_ctx + row_pool), "flops": 0}
    Lc = S * L
    qo = 2 * Bn * Nq * Hq * D * es
    fresh = Bn * Nq * row_ctx
    n_mass = {"rows": Bn * Nq * Hq * (S + 1), "reduced": Bn * (S + 1), "none": 0}[case["mass"]]
    flops = 4 * Hq * D * Bn * (Nq * Lc + Nq * (Nq + 1) / 2)
    if case["kind"] == "decode":
        # every token reads the context before it once
        ctx = Bn * (Nq * Lc + Nq * (Nq + 1) / 2) * row_ctx
        return {"bytes": ctx + 2 * fresh + qo + 4 * n_mass, "flops": flops}
    distinct = case["groups"] * (1 - (1 - S / case["groups"]) ** Bn)
    n = distinct * L * row_pool + fresh + qo + 4 * n_mass
    if case["kind"] == "plan":
        n += Bn * (Lc + Nq) * row_ctx
    elif case["kind"] == "cluster":
        n += 4 * Bn * case["objects"] * (S + 2)
    return {"bytes": n * case["steps"], "flops": flops * case["steps"]}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    # keys, queries, probabilities and outputs are rounded to bf16; the objects' groups are told apart by far more
    return {"rel": 1e-2}
