"""Gathers whose workgroups take several heads one after the other, and long contexts of agents that share groups, whose
tiles are gathered in the order of the groups: bit for bit the contexts of the agents gathered one by one."""
import numpy as np
import pytest

from paper_2510_18546_amd import binding as B

pytestmark = pytest.mark.gpu


def make(agents, kv, groups, cap, lo, hi, picks, n_new, seed=5, ratio=8, d=128):
    import torch
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    lens = rng.integers(lo, hi + 1, groups).astype(np.int32)
    lens[:: 7] = 0
    k, v = (torch.randn((groups, kv, cap, d), device="cuda:0", generator=gen).to(torch.bfloat16) for _ in range(2))
    # agents of different numbers of groups, one of them without any
    sel = [rng.choice(groups, 0 if b == 1 else int(rng.integers(picks // 2, picks + 1)), replace=False).astype(np.int32)
           for b in range(agents)]
    k_new, v_new = (torch.randn((agents, n_new, kv, d), device="cuda:0", generator=gen).to(torch.bfloat16) for _ in range(2))
    q = torch.randn((agents, n_new, kv * ratio, d), device="cuda:0", generator=gen).to(torch.bfloat16)
    pool = B.kv_pool_create(k, v, lens, kv * ratio, 5e5, picks * cap + n_new)
    return pool, lens, sel, k_new, v_new, q


def gather(pool, sel, k_new, v_new, q, from_pool):
    import torch
    plan = B.segment_select(pool, np.concatenate(sel), np.cumsum([0] + [len(x) for x in sel]), k_new.shape[1])
    if from_pool:
        plan.values_from_pool(True)
    kc, vt = B.alloc_context(pool, plan)
    kc, vt = kc.view(torch.int16).fill_(7), vt.view(torch.int16).fill_(7)
    q_prep = torch.empty_like(q)
    B.gather_rope_queries(pool, plan, k_new, v_new, q, kc, vt, q_prep)
    return plan, kc, vt, q_prep


def n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def route(plan, kv, lens, sel, n_new, q_heads, from_pool):
    """How a bf16 gather of rows of 128 values goes, by the rules of the library: in the order of the groups or not, past the
    caches or not, heads a workgroup, with loads ahead or not."""
    agents, tiles = len(sel), -(-plan.info.max_ctx_len // 64)
    cached = [sum(int(lens[g]) for g in s) for s in sel]
    tokens, used = sum(cached) + agents * n_new, np.bincount(np.concatenate(sel), minlength=len(lens))
    size = 512 * agents * kv * plan.info.ctx_stride
    distinct, own = lens[used > 0].sum(), agents * n_new + lens[used == 1].sum()
    stream, rows, queries = size > 256 << 20, tokens * kv * (1 if from_pool else 2), agents * n_new * q_heads
    saved = (sum(cached) - distinct) * kv * (256 if from_pool else 512)
    order = (size >= 768 << 20 and 3 * own <= tokens and saved >= 400000 * (used > 0).sum() * (1 + 10 * queries / rows) and
             sum(cached) >= (2 if size < 1 << 30 else 1.5) * distinct and
             not (from_pool and sum(cached) * kv * 256 < 160000 * sum(map(len, sel))))
    work = (1 if from_pool else 2) * kv * tiles * agents
    heads = 8 if 6 * queries < rows else 4
    if not stream:
        heads = 2 if work > 32 * n_cu() else 1 if tiles < 24 else 2 if agents >= 6 and tiles < 60 else 4 if agents > 2 else heads
    while heads > 1 and (kv % heads or 4 * work < 5 * heads * n_cu()):
        heads //= 2
    if (order or size < 768 << 20) and (heads == 1 or 2 * queries < (3 if stream else 2) * rows):
        return order, stream, heads, True
    heads = max(h for h in (1, 2, 4, 8) if h == 1 or kv % h == 0 and kv // h * (1 + h) * tiles * agents >= 32 * n_cu())
    return False, stream, heads, False


# (order, past the caches, heads, ahead) as `route` says it: contexts of 768 MB and more in order; two that share too little,
# agent by agent; smaller ones; and launches that are mostly queries, agent by agent too
@pytest.mark.parametrize("agents,kv,groups,cap,lo,hi,picks,n_new,from_pool,how", [
    (24, 8, 60, 256, 200, 256, 50, 5, False, (True, True, 8, True)), (24, 8, 60, 256, 200, 256, 50, 130, True, (True, True, 8, True)),
    (40, 3, 90, 512, 300, 512, 48, 70, False, (True, True, 1, True)), (100, 1, 80, 1000, 500, 1000, 70, 5, False, (True, True, 1, True)),
    (130, 8, 130, 32, 1, 32, 120, 64, False, (True, True, 4, True)), (90, 2, 60, 256, 200, 256, 50, 5, False, (True, True, 2, True)),
    (14, 8, 700, 512, 300, 512, 42, 5, False, (False, True, 8, False)), (60, 2, 3000, 512, 300, 512, 42, 33, True, (False, True, 2, False)),
    (25, 8, 30, 70, 30, 70, 20, 129, False, (False, False, 1, True)), (4, 8, 64, 130, 60, 130, 40, 100, False, (False, False, 4, True)),
    (3, 2, 40, 64, 10, 64, 33, 17, False, (False, False, 1, True)), (30, 8, 60, 130, 100, 130, 14, 1, False, (False, False, 2, True)),
    (30, 8, 64, 64, 30, 64, 8, 512, False, (False, False, 1, True)), (3, 8, 40, 130, 100, 130, 30, 129, False, (False, False, 4, True)),
    (1, 8, 170, 200, 150, 200, 160, 5, False, (False, False, 8, True)), (7, 8, 60, 130, 100, 130, 20, 1, False, (False, False, 2, True)), (64, 8, 64, 30, 1, 30, 2, 900, False, (False, False, 8, False)),
    (190, 2, 64, 30, 1, 30, 2, 900, False, (False, False, 2, False)), (100, 8, 40, 64, 30, 64, 40, 500, True, (False, True, 8, False))])
def test_same_contexts_as_one_by_one(agents, kv, groups, cap, lo, hi, picks, n_new, from_pool, how):
    import torch
    pool, lens, sel, k_new, v_new, q = make(agents, kv, groups, cap, lo, hi, picks, n_new)
    plan, kc, vt, q_prep = gather(pool, sel, k_new, v_new, q, from_pool)
    assert route(plan, kv, lens, sel, n_new, 8 * kv, from_pool) == how
    T = plan.info.ctx_stride
    kc = kc.view(agents, kv, T, 128)
    table = vt.view(torch.int64)[:agents * kv * T].view(agents, kv, T) if from_pool else None
    vt = vt[:agents * kv * 128 * T].view(agents, kv, 128, T)
    for b in range(agents):
        p1, k1, v1, q1 = gather(pool, [sel[b]], k_new[b:b + 1], v_new[b:b + 1], q[b:b + 1], False)
        t1 = p1.info.ctx_stride
        k1, v1 = k1.view(kv, t1, 128), v1.view(kv, 128, t1)
        assert torch.equal(kc[b, :, :t1], k1), b
        assert bool((kc[b, :, t1:] == 7).all()), b
        assert torch.equal(q_prep[b:b + 1].view(torch.int16), q1.view(torch.int16)), b
        if not from_pool:
            assert torch.equal(vt[b, :, :, :t1], v1), b
            assert bool((vt[b, :, :, t1:] == 7).all()), b
            continue
        # the table of row addresses: the pool's rows, then the new tokens' rows, then one and the same row
        at = [pool.v.data_ptr() + 256 * ((int(g) * kv + h) * cap + t) for h in range(kv) for g in sel[b] for t in range(lens[g])]
        at = np.array(at, np.int64).reshape(kv, -1)
        new = np.array([[v_new.data_ptr() + 256 * ((b * n_new + i) * kv + h) for i in range(n_new)] for h in range(kv)], np.int64)
        want = np.concatenate([at, new], 1)
        got = table[b, :, :t1].cpu().numpy()
        np.testing.assert_array_equal(got[:, :want.shape[1]], want)
        assert len(np.unique(got[:, want.shape[1]:])) <= 1
        p1.close()
    plan.close()


# 8-bit pools: contexts that go past the caches, four, two or one heads a workgroup; the others two heads for the agents
# together, one for each by itself
@pytest.mark.parametrize("agents,kv,d,cap,n_new,heads", [
    (9, 8, 128, 130, 70, 4), (17, 2, 128, 256, 1, 2), (18, 6, 64, 200, 33, 2), (25, 3, 128, 130, 70, 1), (30, 4, 64, 200, 130, 4),
    (3, 8, 128, 130, 40, 2), (4, 6, 64, 130, 129, 2), (2, 8, 64, 130, 1, 2)])
def test_same_contexts_from_8_bit_pools(agents, kv, d, cap, n_new, heads):
    import torch
    rng = np.random.default_rng(agents)
    gen = torch.Generator(device="cuda:0").manual_seed(agents)
    groups, picks = 140, 90
    lens = rng.integers(cap - 30, cap + 1, groups).astype(np.int32)
    lens[::9] = 0
    k, v = (torch.randint(-127, 128, (groups, kv, cap, d), dtype=torch.int8, device="cuda:0", generator=gen) for _ in range(2))
    scales = [torch.rand((groups, kv, cap), device="cuda:0", generator=gen) + 0.01 for _ in range(2)]
    k_new, v_new = (torch.randn((agents, n_new, kv, d), device="cuda:0", generator=gen).to(torch.bfloat16) for _ in range(2))
    q = torch.randn((agents, n_new, kv, d), device="cuda:0", generator=gen).to(torch.bfloat16)
    pool = B.kv_pool_create(k, v, lens, kv, 1e4, picks * cap + n_new)
    B.kv_pool_set_scales(pool, *scales)
    sel = [rng.choice(groups, 0 if b == 1 else picks - b % 3, replace=False).astype(np.int32) for b in range(agents)]
    plan, kc, vt, q_prep = gather(pool, sel, k_new, v_new, q, False)
    T = plan.info.ctx_stride
    past = 4 * agents * kv * T * d > 256 << 20
    assert heads == max(h for h in (1, 2, 4) if h == 1 or kv % h == 0 and (past if h == 4 else past or 2 * kv * T // 64 * agents >= (18 if d == 128 else 16) * n_cu()))
    kc, vt = kc.view(agents, kv, T, d), vt.view(agents, kv, d, T)
    # the values of agent 0 are code x scale in float32, rounded once; token j in the column with its bits 2 and 3 exchanged
    rows = torch.from_numpy(np.concatenate([g * cap + np.arange(lens[g]) for g in sel[0]])).cuda()
    v0 = (v.float() * scales[1][..., None]).to(torch.bfloat16).transpose(0, 1).reshape(kv, groups * cap, d)[:, rows]
    v0 = torch.cat([v0, v_new[0].transpose(0, 1)], 1)
    j = torch.arange(v0.shape[1], device="cuda:0")
    col = (j & ~12) | ((j & 4) << 1) | ((j & 8) >> 1)
    assert torch.equal(vt[0][:, :, col], v0.transpose(1, 2).contiguous().view(torch.int16))
    for b in range(agents):
        p1, k1, v1, q1 = gather(pool, [sel[b]], k_new[b:b + 1], v_new[b:b + 1], q[b:b + 1], False)
        t1 = p1.info.ctx_stride
        assert torch.equal(kc[b, :, :t1], k1.view(kv, t1, d)), b
        assert torch.equal(vt[b, :, :, :t1], v1.view(kv, d, t1)), b
        assert torch.equal(q_prep[b:b + 1].view(torch.int16), q1.view(torch.int16)), b
        assert bool((kc[b, :, t1:] == 7).all()) and bool((vt[b, :, :, t1:] == 7).all()), b
        p1.close()
    plan.close()
