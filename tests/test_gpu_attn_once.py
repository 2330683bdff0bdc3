"""Decode steps whose splits are whole in LDS (attn_once_kernel): one to five tiles a split, both head widths, rows up to
16, segments that end anywhere in a wave's 32 keys, more of them than a wave has lanes, agents with fewer tiles than
splits; and steps whose rows cross the borders of 32-key blocks, tiles and splits. Against the oracle, to the tolerances of
every other bf16 case (outputs 2e-2: P and O rounded to bf16, 2^-9 each; masses 1e-2)."""
import numpy as np
import pytest

from paper_2510_18546_amd import inputs as I

pytestmark = pytest.mark.gpu


def workload(seed, agents, r, kv, d, nq, lens, n_sel):
    cap = max(lens)
    cfg = I.Config("once", seed, I.BF16, agents, r * kv, kv, d, len(lens), cap, cap, cap, n_sel, nq, 500000.0)
    w = I.make_workload(cfg)
    w.lens[:] = lens
    for g, n in enumerate(lens):
        w.k_pool[g, :, n:] = w.v_pool[g, :, n:] = np.nan
    return cfg, w


def tiles_of(st, n_rows=None):
    """Key tiles a split of the plan's step in attn_once_kernel, 0: the streaming kernel."""
    import ctypes as C
    from paper_2510_18546_amd import binding as B
    rule = B.load()["_Z18en_attn_once_tilesPK7en_poolPK7en_planii"]
    return rule(st.pool.handle, st.plan.handle, C.c_int(n_rows or st.cfg.n_new), C.c_int(st.plan.info.n_splits))


def both(step, oracle, w, splits, tiles=None):
    import torch
    st = step.PlanningStep(w, n_splits=splits)
    assert tiles_of(st) == tiles if tiles else tiles_of(st) > 0
    st.ws.fill_(0xFF)                            # a NaN pattern: nothing is read that was not written
    print(f"[case] {w.cfg} splits {splits}", flush=True)
    st.run()
    torch.cuda.synchronize()
    out, mass = oracle.attention(w.k_pool, w.v_pool, w.lens, w.sel, w.sel_ptr, w.q, w.k_new, w.v_new, w.cfg.rope_base)
    assert np.abs(st.out_host() - out).max() <= 2e-2
    assert np.abs(st.mass_host() - mass).max() <= 1e-2
    assert np.abs(st.mass_host().sum(-1) - 1.0).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("total,splits", [(40, None), (64, 1), (65, 1), (160, 1), (192, 1), (193, 1), (320, 1), (321, 2), (300, 5), (640, 2),
                                          (700, 3), (1100, None)])
def test_tiles_per_split(oracle, total, splits, d):
    from paper_2510_18546_amd import step
    # one group as long as it takes, behind groups of 0, 1, 31 and 33 tokens
    lens = [0, 1, 31, 33, total - 1 - 65 if total > 70 else 0]
    cfg, w = workload(total, 2, 3, 2, d, 1, lens if total > 70 else [0, 1, 31, total - 33, 0], 5)
    both(step, oracle, w, splits)


@pytest.mark.parametrize("r,nq,d", [(16, 1, 128), (4, 4, 128), (7, 2, 64), (1, 16, 64), (1, 1, 128), (5, 3, 128)])
def test_rows(oracle, r, nq, d):
    from paper_2510_18546_amd import step
    for seed, lens in ((1, [70, 3, 55]), (2, [200, 120, 129]), (3, [32, 32, 0])):
        cfg, w = workload(10 * r + seed, 2, r, 2, d, nq, lens, 3)
        both(step, oracle, w, None)


@pytest.mark.parametrize("d", [64, 128])
def test_many_short_segments(oracle, d):
    """80 segments of 0 to 5 tokens: the bounds do not fit a wave's lanes; several (bucket, row) pairs for each 16 lanes."""
    from paper_2510_18546_amd import step
    lens = [int(x) for x in np.random.default_rng(7).integers(0, 6, 80)]
    cfg, w = workload(31, 3, 4, 2, d, 2, lens, 80)
    both(step, oracle, w, None)


@pytest.mark.parametrize("agents,kv,d,tokens,splits,tiles", [
    (64, 4, 128, 820, 7, 2),       # 3.5 rounds of two workgroups a compute unit
    (128, 4, 128, 240, 2, 2),      # two
    (32, 4, 128, 560, 3, 3),       # 1.5 rounds of one
    (150, 4, 128, 100, 1, 2),      # one split, 1.2 rounds, written out directly
    (256, 4, 64, 240, 2, 2),       # 1.6 rounds of five
    (200, 4, 64, 170, 1, 3),       # 1.04 rounds of three
    (96, 4, 64, 560, 3, 3),        # 1.5
])
def test_several_rounds(oracle, agents, kv, d, tokens, splits, tiles):
    """More workgroups than the chip holds at once, agents of unequal length among them: outputs, masses, merge."""
    from paper_2510_18546_amd import step
    lens = [tokens - 70, 37, 33, 0]
    cfg, w = workload(agents, agents, 2, kv, d, 1, lens, 4)
    lists = [[0, 1, 2, 3], [3, 1], [2], [1, 0], []]
    lists = [np.array(lists[b % 5], np.int32) for b in range(agents)]
    w.sel = np.concatenate(lists)
    w.sel_ptr = np.cumsum([0] + [len(x) for x in lists]).astype(np.int32)
    both(step, oracle, w, splits, tiles)


def test_agents_of_unequal_length(oracle):
    """Agents of one tile beside one of eleven: most of their splits hold nothing."""
    from paper_2510_18546_amd import step
    cfg, w = workload(41, 3, 4, 2, 128, 1, [600, 70, 9], 3)
    lists = [[0, 1], [2], []]
    w.sel = np.concatenate([np.array(x, np.int32) for x in lists]).astype(np.int32)
    w.sel_ptr = np.cumsum([0] + [len(x) for x in lists]).astype(np.int32)
    for splits in (None, 3, 6):
        both(step, oracle, w, splits)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cached,steps", [(30, (1, 1, 1, 4)), (61, (2, 4, 1)), (126, (4, 4)), (318, (1, 1, 1, 4)), (637, (4, 1, 1, 2))])
def test_steps_across_borders(oracle, cached, steps, d):
    """Rows appended to a gathered context: outputs of every step, and the context as a gather of all rows leaves it."""
    import torch
    from paper_2510_18546_amd import binding as B
    from paper_2510_18546_amd import step
    n = sum(steps)
    cfg, w = workload(cached, 2, 4, 2, d, n, [cached - 20, 20], 2)
    st = step.PlanningStep(w)
    print(f"[case] {cfg} steps {steps}", flush=True)
    ref, _ = oracle.attention(w.k_pool, w.v_pool, w.lens, w.sel, w.sel_ptr, w.q, w.k_new, w.v_new, cfg.rope_base)
    B.gather_rope(st.pool, st.plan, torch.zeros_like(st.k_new), torch.zeros_like(st.v_new), st.kc, st.vt)
    q0 = 0
    for m in steps:
        q, k, v = (t[:, q0:q0 + m].contiguous() for t in (st.q, st.k_new, st.v_new))
        out = torch.empty_like(q)
        ws = torch.empty(max(B.decode_workspace_bytes(st.pool, st.plan, m), 256), dtype=torch.uint8, device="cuda:0").fill_(0xFF)
        B.segmented_decode_step(st.pool, st.plan, q0, q, k, v, st.kc, st.vt, out, ws)
        torch.cuda.synchronize()
        assert np.abs(step._to_host(out) - ref[:, q0:q0 + m]).max() <= 2e-2
        q0 += m
    kc, vt = st.kc.clone(), st.vt.clone()
    B.gather_rope(st.pool, st.plan, st.k_new, st.v_new, st.kc, st.vt)
    assert torch.equal(vt, st.vt)                # values are copies
    # rotated keys differ by which of two products is rounded, then by one rounding to bf16 of values up to 4
    diff = kc.view(torch.bfloat16).float() - st.kc.view(torch.bfloat16).float()
    assert diff.abs().max().item() <= 4e-2


@pytest.mark.parametrize("d", [64, 128])
def test_no_scratch_for_many_short_contexts(oracle, d):
    """As many (agent, KV head) pairs as the streaming kernel gives one split of two waves, over contexts of which this
    kernel would rather have several splits: one, which needs no scratch, still does for a call that brings none."""
    import torch
    from paper_2510_18546_amd import binding as B
    from paper_2510_18546_amd import step
    cfg, w = workload(51, 256, 2, 2, d, 2, [100, 70] if d == 128 else [200, 170], 2)
    print(f"[case] {cfg}", flush=True)
    st = step.PlanningStep(w)
    assert st.plan.info.n_splits > 1
    ref, ref_mass = oracle.attention(w.k_pool, w.v_pool, w.lens, w.sel, w.sel_ptr, w.q, w.k_new, w.v_new, cfg.rope_base)
    st.ws.fill_(0xFF)
    st.run()                                     # in more than one round of workgroups
    torch.cuda.synchronize()
    assert np.abs(st.out_host() - ref).max() <= 2e-2
    assert np.abs(st.mass_host() - ref_mass).max() <= 1e-2
    st.gather()
    B.segmented_prefill_attention(st.pool, st.plan, st.q, st.kc, st.vt, st.out, None)
    torch.cuda.synchronize()
    assert np.abs(st.out_host() - ref).max() <= 2e-2
    q, k, v = (t[:, :1].contiguous() for t in (st.q, st.k_new, st.v_new))
    out = torch.empty_like(q)
    B.segmented_decode_step(st.pool, st.plan, 0, q, k, v, st.kc, st.vt, out, None)
    torch.cuda.synchronize()
    assert np.abs(step._to_host(out) - ref[:, :1]).max() <= 2e-2
    st.plan.set_splits(2)
    with pytest.raises(B.EnError, match="workspace required"):
        B.segmented_prefill_attention(st.pool, st.plan, st.q, st.kc, st.vt, st.out, None)


def _run(step, w, splits):
    import torch
    st = step.PlanningStep(w, n_splits=splits)
    st.ws.fill_(0xFF)
    st.run()
    torch.cuda.synchronize()
    return st.out_host(), st.mass_host()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("splits", [1, 3])
def test_not_finite(oracle, splits, d):
    """NaN and infinity stay in what is computed from them: a query's in its row, a key's in the rows of its KV head, a
    value's in its element of them, whatever the key's weight is. Everything else has the bits of the clean run."""
    from paper_2510_18546_amd import step
    cfg, w = workload(61, 2, 3, 2, d, 1, [150, 149], 2)
    print(f"[case] {cfg} splits {splits}", flush=True)
    out0, mass0 = _run(step, w, splits)
    assert np.isfinite(out0).all() and np.isfinite(mass0).all()

    q = w.q.copy()
    w.q[1, 0, 4, 5] = np.nan
    out, mass = _run(step, w, splits)
    assert np.isnan(out[1, 0, 4]).all() and np.isnan(mass[1, 0, 4]).all()
    out[1, 0, 4], mass[1, 0, 4] = out0[1, 0, 4], mass0[1, 0, 4]
    assert np.array_equal(out, out0) and np.array_equal(mass, mass0)
    w.q[:] = q

    # a key of a group that both agents hold, in KV head 1
    for bad in (np.nan, np.inf):
        k = w.k_pool.copy()
        w.k_pool[0, 1, 40, 7] = bad
        out, mass = _run(step, w, splits)
        rows = slice(3, 6)
        # (an infinite key is turned: infinite in two dimensions; a row's score is either infinity or NaN)
        low = ~np.isnan(out[:, :, rows]).any(-1)
        assert not low.any() or (bad == np.inf and np.isfinite(out[:, :, rows][low]).all())
        assert low.mean() < 1.0
        assert np.array_equal(out[:, :, :3], out0[:, :, :3]) and np.array_equal(mass[:, :, :3], mass0[:, :, :3])
        w.k_pool[:] = k

    # a value, under its key's usual weight and under a weight that underflows
    for bad in (np.nan, np.inf):
        for far in (False, True):
            k, v = w.k_pool.copy(), w.v_pool.copy()
            if far:                                  # (towards no row's query: the slowest pair, against every query)
                w.q[..., d // 2 - 1] = 8.0
                w.k_pool[0, 1, 40] = 0
                w.k_pool[0, 1, 40, d // 2 - 1] = -3000.0
            base, mbase = _run(step, w, splits)
            w.v_pool[0, 1, 40, 9] = bad
            out, mass = _run(step, w, splits)
            assert not np.isfinite(out[:, :, 3:6, 9]).any(), (bad, far)
            out[:, :, 3:6, 9] = base[:, :, 3:6, 9]
            assert np.array_equal(out, base) and np.array_equal(mass, mbase), (bad, far)
            w.q[:], w.k_pool[:], w.v_pool[:] = q, k, v
