"""The reduced masses where their pieces meet: units of 64 query rows of a head, four to a workgroup, eight
buckets each; steps of few rows, whose workgroups hold several heads; heads and buckets that do not fill the last
workgroup; buckets within one split, over two and over more. Against the oracle, to the tolerances of
test_gpu_parity, as part of the attention call and as a call of its own. And the masses of every row, whose sums
are exact where all scores are 0."""
import numpy as np
import pytest

from paper_2510_18546_amd import inputs as I
from test_gpu_parity import run_case, small, step_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,heads,kv,n_new,n_sel,splits", [
    (I.BF16, 10, 2, 7, 6, 2),        # the last step that the kernel for few rows takes
    (I.BF16, 10, 2, 8, 8, 2),        # the first that is added up beside the merge: two idle waves, one bucket more than a group
    (I.BF16, 7, 1, 63, 7, 3),        # units of 63 rows; eight buckets exactly
    (I.BF16, 5, 1, 64, 5, 7),        # buckets over more than two splits
    (I.BF16, 6, 2, 65, 9, 2),        # a second unit of one row per head
    (I.BF16, 6, 2, 40, 3, 1),        # one split: no merge launch
    (I.F32, 3, 1, 8, 9, 2),
    (I.F32, 3, 3, 66, 2, 1),
    (I.BF16, 35, 5, 65, 9, 7),       # more than 2048 (head, row) pairs: the call of its own in two launches
    (I.F32, 33, 3, 66, 8, 1),
])
def test_reduced_masses_of_few_rows(step_mod, oracle, dtype, heads, kv, n_new, n_sel, splits):
    cfg = small(f"reduced-{n_new}-{n_sel}", 800 + n_new, dtype=dtype, n_agents=2, n_q_heads=heads, n_kv_heads=kv,
                head_dim=64, len_lo=0, n_sel=n_sel, n_new=n_new, rope_base=1e4)
    st, _, _, _ = run_case(step_mod, oracle, cfg, n_splits=splits)
    red = st.mass_red_host()
    st.mass_red.fill_(float("nan"))
    st.masses(1)                     # the same sums once more, from the scratch that the attention call left
    # both are sums of the same masses in float32, in another order: the sum of n numbers of one sign is off by at
    # most n 2^-24 of itself (at most 128 terms per float sum, the rest is added up exactly)
    np.testing.assert_allclose(st.mass_red_host(), red, rtol=2.0 ** -16, atol=2.0 ** -30)


@pytest.mark.parametrize("dtype,n_new,n_sel,splits", [
    (I.F32, 15, 5, 1), (I.F32, 16, 5, 1), (I.F32, 70, 18, 2), (I.BF16, 40, 5, 1), (I.BF16, 65, 16, 2),
    (I.BF16, 130, 3, 7)])
def test_masses_of_queries_without_direction(step_mod, dtype, n_new, n_sel, splits):
    """All scores are 0, every exponential is 1, the sums count keys: a mass is the one quotient of the segment's
    keys and the row's, rounded once. (15 and 16 rows per head: either side of the border between the two kernels.)"""
    cfg = small(f"even-{n_new}-{n_sel}", 830 + n_new, dtype=dtype, n_agents=2, n_q_heads=4, head_dim=64, n_groups=24,
                len_lo=0, n_sel=n_sel, n_new=n_new, rope_base=1e4)
    st = step_mod.PlanningStep(I.make_workload(cfg), n_splits=splits)
    st.q.zero_()
    st.run()
    mass = st.mass_host()
    for b in range(cfg.n_agents):
        off = st.plan.offsets(b)
        for i in range(n_new):
            keys = np.append(np.diff(off), i + 1).astype(np.float32)
            want = keys / np.float32(off[-1] + i + 1)
            np.testing.assert_array_equal(mass[b, i], np.broadcast_to(want.astype(np.float64), mass[b, i].shape))


def test_masses_of_many_agents_and_segments(step_mod, oracle):
    # agents x chunks of 16 buckets: 4100 x 16, more than a grid's second and third dimensions hold
    cfg = small("many-agents-segments", 860, dtype=I.F32, n_agents=4100, n_q_heads=1, n_kv_heads=1, head_dim=64,
                n_groups=256, capacity=1, len_lo=0, len_hi=1, n_sel=240, n_new=16, rope_base=1e4)
    rows = np.array([(b, i, 0) for b in (0, 2049, 4095, 4096, 4099) for i in range(16)], dtype=np.int32)
    run_case(step_mod, oracle, cfg, rows=rows)


@pytest.mark.parametrize("dtype,n_new,splits", [
    (I.F32, 3, 1), (I.F32, 9, 1), (I.F32, 70, 3), (I.BF16, 8, 2), (I.BF16, 40, 1), (I.BF16, 130, 2), (I.BF16, 350, 2),
    (I.F32, 350, 1)])
def test_reduced_masses_of_a_segment_far_off(step_mod, dtype, n_new, splits):
    """A segment whose scores lie 30 below the others, masses of about 1e-14 a row: their sum is as exact as that of
    the large ones."""
    cfg = small(f"far-{n_new}", 890 + n_new, dtype=dtype, n_agents=2, n_q_heads=6, head_dim=64, n_new=n_new)
    w = I.make_workload(cfg)
    far, slow = int(w.sel[2]), cfg.head_dim // 2 - 1       # (that pair turns by 3e-6 a token)
    lean = np.float32((30.0 * 8.0) ** 0.5)
    for x, along in ((w.q, lean), (w.k_new, 0), (w.k_pool, 0), (w.k_pool[far], -lean)):
        x[..., slow], x[..., -1] = along, 0
    st = step_mod.PlanningStep(w, n_splits=splits)
    st.gather()
    st.attention()
    st.masses(0)
    st.masses(1)
    red, rows = st.mass_red_host(), st.mass_host().sum(axis=(1, 2))
    assert 1e-16 < rows[0, 2] < 1e-9
    # row masses in float32 (three roundings each, two in the sums), added up in a tree of at most 6 + 2 + 3 levels
    # of a row, then at most four in a line: below 32 roundings
    np.testing.assert_allclose(red, rows, rtol=32 * 2.0 ** -24, atol=0)


@pytest.mark.parametrize("rows,step", [(4032, 2.0 ** -34), (4160, 0.0)])
def test_reduced_masses_of_a_long_step(step_mod, rows, step):
    """64 heads: as many units as an accumulator's count can tell apart (1008 workgroups; sums in steps of 2^-34), and
    more (no accumulators). Every row gives the second segment 2^-38."""
    import torch
    from paper_2510_18546_amd import binding as B
    hq, cached, d, dev = 64, 8192, 64, "cuda:0"
    k = torch.zeros((2, 1, cached, d), dtype=torch.bfloat16, device=dev)
    q = torch.zeros((1, rows, hq, d), dtype=torch.bfloat16, device=dev)
    lean = (25 * np.log(2.0) * d ** 0.5) ** 0.5
    q[..., d // 2 - 1], k[1, 0, 0, d // 2 - 1] = lean, -lean
    pool = B.kv_pool_create(k, k.clone(), np.array([cached, 1], np.int32), hq, 500000.0, cached + 1 + rows)
    plan = B.segment_select(pool, np.array([0, 1], np.int32), np.array([0, 2], np.int32), rows)
    plan.set_splits(2)
    kc, vt = B.alloc_context(pool, plan)
    new, q_prep, out = torch.zeros((1, rows, 1, d), dtype=torch.bfloat16, device=dev), torch.empty_like(q), torch.empty_like(q)
    ws = B.alloc_workspace(pool, plan)
    in_call, by_itself = (torch.zeros((1, 3), device=dev) for _ in range(2))
    of_rows = torch.zeros((1, rows, hq, 3), device=dev)
    B.gather_rope_queries(pool, plan, new, new, q, kc, vt, q_prep)
    B.segmented_prefill_attention_prepared(pool, plan, q_prep, kc, vt, out, ws, in_call)
    B.segment_attention_mass(pool, plan, ws, 1, by_itself)
    B.segment_attention_mass(pool, plan, ws, 0, of_rows)
    want = of_rows.double().sum(dim=(1, 2)).cpu().numpy()[0]
    assert 3e-7 < want[1] < 2e-6
    # 1008 sums rounded to a step; sums in float32 of at most 6 + 2 + 6 levels and 17 terms in a line
    np.testing.assert_allclose(in_call.cpu().numpy()[0], want, rtol=64 * 2.0 ** -24, atol=1008 * step / 2)
    np.testing.assert_allclose(by_itself.cpu().numpy()[0], want, rtol=64 * 2.0 ** -24, atol=0)


@pytest.mark.parametrize("dtype,n_new,splits,in_call", [
    (I.BF16, 7, 2, False), (I.BF16, 40, 1, False), (I.BF16, 40, 2, False), (I.BF16, 65, 7, False), (I.F32, 9, 1, False),
    (I.BF16, 40, 2, True), (I.BF16, 40, 1, True), (I.BF16, 130, 1, True)])
def test_reduced_masses_of_a_query_that_is_no_number(step_mod, dtype, n_new, splits, in_call):
    """The sums that hold its masses are NaN too, the other agent's are as before; the next call, without it, is
    free of it."""
    cfg = small(f"nan-{n_new}", 870 + n_new, dtype=dtype, n_agents=2, n_q_heads=6, head_dim=64, len_lo=8, n_new=n_new,
                rope_base=1e4)
    st = step_mod.PlanningStep(I.make_workload(cfg), n_splits=splits)

    def reduced():
        st.gather()
        st.attention(in_call)
        if not in_call:
            st.masses(1)
        return st.mass_red_host()

    clean = reduced()
    assert np.isfinite(clean).all()
    q = st.q.clone()
    st.q[1, n_new // 2, 3] = float("nan")
    dirty = reduced()
    assert np.isnan(dirty[1]).all()
    np.testing.assert_array_equal(dirty[0], clean[0])
    st.q.copy_(q)
    np.testing.assert_array_equal(reduced(), clean)
