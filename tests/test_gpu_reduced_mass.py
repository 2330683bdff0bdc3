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


@pytest.mark.parametrize("dtype,n_new,splits", [(I.BF16, 7, 2), (I.BF16, 40, 2), (I.BF16, 65, 7), (I.F32, 9, 1)])
def test_reduced_masses_of_a_query_that_is_no_number(step_mod, dtype, n_new, splits):
    """The sums that hold its masses are NaN too, the other agent's are as before; the next call, without it, is
    free of it."""
    cfg = small(f"nan-{n_new}", 870 + n_new, dtype=dtype, n_agents=2, n_q_heads=6, head_dim=64, len_lo=8, n_new=n_new,
                rope_base=1e4)
    st = step_mod.PlanningStep(I.make_workload(cfg), n_splits=splits)

    def reduced():
        st.gather()
        st.attention()
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
