"""Where a gather finds its rows: agents' tables that the lanes of a wave hold (up to 62 segments), that are staged in
LDS (up to 254) and that are read where they are, with empty segments, many to a tile and across tiles, agents without any,
and agents that end within a wave's tokens. Values bit for bit, rotated keys to a rounding of the context's type."""
import numpy as np
import pytest

from paper_2510_18546_amd import inputs as I
from test_gpu_parity import announce, small, step_mod  # noqa: F401
from test_gpu_q8 import Q8Step, quantised_pool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f32", "bf16", "pool", "i8"])
@pytest.mark.parametrize("most,len_hi", [(1, 200), (2, 3), (61, 5), (62, 0), (62, 12), (63, 12), (254, 2), (255, 2)])
def test_every_row_is_found(step_mod, oracle, kind, most, len_hi):
    import torch
    from paper_2510_18546_amd import binding as B
    rng = np.random.default_rng(most + len_hi)
    sel_lists = [list(rng.choice(300, n, replace=False)) for n in (most, 0, most // 2, most, 1)]
    cfg = small(f"tables-{kind}", 1000 + most, dtype=I.F32 if kind == "f32" else I.BF16, n_agents=5, len_lo=0, len_hi=len_hi,
                capacity=max(1, len_hi), n_groups=300, n_sel=most, n_new=40, head_dim=128, n_q_heads=2, n_kv_heads=2)
    announce(f"{cfg}")
    w = I.make_workload(cfg, sel_lists=sel_lists)
    k_pool, v_pool = w.k_pool, w.v_pool
    if kind == "i8":
        kq, vq = quantised_pool(oracle, w)
        k_pool, v_pool = kq[2], vq[2]
        st = Q8Step(step_mod, B, w, kq, vq)
        st.bf16 = True
    else:
        st = step_mod.PlanningStep(w, values_from_pool=kind == "pool")
    st.kc.fill_(0xFF)
    st.vt.fill_(0xFF)
    B.gather_rope(st.pool, st.plan, st.k_new, st.v_new, st.kc, st.vt)
    torch.cuda.synchronize()
    for b in range(cfg.n_agents):
        rk, rv = oracle.gather_rope(k_pool, v_pool, w.lens, w.agent_sel(b), w.k_new[b], w.v_new[b], cfg.rope_base)
        kc, v, kpad, _ = step_mod.PlanningStep.context_host(st, b)
        L = kc.shape[1]
        if kind != "pool":
            want = torch.from_numpy(rv.astype(np.float32))
            np.testing.assert_array_equal(v, (want if kind == "f32" else want.bfloat16().float()).numpy())
        # products and sums to 2^-24 of rows of a few units; bf16: half a step of 2^-8 (and what turns over next to it)
        tol = 2e-6 * max(1.0, np.abs(rk).max()) + (0 if kind == "f32" else 1.01 * 2.0 ** -8 * np.abs(rk))
        assert (np.abs(kc - rk) <= tol).all()
        assert (kpad[:, :-(-L // 64) * 64 - L] == 0).all()
    if kind == "pool":                           # the values are read by their addresses
        st.run()
        torch.cuda.synchronize()
        out, _ = oracle.attention(w.k_pool, w.v_pool, w.lens, w.sel, w.sel_ptr, w.q, w.k_new, w.v_new, cfg.rope_base)
        assert np.abs(st.out_host() - out).max() <= 2e-2
