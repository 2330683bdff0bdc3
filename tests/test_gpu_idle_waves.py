"""Prefill workgroups in which one to eight waves have rows and the others only load tiles: every number of tiles modulo
the four LDS stages, both head widths, values gathered and left in the pool, one split (whose waves meet again for the
reduced masses) and several. Against the oracle, to the tolerances of every other bf16 case."""
import numpy as np
import pytest

from paper_2510_18546_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("values_from_pool", [False, True])
@pytest.mark.parametrize("r,nq,tokens,splits", [(1, 40, 20, 1), (1, 64, 100, 1), (3, 33, 140, 1), (2, 65, 190, 2), (7, 12, 260, 1),
                                                (5, 50, 330, 3), (1, 300, 64, 1)])
def test_waves_without_rows(oracle, r, nq, tokens, splits, values_from_pool, d):
    import torch
    from paper_2510_18546_amd import step
    cfg = I.Config("idle", r + nq, I.BF16, 2, 2 * r, 2, d, 3, tokens, tokens // 2, tokens, 2, nq, 500000.0)
    w = I.make_workload(cfg)
    print(f"[case] {cfg} splits {splits} values from pool {values_from_pool}", flush=True)
    st = step.PlanningStep(w, n_splits=splits, values_from_pool=values_from_pool)
    st.ws.fill_(0xFF)
    st.run()
    torch.cuda.synchronize()
    out, mass = oracle.attention(w.k_pool, w.v_pool, w.lens, w.sel, w.sel_ptr, w.q, w.k_new, w.v_new, cfg.rope_base)
    assert np.abs(st.out_host() - out).max() <= 2e-2
    assert np.abs(st.mass_host() - mass).max() <= 1e-2
    # sums of nq * 2 r masses whose errors have no common sign, and a thousandth of what is summed
    red = mass.sum((1, 2))
    assert (np.abs(st.mass_red_host() - red) <= 1e-2 * np.sqrt(nq * 2 * r) + 1e-3 * red).all()
