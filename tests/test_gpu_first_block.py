"""The first block of keys of a prefill split: its row sums are taken from the probabilities that the products use."""
import numpy as np
import pytest

from paper_2510_18546_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("values_from_pool", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_sums_of_what_the_products_use(d, values_from_pool, splits):
    """32 keys that nearly all rows' weight lies on: one with probability 1, the others a hair under the middle between two
    bf16 numbers, 0.50170 rounded to 0.5. The values are 1, so with sums of the rounded probabilities every output is 1
    exactly (weights beyond the block are 2^-60); sums of the unrounded ones give 0.9968, in bf16 0.99609."""
    import torch
    from paper_2510_18546_amd import step
    cfg = I.Config("first", 5, I.BF16, 1, 4, 1, d, 1, 64, 64, 64, 1, 40, 500000.0)
    w = I.make_workload(cfg)
    # the two pairs of dimensions that turn by 0.4 % of a bf16 step over these positions; queries that are 1 after
    # scaling and rounding
    one, two = d // 2 - 1, d // 2 - 2
    w.q[:] = w.k_new[:] = w.k_pool[:] = 0
    w.v_pool[:] = w.v_new[:] = 1
    a = 7.84375 if d == 128 else 5.5625
    w.q[..., [one, two]] = a
    w.k_pool[0, 0, 1:32, one] = -1.0
    w.k_pool[0, 0, 1:32, two] = 0.0048828125
    w.k_pool[0, 0, 32:, one] = w.k_new[..., one] = -60.0
    st = step.PlanningStep(w, n_splits=splits, values_from_pool=values_from_pool)
    print(f"[case] d {d} values from pool {values_from_pool} splits {splits}", flush=True)
    st.run()
    torch.cuda.synchronize()
    assert (st.out_host() == 1.0).all()
    # the same rounding in the masses: all but 2^-60 of them on the group, to fp32 sums of 64 terms
    assert np.abs(st.mass_host()[..., 0] - 1.0).max() <= 64 * 2.0 ** -24
