"""The decision of the clustering where an object has more segments than a wave has lanes: the lowest segment among equal
scores, wherever their lanes are, segments without tokens left out."""
import numpy as np
import pytest

from paper_2510_18546_amd import inputs as I

pytestmark = pytest.mark.gpu
BIG = 2.0 ** 26            # a mass added to it, at most 1, is less than half a step: such scores stay what they are


@pytest.mark.parametrize("n_sel", [3, 64, 65, 130, 200])
def test_lowest_of_equal_scores(oracle, n_sel):
    import torch
    from paper_2510_18546_amd import binding as B
    from paper_2510_18546_amd import step
    cfg = I.Config("decide", n_sel, I.BF16, 3, 4, 2, 64, n_sel, 3, 0, 3, n_sel, 40, 500000.0)
    w = I.make_workload(cfg)
    rng = np.random.default_rng(n_sel)
    w.lens[:] = rng.integers(0, 4, n_sel)
    w.lens[0] = 0
    st = step.PlanningStep(w)
    print(f"[case] {cfg}", flush=True)
    st.gather()
    st.attention()
    n_obj = 8
    planted = np.zeros((3, n_obj, n_sel + 1), np.float32)
    planted[:, 1] = BIG                              # all equal
    for b in range(3):
        for o in range(2, n_obj):
            at = rng.choice(n_sel, size=min(n_sel, int(rng.integers(2, 6))), replace=False)
            planted[b, o, at] = BIG
            if o >= 5:                               # one above the others, of the second row of lanes where there is one
                planted[b, o, at[int(np.argmax(at))]] = 2 * BIG
    planted[:, 6:] *= -1                             # the equal ones are the lowest; nothing reaches the threshold but masses
    planted[:, 7, :n_sel] -= 4 * BIG
    score = torch.from_numpy(planted).cuda()
    assign = torch.full((3, n_obj), -7, dtype=torch.int32, device="cuda:0")
    B.segment_cluster_assign(st.pool, st.plan, st.ws, np.linspace(0, 40, n_obj + 1).astype(np.int32), score, assign,
                             accumulate=True, threshold=0.0)
    torch.cuda.synchronize()
    got, got_a = score.cpu().numpy(), assign.cpu().numpy()
    for b in range(3):
        lens = [int(w.lens[g]) for g in w.agent_sel(b)]
        assert np.array_equal(got_a[b], oracle.cluster_assign(got[b], lens, np.float32(0.0)))
        assert got_a[b, 1] == (np.flatnonzero(lens)[0] if any(lens) else -1)
        assert got_a[b, 7] == -1
