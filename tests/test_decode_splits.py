"""KV splits of decode steps, on the host: what a step's partial results may be, whichever kernel takes it."""
import numpy as np
import pytest

from paper_2510_18546_amd import binding as B

N_CU, TILE, MAX_SPLITS = 256, 64, 64


def streaming(base, tiles):
    """Splits of the streaming kernel, and partial results per row that it leaves with a workspace."""
    want = max(1, min(-(-2 * N_CU // base), tiles, MAX_SPLITS)) if 2 * N_CU > base or tiles < 64 else 2
    longest = -(-tiles // want)
    if longest <= 2 or 8 * (tiles - (longest - 1) * want) >= want:
        want = -(-tiles // longest)
    return want, want * (2 if base * want <= 2 * N_CU else 1)


def plans(seed, n):
    """Plans of one row an agent and head, or a few, over contexts of every length."""
    rng = np.random.default_rng(seed)
    for _ in range(n):
        agents = int(np.exp(rng.uniform(0, np.log(1200))))
        kv, r, d = int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 2, 4, 7, 8])), int(rng.choice([64, 128]))
        tokens, n_new = int(np.exp(rng.uniform(0, np.log(20000)))), int(rng.choice([1, 1, 2, 4, 16]))
        cap = max(1, min(tokens, 256))
        groups = -(-tokens // cap)
        pool = B.kv_pool_create(None, None, np.full(groups, cap, np.int32), n_q_heads=kv * r, rope_base=1e4,
                                max_ctx=groups * cap + n_new, dtype=int(rng.choice([B.EN_BF16, B.EN_I8])), k_ptr=0x1000,
                                v_ptr=0x2000, shape=(groups, kv, cap, d))
        plan = B.segment_select(pool, np.tile(np.arange(groups, dtype=np.int32), agents),
                                np.arange(agents + 1, dtype=np.int32) * groups, n_new)
        yield pool, plan, agents, kv, r, d, n_new, agents * kv, -(-(groups * cap + n_new) // TILE)
        plan.close()
        pool.close()


def test_steps_written_out_directly_stay_so():
    """Where the streaming kernel has one result a row, whose sums stay in fp32 to the end, no partial results in bf16."""
    met = 0
    for pool, plan, agents, kv, r, d, n_new, base, tiles in plans(1, 400):
        if r * n_new <= 16 and streaming(base, tiles)[1] == 1:
            met += 1
            assert plan.info.n_splits == 1, (agents, kv, r, d, n_new, tiles)
    assert met > 20


def align(n):
    return -(-n // 256) * 256


def scratch(agents, heads, rows, segments, d, partial):
    """Bytes of a step's scratch with `partial` results per row: (reference, sum) pairs of the row and of its buckets,
    accumulators of the reduced masses, and what more than one result needs: the merged pair, the outputs in bf16."""
    n = agents * heads * rows
    at = align(align(partial * n * 8) + partial * n * (segments + 1) * 8)
    at = align(at + agents * (segments + 1) * 8)
    return align(align(at + n * 8) + partial * n * d * 2) if partial > 1 else at


def test_no_more_scratch_than_the_streaming_kernel_needs():
    """Scratch sized for a step of the streaming kernel holds the step whichever kernel takes it, the plan's own workspace
    holds its steps of a row where it held those, and so does the static array."""
    less = 0
    for pool, plan, agents, kv, r, d, n_new, base, tiles in plans(2, 600):
        before = scratch(agents, kv * r, 1, plan.info.max_segments, d, streaming(base, tiles)[1])
        now = B.decode_workspace_bytes(pool, plan, 1)
        assert now <= before, (agents, kv, r, d, n_new, tiles)
        less += now < before
    assert less > 100
