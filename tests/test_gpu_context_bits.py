"""The keys of a context, bit for bit: x1 cos - x2 sin and x1 sin + x2 cos, of each the product of x2 rounded and the
product of x1 inside a fused multiply-add. The other way round in the second half: the 8-bit gather; where a 16-bit gather
is large enough for units of four heads by 32 workgroups for each compute unit, all but the last of four (of eight too,
with D = 64), whatever number of heads its workgroups take; the first row that a wave of the decode kernel appends. These
are the bits that contexts have always had, whichever way the loops are unrolled."""
import math

import numpy as np
import pytest

from paper_2510_18546_amd import binding as B
from paper_2510_18546_amd import inputs as I

pytestmark = pytest.mark.gpu


def rotated(x, pos, base, x1_rounded=False):
    """x [..., len(pos), D] as float32 values; the products of a float32 pair are exact in 64 bits."""
    half = x.shape[-1] // 2
    theta = [base ** (-2.0 * k / x.shape[-1]) for k in range(half)]
    cos, sin = (np.array([[f(float(p) * t) for t in theta] for p in pos]).astype(np.float32) for f in (math.cos, math.sin))
    x1, x2 = x[..., :half].astype(np.float64), x[..., half:].astype(np.float64)
    a, b, c = (p.astype(np.float32) for p in (x2 * sin, x2 * cos, x1 * sin))
    second = x2 * cos + c if x1_rounded else x1 * sin + b
    return np.concatenate([(x1 * cos - a).astype(np.float32), second.astype(np.float32)], -1)


def bf16(x):
    import torch
    return torch.from_numpy(x).to(torch.bfloat16).float().numpy()


@pytest.mark.parametrize("dtype,kv,agents,d", [
    ("f32", 1, 1, 64), ("f32", 2, 3, 128), ("bf16", 1, 1, 128), ("bf16", 3, 1, 64), ("bf16", 2, 256, 64),
    ("bf16", 4, 140, 128), ("bf16", 4, 140, 64), ("bf16", 8, 72, 128), ("bf16", 8, 72, 64), ("f32", 4, 600, 64),
    ("bf16", 8, 3, 128), ("bf16", 2, 1000, 128), ("bf16", 4, 500, 128), ("bf16", 8, 250, 128), ("keys only", 4, 130, 128), ("i8", 2, 2, 128),
    ("i8", 1, 2, 64)])
def test_rotated_keys(dtype, kv, agents, d):
    """keys only: bf16, the values left in the pool, which take one head a workgroup there. agents: enough for 2, 4 and 8 heads a unit (32 workgroups for each of 256 compute units), then for 768 MB of keys and
    values, which are gathered in the order of the groups."""
    import torch
    keys_only, dtype = dtype == "keys only", "bf16" if dtype == "keys only" else dtype
    rng = np.random.default_rng(agents + d)
    g_n, cap, s_n, n_new, base = 12, 96, 9, 34, 1e4
    dev, bits16 = "cuda:0", dtype != "f32"
    act = torch.bfloat16 if bits16 else torch.float32
    lens = rng.integers(80, cap + 1, g_n).astype(np.int32)
    scales = None
    if dtype == "i8":
        k = torch.from_numpy(rng.integers(-127, 128, (g_n, kv, cap, d)).astype(np.int8)).to(dev)
        scales = [torch.from_numpy(rng.uniform(0.005, 0.02, (g_n, kv, cap)).astype(np.float32)).to(dev) for _ in range(2)]
        values = k.cpu().numpy().astype(np.float32) * scales[0].cpu().numpy()[..., None]
    else:
        k = torch.from_numpy(rng.standard_normal((g_n, kv, cap, d)).astype(np.float32)).to(act).to(dev)
        values = k.float().cpu().numpy()
    pool = B.kv_pool_create(k, k.clone(), lens, kv, base, s_n * cap + n_new)
    if scales:
        B.kv_pool_set_scales(pool, *scales)
    sel = [rng.choice(g_n, s_n, replace=False).astype(np.int32) for _ in range(agents)]
    plan = B.segment_select(pool, np.concatenate(sel), np.arange(agents + 1) * s_n, n_new)
    assert (agents in (250, 500, 1000)) == (dtype == "bf16" and 4 * agents * kv * plan.info.ctx_stride * d >= 768 << 20)
    if keys_only:
        plan.values_from_pool(True)
        assert 5 * (kv // 4) * plan.info.ctx_stride // 64 * agents >= 32 * 256 > kv * plan.info.ctx_stride // 64 * agents
    k_new = torch.from_numpy(rng.standard_normal((agents, n_new, kv, d)).astype(np.float32)).to(act).to(dev)
    kc, vt = B.alloc_context(pool, plan)
    B.gather_rope(pool, plan, k_new, k_new, kc, vt)
    T = plan.info.ctx_stride

    def context(b):
        return kc.view(act).view(agents, kv, T, d)[b].float().cpu().numpy()

    for b in sorted({0, agents // 2, agents - 1}):
        src = np.concatenate([values[g, :, :lens[g]] for g in sel[b]] + [k_new[b].float().cpu().numpy().transpose(1, 0, 2)], 1)
        want = rotated(src, range(src.shape[1]), base, dtype == "i8")
        unit = kv if agents > 16 else 1
        if dtype == "bf16" and (unit == 4 or unit == 8 and d == 64):
            want[:-1] = rotated(src[:-1], range(src.shape[1]), base, True)
        np.testing.assert_array_equal(context(b)[:, :src.shape[1]], bf16(want) if bits16 else want)
    if agents > 100:
        return
    # the new tokens once more, as the rows of decode steps: one by one and two at a time (by the decode attention
    # kernel) and together (by a launch of its own)
    offsets = [int(plan.offsets(b)[-1]) for b in range(agents)]
    rows_new = k_new.float().cpu().numpy().transpose(0, 2, 1, 3)
    q = torch.zeros_like(k_new)
    out = torch.empty_like(k_new)
    values_before = vt.clone()
    for n in (1, 2, n_new):
        fused = dtype != "f32" and n < n_new
        ws = torch.empty(max(256, B.decode_workspace_bytes(pool, plan, n)), dtype=torch.uint8, device=dev)
        for b, L in enumerate(offsets):
            kc.view(act).view(agents, kv, T, d)[b, :, L:L + n_new] = 0
        for i in range(0, n_new, n):
            rows = k_new[:, i:i + n].contiguous()
            B.segmented_decode_step(pool, plan, i, q[:, i:i + n].contiguous(), rows, rows, kc, vt, out[:, i:i + n].contiguous(), ws)
        assert torch.equal(vt, values_before), n
        for b, L in enumerate(offsets):
            pos = np.arange(L, L + n_new)
            want = rotated(rows_new[b], pos, base)
            # (a step may meet another wave's range at a multiple of 64)
            first = (np.arange(n_new) % n == 0) & fused
            want[:, first] = rotated(rows_new[b], pos, base, True)[:, first]
            sure = first | (pos % 64 != 0) | (not fused)
            np.testing.assert_array_equal(context(b)[:, L:L + n_new][:, sure], (bf16(want) if bits16 else want)[:, sure], err_msg=str(n))
