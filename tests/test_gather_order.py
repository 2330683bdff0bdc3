"""The order in which long contexts of agents that share groups are gathered, built on the host: every tile of every agent
once, the tiles that agents share one after the other on one XCD, and no XCD with the work of another."""
import os
import subprocess

import numpy as np
import pytest

from paper_2510_18546_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
XCDS, TILE = 8, 64

# reads: heads, query rows in all, keys only, groups, agents, new tokens, capacity, tokens per group, (groups, then their numbers) per agent,
# -1: as the agent before
DRIVER = '''
#include <cstdio>
#include "en_internal.h"
static int num() { int v = 0; if (scanf("%d", &v) != 1) v = -1; return v; }
int main() {
    en_pool_desc d = {};
    d.n_kv_heads = d.n_q_heads = num();
    const int queries = num(), keys_only = num();
    d.n_groups = num();
    const int agents = num(), n_new = num();
    d.capacity = num();
    d.head_dim = 128; d.dtype = EN_BF16; d.max_ctx = 1 << 26; d.rope_base = 1e4;
    std::vector<int32_t> len(d.n_groups), sel, ptr(1, 0);
    for (auto &v : len) v = num();
    for (int b = 0; b < agents; ++b) {
        const int n = num(), prev = b > 0 ? ptr[b - 1] : 0, end = int(sel.size());
        for (int k = 0; k < n; ++k) sel.push_back(num());
        for (int k = prev; n < 0 && k < end; ++k) sel.push_back(sel[k]);
        ptr.push_back(int32_t(sel.size()));
    }
    en_pool *pool = nullptr; en_plan *plan = nullptr;
    if (kv_pool_create(&d, (void *)256, (void *)256, len.data(), &pool) != EN_OK) return 1;
    if (segment_select(pool, agents, sel.data(), ptr.data(), n_new, &plan) != EN_OK) return 2;
    plan->values_from_pool = keys_only;
    en_gather_order(plan, queries);
    if (plan->order_ints != plan->h_desc.size()) return 3;
    const size_t tables = plan->nseg.size() + plan->sel.size() + plan->bnd.size() + plan->hdr.size();
    printf("%d %d %zu", plan->order_ints > 0, plan->order_shift, en_plan_block_bytes(plan, 4 * (tables + plan->order_ints)));
    for (int v : plan->h_desc) printf(" %d", v);
    printf("\\n");
    en_plan_destroy(plan); kv_pool_destroy(pool);
    return 0;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    at = tmp_path_factory.mktemp("order")
    src, exe = at / "order.cpp", at / "order"
    src.write_text(DRIVER)
    csrc, inc = os.path.join(ROOT, "paper_2510_18546_amd", "csrc"), os.path.join(ROOT, "include")
    B.load()
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", inc, "-I", csrc,
                           str(src), "-o", str(exe), B._build.LIB_PATH,
                           "-Wl,-rpath," + os.path.dirname(B._build.LIB_PATH)])
    return str(exe)


def run(driver, kv, lens, sel, n_new, queries=0, keys_only=0):
    nums = [kv, queries, keys_only, len(lens), len(sel), n_new, max(1, int(max(lens)))] + [int(x) for x in lens]
    for b, s in enumerate(sel):
        nums += [-1] if b and s is sel[b - 1] else [len(s)] + [int(x) for x in s]
    out = subprocess.run([driver], input=" ".join(map(str, nums)), capture_output=True, text=True, check=True).stdout
    return np.array(out.split(), np.int64)


def order(driver, kv, lens, sel, n_new):
    """(gathered in order?, tiles an entry, list of (agent, first tile, tiles) per XCD, {(agent, tile): piece it shares})"""
    flat = run(driver, kv, lens, sel, n_new)
    most, e = 1 << flat[1], flat[3:].reshape(-1, XCDS, 2)
    lists = [[(int(b), int(v) >> 2, (int(v) & 3) + 1) for b, v in e[:, x] if b >= 0] for x in range(XCDS)]
    piece = {}
    for b, s in enumerate(sel):
        end = 0
        for g in list(s) + [-1]:
            begin, end = end, end + (int(lens[g]) if g >= 0 else n_new)
            t0, t1 = -(-begin // TILE), -(-end // TILE)
            piece.update({(b, t): (int(g) if g >= 0 else ("new", b), (t - t0) // most) for t in range(t0, t1)})
    return bool(flat[0]), int(most), lists, piece


def check_once(lists, piece, most):
    seen = [(b, t) for l in lists for b, t0, k in l for t in range(t0, t0 + k)]
    assert len(seen) == len(set(seen)) and set(seen) == set(piece)
    assert all(1 <= k <= most and len({piece[b, t] for t in range(t0, t0 + k)}) == 1 for l in lists for b, t0, k in l)


def busiest(lists):
    tiles = [sum(k for _, _, k in l) for l in lists]
    return max(tiles) * XCDS / sum(tiles)


def idle(most, lists):
    """Workgroups without a tile, as a share of those with one."""
    return most * max(map(len, lists)) * XCDS / sum(k for l in lists for _, _, k in l) - 1


def picks(rng, groups, agents, n):
    return [rng.choice(groups, n, replace=False) for _ in range(agents)]


# (groups, tokens of a group, agents, groups per agent): few groups, so long or so shared that a whole group, or a piece
# of it, is more than an XCD's share of the work
@pytest.mark.parametrize("groups,lo,hi,agents,per", [(1, 2048, 2048, 128, 1), (3, 1024, 2048, 128, 2), (9, 1024, 2048, 64, 8),
                                                     (20, 700, 1024, 64, 16), (1, 256, 256, 1000, 1), (2, 100, 256, 2000, 2)])
def test_few_shared_groups_use_every_xcd(driver, groups, lo, hi, agents, per):
    rng = np.random.default_rng(groups)
    lens = rng.integers(lo, hi + 1, groups)
    in_order, most, lists, piece = order(driver, 8, lens, picks(rng, groups, agents, per), 1)
    assert in_order
    check_once(lists, piece, most)
    # (whole groups on one XCD: 7.8, 3.4, 1.5, 1.2, 6.4, 4.7.) A run of entries is a 32nd of the tiles at most and joined
    # the list with the fewest entries
    assert busiest(lists) <= 1.25


@pytest.mark.parametrize("groups,cap,agents,per,n_new", [(60, 256, 24, 50, 5), (80, 1000, 100, 70, 5), (130, 32, 130, 120, 64),
                                                         (40, 64, 9, 30, 130), (5, 700, 3, 4, 1)])
def test_every_tile_once_and_shared_pieces_together(driver, groups, cap, agents, per, n_new):
    rng = np.random.default_rng(agents)
    lens = rng.integers(cap // 2, cap + 1, groups)
    lens[::7] = 0
    sel = [s[:0] if b == 1 else s[b % 3:] for b, s in enumerate(picks(rng, groups, agents, per))]
    in_order, most, lists, piece = order(driver, 4096, lens, sel, n_new)      # (enough heads for any of them to be long)
    assert in_order
    check_once(lists, piece, most)
    # a piece that agents share is one run of entries in one list, unless it is more than a 32nd of the tiles
    runs = [piece[b, t0] for l in lists for i, (b, t0, _) in enumerate(l) if i == 0 or piece[b, t0] != piece[l[i - 1][0], l[i - 1][1]]]
    size = {}
    for p in piece.values():
        size[p] = size.get(p, 0) + 1
    twice = {p for p in runs if runs.count(p) > 1}
    assert all(32 * size[p] > len(piece) for p in twice)


@pytest.mark.parametrize("groups,lo,hi,agents,per,n_new", [(130, 1, 32, 130, 120, 64), (60, 32, 64, 128, 40, 512),
                                                           (40, 100, 256, 300, 12, 200), (1, 256, 256, 1000, 1, 1)])
def test_new_tokens_go_round_the_xcds(driver, groups, lo, hi, agents, per, n_new):
    """New tokens are shared with nobody: their entries go to the XCDs in turn, those of an agent one after the other."""
    rng = np.random.default_rng(groups)
    in_order, most, lists, piece = order(driver, 64, rng.integers(lo, hi + 1, groups), picks(rng, groups, agents, per), n_new)
    assert in_order
    check_once(lists, piece, most)
    assert busiest(lists) <= 1.25               # (as pieces of one more group: up to 1.34)
    new = [[(b, t) for b, t, _ in l if piece[b, t][0] == ("new", b)] for l in lists]
    assert all(x == sorted(x) for x in new)


# agents, tokens of each agent's own group, shared groups, their tokens, of them per agent, new tokens
@pytest.mark.parametrize("agents,own,groups,tokens,per,n_new,want", [
    (60, 4096, 20, 160, 9, 1, False), (100, 2048, 20, 160, 8, 1, False), (120, 0, 32, 192, 8, 1024, False),
    (100, 0, 32, 384, 4, 1024, False), (128, 0, 16, 48, 8, 512, False), (64, 0, 1024, 256, 64, 1, True),
    (500, 0, 16, 48, 8, 120, True), (64, 0, 2560, 96, 64, 1, False), (64, 512, 64, 256, 16, 1, True), (16, 0, 4000, 256, 64, 1, False),
    (64, 0, 2545, 48, 87, 1, False), (64, 0, 1326, 48, 87, 1, True), (16, 0, 139, 256, 47, 1, False), (16, 0, 139, 256, 49, 1, True)])
def test_order_goes_by_the_tokens_that_agents_share(driver, agents, own, groups, tokens, per, n_new, want):
    rng = np.random.default_rng(groups)
    sel = [np.r_[s, groups + b] if own else s for b, s in enumerate(picks(rng, groups, agents, per))]
    in_order, most, lists, piece = order(driver, 8, [tokens] * groups + [own] * (agents if own else 0), sel, n_new)
    assert in_order == want
    if want:
        check_once(lists, piece, most)


def test_no_order_of_more_workgroups_than_a_launch_may_have(driver):
    """4.4 million entries of three tiles, four tiles' workgroups each: 17.6 million of them, 2^24 - 1 fit."""
    nums = [1, 0, 0, 4000, 1100, 1, 192] + [192] * 4000 + [4000] + list(range(4000)) + [-1] * 1099
    out = subprocess.run([driver], input=" ".join(map(str, nums)), capture_output=True, text=True, check=True).stdout
    assert out.split()[0] == "0" and len(out.split()) == 3


def test_a_planner_of_one_kind_of_step_allocates_its_device_block_once(driver):
    """The order's length differs between selections of the same agents and groups; the block's size does not follow it."""
    rng = np.random.default_rng(3)
    lens = rng.integers(150, 257, 200)
    out = [run(driver, 8, lens, picks(rng, 200, 48, 30), 1) for _ in range(12)]
    assert all(o[0] for o in out) and len({len(o) for o in out}) > 3
    assert len({int(o[2]) for o in out}) == 1


# 64 agents, 8 heads, 32 new tokens: 256 query rows of each for 4 K tokens of 2 x 8 rows are 0.12 of the rows
@pytest.mark.parametrize("tokens,agents_a_group,queries,keys_only,want", [
    (96, 3, 0, 0, True), (96, 2.6, 64 * 256 * 32, 0, False), (96, 8, 64 * 256 * 32, 0, True), (256, 3, 64 * 256 * 32, 0, True),
    (48, 2.2, 0, 0, False), (96, 4.2, 0, 1, True), (96, 2.6, 0, 1, False), (256, 2.6, 64 * 256 * 32, 1, False), (64, 30, 0, 1, False),
    (64, 30, 0, 0, True)])
def test_the_order_has_to_save_more_beside_queries_and_of_keys_only(driver, tokens, agents_a_group, queries, keys_only, want):
    rng = np.random.default_rng(tokens)
    per = 4096 // tokens
    groups = int(64 * per / agents_a_group)
    assert run(driver, 8, [tokens] * groups, picks(rng, groups, 64, per), 32, queries, keys_only)[0] == want


@pytest.mark.parametrize("kv,lo,hi,most", [(8, 56, 136, 1), (8, 120, 200, 1), (8, 250, 256, 4), (8, 256, 256, 4), (8, 128, 128, 2),
                                           (2, 64, 128, 2), (2, 48, 48, 1)])
def test_entries_leave_few_workgroups_idle(driver, kv, lo, hi, most):
    """Also where one group is longer than most."""
    rng = np.random.default_rng(lo)
    per = 5000 // hi
    lens = rng.integers(lo, hi + 1, 16 * per)
    lens[0] = 300
    in_order, got, lists, piece = order(driver, kv, lens, picks(rng, 16 * per, 512 // kv, per), 1)
    assert in_order and got == most
    check_once(lists, piece, got)
    assert idle(got, lists) <= (0.2 if kv > 2 else 0.55)
