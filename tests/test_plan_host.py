"""CPU-only tests of the C-ABI library: it loads, exports every declared symbol,
validates its inputs, and its integer plan agrees bit-exactly with the oracle's
integer side.  No device call is made (host-only contexts)."""
import ctypes
import os
import re
import time

import numpy as np
import pytest

import oracle
from paper_2605_06914_amd import (Context, EXPORTED, LIB_PATH, TaperError, load_library, TAPER_EBLOCK, TAPER_EGROUP,
                                  TAPER_EHIP, TAPER_EINVAL, TAPER_ELEN)
from taper_inputs import (AttnShape, structure_config1, structure_config2, structure_config3, structure_config4,
                          structure_config5, structure_custom)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
QWEN = AttnShape(64, 8, 128, 16)


def test_library_exports_every_declared_symbol():
    lib = load_library()
    header = "".join(open(os.path.join(ROOT, "include", f)).read() for f in sorted(os.listdir(os.path.join(ROOT, "include"))))
    declared = set(re.findall(r"TAPER_API\s+[\w\s\*]+?\b(taper_\w+)\s*\(", header))
    assert declared == set(EXPORTED), declared ^ set(EXPORTED)
    for name in declared:
        assert getattr(lib, name) is not None
    assert os.path.exists(LIB_PATH)
    assert lib.taper_strerror(-3) == b"malformed request grouping"


def host_ctx(sh=QWEN):
    return Context(sh.n_q_heads, sh.n_kv_heads, sh.head_dim, sh.page_size, device=-1)


def build(st, ctx=None, **kw):
    ctx = ctx or host_ctx(st.shape)
    return ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **kw)


@pytest.mark.parametrize("bad", [dict(n_q_heads=64, n_kv_heads=7), dict(head_dim=96), dict(page_size=32),
                                 dict(n_q_heads=64, n_kv_heads=2), dict(scale=0.0)])
def test_create_rejects_unsupported_shapes(bad):
    kw = dict(n_q_heads=64, n_kv_heads=8, head_dim=128, page_size=16, scale=None, device=-1)
    kw.update(bad)
    with pytest.raises(TaperError) as e:
        Context(**kw)
    assert e.value.status == TAPER_EINVAL


def test_validation_errors():
    st = structure_config1()
    ctx = host_ctx(st.shape)

    def expect(code, **over):
        args = dict(block_table=st.block_table.copy(), branch_group=st.branch_group.copy(),
                    prefix_len=st.prefix_len.copy(), suffix_len=st.suffix_len.copy(), n_pool_pages=st.n_pool_pages)
        for k, f in over.items():
            args[k] = f(args[k])
        with pytest.raises(TaperError) as e:
            ctx.plan_build(**args)
        assert e.value.status == code, (e.value, code)

    def setv(i, v):
        def f(a):
            a = a.copy()
            a[i] = v
            return a
        return f

    expect(TAPER_EBLOCK, block_table=setv((0, 3), -1))
    expect(TAPER_EBLOCK, block_table=setv((4, 13), 64))
    expect(TAPER_EBLOCK, n_pool_pages=lambda n: 10)
    expect(TAPER_EGROUP, branch_group=setv(0, 1))
    expect(TAPER_EGROUP, branch_group=setv(2, 3))
    expect(TAPER_EGROUP, branch_group=lambda a: np.array([0, 1, 1, 0, 1], np.int32))
    expect(TAPER_EGROUP, prefix_len=setv(3, 191))
    expect(TAPER_EGROUP, block_table=setv((2, 5), int(st.block_table[0, 0])))  # a member's prefix page differs
    expect(TAPER_ELEN, suffix_len=setv(2, -1))
    expect(TAPER_ELEN, prefix_len=lambda a: np.array([0, 192, 192, 192, 192], np.int32))  # serial request left empty
    expect(TAPER_ELEN, suffix_len=setv(4, 16 * 10))  # row too short for its pages
    expect(TAPER_EINVAL, n_pool_pages=lambda n: 0)
    # unused block-table entries may hold anything
    bt = st.block_table.copy()
    bt[bt < 0] = 123456
    ctx.plan_build(bt, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages).free()


def test_host_only_context_refuses_device_work():
    st = structure_config1()
    ctx = host_ctx(st.shape)
    plan = build(st, ctx)
    with pytest.raises(TaperError) as e:
        load = load_library()
        rc = load.taper_decode_step_attention(ctx._h, plan._h, 8, 8, 8, None, None)
        if rc != 0:
            raise TaperError(rc, load.taper_last_error().decode())
    assert e.value.status == TAPER_EHIP


def check_plan_against_oracle(st, **kw):
    sh = st.shape
    g = sh.gqa
    plan = build(st, **kw)
    e = plan.export()
    ints = oracle.resolve(sh.page_size, st.block_table, st.branch_group, st.prefix_len, st.suffix_len,
                          want_slots=st.logical_tokens < 2_000_000)
    assert e["n_groups"] == ints.n_groups and e["n_seqs"] == st.n_seqs
    for key in ("ctx_len", "n_prefix_pages", "n_suffix_pages", "group_start"):
        assert np.array_equal(e[key], getattr(ints, key)), key
    assert e["tokens_unique"] == st.unique_tokens and e["tokens_logical"] == st.logical_tokens
    if ints.slots is not None:
        assert np.array_equal(plan.resolve_slots_host(ints.slots.shape[1]), ints.slots)
    # every (sequence, logical position) is covered by exactly one work item
    F = {n: i for i, n in enumerate(e["item_fields"])}
    items = e["items"]
    cover = [np.zeros(int(c), np.int32) for c in ints.ctx_len]
    for it in items:
        seq0, nb, page0, ntok, kind = (int(it[F[k]]) for k in ("seq0", "n_branch", "page0", "n_tokens", "kind"))
        assert ntok >= 1 and nb >= 1 and (kind == 0) == (nb >= 2)
        assert nb * g <= 12 * 16
        npp = int(ints.n_prefix_pages[seq0])
        for b in range(nb):
            s = seq0 + b
            assert st.branch_group[s] == st.branch_group[seq0]
            if page0 < npp or ints.n_suffix_pages[seq0] == 0 and st.suffix_len[seq0] == 0:
                lo = page0 * 16  # inside the prefix
                assert lo + ntok <= st.prefix_len[s]
            else:
                assert nb == 1
                lo = int(st.prefix_len[s]) + (page0 - npp) * 16
            cover[s][lo : lo + ntok] += 1
    for s, c in enumerate(cover):
        assert np.all(c == 1), f"sequence {s} not covered exactly once"
    # parts partition the items; partial rows are disjoint; merge map lists each sequence's items
    # after them the pool: private items that belong to no share
    ps = e["part_start"]
    n_pool = e["n_pool_items"]
    assert ps[0] == 0 and ps[-1] + n_pool == len(items) and np.all(np.diff(ps) >= 1)
    assert np.array_equal(items[: ps[-1], F["part"]], np.repeat(np.arange(len(ps) - 1), np.diff(ps)))
    assert np.all(items[ps[-1] :, F["part"]] == len(ps) - 1) and np.all(items[ps[-1] :, F["n_branch"]] == 1)
    pool_cap = max(32, (kw.get("pool_item_tokens", 0) or 1536) // 32 * 32)
    assert np.all(items[ps[-1] :, F["n_tokens"]] <= pool_cap)
    nsh = e["n_parts_shared"]
    assert np.all(items[: ps[nsh], F["kind"]] == 0) and np.all(items[ps[nsh] :, F["kind"]] >= 1)
    rows = items[:, F["n_branch"]].astype(np.int64) * g * sh.n_kv_heads
    assert np.array_equal(items[:, F["part_base"]], np.concatenate([[0], np.cumsum(rows)[:-1]]))
    assert e["n_partial_rows"] == rows.sum()
    ms, merge = e["merge_start"], e["merge"]
    for s in range(st.n_seqs):
        its = [it for it in items if it[F["seq0"]] <= s < it[F["seq0"]] + it[F["n_branch"]]]
        mine = [(int(it[F["part_base"]]) + (s - int(it[F["seq0"]])) * g, int(it[F["n_branch"]]) * g) for it in its]
        assert [tuple(x) for x in merge[ms[s] : ms[s + 1]]] == mine
        # kind 2 marks exactly the private items that are their sequence's only item
        assert all((int(it[F["kind"]]) >= 2) == (len(its) == 1 and it[F["n_branch"]] == 1) for it in its)
    plan.free()
    return e


@pytest.mark.parametrize("maker", [structure_config1, structure_config2, structure_config3,
                                   lambda: structure_config5(k=16, n_serial=12, n_parallel=5)])
def test_plan_integers_match_oracle(maker):
    check_plan_against_oracle(maker())


@pytest.mark.parametrize("kw", [dict(share_prefix=False), dict(target_workgroups=8), dict(target_workgroups=100000), dict(target_workgroups=100000, min_share_tokens=1),
                                dict(max_branches_per_item=3), dict(scatter_sub_groups=True), dict(max_branches_per_item=4, scatter_sub_groups=True), dict(pool_pct=-1), dict(pool_pct=90, pool_item_tokens=64), dict(pool_pct=100, pool_item_tokens=200),
                                dict(shared_cost_pct=300, shared_item_cost=5000, private_item_cost=1)])
def test_plan_options(kw):
    reqs = [(37, [0]), (50, [0, 7, 16, 21]), (16, [1]), (700, [0, 33, 64, 65, 129, 300]), (1, [0]), (0, [45]),
            (333, list(range(30)))]
    e = check_plan_against_oracle(structure_custom(QWEN, reqs, seed=1), **kw)
    if kw.get("share_prefix") is False:
        assert e["n_parts_shared"] == 0
    if kw.get("pool_pct") == -1:
        assert e["n_pool_items"] == 0
    if kw.get("pool_pct") == 90:
        F = {n: i for i, n in enumerate(e["item_fields"])}
        it = e["items"]
        priv = it[it[:, F["kind"]] >= 1]
        pooled = it[e["part_start"][-1] :, F["n_tokens"]].sum()
        assert 0.85 * priv[:, F["n_tokens"]].sum() <= pooled <= 0.9 * priv[:, F["n_tokens"]].sum() + 64


def test_config4_plan_is_balanced():
    st = structure_config4()
    e = check_plan_against_oracle(st)
    F = {n: i for i, n in enumerate(e["item_fields"])}
    ps = e["part_start"]
    tok = np.array([e["items"][ps[i] : ps[i + 1], F["n_tokens"]].sum() for i in range(len(ps) - 1)])
    nsh = e["n_parts_shared"]
    assert nsh > 0 and (nsh + e["n_parts_private"]) * 8 <= 600
    for t in (tok[:nsh], tok[nsh:]):
        assert t.max() <= 1.25 * t.sum() / len(t) + 64


@pytest.mark.parametrize("width,target", [(32, 0), (64, 0), (64, 4096), (100, 64)])
def test_sub_groups_of_a_wide_request_stream_the_prefix_side_by_side(width, target):
    """A request wider than one item is cut into sub-groups that each read the whole prefix.  Their items
    have the same cuts, a share each, and neighbouring shares (workgroups that start together and, for one
    kv head, sit on one XCD), chunk by chunk; with scatter_sub_groups they are placed like unrelated requests."""
    from taper_inputs import structure_wide

    st = structure_wide(width) if width <= 64 else structure_custom(QWEN, [(900, [0]), (5000, [7] * width), (70, [1, 2])], seed=3)
    e = check_plan_against_oracle(st, target_workgroups=target)
    F = {n: i for i, n in enumerate(e["item_fields"])}
    items, ps = e["items"], e["part_start"]
    shared = items[items[:, F["kind"]] == 0]
    sizes = np.bincount(st.branch_group)
    first = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    checked = 0
    for g in np.flatnonzero(sizes > 24):
        mine = shared[(shared[:, F["seq0"]] >= first[g]) & (shared[:, F["seq0"]] < first[g] + sizes[g])]
        n_sub = -(-int(sizes[g]) // 24)
        assert len(mine) % n_sub == 0 and len(np.unique(mine[:, F["seq0"]])) == n_sub
        parts = mine[:, F["part"]]
        assert np.array_equal(parts, parts[0] + np.arange(len(mine))), "neighbouring shares, in order"
        assert np.all(np.diff(ps)[parts] == 1), "a share each"
        for c in range(len(mine) // n_sub):  # chunk c of every sub-group: the same pages
            chunk = mine[c * n_sub : (c + 1) * n_sub]
            assert len(set(chunk[:, F["page0"]])) == 1 and len(set(chunk[:, F["n_tokens"]])) == 1
            assert sorted(chunk[:, F["seq0"]]) == sorted(np.unique(mine[:, F["seq0"]]))
        checked += 1
    assert checked >= 1


def test_small_steps_without_shared_work_take_half_the_grid_when_that_saves_pieces():
    """With the grid left to the library, a step of serial requests is cut for one workgroup per compute unit
    instead of two when that cuts sequences into so many fewer pieces that it pays; never with shared-prefix
    work, never for an explicit grid (unless asked), never when nothing is saved; the plan is a full cover
    either way."""
    F = None

    def pieces(e):
        nonlocal F
        F = {n: i for i, n in enumerate(e["item_fields"])}
        return int((e["items"][:, F["kind"]] == 1).sum())

    irp = structure_config2()
    auto, never, explicit = (check_plan_against_oracle(irp, **kw) for kw in ({}, dict(small_step_grid=-1), dict(target_workgroups=512)))
    assert never["n_parts_private"] == explicit["n_parts_private"] == 64 and auto["n_parts_private"] == 32
    assert pieces(auto) < pieces(never) == pieces(explicit)
    asked = check_plan_against_oracle(irp, target_workgroups=512, small_step_grid=1)
    assert asked["n_parts_private"] == 32
    equal = structure_custom(QWEN, [(1024, [0])] * 32, seed=1)  # 256 (sequence, kv head) pairs: a workgroup each, nothing cut
    e = check_plan_against_oracle(equal)
    assert e["n_parts_private"] == 32 and pieces(e) == 0
    uncut = structure_custom(QWEN, [(1024, [0])] * 128, seed=1)  # nothing is cut at the full grid: nothing to save
    assert check_plan_against_oracle(uncut)["n_parts_private"] == 64
    big = structure_config5(k=0)  # long shares: the pieces saved do not pay for the slower grid
    assert check_plan_against_oracle(big)["n_parts_private"] == 64
    mixed = check_plan_against_oracle(structure_config3())
    assert mixed["n_parts_shared"] + mixed["n_parts_private"] == 64


@pytest.mark.parametrize("head_shape,width,pct", [((64, 8, 128), 2, 80), ((64, 8, 128), 8, 80), ((64, 8, 128), 9, 120), ((64, 8, 128), 24, 120),
                                                  ((64, 8, 128), 25, 110), ((64, 8, 128), 64, 110), ((32, 8, 64), 16, 80), ((32, 8, 64), 17, 120),
                                                  ((64, 4, 128), 5, 120), ((64, 4, 128), 24, 110)])
def test_a_shared_token_weighs_more_in_items_of_more_row_tiles(head_shape, width, pct):
    """Items of up to 4 row tiles 80 %, wider ones 120, wider sub-groups of one request 110 (steps of long shares)."""
    st = structure_custom(AttnShape(*head_shape, 16), [(3000, [0])] * 30 + [(8000 + 500 * i, [700] * width) for i in range(8)], seed=5)
    ctx = Context(*head_shape, device=-1)
    a, b = (ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **kw).export()
            for kw in ({}, dict(shared_cost_pct=pct)))
    assert np.array_equal(a["items"], b["items"]) and np.array_equal(a["part_start"], b["part_start"])
    ctx.close()


@pytest.mark.parametrize("width,pct", [(8, 80), (24, 120), (25, 160), (60, 160)])
def test_a_shared_token_of_sub_groups_weighs_more_in_short_shares(width, pct):
    st = structure_custom(QWEN, [(700, [0])] * 48 + [(1200 + 100 * i, [100] * width) for i in range(5)], seed=6)
    ctx = Context(64, 8, 128, device=-1)
    assert 350 <= (st.unique_tokens + 7000 * (width > 24)) // 64 < 2000
    a, b = (ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **kw).export()
            for kw in ({}, dict(shared_cost_pct=pct)))
    assert np.array_equal(a["items"], b["items"]) and np.array_equal(a["part_start"], b["part_start"])
    ctx.close()


@pytest.mark.parametrize("seed", range(4))
def test_pool_items_stay_within_their_default_size(seed):
    """A quarter of a share, between 512 and 1536 tokens, also where a quarter of a share is more."""
    rng = np.random.default_rng(seed)
    st = structure_custom(QWEN, [(int(x), [0]) for x in rng.integers(20000, 40000, 64)] + [(20000, [3000] * 6)] * 4, seed=seed)
    ctx = Context(64, 8, 128, device=-1)
    e = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages).export()
    F = {n: i for i, n in enumerate(e["item_fields"])}
    pool = e["items"][e["part_start"][-1]:, F["n_tokens"]]
    assert e["n_pool_items"] > 0 and 1024 < pool.max() <= 1536, pool.max()
    ctx.close()


@pytest.mark.parametrize("shape,share_tokens,pct", [("serial", 2040, 25), ("serial", 2600, 31), ("serial", 3584, 42), ("serial", 5120, 60),
                                                    ("serial", 12000, 60), ("sub_groups", 5120, 60)])
def test_the_pools_part_of_the_private_tokens_follows_the_length_of_the_shares(shape, share_tokens, pct):
    """A quarter for shares of up to 2048 tokens, 60 % from 5120 on, in proportion between; whether requests have sub-groups makes no
    difference.  One prefix of 4 (or 64) branches beside 200 equal serial requests that fill the rest."""
    total, prefix, n, width = share_tokens * 64, 4096, 200, 64 if shape == "sub_groups" else 4
    listed = prefix * (1 if width == 4 else 3)  # (three sub-groups of at most 24 branches each stream the prefix)
    each = (total - listed - 64 * width) // n
    reqs = [(prefix, [64] * width)] + [(0, [each + (1 if i < total - listed - 64 * width - each * n else 0)]) for i in range(n)]
    e = build(structure_custom(QWEN, reqs, seed=3)).export()
    F = {k: i for i, k in enumerate(e["item_fields"])}
    it = e["items"]
    private = it[it[:, F["kind"]] != 0][:, F["n_tokens"]].sum()
    pooled = it[e["part_start"][-1]:, F["n_tokens"]].sum()
    assert abs(pooled - private * pct / 100) <= private / 100 + 64, (pooled / private, pct)  # (whole percents, cut at 32 tokens)


def test_where_merges_are_made_can_be_set():
    """The rule's choice, the other one, and back; nothing else of the plan changes."""
    st = structure_config3()
    ctx = Context(64, 8, 128, device=-1)
    args = (st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages)
    rule = ctx.plan_build(*args).export()
    for on in (False, True):
        for plan in (ctx.plan_build(*args, merge_launch=on),
                     ctx.plan_build_segments(*args[:3], np.arange(st.n_seqs + 1), st.suffix_len, st.n_pool_pages, merge_launch=on)):
            e = plan.export()
            assert e["merge_launch"] == on
            assert all(np.array_equal(e[k], rule[k]) for k in ("items", "part_start", "merge_start", "merge"))
            plan.set_merge_launch(not on)
            assert plan.export()["merge_launch"] == (not on)
            plan.free()
    plan = ctx.plan_build(*args)
    with pytest.raises(TaperError) as err:
        plan.set_merge_launch(2)
    assert err.value.status == TAPER_EINVAL and plan.export()["merge_launch"] == rule["merge_launch"]
    plan.free()
    ctx.close()


def test_short_steps_keep_their_merges_inside_the_attention_launch():
    """A second launch per layer costs the host more than it saves the GPU there; the mixed batch on one kv head has it."""
    small = structure_custom(AttnShape(32, 8, 64, 16), [(1246, [0]), (1135, [0]), (912, [104, 251, 451, 370, 119]), (376, [145, 272, 316, 135]),
                                                        (607, [97, 191, 195, 413])], seed=4)
    ctx = Context(32, 8, 64, device=-1, partial_format="f32")
    e = build(small, ctx).export()
    assert np.diff(e["merge_start"]).max() > 8 and e["merge_launch"] == 0  # (three rounds of 4 entries, 10.6 us either way)
    ctx.close()
    ctx = Context(8, 1, 128, device=-1)
    assert build(structure_config3(), ctx).export()["merge_launch"] == 1
    ctx.close()


@pytest.mark.parametrize("shape,partial,reqs,launch", [
    # a chain of 14 to 18 blocks of one row tile and three rounds: 9.4 us a call (8.5 with the launch), 19.3 a layer in a loop (22.7)
    ((4, 1, 64), "f32", [(868, [1, 3, 3, 0, 3]), (823, [0, 2, 1, 2, 2]), (877, [1, 4, 1, 1, 4, 3, 4]), (851, [1, 3, 1, 3, 1, 1, 4]),
                         (861, [0, 1, 0, 4, 5, 3, 4]), (875, [0, 4, 1, 2, 0, 4])], 0),
    # four rounds: 14.0 us a call (9.2), 21.1 a layer (21.4)
    ((32, 8, 64), "f32", [(2685, [16, 6, 10, 3, 19, 29, 11]), (2449, [13, 14, 7, 27, 3, 6, 15, 21])], 1)])
def test_the_line_between_merges_inside_and_a_launch_of_their_own(shape, partial, reqs, launch):
    """Steps of three and four rounds on either side of it, by what the present kernels take for them."""
    ctx = Context(*shape, device=-1, partial_format=partial)
    assert build(structure_custom(AttnShape(*shape, 16), reqs, seed=5), ctx).export()["merge_launch"] == launch
    ctx.close()


def test_a_callers_costs_hold_for_short_items_too():
    """100 sequences of 20 tokens (a block of 32 each): as many to a share as its size and the caller's item cost say."""
    st = structure_custom(QWEN, [(20, [0])] * 100, seed=6)
    full = lambda cost, share_cost: (1000 + share_cost) // (cost + 32)  # whole items in a share of 1000 tokens and an item's cost
    for kw, per_share in ((dict(private_item_cost=1), full(1, 1)), (dict(private_item_cost=64), full(64, 64)),
                          (dict(private_merge_cost=-1), full(128, 128)), (dict(solo_item_tokens=-1), full(128, 128)),
                          (dict(solo_item_tokens=19), full(128, 128)), (dict(), full(160, 128))):
        e = check_plan_against_oracle(st, min_share_tokens=1000, **kw)
        assert len(e["part_start"]) - 1 == -(-100 // per_share), (kw, np.diff(e["part_start"]))


def test_a_pool_taken_from_before_many_short_segments_costs_no_more_time():
    """1500 sequences of 129 tokens, a quarter of which go to the pool, before 150000 branches of one token, which stay: the plan takes
    about as long as with the sequences behind the branches, not a move of all branches for each."""
    n_long, n_req, width = 1500, 12500, 12
    ctx = Context(1, 1, 64, device=-1)

    def best(long_first):
        long_ = (np.full(n_long, 129), np.zeros(n_long), np.ones(n_long))
        short = (np.ones(n_req * width), np.ones(n_req * width), np.tile([1] + [0] * (width - 1), n_req))
        parts = [long_, short] if long_first else [short, long_]
        prefix, suffix, opens = (np.concatenate([p[i] for p in parts]).astype(np.int32) for i in range(3))
        table, times = np.zeros((len(prefix), 9), np.int32), []
        for _ in range(3):
            t0 = time.perf_counter()
            plan = ctx.plan_build(table, np.cumsum(opens) - 1, prefix, suffix, 1)
            times.append(time.perf_counter() - t0)
            assert plan.export()["n_pool_items"] > 300
            plan.free()
        return min(times)

    ahead, behind = best(True), best(False)
    assert ahead < 2 * behind, (ahead, behind)
    ctx.close()


def shared_shares(st, **kw):
    """Requests whose prefix each shared share has items of, and the number of shares in all."""
    e = build(st, **kw).export()
    F = {k: i for i, k in enumerate(e["item_fields"])}
    it, ps = e["items"], e["part_start"]
    return [{int(st.branch_group[s]) for s in it[ps[q]:ps[q + 1], F["seq0"]]} for q in range(e["n_parts_shared"])], len(ps) - 1


@pytest.mark.parametrize("serial,requests,apart", [(6600, 20, True), (6700, 20, False), (10, 32, True), (10, 33, False)])
def test_short_prefixes_get_shares_of_their_own_where_there_are_enough(serial, requests, apart):
    """Below 128 tokens per share (64 shares: 8192 tokens; 20 prefixes of 60 tokens and 3 branches of 5 make 1500) and up to half the shares."""
    st = structure_custom(QWEN, [(60, [5, 5, 5])] * requests + [(0, [serial])], seed=6)
    held, n = shared_shares(st)
    assert n <= 64 and set().union(*held) == set(range(requests))
    assert all(len(h) == 1 for h in held) == apart, held


@pytest.mark.parametrize("heads,branches,pct", [(2, 32, 140), (1, 64, 140), (8, 9, 220), (8, 16, 220), (8, 17, 300), (8, 24, 300)])
def test_prices_of_shared_items_in_short_shares(heads, branches, pct):
    """A shared token's price by the item's row tiles and 20 per branch below 128 tokens per share, 180 % and 32 per branch up to 350: the default cuts
    are those of these prices given by hand, and not those of the other range.  (4, 4, 5, 8, 9 and 12 row tiles; 512 shares.)"""
    sh = AttnShape(heads, 1, 128, 16)
    cuts = lambda n, **kw: build(structure_custom(sh, [(n * (1 + i) // 12, [3 + i] * branches) for i in range(24)], seed=7), Context(heads, 1, 128, device=-1), **kw).export()["items"][:, :8].tolist()
    below, above = dict(shared_cost_pct=pct, shared_item_cost=60 + 20 * branches), dict(shared_cost_pct=180, shared_item_cost=60 + 32 * branches)
    for lengths, right, wrong in (((400, 800, 1000), below, above), ((3000, 3500, 4500), above, below)):
        default = [cuts(n) for n in lengths]
        assert default == [cuts(n, **right) for n in lengths]
        assert default != [cuts(n, **wrong) for n in lengths]


@pytest.mark.parametrize("shape,n,shares", [((8, 1, 128), 3500, 240), ((8, 1, 128), 4500, 228), ((8, 1, 64), 4500, 300)])
def test_short_shares_are_cut_finer_only_while_shared_ones_are_half_of_them(shape, n, shares):
    """12 requests of 9 branches (5 row tiles) below 128 tokens per share, of 512: by the finer prices they take 240 and 300 shares; beyond half, at head_dim 128,
    the prices are those of 128 tokens per share and more (180 %, 60 and 32 per branch)."""
    st = structure_custom(AttnShape(*shape, 16), [(n, [3] * 9)] * 12, seed=8)
    ctx = Context(*shape, device=-1)
    prefix_cuts = lambda e: sorted(int(t) for t in e["items"][:, 3] if t > 3)
    default = build(st, ctx).export()
    fine = build(st, ctx, shared_cost_pct=220, shared_item_cost=60 + 20 * 9).export()
    coarse = build(st, ctx, shared_cost_pct=180, shared_item_cost=60 + 32 * 9).export()
    right, wrong = (coarse, fine) if shares == 228 else (fine, coarse)
    assert default["n_parts_shared"] == shares and fine["n_parts_shared"] == (240 if n == 3500 else 300)
    assert prefix_cuts(default) == prefix_cuts(right) != prefix_cuts(wrong)
    ctx.close()
