"""The streaming loops, the merge rounds and the plan's cuts at the sizes where they can go wrong: numbers of
16 KiB blocks around the ring's length, ragged last blocks, every number of row tiles per wave, numbers of
partials around the merge rounds and beyond the window of merge entries kept on chip."""
import numpy as np
import pytest

from taper_inputs import AttnShape, fill_values_numpy, structure_custom
from tests.gpu_util import assert_parity, both_merges, run_gpu, run_oracle

# tokens per block are 32 at head_dim 128 and 64 at 64; the ring holds four blocks
PREFIXES = [1, 16, 17, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160, 193, 255, 256, 257, 321]
SHAPES = [(64, 8, 128), (32, 8, 64), (6, 2, 128), (16, 1, 64)]


def context(sh, **kw):
    from paper_2605_06914_amd import Context

    return Context(sh.n_q_heads, sh.n_kv_heads, sh.head_dim, device=0, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("tiles", [1, 2, 4, 5, 8, 9, 12])
def test_shared_items_of_few_blocks(shape, tiles, partial_format):
    sh = AttnShape(*shape, 16)
    width = max(2, 16 * tiles // sh.gqa)
    if (width * sh.gqa + 15) // 16 > 12:
        pytest.skip("wider than one item")
    reqs = [(p, [(7 * i + p) % 41 for i in range(width)]) for p in PREFIXES]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=300 + tiles))
    ctx = context(sh, partial_format=partial_format)
    got, lse, _ = run_gpu(ctx, b, max_branches_per_item=width)
    ref, ref_lse = run_oracle(b)
    assert_parity(got, ref, f"{shape} tiles {tiles}")
    assert np.max(np.abs(lse - ref_lse)) < 2e-3  # (fp32 sums of fp32 exponentials of scores that are exact to 2^-20)
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_private_items_of_few_blocks(shape, partial_format):
    """Serial contexts that give the four waves of a workgroup 0, 1, 2, 3 ... blocks, whole and ragged."""
    sh = AttnShape(*shape, 16)
    reqs = [(n, [0]) for n in PREFIXES + [127, 383, 384, 385, 511, 513, 640, 777, 1025]]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=401))
    ref, ref_lse = run_oracle(b)
    for kw in ({}, dict(solo_item_tokens=-1)):
        ctx = context(sh, partial_format=partial_format)
        got, lse, _ = run_gpu(ctx, b, **kw)
        assert_parity(got, ref, f"{shape} {kw}")
        assert np.max(np.abs(lse - ref_lse)) < 2e-3
        ctx.close()


@pytest.mark.gpu
@both_merges
@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
def test_merges_of_few_and_of_very_many_partials(partial_format, merge_launch):
    """1 to 9 partials per sequence (rounds of 2, 4, 8), and more than the 128 entries a workgroup keeps on chip."""
    sh = AttnShape(16, 1, 128, 16)
    reqs = [(32 * k, [0]) for k in range(1, 11)] + [(6000, [0]), (96, [5] * 5), (64, [40, 0, 33])]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=511))
    ctx = context(sh, partial_format=partial_format)
    st = b.structure
    kw = dict(target_workgroups=4096, min_share_tokens=1, private_item_cost=1, solo_item_tokens=-1, merge_launch=merge_launch)
    e = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **kw).export()
    counts = np.diff(e["merge_start"])
    print("[merge] partials per sequence:", counts.tolist(), flush=True)
    assert e["merge_launch"] == merge_launch and counts.max() > 128 and len(set(counts.tolist()) & {1, 2, 3, 4, 5, 6}) >= 4
    ref, _ = run_oracle(b)
    got, _, bits = run_gpu(ctx, b, **kw)
    assert_parity(got, ref, "many partials")
    for _ in range(10):  # whoever merges, the rounds are the same
        assert np.array_equal(run_gpu(ctx, b, **kw)[2], bits)
    ctx.close()


def test_a_prefix_is_not_cut_into_more_items_than_its_merge_is_worth():
    """One request alone on one kv head: the grid would allow hundreds of cuts of its prefix, each of which one workgroup
    would have to merge for every branch."""
    from paper_2605_06914_amd import Context

    sh = AttnShape(16, 1, 128, 16)
    for width in (2, 5, 12):
        st = structure_custom(sh, [(24000, [600] * width)], seed=9)
        ctx = Context(16, 1, 128, device=-1)
        e = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages).export()
        F = {n: i for i, n in enumerate(e["item_fields"])}
        shared = e["items"][e["items"][:, F["kind"]] == 0]
        k, rows = len(shared), width * sh.gqa
        assert int(shared[:, F["n_tokens"]].sum()) == 24000
        assert 4 <= k and k * k <= 1.5 * 4.0 * 24000 / rows, (width, k)
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("elements", [1, 4])
def test_a_pool_that_starts_anywhere(shape, elements):
    """Pool, queries and results as views 2 and 8 bytes into larger buffers, over items of every number of tiles per wave: the
    bits are those of aligned buffers."""
    import torch

    from tests.gpu_util import bits_from_torch, torch_bf16

    sh = AttnShape(*shape, 16)
    widths = sorted({max(2, 16 * t // sh.gqa) for t in (1, 4, 8, 12)})
    reqs = [(p, [(7 * i + p) % 41 for i in range(w)]) for w in widths if (w * sh.gqa + 15) // 16 <= 12 for p in (1, 31, 64, 97, 161, 321)]
    b = fill_values_numpy(structure_custom(sh, reqs + [(n, [0]) for n in (5, 77, 300, 1500)], seed=71))
    ctx = context(sh)
    _, _, want = run_gpu(ctx, b, max_branches_per_item=max(widths))

    def shifted(t):
        big = torch.zeros(t.numel() + 16, dtype=t.dtype, device=t.device)
        view = big[elements:elements + t.numel()]
        view.copy_(t.reshape(-1))
        return big, view

    st = b.structure
    (_, q), (_, kv) = shifted(torch_bf16(b.q)), shifted(torch_bf16(b.kv))
    whole, out = shifted(torch.zeros(b.q.size, dtype=torch.bfloat16, device="cuda:0"))
    assert kv.data_ptr() % 16 == 2 * elements
    print(f"[offset] {shape} {elements} elements: S={st.n_seqs}", flush=True)
    plan = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, max_branches_per_item=max(widths))
    ctx.decode_step_attention(plan, q, kv, out)
    torch.cuda.synchronize()
    same = np.array_equal(bits_from_torch(out).reshape(want.shape), want)
    assert same
    assert not whole[:elements].any() and not whole[elements + out.numel():].any()
    plan.free()
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("lens,pct", [([40], 90), ([100], 70), ([100, 100], 90), ([64] * 5, 90), ([3000], 90)])
def test_steps_whose_pool_would_take_everything(lens, pct):
    sh = AttnShape(64, 8, 128, 16)
    b = fill_values_numpy(structure_custom(sh, [(n, [0]) for n in lens], seed=611))
    ctx = context(sh)
    got, _, _ = run_gpu(ctx, b, pool_pct=pct)
    ref, _ = run_oracle(b)
    assert_parity(got, ref, f"{lens} {pct} %")
    ctx.close()
