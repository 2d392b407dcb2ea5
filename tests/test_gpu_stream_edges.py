"""Streaming loops at their edges: shared items of one block, of as many as the ring holds and a few more, with remainders of every kind, one after
the other in one workgroup's ring; private items that follow each other."""
import pytest

from taper_inputs import AttnShape, fill_values_numpy, structure_custom
from tests.gpu_util import assert_parity, both_merges, run_gpu, run_oracle, torch_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
@pytest.mark.parametrize("branches", [2, 9, 24])
@pytest.mark.parametrize("shape", [(8, 1, 128), (16, 2, 128), (8, 2, 64), (16, 1, 64)])
def test_shared_items_of_few_blocks(shape, branches, partial_format):
    """Prefixes of 1 to 9 blocks (32 tokens at head_dim 128, 64 at 64), a token less and a token more, half blocks and whole pages; rows of 1 to 12
    tiles, so that waves of one workgroup hold different numbers of them.  Bits repeat, and the whole workgroup's ring is used by item after item."""
    from paper_2605_06914_amd import Context

    sh, block = AttnShape(*shape, 16), 32 if shape[2] == 128 else 64
    lengths = [1, 15, 16, 17] + [n * block + d for n in (1, 2, 3, 4, 5, 6, 9) for d in (-1, 0, 1)] + [3 * block + block // 2, 7 * block + 16]
    reqs = [(n, [(i + k) % 3 for k in range(branches)]) for i, n in enumerate(lengths)]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=81))
    ref, ref_lse = run_oracle(b)
    ctx = Context(*shape, device=0, partial_format=partial_format)
    for kw in (dict(), dict(target_workgroups=shape[1]), dict(target_workgroups=5 * shape[1])):
        got, lse, bits = run_gpu(ctx, b, **kw)
        assert_parity(got, ref, f"few blocks {shape} {branches} {partial_format} {kw}")
        assert abs(lse - ref_lse).max() <= 1e-3  # (fp32 sums of at most 580 terms)
        assert (run_gpu(ctx, b, **kw)[2] == bits).all()
    ctx.close()


@both_merges
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("shape", [(8, 1, 128), (6, 2, 128), (8, 2, 64)])
def test_items_that_follow_each_other(shape, offset, merge_launch):
    """Long private items, behind which a share's next item is brought closer, followed by items of one block, of fewer blocks than waves, of as many, of
    long ones; whole sequences and pieces, alone in a workgroup and dealt to single waves; pools that start at multiples of 2 and 4 bytes."""
    import torch

    from paper_2605_06914_amd import Context

    sh = AttnShape(*shape, 16)
    reqs = [(n, [0]) for n in (600, 1, 513, 33, 700, 64, 545, 97, 512, 520, 640, 128, 1100, 2, 513, 513, 129, 1030, 31, 96, 97, 95, 32, 5, 65, 98)] + [(40, [600, 20, 530, 0, 900, 3])]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=82))
    ref, ref_lse = run_oracle(b)
    st = b.structure
    room = torch.empty(st.n_pool_pages * sh.page_elems + 8, dtype=torch.bfloat16, device="cuda:0")
    kv = room[offset:offset + st.n_pool_pages * sh.page_elems]
    kv.copy_(torch_bf16(b.kv).view(-1))
    ctx = Context(*shape, device=0)
    one = dict(target_workgroups=shape[1])
    for kw in (dict(), one, dict(one, solo_item_tokens=-1), dict(one, solo_item_tokens=4096), dict(target_workgroups=3 * shape[1], solo_item_tokens=-1, pool_pct=30)):
        got, lse, bits = run_gpu(ctx, b, kv_dev=kv, merge_launch=merge_launch, **kw)
        assert_parity(got, ref, f"items in a row {shape} {offset} {kw}")
        assert abs(lse - ref_lse).max() <= 1e-3  # (fp32 sums of at most 1100 terms)
        assert (run_gpu(ctx, b, kv_dev=kv, merge_launch=merge_launch, **kw)[2] == bits).all()
    ctx.close()


@pytest.mark.parametrize("n", [5, 10, 11])
@pytest.mark.parametrize("shape", [(8, 1, 128), (6, 2, 128), (8, 2, 64)])
def test_runs_of_solo_items_and_rows_of_long_ones(shape, n):
    """Runs of as many single-wave items as the next one's first block is brought closer for, and one more, behind items of 96 and 97 tokens; whole
    workgroup's items of 768 and 769 tokens behind each other in a launch of private work alone.  One share per kv head, bits repeat."""
    from paper_2605_06914_amd import Context

    sh = AttnShape(*shape, 16)
    ctx = Context(*shape, device=0)
    one = dict(target_workgroups=shape[1], pool_pct=-1)
    for lengths, solo in (([97] * n, 512), ([96] * (n - 1) + [130], 512), ([97 + 31 * i for i in range(n)], 512), ([769, 768, 769, 1, 1000, 33, 769], -1)):
        b = fill_values_numpy(structure_custom(sh, [(k, [0]) for k in lengths], seed=83))
        ref, ref_lse = run_oracle(b)
        st = b.structure
        plan = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, solo_item_tokens=solo, **one)
        e = plan.export()
        plan.free()
        assert e["n_parts_private"] == 1 and e["solo_items"][0] == (0 if solo < 0 else n), lengths
        got, lse, bits = run_gpu(ctx, b, solo_item_tokens=solo, **one)
        assert_parity(got, ref, f"rows of items {shape} {lengths}")
        assert abs(lse - ref_lse).max() <= 1e-3  # (fp32 sums of at most 1000 terms)
        assert (run_gpu(ctx, b, solo_item_tokens=solo, **one)[2] == bits).all()
    ctx.close()
