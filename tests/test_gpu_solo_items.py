"""Short private items that single waves run side by side: results and partial rows, alone and in runs of every length around
the four waves and the 64 items that are announced at once; sequences all of whose partials come from such runs."""
import numpy as np
import pytest

import oracle
from taper_inputs import AttnShape, f32_from_bf16_bits, fill_values_numpy, reduce_structure, structure_custom
from tests.gpu_util import assert_parity, bits_from_torch, both_merges, run_gpu, run_oracle, torch_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
@pytest.mark.parametrize("shape", [(16, 2, 128), (6, 2, 128), (8, 8, 64), (16, 1, 64)])
def test_short_branches_beside_their_prefix(shape, partial_format):
    """Branches of 0, 1, a block less, a block, a block more ... tokens; shares of one item, of two, three, and of all."""
    from paper_2605_06914_amd import Context

    sh = AttnShape(*shape, 16)
    reqs = [(40, [1, 31, 32, 33, 0, 64, 127]), (200, [128, 129, 255, 256, 257, 511]), (512, [0]), (17, [0]), (513, [0]), (90, [3, 5])]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=71))
    ref, ref_lse = run_oracle(b)
    ctx = Context(*shape, device=0, partial_format=partial_format)
    hkv = shape[1]
    st, runs = b.structure, set()
    for kw in (dict(), dict(target_workgroups=hkv), dict(target_workgroups=3 * hkv), dict(target_workgroups=7 * hkv), dict(target_workgroups=6 * hkv, solo_item_tokens=100),
               dict(min_share_tokens=1, private_item_cost=1), dict(solo_item_tokens=-1)):
        got, lse, bits = run_gpu(ctx, b, **kw)
        assert_parity(got, ref, f"solo {shape} {partial_format} {kw}")
        e = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **kw).export()
        kind = e["items"][:, e["item_fields"].index("kind")]
        runs |= {int(n) for q, n in enumerate(e["solo_items"]) if (kind[e["part_start"][q]:e["part_start"][q] + n] == 1).any()}
        assert np.abs(lse - ref_lse).max() <= 1e-3  # (fp32 sums of at most 768 terms)
        assert np.array_equal(run_gpu(ctx, b, **kw)[2], bits)
    assert {1, 2, 3, 4, 5} <= runs  # (runs with partials among them, of fewer items than waves and of more)
    ctx.close()


@both_merges
@pytest.mark.parametrize("shape", [(16, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("batch", ["branches", "reduced"])
def test_more_partials_in_a_run_than_are_announced_at_once(shape, batch, merge_launch):
    """180 and 200 partials run by the waves of one workgroup per kv head: lots of 64 announcements.  Branches wait for their prefix's
    item besides; the partials of reduced sequences all come from the run, and every merge is made behind one of its lots."""
    import torch

    from paper_2605_06914_amd import Context

    sh = AttnShape(*shape, 16)
    rng = np.random.default_rng(8)
    if batch == "branches":
        base = st = structure_custom(sh, [(3, [1, 2, 1, 2])] * 45, seed=72)
        seg_start, seg_len = np.arange(st.n_seqs + 1, dtype=np.int32), st.suffix_len
    else:
        base = structure_custom(sh, [(int(rng.integers(1, 5)), [int(x) for x in rng.integers(1, 5, size=6)]) for _ in range(25)], seed=72,
                                n_pool_pages=256)
        st = reduce_structure(base, z_len=[int(x) for x in rng.integers(1, 3, size=25)], seed=73)
        seg_start, seg_len = st.seg_start, st.seg_len
    b = fill_values_numpy(base)
    q, kv = b.q[: st.n_seqs], b.kv
    ctx = Context(*shape, device=0)
    ref, _ = oracle.attention_segments(sh.n_q_heads, sh.n_kv_heads, sh.head_dim, 16, sh.scale, q, kv, st.block_table, st.prefix_len,
                                       seg_start, seg_len)
    qd, kvd = torch_bf16(q), torch_bf16(kv)
    plan = ctx.plan_build_segments(st.block_table, st.branch_group, st.prefix_len, seg_start, seg_len, st.n_pool_pages,
                                   target_workgroups=shape[1], merge_launch=merge_launch)
    e = plan.export()
    q0, n = int(np.argmax(e["solo_items"])), int(e["solo_items"].max())
    kinds = e["items"][e["part_start"][q0]:e["part_start"][q0] + n, e["item_fields"].index("kind")]
    assert n == (180 if batch == "branches" else 200) and (kinds == 1).all() and e["merge_launch"] == merge_launch
    outs = []
    for _ in range(3):
        out = torch.full_like(qd, float("nan"))
        ctx.decode_step_attention(plan, qd, kvd, out)
        torch.cuda.synchronize()
        outs.append(bits_from_torch(out))
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])
    assert_parity(f32_from_bf16_bits(outs[0]).astype(np.float64), ref, f"run of {n} {shape} {batch}")
    plan.free()
    ctx.close()
