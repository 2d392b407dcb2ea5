"""The merges as a launch behind the attention launch: partials per sequence at the edges of what a wave takes at once (32 in
flight, 64 per pass), head counts that do not fill a workgroup, a branch whose only partial is its prefix's, sequences
that are one item and must stay as their item wrote them."""
import numpy as np
import pytest

from taper_inputs import AttnShape, fill_values_numpy, structure_custom
from tests.gpu_util import assert_parity, run_gpu, run_oracle, torch_bf16

pytestmark = pytest.mark.gpu

FINE = dict(target_workgroups=4096, min_share_tokens=1, private_item_cost=1, solo_item_tokens=-1, pool_pct=-1)


@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
@pytest.mark.parametrize("shape", [(6, 2, 128), (16, 1, 128), (8, 8, 64), (32, 4, 64)])
def test_merge_launch_at_its_edges(shape, partial_format):
    from paper_2605_06914_amd import Context

    sh = AttnShape(*shape, 16)
    # private sequences of 1 ... 70 blocks of 32 tokens (64 with some heads), shared prefixes of one item and of several
    reqs = [(32 * k, [0]) for k in (1, 2, 31, 32, 33, 63, 64, 65, 70)] + [(16, [0, 0, 5]), (640, [0, 40, 0]), (33, [90, 0])]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=611))
    st = b.structure
    ctx = Context(*shape, device=0, partial_format=partial_format)
    e = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **FINE).export()
    counts = np.diff(e["merge_start"])
    print("[merge launch]", shape, "partials per sequence:", counts.tolist(), flush=True)
    assert e["merge_launch"] == 1 and counts.max() > 64 and counts.min() == 1 and ((counts > 32) & (counts < 64)).any()
    ref, ref_lse = run_oracle(b)
    got, lse, bits = run_gpu(ctx, b, **FINE)
    assert_parity(got, ref, f"merge launch {shape} {partial_format}")
    # (fp32 sums of at most 2240 terms: some 1e-5 of a value near 8, scores rounded in fp32 alike)
    assert np.abs(lse - ref_lse).max() <= 1e-3
    for _ in range(3):
        assert np.array_equal(run_gpu(ctx, b, **FINE)[2], bits)
    ctx.close()


@pytest.mark.parametrize("partial_format", ["f16_scaled", "f32"])
@pytest.mark.parametrize("shape", [(16, 2, 128), (8, 8, 64)])
def test_merge_launch_gives_what_merges_inside_the_launch_give(shape, partial_format):
    """One plan merged both ways, which only the order of fp32 sums tells apart: up to 70 rows of values below 6, each sum off by at
    most 70 x 6 x 2^-23 = 5e-5 before both round to bf16, to the same value or to neighbours."""
    import torch

    from paper_2605_06914_amd import Context

    sh = AttnShape(*shape, 16)
    reqs = [(32 * k, [0]) for k in (1, 2, 7, 8, 9, 16, 17, 33, 70)] + [(640, [0, 40, 0]), (200, [90, 3, 5, 7, 1, 64])]
    b = fill_values_numpy(structure_custom(sh, reqs, seed=5))
    st = b.structure
    ctx = Context(*shape, device=0, partial_format=partial_format)
    plan = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages, **FINE)
    counts = np.diff(plan.export()["merge_start"])
    assert counts.max() == 70 and len(set(counts.tolist())) >= 8
    q, kv = torch_bf16(b.q), torch_bf16(b.kv)
    got = []
    for on in (False, True):
        plan.set_merge_launch(on)
        out = torch.full_like(q, float("nan"))
        lse = torch.full(q.shape[:2], float("nan"), device=q.device)
        ctx.decode_step_attention(plan, q, kv, out, lse)
        torch.cuda.synchronize()
        got.append((out.double().cpu().numpy(), lse.cpu().numpy()))
    (x, lx), (y, ly) = got
    step = 2.0 ** -7 * np.maximum(np.abs(x), np.abs(y))  # (a bf16 step is at most this much of the value)
    assert np.abs(kv.float().abs().max().item()) < 6
    assert (np.abs(x - y) <= step + 5e-5).all(), np.abs(x - y).max()
    assert np.abs(lx - ly).max() <= 1e-5 * np.abs(lx).max()  # (fp32 sums of positive numbers, their logarithm)
    plan.free()
    ctx.close()


def test_two_threads_on_one_stream():
    """Two threads call on one context and one stream, each a plan with a merge launch: every result is the one the plan gives alone."""
    import threading

    import torch

    from paper_2605_06914_amd import Context

    sh = AttnShape(8, 1, 128, 16)
    ctx = Context(8, 1, 128, device=0)
    work = []
    for seed, reqs in ((1, [(15000, [0])]), (2, [(9000, [0, 30, 700]), (5000, [0])])):
        b = fill_values_numpy(structure_custom(sh, reqs, seed=seed))
        st = b.structure
        plan = ctx.plan_build(st.block_table, st.branch_group, st.prefix_len, st.suffix_len, st.n_pool_pages)
        assert plan.export()["merge_launch"] == 1
        q, kv = torch_bf16(b.q), torch_bf16(b.kv)
        alone = torch.empty_like(q)
        ctx.decode_step_attention(plan, q, kv, alone)
        work.append((plan, q, kv, alone, [torch.full_like(q, float("nan")) for _ in range(200)]))
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream().cuda_stream

    def calls(plan, q, kv, _, outs):
        for out in outs:
            ctx.decode_step_attention(plan, q, kv, out, stream=stream)

    threads = [threading.Thread(target=calls, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for plan, _, _, alone, outs in work:
        assert all(torch.equal(out.view(torch.int16), alone.view(torch.int16)) for out in outs)
        plan.free()
    ctx.close()
