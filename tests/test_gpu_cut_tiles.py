"""Attention tiles cut along the keys into pieces of unequal length, and the device blocks that plans
hand on to each other (needs an MI355X)."""
import pytest
import torch

import paper_2502_01960_amd as mpic
from test_gpu_lazy import _run_lazy
from test_gpu_parity import _custom, _run_sampled, _sampled_rows

pytestmark = pytest.mark.gpu

# a recomputed chunk in front of a stored one; requests whose number is no divisor of the L2 domains
LAYOUTS = [
    [[("chunk", 0, 333, 333), ("text", 65), ("chunk", 1, 1500, 32), ("text", 91)]],
    [[("chunk", 1, 1500, 8), ("text", 40 + b), ("chunk", 0, 333, 100), ("text", 7)] for b in range(3)],
]


@pytest.mark.parametrize("reqs", LAYOUTS, ids=["one_request", "three_requests"])
@pytest.mark.parametrize("lazy", [False, True])
def test_cut_tiles(reqs, lazy):
    p = _custom(reqs, 2, [333, 1500], 0)
    if lazy:
        _run_lazy(p, rows=_sampled_rows(p))
    else:
        _run_sampled(p, False)
    tiles = p.plan.get("attn_tiles")
    assert (tiles[:, 6] >= 0).any()


@pytest.mark.parametrize("side", [False, True], ids=["default_stream", "side_stream"])
def test_blocks_of_destroyed_plans(side):
    """Plans of different sizes that come and go on one context while the work of the plan before is
    still enqueued: every pass gives the bits of the first one of its layout."""
    probs = [_custom(reqs, 2, [333, 1500], 0) for reqs in LAYOUTS]
    ctx = None
    for p in probs:
        p.gpu_setup(False)
        ctx = ctx or p.ctx
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    first, last = {}, None
    for i in range(14):
        j = (i // 2) % 2
        p = probs[j]
        plan = mpic.Plan(ctx, p.requests, p.k)
        stream = other if side and i % 3 == 0 else torch.cuda.default_stream()
        out, k_ctx, v_ctx = torch.zeros_like(p.out), torch.zeros_like(p.k_ctx), torch.zeros_like(p.v_ctx)
        stream.wait_stream(torch.cuda.default_stream())
        mpic.mpic_assemble_kv(ctx.handle, plan.handle, p.srcs, p.d_fk, p.d_fv, k_ctx, v_ctx, stream.cuda_stream)
        mpic.mpic_selective_attn(ctx.handle, plan.handle, p.d_q, k_ctx, v_ctx, p.sh.softmax_scale, out, None, stream.cuda_stream)
        if last is not None:
            last.close()
        last = plan
        torch.cuda.default_stream().wait_stream(stream)
        got = (out, k_ctx, v_ctx)
        if j not in first:
            first[j] = got
        else:
            for a, b in zip(got, first[j]):
                assert torch.equal(a.view(torch.int16), b.view(torch.int16)), i
    last.close()


def test_cut_tiles_on_two_streams_at_once():
    """Attention calls of one context that overlap on two streams do not meet in a workspace: every call
    gives the bits it gives alone."""
    probs = [_custom(reqs, 2, [333, 1500], 0) for reqs in LAYOUTS]
    for p in probs:
        p.gpu_setup(False)
    ctx = probs[0].ctx
    plans = [mpic.Plan(ctx, p.requests, p.k) for p in probs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    want = []
    for p, plan in zip(probs, plans):
        assert (plan.get("attn_tiles")[:, 6] >= 0).any()
        mpic.mpic_assemble_kv(ctx.handle, plan.handle, p.srcs, p.d_fk, p.d_fv, p.k_ctx, p.v_ctx)
        mpic.mpic_selective_attn(ctx.handle, plan.handle, p.d_q, p.k_ctx, p.v_ctx, p.sh.softmax_scale, p.out, None)
        torch.cuda.synchronize()
        want.append(p.out.clone())
    outs = [[torch.zeros_like(p.out) for _ in range(25)] for p in probs]
    torch.cuda.synchronize()
    for i in range(25):
        for p, plan, out, s in zip(probs, plans, outs, streams):
            mpic.mpic_selective_attn(ctx.handle, plan.handle, p.d_q, p.k_ctx, p.v_ctx, p.sh.softmax_scale, out[i], None, s.cuda_stream)
    torch.cuda.synchronize()
    for w, of in zip(want, outs):
        for out in of:
            assert torch.equal(out.view(torch.int16), w.view(torch.int16))
    for plan in plans:
        plan.close()
