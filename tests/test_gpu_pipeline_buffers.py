"""Buffers that layers share in mpic_prefill_layers (needs an MI355X): a call for all layers gives what one
call per layer and step gives, bit for bit, whichever of them overlap."""
import pytest
import torch

import paper_2502_01960_amd as mpic
from helpers import LayeredProblem

pytestmark = pytest.mark.gpu

SMALL = {1: {}, 3: dict(n_chunks=3, chunk_len=150, text_len=21, batch=2)}


def _tensors(p, shared):
    """Per layer q, fresh k, fresh v, context k, context v, output, log-sum-exp."""
    dev, sh, n = torch.device("cuda:0"), p.sh, len(p.oplan["q_pos"])
    new = lambda *shape: torch.full(shape, float("nan"), dtype=sh.torch_dtype, device=dev)
    kv = (sh.n_kv_heads, sh.head_dim)
    layers = []
    for l in range(p.n_layers):
        q, k, v = (t.to(dev) for t in p.fresh[l])
        out, kc, vc = new(n, sh.n_q_heads, sh.head_dim), new(p.n_slots, *kv), new(p.n_slots, *kv)
        lse = torch.full((n, sh.n_q_heads), float("nan"), dtype=torch.float32, device=dev)
        before = layers[-1] if l else None
        if l and shared == "output is the next fresh keys":
            k = before[5].view(-1)[:n * kv[0] * kv[1]].view(n, *kv)
        if l and shared == "log-sum-exp is in the next fresh values":
            v.copy_(p.fresh[l][2])
            before[6] = v.view(-1).view(torch.float32)[:n * sh.n_q_heads].view(n, -1)
        if l and shared == "contexts":
            kc, vc = layers[0][3], layers[0][4]
        if l and shared in ("query is in the next context", "output is in the next context"):
            i = 0 if shared.startswith("query") else 5
            room = new(max(before[i].numel(), kc.numel()))
            room[:before[i].numel()] = before[i].view(-1)
            before[i], kc = room[:before[i].numel()].view(before[i].shape), room[:kc.numel()].view(kc.shape)
        layers.append([q, k, v, kc, vc, out, lse])
    return layers


@pytest.mark.parametrize("config", [1, 3])
@pytest.mark.parametrize("shared", ["nothing", "contexts", "output is the next fresh keys", "log-sum-exp is in the next fresh values",
                                    "query is in the next context", "output is in the next context"])
def test_layers_in_one_call_equal_layers_one_by_one(config, shared):
    p = LayeredProblem(config, 3, (mpic.MPIC_TIER_HBM,), None, **SMALL[config])
    p.plan_for()
    h, plan, scale = p.ctx.handle, p.plan.handle, p.sh.softmax_scale
    one = _tensors(p, shared)
    assert mpic.mpic_prefill_layers(h, plan, p.store.handle, p.ids, *([t[i] for t in one] for i in range(5)), scale,
                                    [t[5] for t in one], [t[6] for t in one]) is None
    ref = _tensors(p, shared)
    for l, (q, k, v, kc, vc, out, lse) in enumerate(ref):
        srcs = [mpic.mpic_store_layer(h, p.store.handle, i, l) for i in p.ids]
        mpic.mpic_assemble_kv(h, plan, srcs, k, v, kc, vc)
        mpic.mpic_selective_attn(h, plan, q, kc, vc, scale, out, lse)
    torch.cuda.synchronize()
    for got, want in zip(one, ref):
        for a, b in zip(got[3:], want[3:]):
            assert torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)) and torch.equal(torch.isnan(a), torch.isnan(b))
    if not shared.startswith("log"):  # (halves of fp32 numbers read as bf16 may be anything)
        assert not torch.isnan(one[-1][5]).any()
    p.close()
