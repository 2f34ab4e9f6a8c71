"""Decode steps at the sizes where their route changes (needs an MI355X): contexts that stay in one
piece and write the output themselves, contexts one key longer that are split and merged, both next
to a request without any context; against the oracle at the gates of the decode tests."""
import dataclasses

import pytest
import torch

import workloads
from test_gpu_f32 import _f32
from test_gpu_lazy import _run_lazy
from test_gpu_parity import _check_decode, _custom

pytestmark = pytest.mark.gpu


def _bf16(lens, hq, hkv):
    p = _custom([[("chunk", i, n - 3, 5), ("text", 3)] if n > 3 else [("text", n)] for i, n in enumerate(lens)],
                len(lens), [max(1, n - 3) for n in lens], 5)
    p.sh = dataclasses.replace(p.sh, n_q_heads=hq, n_kv_heads=hkv)
    p.chunks = {s: workloads.gen_chunk(p.sh, 0, s, p.src_len[s]) for s in p.chunks}
    q_off = p.oplan["q_off"]
    fresh = [workloads.gen_fresh(p.sh, 0, b, int(q_off[b + 1] - q_off[b])) for b in range(len(lens))]
    p.q, p.fresh_k, p.fresh_v = (torch.cat([f[i] for f in fresh]) for i in range(3))
    return p


# one key; edges of a wavefront's block and of a workgroup's four; the longest unsplit context; the shortest split one
@pytest.mark.parametrize("heads", [(4, 4), (14, 2), (40, 1)])
@pytest.mark.parametrize("lens", [(1,), (31, 32, 33), (127, 0, 129), (256, 200), (257, 0, 7)])
def test_bf16_context_lengths(lens, heads):
    p = _bf16(lens, *heads)
    p.gpu_setup(False)
    p.gpu_assemble()
    _check_decode(p, True)
    _check_decode(p, False)


@pytest.mark.parametrize("n", [64, 224, 256, 290])     # (slots of key blocks: up to 31 more per source than keys)
def test_lazy_context_lengths(n):
    _run_lazy(_bf16((n, 50), 14, 2))


@pytest.mark.parametrize("heads", [(6, 2, 128), (4, 4, 64), (40, 1, 64)])
@pytest.mark.parametrize("lens", [(1, 0), (255, 256), (257, 0, 3)])
def test_fp32_context_lengths(lens, heads):
    p = _f32([[("text", n)] for n in lens], [], 0, *heads)
    p.gpu_setup(False)
    p.gpu_assemble()
    _check_decode(p, True)
    _check_decode(p, False)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_new_token_that_is_no_number(dtype):
    """A NaN in the key of the new token reaches its request's rows, whether or not the request has a context."""
    p = _bf16((5, 0, 0), 14, 2) if dtype == "bf16" else _f32([[("text", n)] for n in (5, 0, 0)], [], 0, 6, 2, 128)
    p.gpu_setup(False)
    p.gpu_assemble()
    q, nk, nv = p.decode_inputs()
    nk[:2, :, 3] = float("nan")
    out, lse = p.gpu_decode(q, nk, nv)
    assert torch.isnan(torch.from_numpy(out[:2])).all() and torch.isnan(torch.from_numpy(lse[:2])).all()
    assert (out[2] == nv[2].double().repeat_interleave(p.sh.n_q_heads // p.sh.n_kv_heads, 0).numpy()).all()
