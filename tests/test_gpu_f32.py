"""fp32 attention and decode on the matrix cores (needs an MI355X): sizes at the edges of the
32-column tiles, the 32-key blocks, the eight wavefronts and the key splits, against the oracle at
the fp32 gates (1e-5 relative)."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads
from helpers import assert_f32_close
from oracle import build_plan
from test_gpu_parity import _check_decode, _custom
from test_gpu_lazy import _run_lazy

pytestmark = pytest.mark.gpu


def _f32(requests, src_len, k, hq, hkv, d, **options):
    p = _custom([[("text", 1)]], 0, [], 0, sh_id=1)
    p.sh = sh = dataclasses.replace(p.sh, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, softmax_scale=float(1 / np.sqrt(d)))
    p.requests, p.n_src, p.src_len, p.k = requests, len(src_len), src_len, k
    p.n_slots = sum(workloads.request_len(r) for r in requests)
    p.oplan = build_plan(requests, k, 0, None)
    p.chunks = {s: workloads.gen_chunk(sh, 0, s, src_len[s]) for s in sorted(set(p.oplan["inst_src"].tolist()))}
    q_off = p.oplan["q_off"]
    fresh = [workloads.gen_fresh(sh, 0, b, int(q_off[b + 1] - q_off[b])) for b in range(len(requests))]
    p.q, p.fresh_k, p.fresh_v = (torch.cat([f[i] for f in fresh]) for i in range(3))
    for name, value in options.items():
        setattr(p, name, value)
    return p


# one key; one row past a tile; one key past a block; all wavefronts and one block more; several splits
_LAYOUTS = {
    "single": ([[("text", 1)]], [], 0),
    "row_edges": ([[("text", 31)], [("text", 32)], [("text", 33)], [("text", 65)]], [], 0),
    "key_edges": ([[("chunk", 0, 32, 0), ("text", 1)], [("chunk", 1, 255, 0), ("text", 2)], [("chunk", 2, 256, 0), ("text", 1)]],
                  [32, 255, 256], 0),
    "mixed": ([[("text", 5), ("chunk", 0, 300, None), ("text", 3), ("chunk", 1, 77, None), ("text", 41)],
               [("chunk", 1, 77, None), ("text", 0), ("chunk", 0, 300, None), ("text", 9)]], [300, 77], 7),
}


@pytest.mark.parametrize("heads", [(4, 4, 64), (6, 2, 128), (40, 1, 64)])
@pytest.mark.parametrize("layout", sorted(_LAYOUTS))
def test_fp32_tiles(layout, heads):
    requests, src_len, k = _LAYOUTS[layout]
    p = _f32(requests, src_len, k, *heads)
    p.gpu_setup(False)
    p.gpu_assemble()
    p.gpu_attend()
    torch.cuda.synchronize()
    K, V = p.oracle_link()
    O_ref, L_ref = p.oracle_attend(K, V)
    assert_f32_close(p.out.to(torch.float64).cpu().numpy(), O_ref, "attention output")
    L = p.lse.to(torch.float64).cpu().numpy()
    assert np.abs(L - L_ref).max() <= 1e-5 * max(1.0, np.abs(L_ref).max())
    _check_decode(p, True, (K, V))
    _check_decode(p, False, (K, V))


@pytest.mark.parametrize("heads", [(4, 4, 64), (6, 2, 128)])
@pytest.mark.parametrize("interleaved,pre_rope", [(False, False), (True, True)])
def test_fp32_tiles_turn_stored_keys_as_they_read_them(heads, interleaved, pre_rope):
    requests, src_len, k = _LAYOUTS["mixed"]
    _run_lazy(_f32(requests, src_len, k, *heads, interleaved=interleaved, pre_rope=pre_rope))
    _run_lazy(_f32(requests, src_len, k, *heads, interleaved=not interleaved, pre_rope=pre_rope))
