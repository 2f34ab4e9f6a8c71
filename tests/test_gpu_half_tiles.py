"""Attention over caches read in place in half tiles (needs an MI355X): tiles with no second half, with
one row in it, rows that straddle it, pieces that a half sees nothing of, and head groupings whose heads
split over the halves; both lazy routes against the oracle at the gates of the lazy tests."""
import numpy as np
import pytest

import paper_2502_01960_amd as mpic
from test_gpu_decode_sizes import _bf16
from test_gpu_lazy import _run_lazy
from test_gpu_parity import _custom

pytestmark = pytest.mark.gpu


# fresh rows per request (one kv head: as many flattened rows): up to the half, one more, a whole tile, one more
@pytest.mark.parametrize("heads", [(1, 1), (3, 1), (28, 4)])
@pytest.mark.parametrize("fresh", [1, 127, 128, 129, 256, 257])
def test_rows_around_the_half(fresh, heads):
    p = _bf16((fresh + 300, 40), *heads)
    requests = [[("text", fresh // 2), ("chunk", 0, p.src_len[0], 0), ("text", fresh - fresh // 2)], p.requests[1]]
    q = _custom(requests, 2, p.src_len, 5)
    q.sh = p.sh
    import torch
    import workloads
    q.chunks = {s: workloads.gen_chunk(q.sh, 0, s, q.src_len[s]) for s in q.chunks}
    q_off = q.oplan["q_off"]
    rows = [workloads.gen_fresh(q.sh, 0, b, int(q_off[b + 1] - q_off[b])) for b in range(2)]
    q.q, q.fresh_k, q.fresh_v = (torch.cat([r[i] for r in rows]) for i in range(3))
    _run_lazy(q)


@pytest.mark.parametrize("pre_rope,interleaved", [(False, False), (True, True)])
def test_halves_of_cut_tiles(pre_rope, interleaved):
    """One long request: pieces along the keys, the first half of whose rows sits at the start of the context."""
    requests = [[("text", 40), ("chunk", 0, 1900, 7), ("text", 30), ("chunk", 1, 700, None), ("text", 9)]]
    p = _custom(requests, 2, [1900, 700], 3)
    p.pre_rope, p.interleaved = pre_rope, interleaved
    _run_lazy(p)


@pytest.mark.parametrize("k", [16, 64])
def test_error_is_no_larger_than_in_whole_tiles(k):
    """Against float64: both round their weights to bf16, relative to reference points that halves take from more keys."""
    p = _custom([[("text", 190), ("chunk", i, 400, k), ("text", 160)] for i in range(4)], 4, [400] * 4, 3)
    p.lazy = True
    p.gpu_setup(False)
    p.gpu_assemble()
    ref, _ = p.oracle_attend(*p.oracle_link())
    outs, err = {}, {}
    for block_keys in (0, 96):
        p.ctx.set_option(mpic.MPIC_OPT_ATTN_BLOCK_KEYS, block_keys)
        p.gpu_attend()
        outs[block_keys] = p.out.double().cpu().numpy()
        err[block_keys] = np.linalg.norm(outs[block_keys] - ref) / np.linalg.norm(ref)
    assert not np.array_equal(outs[0], outs[96]), "the launch is to run in half tiles"
    assert err[0] <= err[96], err
