"""Attention tiles cut along the keys into pieces of unequal length (needs an MI355X)."""
import pytest

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
