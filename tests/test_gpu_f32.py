"""fp32 attention and decode on the matrix cores (needs an MI355X): sizes at the edges of the
32-column tiles, the 32-key blocks, the eight wavefronts and the key splits, against the oracle at
the fp32 gates (1e-5 relative)."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads
from helpers import assert_f32_close
from oracle import attend, build_plan
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


# tiles cut along the keys (more than 8 blocks of 32): one block more than stays whole, a ragged last piece, rows at
# both ends of the context in one tile (the early ones see nothing of the later pieces), a short request beside
_CUT_LAYOUTS = {
    "one_more": ([[("chunk", 0, 256, 0), ("text", 1)]], [256], 0),
    "ragged": ([[("text", 7), ("chunk", 0, 700, None), ("text", 11)]], [700], 9),
    "both_ends": ([[("text", 9), ("chunk", 0, 1003, 0), ("text", 5)], [("text", 3)]], [1003], 0),
}


@pytest.mark.parametrize("heads", [(4, 4, 64), (6, 2, 128), (40, 1, 64)])
@pytest.mark.parametrize("layout", sorted(_CUT_LAYOUTS))
def test_fp32_tiles_cut_along_the_keys(layout, heads):
    requests, src_len, k = _CUT_LAYOUTS[layout]
    p = _f32(requests, src_len, k, *heads)
    p.gpu_setup(False)
    p.gpu_assemble()
    p.gpu_attend()
    torch.cuda.synchronize()
    K, V = p.oracle_link()
    O_ref, L_ref = p.oracle_attend(K, V)
    assert_f32_close(p.out.to(torch.float64).cpu().numpy(), O_ref, "attention output")
    assert np.abs(p.lse.to(torch.float64).cpu().numpy() - L_ref).max() <= 1e-5 * max(1.0, np.abs(L_ref).max())
    _run_lazy(_f32(requests, src_len, k, *heads, pre_rope=True))


@pytest.mark.parametrize("heads", [(4, 4, 64), (6, 2, 128)])
@pytest.mark.parametrize("interleaved,pre_rope", [(False, False), (True, True)])
def test_fp32_tiles_turn_stored_keys_as_they_read_them(heads, interleaved, pre_rope):
    requests, src_len, k = _LAYOUTS["mixed"]
    _run_lazy(_f32(requests, src_len, k, *heads, interleaved=interleaved, pre_rope=pre_rope))
    _run_lazy(_f32(requests, src_len, k, *heads, interleaved=not interleaved, pre_rope=pre_rope))


def _plain_loops(q, K, V, seen, scale):
    """One head in fp32 the plain way: every logit one chain of fused multiply-adds, weights rounded
    once, 64 partial sums over the keys and a tree over them.  q [R][D], K, V [n][D], seen [R]: keys a
    row sees."""
    f32, f64 = np.float32, np.float64
    R, (n, d) = len(q), K.shape
    s = np.zeros((R, n), f32)
    for i in range(d):
        s = (s.astype(f64) + q[:, i, None].astype(f64) * K[None, :, i]).astype(f32)
    s = np.where(np.arange(n)[None] < seen[:, None], s * f32(scale), f32(-np.inf))
    w = np.exp((s - s.max(1, keepdims=True)).astype(f64)).astype(f32)
    pad = -n % 64
    w = np.pad(w, ((0, 0), (0, pad))).reshape(R, -1, 64)
    Vp = np.pad(V, ((0, pad), (0, 0))).reshape(-1, 64, d)
    z, o = np.zeros((R, 64), f32), np.zeros((R, 64, d), f32)
    for t in range(w.shape[1]):
        z = z + w[:, t]
        o = (o.astype(f64) + w[:, t, :, None].astype(f64) * Vp[t]).astype(f32)
    while z.shape[1] > 1:
        half = z.shape[1] // 2
        z, o = z[:, :half] + z[:, half:], o[:, :half] + o[:, half:]
    return o[:, 0] * (f32(1) / z)


@pytest.mark.parametrize("heads,text,chunk", [((8, 8, 128), 77, 576), ((4, 4, 64), 80, 1500)])
def test_fp32_error_is_no_larger_than_that_of_plain_loops(heads, text, chunk):
    """Against float64 over the context as it was linked: the matrix instructions and the split of the
    keys may not cost accuracy.  Both sides are root mean squares over thousands of outputs; the
    kernels are at 0.7 to 0.8 of the plain loops' error in prefill and 0.7 to 0.95 in decode."""
    p = _f32([[("text", text // 2), ("chunk", 0, chunk, None), ("text", text - text // 2)]], [chunk], 32, *heads)
    p.gpu_setup(False)
    p.gpu_assemble()
    p.gpu_attend()
    K, V = p.gpu_logical_kv()
    f32 = lambda x: x.astype(np.float32)
    group, scale = heads[0] // heads[1], p.sh.softmax_scale

    def rms(got, ref):
        return np.sqrt(((got.astype(np.float64) - ref) ** 2).mean())

    def plain(q, seen):
        q = q.to(torch.float32).numpy()
        return np.stack([_plain_loops(q[:, h], f32(K[:, h // group]), f32(V[:, h // group]), seen, scale)
                         for h in range(heads[0])], axis=1)

    ref, _ = attend(p.q.to(torch.float64).numpy(), K, V, p.oplan, np.float32(scale))
    assert rms(p.out.cpu().numpy(), ref) <= rms(plain(p.q, p.oplan["q_pos"] + 1), ref)
    if heads[2] == 128:   # (four rows of 64 coordinates are too few to compare)
        q = p.decode_inputs()[0]
        got, _ = p.gpu_decode(q, None, None)
        ref, _ = p.oracle_decode(K, V, q, None, None)
        assert rms(got, ref) <= rms(plain(q, np.array([len(K)])), ref)


@pytest.mark.parametrize("heads", [(4, 4, 64), (6, 2, 128)])
@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("source", ["fresh", "stored"])
def test_fp32_rows_keep_clear_of_values_behind_them(heads, lazy, source):
    """An infinity and a NaN in the value row of one position: the rows in front of it do not notice,
    the others (and a decode step, whose last block repeats the last row as padding) notice in those
    coordinates only; a NaN in its key row reaches none of the rows in front of it."""
    requests = [[("text", 20), ("chunk", 0, 300, None), ("text", 3), ("chunk", 1, 77, None), ("text", 30)]]
    p = _f32(requests, [300, 77], 7, *heads)
    p.lazy = lazy
    at, row = (409, int(np.flatnonzero(p.oplan["q_pos"] == 409)[0])) if source == "fresh" else (200, 180)
    q, nk, nv = p.decode_inputs()

    def run():
        p.gpu_setup(False)
        if lazy:
            p.gpu_link_fresh_only()
            p.gpu_attend_in_place()
            decode = p.gpu_decode_in_place(q, None, None)[0]
        else:
            p.gpu_assemble()
            p.gpu_attend()
            decode = p.gpu_decode(q, None, None)[0]
        torch.cuda.synchronize()
        return p.out.to(torch.float64).cpu().numpy(), p.lse.to(torch.float64).cpu().numpy(), decode

    K, V = p.oracle_link()
    O_ref, L_ref = p.oracle_attend(K, V)
    D_ref, _ = p.oracle_decode(K, V, q, None, None)
    values = p.fresh_v if source == "fresh" else p.chunks[0][1]
    keys = p.fresh_k if source == "fresh" else p.chunks[0][0]
    before = p.oplan["q_pos"] < at
    assert before.any() and not before.all()
    values[row, :, 5], values[row, :, 40] = float("inf"), float("nan")
    out, lse, decode = run()
    assert np.abs(lse - L_ref).max() <= 1e-5 * np.abs(L_ref).max()
    assert_f32_close(out[before], O_ref[before], "rows in front of the spoiled position")
    assert np.isposinf(out[~before][..., 5]).all() and np.isnan(out[~before][..., 40]).all()
    assert np.isposinf(decode[..., 5]).all() and np.isnan(decode[..., 40]).all()
    rest = np.ones(heads[2], dtype=bool)
    rest[[5, 40]] = False
    assert_f32_close(out[~before][..., rest], O_ref[~before][..., rest], "other coordinates")
    assert_f32_close(decode[..., rest], D_ref[..., rest], "other coordinates of the decode step")
    keys[row, :, 7] = float("nan")
    out, lse, decode = run()
    assert_f32_close(out[before], O_ref[before], "rows in front of the spoiled key")
    assert np.abs(lse - L_ref)[before].max() <= 1e-5 * np.abs(L_ref).max()
    assert np.isnan(out[~before]).all() and np.isnan(lse[~before]).all() and np.isnan(decode).all()
