"""Performance cases of the selective-recompute prefill path, as a serving program calls it.

A case is a dict of plain values.  What it does, by "kind":
  layer     link one layer's context (mpic_assemble_kv), then attend (mpic_selective_attn)
  next      scatter the fresh rows of a layer whose stored rows are linked already, attend and link
            the stored rows of the next layer in the same launch (mpic_selective_attn_link_next)
  in_place  lazy_rope context: scatter the fresh rows, attend with the caches read where they are
            stored (mpic_selective_attn_in_place)
  decode    one decode step over the linked context (mpic_decode_attn)
  decode_in_place  the same with the caches read where they are stored
  request   a new request from its plan to the last layer: Plan, then mpic_prefill_layers with the
            caches fetched from the store (GPU memory or pinned host memory)

Model shapes and layouts are those of the repository's workloads (tiny fp32, LLaVA-1.5-like,
LLaVA-1.6-like, retrieval with a shared pool, long paged context) and ragged variants of them.
"""
import math
import random

import torch

import paper_2502_01960_amd as mpic

# (query heads, kv heads, head dim, rotary base) of the workloads' model shapes
MODELS = {
    "tiny": (4, 4, 64, 1.0e4),
    "llava15": (32, 32, 128, 1.0e4),
    "llava16": (28, 4, 128, 1.0e6),
    "mrag": (32, 8, 128, 5.0e5),
    "long": (64, 8, 128, 1.0e6),
}

DEFAULTS = dict(kind="layer", model="llava16", dtype="bf16", batch=1, chunks=4, chunk_len=576, text_len=64,
                tail=0,            # tokens of the question after the last text segment
                lead=True,         # text in front of every chunk (False: references back to back)
                k=32,              # tokens recomputed at the head of every chunk
                listed=False,      # the k tokens of a chunk are drawn all over it and named one by one
                missing=0,         # chunks per request whose cache is missing: recomputed as a whole
                pool=0,            # > 0: the requests draw their chunks from this many shared ones
                ragged=False,      # every length drawn from half the stated one up to it
                page=0, interleaved=False, pre_rope=False, lse=False, layers=1, tier="hbm",
                layout=1)          # number of the drawn layout


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # the smallest call: the tiny fp32 configuration (152 tokens, 40 fresh rows), launches and latency
        _case("tiny_f32", model="tiny", dtype="f32", chunks=2, chunk_len=64, text_len=8, k=8),
        # the validation precision on one image of a full-size model shape
        _case("f32_image", model="llava15", dtype="f32", chunks=1, chunk_len=576, text_len=40, tail=37, k=32, lse=True),
        # an ordinary single request: four 576-token images, multi-head attention
        _case("llava15_layer", model="llava15", chunks=4, chunk_len=576, text_len=64, k=32),
        # the headline batch: 4 requests x 8 images of 2304 tokens, steady state of the layer loop
        _case("llava16_next", kind="next", batch=4, chunks=8, chunk_len=2304, text_len=128, tail=256, k=64),
        # one turn of a conversation: odd lengths, fresh rows before positional embedding, interleaved
        # pairing, one cache missing
        _case("turn_ragged", chunks=3, chunk_len=2304, text_len=90, tail=61, k=32, missing=1, ragged=True,
              interleaved=True, pre_rope=True, lse=True, layout=7),
        # retrieval: 8 requests x 16 references of 1024 tokens out of a pool of 64
        _case("mrag_layer", model="mrag", batch=8, chunks=16, chunk_len=1024, text_len=512, lead=False, pool=64, k=64),
        # one long request into 16-token pages
        _case("long_paged", model="long", chunks=32, chunk_len=2304, text_len=64, k=32, page=16),
        # caches linked by reference, recompute set named token by token
        _case("listed_in_place", kind="in_place", model="mrag", batch=2, chunks=6, chunk_len=1024, text_len=120, k=48,
              listed=True, ragged=True, layout=5),
        # decode steps after those prefills
        _case("decode_llava15", kind="decode", model="llava15", chunks=4, chunk_len=576, text_len=64, k=32),
        _case("decode_llava16", kind="decode", batch=4, chunks=8, chunk_len=2304, text_len=128, tail=256, k=64),
        _case("decode_mrag_in_place", kind="decode_in_place", model="mrag", batch=8, chunks=16, chunk_len=1024,
              text_len=512, lead=False, pool=64, k=64),
        # a new request through the cache library: plan and four layers
        _case("request_hbm", kind="request", chunks=4, chunk_len=576, text_len=64, tail=100, k=32, layers=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: model shapes of the workloads, 1 to 8 requests of 1 to 32
    chunks of 64 to 2304 tokens, texts of 8 to 512 tokens, k from none to 128."""
    biggest = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["layer", "layer", "next", "in_place", "decode", "decode", "decode_in_place", "request"])
        f32 = rng.random() < 0.15
        model = rng.choice(["tiny", "llava15"] if f32 else ["llava15", "llava16", "llava16", "mrag", "long"])
        chunks = _log(rng, 1, 4 if f32 else 32)
        pooled = rng.random() < 0.25
        c = _case(kind=kind, model=model, dtype="f32" if f32 else "bf16", batch=1 if f32 else rng.randint(1, 8), chunks=chunks,
                  chunk_len=_log(rng, 64, 576 if f32 else 2304), text_len=_log(rng, 8, 128 if f32 else 512),
                  tail=rng.choice([0, _log(rng, 8, 256)]), lead=rng.random() < 0.8,
                  k=rng.choice([0, 8, 16, 32, 32, 64, 64, 128]), listed=rng.random() < 0.15,
                  missing=1 if rng.random() < 0.1 else 0, pool=chunks * rng.randint(1, 4) if pooled else 0,
                  ragged=rng.random() < 0.7, page=rng.choice([0, 0, 16, 64]), interleaved=rng.random() < 0.2,
                  pre_rope=rng.random() < 0.25, lse=rng.random() < 0.3,
                  layers=rng.randint(2, 4) if kind == "request" else 1,
                  tier=rng.choice(["hbm", "hbm", "host"]) if kind == "request" else "hbm", layout=rng.randint(1, 1 << 20))
        # chunk instances of a batch read in place: at most 128; caches put into a store: at most 1 GB
        if kind in ("in_place", "decode_in_place") and c["batch"] * chunks > 128:
            continue
        if kind == "request" and _store_bytes(c) > 1 << 30:
            continue
        if _cost(c) <= biggest and _context_bytes(c) <= 2 << 30:
            return c


# ---------------------------------------------------------------- sizes
def _layout(case):
    """(requests as the planner takes them, token counts of the chunk sources)."""
    rng = random.Random(case["layout"])

    def length(n):
        return rng.randint(max(1, n // 2), n) if case["ragged"] else n

    n_src = case["pool"] or case["batch"] * case["chunks"]
    src_len = [length(case["chunk_len"]) for _ in range(n_src)]
    requests = []
    for b in range(case["batch"]):
        first = b * case["chunks"]
        ids = rng.sample(range(n_src), case["chunks"]) if case["pool"] else range(first, first + case["chunks"])
        segs = []
        for i, s in enumerate(ids):
            if case["lead"]:
                segs.append(("text", length(case["text_len"])))
            if i < case["missing"]:
                k = src_len[s]
            elif case["listed"]:
                k = sorted(rng.sample(range(src_len[s]), min(case["k"], src_len[s])))
            else:
                k = case["k"]
            segs.append(("chunk", s, src_len[s], k))
        segs.append(("text", length(case["text_len"])))
        if case["tail"]:
            segs.append(("text", length(case["tail"])))
        requests.append(segs)
    return requests, src_len


def _counts(case):
    """Per request (context tokens, positions of the fresh rows), and the stored rows read, each
    distinct source counted once (a row that any request takes from its cache is read)."""
    requests, src_len = _layout(case)
    per, used = [], {}
    for segs in requests:
        pos, fresh = 0, []
        for s in segs:
            if s[0] == "text":
                fresh.extend(range(pos, pos + s[1]))
                pos += s[1]
            else:
                again = set(s[3]) if isinstance(s[3], list) else set(range(min(s[3], s[2])))
                fresh.extend(pos + t for t in sorted(again))
                used[s[1]] = max(used.get(s[1], 0), s[2] - len(again))
                pos += s[2]
        per.append((pos, fresh))
    return per, sum(used.values())


def _row_bytes(case):
    _, hkv, d, _ = MODELS[case["model"]]
    return hkv * d * (4 if case["dtype"] == "f32" else 2)


def _store_bytes(case):
    n_src = case["pool"] or case["batch"] * case["chunks"]
    return 2 * case["layers"] * n_src * case["chunk_len"] * _row_bytes(case)


def _context_bytes(case):
    return 2 * sum(n for n, _ in _counts(case)[0]) * _row_bytes(case) * case["layers"]


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def work(case):
    """Bytes and flops of one pass: every input row read once, every output row written once; 4*D
    flops per (query, head, visible key)."""
    hq, hkv, d, _ = MODELS[case["model"]]
    per, stored = _counts(case)
    row = _row_bytes(case)
    qrow = row * hq // hkv
    n = sum(p[0] for p in per)
    nq = sum(len(p[1]) for p in per)
    if case["kind"].startswith("decode"):
        # the context (or the caches and the fresh rows) once, the new rows, the output
        rows = n if case["kind"] == "decode" else stored + nq
        return {"bytes": 2 * rows * row + case["batch"] * (2 * qrow + 2 * row), "flops": 4 * d * hq * (n + case["batch"])}
    flops = 4 * d * hq * sum(p + 1 for _, fresh in per for p in fresh)
    attend = 2 * nq * qrow                     # queries in, output out
    fresh = 4 * nq * row                       # fresh K and V in, their context rows out
    linked = 2 * (stored + n - nq) * row       # caches in, stored context rows out
    if case["kind"] == "in_place":
        total = attend + fresh + 2 * stored * row
    elif case["kind"] == "next":
        total = attend + fresh + linked + 2 * (n - nq) * row  # this layer's stored rows are read too
    else:
        total = attend + fresh + linked
    return {"bytes": case["layers"] * total, "flops": case["layers"] * flops}


# Measured against the same path in float64 over the listed cases: bf16 outputs are off by 2.9e-3 at most
# (rounded to 8 bits, probabilities rounded before the second product; the largest difference is 3.9e-2 of the
# root mean square), fp32 outputs by 2.4e-7 (3.3e-6).  About four times that is allowed.
def tolerance(case):
    return {"rel": 1e-6, "max": 1.5e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.15}


# ---------------------------------------------------------------- state
def prepare(case, seed):
    hq, hkv, d, theta = MODELS[case["model"]]
    f32 = case["dtype"] == "f32"
    dtype = torch.float32 if f32 else torch.bfloat16
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32).to(dtype)

    requests, src_len = _layout(case)
    per, _ = _counts(case)
    lens = [n for n, _ in per]
    nq = sum(len(fresh) for _, fresh in per)
    page = case["page"]
    tables, n_pages, n_slots = None, 0, sum(lens)
    if page:
        need = [(n + page - 1) // page for n in lens]
        n_pages = -(-5 * sum(need) // 4)
        ids = list(range(n_pages))
        random.Random(case["layout"] + 1).shuffle(ids)
        tables = [ids[sum(need[:b]):sum(need[:b + 1])] for b in range(len(need))]
        n_slots = n_pages * page

    kind = case["kind"]
    ctx = mpic.Context(hq, hkv, d, mpic.MPIC_F32 if f32 else mpic.MPIC_BF16, theta, int(case["interleaved"]), page,
                       int(case["pre_rope"]), int(kind in ("in_place", "decode_in_place")))
    s = dict(case, ctx=ctx, scale=1.0 / math.sqrt(d), plan_args=(requests, case["k"], tables, n_pages), event=None)
    n_layers = case["layers"]
    zeros = lambda *shape: torch.zeros(shape, device=dev, dtype=dtype)
    s["q"] = [normal(nq, hq, d) for _ in range(n_layers)]
    s["fk"] = [normal(nq, hkv, d) for _ in range(n_layers)]
    s["fv"] = [normal(nq, hkv, d) for _ in range(n_layers)]
    n_ctx = 2 if kind == "next" else n_layers
    s["kc"] = [zeros(n_slots, hkv, d) for _ in range(n_ctx)]
    s["vc"] = [zeros(n_slots, hkv, d) for _ in range(n_ctx)]
    s["out"] = [zeros(nq, hq, d) for _ in range(n_layers)]
    s["lse"] = [torch.zeros((nq, hq), device=dev, dtype=torch.float32) for _ in range(n_layers)] if case["lse"] else None

    if kind == "request":
        s["store"] = mpic.Store(ctx, n_layers)
        s["ids"] = [1000 + i for i in range(len(src_len))]
        tier = mpic.MPIC_TIER_HOST if case["tier"] == "host" else mpic.MPIC_TIER_HBM
        for i, n in zip(s["ids"], src_len):
            s["store"].put(i, normal(n_layers, n, hkv, d).cpu(), normal(n_layers, n, hkv, d).cpu(), tier)
        s["plan"] = None
        return s

    s["plan"] = mpic.Plan(ctx, *s["plan_args"])
    s["srcs"] = mpic.ChunkSources([(normal(n, hkv, d), normal(n, hkv, d)) for n in src_len])
    h, p = ctx.handle, s["plan"].handle
    if kind == "next":
        # this layer's stored rows come from the launch of the layer before
        before = mpic.ChunkSources([(normal(n, hkv, d), normal(n, hkv, d)) for n in src_len])
        mpic.mpic_assemble_kv_parts(h, p, before, None, None, s["kc"][0], s["vc"][0], mpic.MPIC_PART_CACHED)
    elif kind == "decode":
        mpic.mpic_assemble_kv(h, p, s["srcs"], s["fk"][0], s["fv"][0], s["kc"][0], s["vc"][0])
    elif kind == "decode_in_place":
        mpic.mpic_assemble_kv_parts(h, p, None, s["fk"][0], s["fv"][0], s["kc"][0], s["vc"][0], mpic.MPIC_PART_FRESH)
    if kind.startswith("decode"):
        b = len(lens)
        s["q"], s["nk"], s["nv"] = normal(b, hq, d), normal(b, hkv, d), normal(b, hkv, d)
        s["out"] = zeros(b, hq, d)
        s["lse"] = torch.zeros((b, hq), device=dev, dtype=torch.float32) if case["lse"] else None
    torch.cuda.synchronize()
    return s


def run(s):
    kind, h, scale, kc, vc = s["kind"], s["ctx"].handle, s["scale"], s["kc"], s["vc"]
    if kind == "request":
        # the plan of the request before this one is given back once its GPU work is done
        plan = mpic.Plan(s["ctx"], *s["plan_args"])
        failed = mpic.mpic_prefill_layers(h, plan.handle, s["store"].handle, s["ids"], s["q"], s["fk"], s["fv"], kc, vc,
                                          scale, s["out"], s["lse"])
        if s["plan"] is not None:
            s["event"].synchronize()
            s["plan"].close()
        s["plan"], s["event"] = plan, torch.cuda.Event()
        s["event"].record()
        return {"out": s["out"], "lse": s["lse"], "k_ctx": kc, "v_ctx": vc, "failed": 0 if failed is None else len(failed)}
    p = s["plan"].handle
    if kind == "decode":
        mpic.mpic_decode_attn(h, p, s["q"], s["nk"], s["nv"], kc[0], vc[0], scale, s["out"], s["lse"])
        return {"out": s["out"], "lse": s["lse"]}
    if kind == "decode_in_place":
        mpic.mpic_decode_attn_in_place(h, p, s["q"], s["nk"], s["nv"], s["srcs"], kc[0], vc[0], scale, s["out"], s["lse"])
        return {"out": s["out"], "lse": s["lse"]}
    q, fk, fv, out, lse = s["q"][0], s["fk"][0], s["fv"][0], s["out"][0], s["lse"][0] if s["lse"] else None
    if kind == "layer":
        mpic.mpic_assemble_kv(h, p, s["srcs"], fk, fv, kc[0], vc[0])
        mpic.mpic_selective_attn(h, p, q, kc[0], vc[0], scale, out, lse)
    else:
        mpic.mpic_assemble_kv_parts(h, p, None, fk, fv, kc[0], vc[0], mpic.MPIC_PART_FRESH)
        if kind == "next":
            mpic.mpic_selective_attn_link_next(h, p, q, kc[0], vc[0], scale, out, s["srcs"], kc[1], vc[1], lse)
        else:
            mpic.mpic_selective_attn_in_place(h, p, q, s["srcs"], kc[0], vc[0], scale, out, lse)
    return {"out": out, "lse": lse, "k_ctx": kc, "v_ctx": vc}
