"""Workloads that the library's speed is measured on: what a program that serves long-context or vision-language
models has it do, from one layer's call to a whole long-video cache, through the public entry points of
`paper_2510_20707_amd.binding`.

A case is a dict of plain values; `op` is the entry point it goes through:

  compress    the whole compression step after a prefill
  score       the mixed scores alone
  select      the selection on scores that the caller brings
  similarity  the redundancy analysis of cached keys
  decode      one decoding step on a compacted cache: the new token's rows appended, then its attention

Caches are synthetic, with the statistics of the seeded recipe in `paper_2510_20707_amd.synth`, drawn on the device:
text keys share a mean direction, visual keys lie around centroids in a 16-dimensional subspace (drifting from frame
to frame in a video), values are normal, window queries carry 1/sqrt(D).
"""
import torch

from paper_2510_20707_amd import binding as B

DEV = "cuda:0"
FRAME = 510                  # visual tokens per video frame
TEXT = 64                    # text tokens before and after the visual block


# ------------------------------------------------------------------------------------------------- the cases
def _compress(**kw):
    c = dict(op="compress", dtype="bf16", layers=28, batch=1, hq=28, hkv=4, d=128, n=8192, w=32, b=64, keys="image",
             pool="max", pool_k=7, mode="fixed", floor=0, intrinsic="vnorm", mix="head_adaptive", lse=False,
             room=0, scores=False, prepared=True)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one fp32 layer of 512 tokens, arguments marshalled per call; latency and launches
        _compress(name="compress_tiny_f32", dtype="f32", layers=1, hq=4, hkv=2, d=64, n=512, w=8, b=64, keys="iid",
                  scores=True, prepared=False),
        # one layer of a 4K image prompt, compressed as soon as that layer's prefill attention is done
        _compress(name="compress_layer_4k", layers=1, n=4096, prepared=False),
        # the headline: a whole 28-layer cache of an 8K image prompt, smallest budget
        _compress(name="compress_image_8k"),
        # the same model on a prompt of odd length, inside buffers allocated for 8192 tokens, softmax normalisers handed
        # over by the prefill attention, per-layer (pyramid) budgets of 256 rows on average
        _compress(name="compress_lse_pyramid_7k", n=7013, room=8192, b=256, mode="per_head", lse=True),
        # text-only 16K cache of a 32-layer, 8-KV-head model
        _compress(name="compress_text_16k", layers=32, hq=32, hkv=8, n=16384, b=256, keys="text"),
        # four 32K video prompts, head-adaptive budgets
        _compress(name="compress_video_32k", batch=4, n=32768, b=128, keys="video", mode="adaptive", floor=32),
        # one two-hour video: 256 frames in one prompt, beyond what fits one workgroup's selection
        _compress(name="compress_video_130k", n=2 * TEXT + 256 * FRAME, b=128, keys="video", mode="adaptive", floor=32),
        # fp32 scores of a small model with 64-element heads, odd length, average pooling (an analysis run)
        _compress(name="score_f32_3k", op="score", dtype="f32", layers=8, batch=2, hq=16, hkv=8, d=64, n=3001, w=16,
                  keys="text", pool="avg", pool_k=5, scores=True),
        # head-adaptive selection at the largest budget on an importance score computed elsewhere
        dict(name="select_adaptive_8k", op="select", layers=28, batch=1, hkv=4, n=8192, w=32, b=512, mode="adaptive", floor=128),
        # redundancy and 64-token heat-map of every head's keys of the 8K cache
        dict(name="similarity_8k", op="similarity", dtype="bf16", layers=28, batch=1, hkv=4, d=128, n=8192, block=64, keys="image"),
        # a decoding step of one sequence, one layer at a time, right after compression to 64 rows
        dict(name="decode_layer_64", op="decode", dtype="bf16", layers=1, batch=1, hq=28, hkv=4, d=128, b=64, tail=17, mode="fixed"),
        # a decoding step of a batch of 32 sequences on caches of 1024 rows, heads keeping unequal numbers of rows
        dict(name="decode_batch_1024", op="decode", dtype="bf16", layers=1, batch=32, hq=32, hkv=8, d=128, b=1024, tail=65,
             mode="adaptive"),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the same ranges: 256 to 131072 tokens, one to 32 layers, budgets up to 2048 rows."""
    heads = [(28, 4), (32, 8), (16, 8), (12, 2), (4, 2), (40, 8), (8, 8)]
    op = rng.choice(["compress"] * 6 + ["score", "select", "similarity", "decode", "decode", "decode"])
    hq, hkv = rng.choice(heads)
    d = rng.choice([128, 128, 128, 64])
    dtype = rng.choice(["bf16"] * 5 + ["f32"])
    if op == "decode":
        b = _log(rng, 48, 2048)
        layers = rng.choice([1, 1, 1, 28])
        batch = _log(rng, 1, 48) if layers == 1 else _log(rng, 1, 3)
        return dict(op=op, dtype=dtype, layers=layers, batch=batch, hq=hq, hkv=hkv, d=d, b=b, tail=_log(rng, 1, 300),
                    mode=rng.choice(["fixed", "adaptive"]))
    layers = rng.choice([1, _log(rng, 1, 32), 28, 32])
    batch = _log(rng, 1, 4)
    n = _log(rng, 256, 131072)
    # no dearer than the 32K video cache: 448 heads of 32768 keys
    limit = 448 * 32768 // (4 if dtype == "f32" and op in ("compress", "score") else 1)
    while layers * batch * hkv * n > limit:
        layers, batch = max(1, layers // 2), max(1, batch - 1)
        if layers == batch == 1:
            break
    if op == "similarity":
        block = _log(rng, max(8, -(-n // 512)), min(n, 512))
        return dict(op=op, dtype=dtype, layers=layers, batch=batch, hkv=hkv, d=d, n=n, block=block, keys=rng.choice(["text", "image"]))
    w = rng.choice([32, 32, 16, 8])
    b = _log(rng, w + 1, max(w + 2, min(2048, n // 2)))
    mode = rng.choice(["fixed", "fixed", "adaptive"])
    floor = rng.randrange((b - w) // 2 + 1) if mode == "adaptive" else 0
    if op == "select":
        return dict(op=op, layers=layers, batch=batch, hkv=hkv, n=n, w=w, b=b, mode=mode, floor=floor)
    if mode == "fixed" and rng.random() < 0.3:
        mode = "per_head"
    pool, pool_k = rng.choice([("max", 7), ("max", 7), ("avg", 5), ("none", 1)])
    intrinsic, mix = rng.choice([("vnorm", "head_adaptive")] * 4 + [("none", "imp_only"), ("knorm", "head_adaptive"), ("vnorm", "sum")])
    return _compress(op=op, dtype=dtype, layers=layers, batch=batch, hq=hq, hkv=hkv, d=d, n=n, w=w, b=b,
                     keys=rng.choice(["text", "image"]), pool=pool, pool_k=pool_k, mode=mode, floor=floor,
                     intrinsic=intrinsic, mix=mix, lse=rng.random() < 0.25, room=rng.choice([0, 0, n + 1 + rng.randrange(n)]),
                     scores=op == "score" or rng.random() < 0.3, prepared=op == "score" or layers > 1)


# ------------------------------------------------------------------------------------------------- inputs
def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _keys(c, g):
    """Keys of one layer, fp32 [batch, hkv, n, d]."""
    bt, h, n, d = c["batch"], c["hkv"], c["n"], c["d"]
    rand = lambda *shape: torch.randn(shape, generator=g, device=DEV)  # noqa: E731
    z = rand(bt, h, n, d)
    if c["keys"] == "iid":
        return z
    mu = rand(bt, h, 1, d)
    mu /= mu.norm(dim=-1, keepdim=True)
    if c["keys"] == "text":
        return z.add_(0.5 * mu)
    # text spans (mean pairwise cosine about 0.3) around clustered visual keys (0.4 to 0.8)
    k = z
    p0, p1 = min(TEXT, n // 4), n - min(TEXT, n // 4)
    k[:, :, :p0] += 7.4 * mu
    k[:, :, p1:] += 7.4 * mu
    nv = p1 - p0
    frames = max(1, nv // FRAME) if c["keys"] == "video" else 1
    sub = rand(bt, h, 16, d) / d ** 0.5
    cent = (rand(bt, h, 64, 16).unsqueeze(-1) * sub.unsqueeze(2)).sum(3)             # [bt, h, 64, d]
    which = torch.randint(0, 64, (bt, h, nv), generator=g, device=DEV)
    sigma = 0.3 if c["keys"] == "video" else 0.1 + 0.7 * torch.rand((bt, h, 1, 1), generator=g, device=DEV)
    vis = k[:, :, p0:p1]
    vis.mul_(sigma).add_(8.0 * mu)
    step = -(-nv // frames)
    for f in range(frames):
        lo, hi = f * step, min(nv, (f + 1) * step)
        if lo >= hi:
            break
        if f:
            cent = cent + 0.1 * rand(bt, h, 64, d)
        vis[:, :, lo:hi] += cent.gather(2, which[:, :, lo:hi, None].expand(-1, -1, -1, d))
    return k


def _params(c, **kw):
    args = dict(dtype=c.get("dtype", "bf16"), batch=c["batch"], n_q_heads=c.get("hq", c["hkv"]), n_kv_heads=c["hkv"],
                head_dim=c.get("d", 128), seq_len=c["n"], window=c["w"], budget=c["b"], budget_mode=c["mode"],
                budget_floor=c["floor"])
    args.update(kw)
    return B.make_params(**args)


def _outputs(p, c, gather):
    """The program's output buffers: one tensor per kind for all layers, and each layer's views of them."""
    L, bt, h, n, b, d = c["layers"], c["batch"], c["hkv"], c["n"], p.budget, c.get("d", 128)
    t = {}
    if gather or c["op"] == "select":
        t["indices"] = torch.zeros((L, bt, h, b), dtype=torch.int32, device=DEV)
        t["counts"] = torch.zeros((L, bt, h), dtype=torch.int32, device=DEV)
        t["offsets"] = torch.zeros((L, bt, h + 1), dtype=torch.int32, device=DEV)
    if gather:
        t["K_out"] = torch.zeros((L, bt, h, b, d), dtype=_dtype(c), device=DEV)
        t["V_out"] = torch.zeros((L, bt, h, b, d), dtype=_dtype(c), device=DEV)
    if c["op"] != "select":
        if c["scores"]:
            t["scores"] = torch.zeros((L, bt, h, n), dtype=torch.float32, device=DEV)
        if c["mix"] != "imp_only":
            t["redundancy"] = torch.zeros((L, bt, h), dtype=torch.float32, device=DEV)
    return t, [B.LayerOut(**{k: v[l] for k, v in t.items()}) for l in range(L)]


_ROWS = ("K_out", "V_out", "K_tail", "V_tail")


def _as_bits(t):
    """Rows copied bit for bit, to be compared as such."""
    return {k: (v.view(torch.int16 if v.dtype == torch.bfloat16 else torch.int32) if k in _ROWS else v)
            for k, v in t.items()}


def prepare(case, seed):
    c = case
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 13)
    s = {"case": c}
    if c["op"] == "decode":
        return _prepare_decode(c, g, s)
    if c["op"] == "select":
        p = _params(c)
        t, outs = _outputs(p, c, False)
        # attention-like scores: a few heavy keys above a broad background
        sc = torch.empty((c["layers"], c["batch"], c["hkv"], c["n"]), device=DEV)
        sc.normal_(0.0, 1.5, generator=g).exp_().div_(c["n"])
        for l, o in enumerate(outs):
            o.scores = sc[l]
        s.update(p=p, outs=outs, ws=B.alloc_workspace(p, c["layers"], DEV), out=t)
        return s
    if c["op"] == "similarity":
        p = _params(dict(c, w=1, b=1, mode="fixed", floor=0))
        Ks = [_keys(c, g).to(_dtype(c)) for _ in range(c["layers"])]
        nb = -(-c["n"] // c["block"])
        red = torch.zeros((c["layers"], c["batch"], c["hkv"]), device=DEV)
        maps = torch.zeros((c["layers"], c["batch"], c["hkv"], nb, nb), device=DEV)
        ws = torch.empty(B.mixkv_similarity_workspace_size(p, c["layers"], c["block"]), dtype=torch.uint8, device=DEV)
        s.update(call=B.PreparedSimilarity(p, Ks, list(red), list(maps), c["block"], ws), out={"redundancy": red, "map": maps})
        return s
    L, bt, h, n, d, w, dt = c["layers"], c["batch"], c["hkv"], c["n"], c["d"], c["w"], _dtype(c)
    kw = dict(pool=c["pool"], pool_kernel=c["pool_k"], intrinsic=c["intrinsic"], mix=c["mix"])
    if c["mode"] == "per_head":
        # budgets falling linearly over the layers from 2B - W to W, the same for a layer's heads
        top, steps = min(2 * c["b"] - w, n), max(1, L - 1)
        kw["head_budgets"] = [[round(top + (w - top) * l / steps)] * h for l in range(L)]
        kw["budget"] = top
    p = _params(c, **kw)
    Ks, Vs, Qs, lse = [], [], [], []
    room = max(n, c["room"])
    for _ in range(L):
        K = torch.empty((bt, h, room, d), dtype=dt, device=DEV)[:, :, :n]
        K.copy_(_keys(c, g))
        V = torch.empty((bt, h, room, d), dtype=dt, device=DEV)[:, :, :n]
        V.copy_(torch.randn((bt, h, n, d), generator=g, device=DEV, dtype=dt))
        Q = (torch.randn((bt, c["hq"], w, d), generator=g, device=DEV) / d ** 0.5).to(dt)
        Ks.append(K), Vs.append(V), Qs.append(Q)
        if c["lse"]:
            lse.append(_window_lse(c, K, Q))
    t, outs = _outputs(p, c, c["op"] == "compress")
    ws = B.alloc_workspace(p, L, DEV)
    s.update(p=p, Ks=Ks, Vs=Vs, Qs=Qs, lse=lse or None, outs=outs, ws=ws, out=_as_bits(t))
    if c["prepared"]:
        s["call"] = B.PreparedCall(p, Ks, Vs, Qs, outs, ws, window_lse=s["lse"])
    return s


def _window_lse(c, K, Q):
    """What the prefill attention hands over: every window row's log-sum-exp over the keys it attends to."""
    n, w, grp = c["n"], c["w"], c["hq"] // c["hkv"]
    vis = torch.arange(n, device=DEV)[None] <= (n - w + torch.arange(w, device=DEV))[:, None]
    out = torch.empty((c["batch"], c["hq"], w), device=DEV)
    for b in range(c["batch"]):
        for h in range(c["hkv"]):
            x = (Q[b, h * grp:(h + 1) * grp].reshape(-1, c["d"]).float() @ K[b, h].float().t().contiguous()).view(grp, w, n)
            out[b, h * grp:(h + 1) * grp] = torch.logsumexp(x.masked_fill(~vis, float("-inf")), dim=-1)
    return out


def _counts(c, g):
    """Rows every head keeps: B each, or unequal shares of the batch item's hkv * B."""
    bt, h, b = c["batch"], c["hkv"], c["b"]
    if c["mode"] == "fixed":
        return torch.full((bt, h), b, dtype=torch.int32, device=DEV)
    share = torch.rand((bt, h), generator=g, device=DEV) + 0.5
    cnt = (share / share.sum(-1, keepdim=True) * (h * b)).floor().to(torch.int32)
    cnt[:, -1] += h * b - cnt.sum(-1)
    return cnt


def _prepare_decode(c, g, s):
    L, bt, hq, h, d, b, tail, dt = c["layers"], c["batch"], c["hq"], c["hkv"], c["d"], c["b"], c["tail"], _dtype(c)
    p = B.make_params(c["dtype"], bt, hq, h, d, max(2, b), min(32, b - 1), b, budget_mode=c["mode"])
    cap = -(-tail // 64) * 64
    rand = lambda *shape: torch.randn(shape, generator=g, device=DEV).to(dt)  # noqa: E731
    out = torch.zeros((L, bt, hq, d), dtype=dt, device=DEV)
    kt, vt = rand(L, bt, h, cap, d) + 0.3, rand(L, bt, h, cap, d)
    tails, caches, new, Qs = list(zip(kt, vt)), [], [], []
    for _ in range(L):
        cnt = _counts(c, g)
        off = torch.zeros((bt, h + 1), dtype=torch.int32, device=DEV)
        off[:, 1:] = cnt.cumsum(-1)
        caches.append(B.LayerOut(counts=cnt, offsets=off, K_out=rand(bt, h, b, d) + 0.3, V_out=rand(bt, h, b, d)))
        new.append((rand(bt, h, d) + 0.3, rand(bt, h, d)))
        Qs.append((torch.randn((bt, hq, d), generator=g, device=DEV) * (4.0 / d ** 0.5)).to(dt))
    s.update(p=p, new=new, tails=tails, position=tail - 1, out=_as_bits({"out": out, "K_tail": kt, "V_tail": vt}),
             call=B.PreparedDecode(p, caches, tails, Qs, list(out), tail))
    return s


# ------------------------------------------------------------------------------------------------- one pass
def run(state):
    s, c = state, state["case"]
    if c["op"] == "decode":
        B.mixkv_append(s["p"], s["new"], s["tails"], s["position"])
        s["call"].run()
    elif c["op"] == "similarity":
        s["call"].run()
    elif c["op"] == "select":
        B.mixkv_select(s["p"], s["outs"], s["ws"])
    elif c["op"] == "score":
        s["call"].score()
    elif c["prepared"]:
        s["call"].compress()
    else:
        B.mixkv_compress(s["p"], s["Ks"], s["Vs"], s["Qs"], s["outs"], s["ws"], window_lse=s["lse"])
    return s["out"]


# ------------------------------------------------------------------------------------------------- what it cannot do without
def work(case):
    c = case
    e = 4 if c.get("dtype") == "f32" else 2
    if c["op"] == "decode":
        heads = c["layers"] * c["batch"] * c["hkv"]
        rows = heads * (c["b"] + c["tail"])                                  # read, K and V each
        q = c["layers"] * c["batch"] * c["hq"] * c["d"]
        return {"bytes": 2 * rows * c["d"] * e + 2 * q * e + 4 * heads * c["d"] * e,
                "flops": 4 * (c["hq"] // c["hkv"]) * rows * c["d"]}
    units, n = c["layers"] * c["batch"] * c["hkv"], c["n"]
    if c["op"] == "select":
        return {"bytes": units * (4 * (n - c["w"]) + 4 * c["b"]), "flops": 0}
    if c["op"] == "similarity":
        nb = -(-n // c["block"])
        return {"bytes": units * (n * c["d"] * e + 4 * nb * nb), "flops": units * (4 * n * c["d"] + 2 * nb * nb * c["d"])}
    gw = c["hq"] // c["hkv"] * c["w"]
    reads = 2 if c["intrinsic"] == "vnorm" else 1
    by = units * (reads * n * c["d"] * e + gw * c["d"] * e)
    if c["scores"]:
        by += 4 * units * n
    if c["op"] == "compress":
        by += units * (4 * c["b"] * c["d"] * e + 4 * c["b"])                 # kept rows read and written, indices
    return {"bytes": by, "flops": 2 * units * gw * n * c["d"]}


def tolerance(case):
    """About four times what was measured: the scoring path against itself with its work dealt differently over the
    chip (another order of the fp32 sums), decode and similarity against float64 (rounded to the output's type)."""
    c = case
    if c["op"] == "select":
        return "exact"                                       # a total order on the caller's scores
    if c["op"] == "decode":
        # bf16: 1.4e-4 and one unit in the last place (6.8e-3) on a few outputs; fp32: 3.9e-7, 2.9e-6
        return {"rel": 6e-4, "max": 8e-3} if c["dtype"] == "bf16" else {"rel": 1.6e-6, "max": 1.2e-5}
    if c["op"] == "similarity":
        return {"rel": 1e-6, "max": 4e-6}                    # 1.7e-7, 9e-7
    # scores: 2.3e-7 and 2.5e-6 between orders, up to 3e-6 of the mean against float64.  Two candidates within that
    # of each other may change places at the edge of a budget, which moves the rows between them: one head of 112.
    # Keys without a common direction leave a redundancy near 0, the difference of two equal sums of squares: 1.4e-6.
    if c["keys"] == "iid":
        return {"rel": 1e-5, "max": 4e-5, "differ": 0.01}
    return {"rel": 2e-6, "max": 1.2e-5, "differ": 0.01}
