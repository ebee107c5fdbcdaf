"""Launches long enough for the kernels that serve whole caches (keys in registers for the second pass, queries in the
registers of two waves for the first) against the same layers called one at a time, which take the kernels of short
launches; those are compared with the oracle in test_gpu_parity.py.  Then launches whose workgroups take several runs, with the oracle."""
import pytest
import torch

from oracle import mixkv_oracle as O
from paper_2510_20707_amd import binding as B
from tests import harness as H
from tests import routes

# Query tiles 2 to 8 (and 16 with 64-element rows), full and ragged; 4090 keys end in a tile of 26 rows; 8 layers of 32 heads are 8192
# chunks and 8 even rounds of blocks per wave on 256 compute units.
CASES = [  # q heads, window, head dim, causal, layout, intrinsic
    (40, 32, 128, True, "bhnd", "vnorm"),     # 5 tiles: 3 + 2
    (48, 31, 128, True, "bnhd", "vnorm"),     # 186 rows: 6 tiles
    (56, 31, 128, True, "bhnd", "vnorm"),     # 217 rows: 7 tiles, the last with 7 spare rows
    (64, 32, 128, False, "bnhd", "vnorm"),    # 8 tiles
    (56, 32, 128, True, "bhnd", "none"),      # no value rows
    (32, 32, 128, True, "bhnd", "knorm"),     # 4 tiles: second pass only
    (16, 24, 128, True, "bnhd", "vnorm"),     # 48 rows: 2 tiles
    (56, 16, 64, True, "bhnd", "vnorm"),      # 4 tiles of 64-element rows
    (128, 32, 64, False, "bhnd", "vnorm"),    # 16 tiles
]


@pytest.mark.gpu
@pytest.mark.parametrize("hq,w,d,causal,layout,intrinsic", CASES)
def test_long_launch_agrees_with_single_layers(hq, w, d, causal, layout, intrinsic):
    L, bt, hkv, n = 8, 4, 8, 4090
    g = torch.Generator(device="cuda:0").manual_seed(hq * 100 + w)
    p = B.make_params("bf16", bt, hq, hkv, d, n, w, 64, causal_window=causal, intrinsic=intrinsic, pool="none", pool_kernel=1)
    rand = lambda *shape: torch.randn(shape, generator=g, device="cuda:0")  # noqa: E731
    Ks, Vs, Qs = [], [], []
    for _ in range(L):
        mu = rand(bt, hkv, 1, d)
        kv = []
        for x in (rand(bt, hkv, n, d) + 0.5 * mu, rand(bt, hkv, n, d)):
            x = x.to(torch.bfloat16)
            kv.append(x if layout == "bhnd" else x.transpose(1, 2).contiguous().transpose(1, 2))
        Ks.append(kv[0]), Vs.append(kv[1])
        Qs.append((rand(bt, hq, w, d) * (3.0 / d ** 0.5)).to(torch.bfloat16))

    def outs(k):
        return [B.LayerOut(scores=torch.zeros((bt, hkv, n), device="cuda:0"), redundancy=torch.zeros((bt, hkv), device="cuda:0")) for _ in range(k)]

    whole = outs(L)
    B.mixkv_score(p, Ks, Vs, Qs, whole, B.alloc_workspace(p, L, "cuda:0"))
    ws1 = B.alloc_workspace(p, 1, "cuda:0")
    nc = n - w
    for l in range(L):
        one = outs(1)
        B.mixkv_score(p, Ks[l:l + 1], Vs[l:l + 1], Qs[l:l + 1], one, ws1)
        a, b = whole[l].scores[..., :nc].double(), one[0].scores[..., :nc].double()
        assert torch.isfinite(a).all()
        # fp32 sums of up to 2^12 terms in another order: 2^6 * 2^-24 = 4e-6 of a score's own terms, a few such sums per score
        ref = torch.maximum(b.abs(), b.abs().mean(-1, keepdim=True))
        assert ((a - b).abs() / ref).max() <= 2e-5
        assert (whole[l].redundancy - one[0].redundancy).abs().max() <= 1e-6
        assert torch.isposinf(whole[l].scores[..., nc:]).all()


# Launches whose workgroups walk several runs: heads and their blocks do not divide evenly, so runs start and end inside heads, some have fewer
# blocks than waves, and the image, the ring and the queries in LDS are taken over from the run before.  The kernels that the launch goes to
# are asserted, both kinds of loads among them (below and above 180 MB).
ROOMY = dict(g=5, w=32, d=128, bt=53, L=8, n=2500)
RUNS = {  # query heads per KV head (one KV head), window, head dim, batch, layers, keys; first pass, second pass; options
    "5 tiles, 8.3 chunks and 66 blocks a workgroup": (ROOMY, "qs_stats", "kst_attn", {}),
    "6 tiles, the offset moves mid-run": (dict(ROOMY, g=6, w=31), "qs_stats", "kst_attn", dict(softmax_scale=20.0)),
    "7 tiles, zero and tiny keys, zero values": (dict(ROOMY, g=7, bt=37, n=4090), "qs_stats", "kst_attn", dict(odd_rows=True)),
    "8 tiles, no causal mask": (dict(ROOMY, g=8, bt=89, n=1500), "qs_stats", "kst_attn", dict(causal_window=False)),
    "7 tiles, heads of 289 keys": (dict(ROOMY, g=7, bt=344, n=289), "qs_stats", "attn", dict(odd_rows=True)),
    "8 tiles, heads of 200 keys, key norms": (dict(ROOMY, g=8, bt=520, n=200), "qs_stats", "attn", dict(intrinsic="knorm")),
    "8 tiles, heads of 130 keys alone, cacheable loads": (dict(ROOMY, g=8, bt=520, n=130), "qs_stats", "attn", dict(intrinsic="none")),
    "5 tiles, a second launch group of two layers": (dict(ROOMY, bt=13, L=34, n=2600), "qs_stats", "kst_attn", {}),
    "5 tiles, given normalisers": (ROOMY, "stats", "kst_attn", dict(lse=True)),
    "4 tiles, keys alone, cacheable loads": (dict(ROOMY, g=4, bt=31), "stats", "kst_attn", dict(intrinsic="none", mix="imp_only", redundancy=False)),
    "5 tiles of 64-element rows, cacheable loads": (dict(ROOMY, d=64, bt=31), "stats", "kst_attn", dict(odd_rows=True)),
    "12 tiles of 64-element rows, heads of 11 blocks": (dict(ROOMY, g=12, d=64, bt=110, n=700), "stats", "kst_attn", dict(softmax_scale=20.0)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", RUNS)
def test_runs_that_straddle_heads_against_the_oracle(name):
    c, first, second, opt = RUNS[name]
    g, w, d, bt, L, n = (c[k] for k in ("g", "w", "d", "bt", "L", "n"))
    opt = dict(opt)
    odd_rows, with_lse, want_r = opt.pop("odd_rows", False), opt.pop("lse", False), opt.pop("redundancy", True)
    p = B.make_params("bf16", bt, g, 1, d, n, w, w + 1, pool="none", pool_kernel=1, **opt)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert routes.passes(p, min(L, 32), cus, given_lse=with_lse) == (first, second)
    print(f"[case] {name}", flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(g * 10000 + n)
    rand = lambda *shape: torch.randn(shape, generator=gen, device="cuda:0")  # noqa: E731
    Ks, Vs, Qs, lse = [], [], [], []
    for l in range(L):
        K, V = rand(bt, 1, n, d) + 0.5 * rand(bt, 1, 1, d), rand(bt, 1, n, d)
        if odd_rows:
            K[:, :, 3::11] = 0.0
            K[:, :, 5::13] *= 1e-12
            V[:, :, 7::17] = 0.0
        Ks.append(K.to(torch.bfloat16)), Vs.append(V.to(torch.bfloat16))
        Qs.append((rand(bt, g, w, d) * (3.0 / d ** 0.5)).to(torch.bfloat16))
        if with_lse:
            x = Qs[l].float().view(bt, g * w, d) @ Ks[l][:, 0].float().transpose(1, 2).contiguous()
            vis = torch.arange(n, device="cuda:0")[None] <= (n - w + torch.arange(w, device="cuda:0"))[:, None]
            lse.append(torch.logsumexp(x.view(bt, g, w, n).masked_fill(~vis, float("-inf")), dim=-1).contiguous())
    ws = B.alloc_workspace(p, L, "cuda:0")
    got = []
    for fill in (0x00, 0xff):                          # the same bits again, whatever the workspace held
        outs = [B.LayerOut(scores=torch.zeros((bt, 1, n), device="cuda:0"), redundancy=torch.zeros((bt, 1), device="cuda:0") if want_r else None)
                for _ in range(L)]
        ws.fill_(fill)
        B.mixkv_score(p, Ks, Vs, Qs, outs, ws, window_lse=lse or None)
        got.append(outs)
    for a, b in zip(*got):
        assert torch.equal(a.scores, b.scores) and (not want_r or torch.equal(a.redundancy, b.redundancy))
        assert torch.isfinite(a.scores[..., :n - w]).all() and torch.isposinf(a.scores[..., n - w:]).all()
    # as above; with a scale of 20 the logits reach 2^9 in the log2 domain and are rounded three times: 3 * 2^-16 * ln 2 = 3.2e-5 more
    bound = 2e-5 + (3.2e-5 if opt.get("softmax_scale", 1.0) > 1 else 0)
    op = O.Params(g, 1, w, w + 1, pool="none", pool_kernel=1, **opt)
    for l, b in ((0, 0), (0, 1), (L // 2, bt // 2), (L - 1, bt - 1)):
        host = lambda t: t.double().cpu().numpy()  # noqa: E731
        u = O.score_unit(host(Ks[l][b, 0]), host(Vs[l][b, 0]), host(Qs[l][b]), op, None, host(lse[l][b]) if with_lse else None)
        err = H.check_scores("bf16", got[0][l].scores[b, 0, :n - w].cpu().numpy(), u["s_comp"], f"layer {l} item {b}")
        assert err <= bound, (l, b, err)
        if want_r:
            assert abs(float(got[0][l].redundancy[b, 0]) - float(u["r"])) <= H.RTOL_R["bf16"]
