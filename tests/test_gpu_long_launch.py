"""Launches long enough for the kernels that serve whole caches (keys in registers for the second pass, queries in the
registers of two waves for the first) against the same layers called one at a time, which take the kernels of short
launches; those are compared with the oracle in test_gpu_parity.py."""
import pytest
import torch

from paper_2510_20707_amd import binding as B

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
