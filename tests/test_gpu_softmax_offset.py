"""The running softmax of the first pass where its offset moves a long way in the middle of a run: a key whose logit is
87.5, in rows whose first logits are up to 1 (its term, 2^125, fits a float), and a few tiles later one at 90 (2^128.4, which does
not).  The first must keep its weight exp(-2.5) beside the second's."""
import pytest
import torch

from paper_2510_20707_amd import binding as B
from tests import routes

CASES = [  # dtype, head dim, query tiles, layers, first pass
    ("bf16", 128, 1, 4, "ks_stats"), ("bf16", 64, 2, 4, "ks_stats"), ("f32", 128, 2, 2, "ks_stats"),
    ("bf16", 128, 7, 4, "stats"), ("bf16", 128, 12, 4, "stats"), ("bf16", 64, 3, 4, "stats"), ("f32", 128, 4, 2, "stats"),
    ("bf16", 128, 5, 8, "qs_stats"), ("bf16", 128, 8, 8, "qs_stats"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,tiles,L,route", CASES)
def test_a_far_move_of_the_offset_keeps_what_was_summed(dtype, d, tiles, L, route):
    bt, hkv, n, w = 4, 8, 4090, 32
    nc = n - w
    p = B.make_params(dtype, bt, hkv * tiles, hkv, d, n, w, 64, mix="imp_only", intrinsic="none", pool="none", pool_kernel=1)
    assert routes.passes(p, L)[0] == route
    dt, dev = B.TORCH_DTYPE[p.dtype], "cuda:0"
    g = torch.Generator(device=dev).manual_seed(tiles * 1000 + d)
    Ks, Qs = [], []
    for l in range(L):
        K = torch.rand((bt, hkv, n, d), generator=g, device=dev).mul_(2).sub_(1)
        for u in range(bt * hkv):
            # both keys past the first tile of one wave and half-wave, in one run, whichever way the tiles are dealt
            first = 32 * (32 * (u % 3) + 4 + u % 4) + 8 * (u % 4) + 4 * (u & 1)
            K[u // hkv, u % hkv, first, 0] = 87.5
            K[u // hkv, u % hkv, first + 32 * 4 * (1 + u % 2) + 1, 0] = 90.0
        Ks.append(K.to(dt))
        Q = torch.zeros((bt, hkv * tiles, w, d), dtype=dt, device=dev)
        Q[..., 0] = 1.0
        Qs.append(Q)
    out = [B.LayerOut(scores=torch.zeros((bt, hkv, n), device=dev)) for _ in range(L)]
    print(f"[case] {dtype} D={d} tiles={tiles} L={L}", flush=True)
    B.mixkv_score(p, Ks, Ks, Qs, out, B.alloc_workspace(p, L, dev))
    for l in range(L):
        term = (Ks[l][..., 0].double() - 90.0).exp()
        z = term[..., :nc].sum(-1, keepdim=True) + term[..., nc:].cumsum(-1)          # [bt, hkv, w]: what row i of the window sums
        want = term[..., :nc] * (1.0 / z).mean(-1, keepdim=True)
        got = out[l].scores[..., :nc].double()
        err = ((got - want).abs() / torch.maximum(want, want.mean(-1, keepdim=True))).max().item()
        # logits of up to 130 in the log2 domain, rounded three times by up to half a unit: 3 * 2^-17 * ln 2 = 1.6e-5
        assert err <= 3e-5, (l, err)
