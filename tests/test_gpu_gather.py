"""The kept rows of a fused selection, copied by the selecting workgroup or by a kernel behind it (many rows, few heads):
bit for bit the source rows, on either side of that rule, with row counts around the pieces a workgroup has in flight,
the window alone, everything kept, unequal budgets per head and more heads than a wave has lanes."""
import numpy as np
import pytest
import torch

from paper_2510_20707_amd import binding as B
from paper_2510_20707_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu
WL = synth.WORKLOADS


# dtype, D, N, W, Hkv, B
INSIDE = [("bf16", 128, 700, 8, 2, 8), ("bf16", 128, 700, 8, 2, 64), ("bf16", 64, 700, 8, 2, 129), ("f32", 128, 700, 8, 2, 33)]
APART = [("bf16", 128, 900, 8, 2, 900), ("f32", 64, 3000, 16, 1, 2900), ("bf16", 64, 9000, 8, 1, 1031), ("f32", 128, 2500, 8, 3, 511)]
# Hkv, B, rows of the best-endowed head
TABLE_INSIDE = [(3, 40, 90), (66, 30, 400), (66, 30, 60)]
TABLE_APART = [(3, 900, 1900), (66, 60, 1500)]


@pytest.mark.parametrize("dtype,D,N,W,Hkv,B", INSIDE + APART)
def test_gathered_rows_of_equal_budgets(dtype, D, N, W, Hkv, B):
    print(f"[case] gather {dtype} D={D} N={N} W={W} Hkv={Hkv} B={B}", flush=True)
    wl = WL["c2"].with_(name="gather", dtype=dtype, head_dim=D, seq_len=N, window=W, n_q_heads=Hkv, n_kv_heads=Hkv, budget=B,
                        text_suffix_start=N - 50)
    lay = synth.make_layer(wl, 0)
    p, outs = H.run_compress(wl, [lay])
    H.check_layer(wl, lay, p, outs[0])


@pytest.mark.parametrize("Hkv,B,top", TABLE_INSIDE + TABLE_APART)
def test_gathered_rows_of_unequal_budgets(Hkv, B, top):
    N, W = 2000, 8
    print(f"[case] gather per head Hkv={Hkv} B={B} top={top}", flush=True)
    wl = WL["c2"].with_(name="gather-table", head_dim=64, seq_len=N, window=W, n_q_heads=Hkv, n_kv_heads=Hkv, budget=B,
                        text_suffix_start=N - 50)
    hb = np.full((1, Hkv), W, dtype=np.int32)
    hb[0, 1], hb[0, -1] = top, W + 3
    lay = synth.make_layer(wl, 0)
    p, outs = H.run_compress(wl, [lay], head_budgets=hb, budget_mode="per_head")
    H.check_layer(wl, lay, p, outs[0], head_budgets=hb[0], budget_mode="per_head", units=[(0, 0), (0, 1)])


# The budget table travels with the fold's arguments up to 256 entries per launch, else in a launch of its own: on either side of that,
# over more layers than one launch takes, the rows are those that the selection alone keeps of the same scores.
@pytest.mark.parametrize("L,Hkv", [(1, 3), (32, 8), (33, 8), (35, 7), (29, 9), (4, 65)])
def test_budget_tables_on_either_side_of_the_fold(L, Hkv):
    N, W, D, Bud = 200, 8, 64, 40
    print(f"[case] budget table L={L} Hkv={Hkv}", flush=True)
    rng = np.random.default_rng([11, L, Hkv])
    hb = rng.integers(W, 2 * Bud - W, size=(L, Hkv)).astype(np.int32)
    hb[hb.sum(1) > Hkv * Bud] = Bud
    p = B.make_params("f32", 1, Hkv, Hkv, D, N, W, Bud, budget_mode="per_head", head_budgets=hb)
    g = torch.Generator(device="cuda:0").manual_seed(5)
    K, V = (torch.randn((1, Hkv, N, D), generator=g, device="cuda:0") for _ in range(2))
    Q = torch.randn((1, Hkv, W, D), generator=g, device="cuda:0") / D ** 0.5
    outs, alone = ([B.alloc_layer_out(p, "cuda:0", scores=True) for _ in range(L)] for _ in range(2))
    ws = B.alloc_workspace(p, L, "cuda:0")
    ws.fill_(0xff)                                       # no table is there yet
    B.mixkv_compress(p, [K] * L, [V] * L, [Q] * L, outs, ws)
    for a, o in zip(alone, outs):
        a.scores.copy_(o.scores)
    B.mixkv_select(p, alone, B.alloc_workspace(p, L, "cuda:0"))
    torch.cuda.synchronize()
    for l in range(L):
        assert outs[l].counts.cpu().numpy().ravel().tolist() == hb[l].tolist()
        kept = int(hb[l].sum())
        assert torch.equal(outs[l].indices.view(-1)[:kept], alone[l].indices.view(-1)[:kept])
        assert torch.equal(outs[l].offsets, alone[l].offsets)
