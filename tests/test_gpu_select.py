"""mixkv_select on given scores is exact integer work: bit-exact against the oracle's selection
when both read the same float32 scores (ties included)."""
import numpy as np
import pytest
import torch

from oracle import mixkv_oracle as O
from paper_2510_20707_amd import binding as B

pytestmark = pytest.mark.gpu


def _scores(kind, rng, Bt, Hkv, N, W):
    Nc = N - W
    if kind == "normal":
        s = rng.standard_normal((Bt, Hkv, N))
    elif kind == "ties":                       # heavy exact ties, including +0 / -0
        s = rng.integers(-3, 4, size=(Bt, Hkv, N)).astype(np.float64) * 0.25
        s[s == 0] = np.where(rng.random((s == 0).sum()) < 0.5, 0.0, -0.0)
    elif kind == "tiny-positive":              # attention-like: all in one narrow exponent range
        s = 1e-4 * (1.0 + 1e-3 * rng.random((Bt, Hkv, N)))
    elif kind == "constant":
        s = np.full((Bt, Hkv, N), 0.5)
    else:
        raise ValueError(kind)
    s = s.astype(np.float32)
    s[:, :, Nc:] = np.inf
    return s


@pytest.mark.parametrize("kind", ["normal", "ties", "tiny-positive", "constant"])
@pytest.mark.parametrize("N,W,Bud,Hkv", [(512, 8, 64, 2), (4099, 32, 300, 4), (70, 3, 70, 1), (33000, 32, 128, 2)])
def test_fixed_budget_selection_is_bit_exact(kind, N, W, Bud, Hkv):
    print(f"[case] select fixed kind={kind} N={N} W={W} B={Bud} Hkv={Hkv}", flush=True)
    rng = np.random.default_rng([1, N, Bud])
    Bt = 2
    s = _scores(kind, rng, Bt, Hkv, N, W)
    p = B.make_params("bf16", Bt, Hkv, Hkv, 128, N, W, Bud)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    out.indices.fill_(-1)
    B.mixkv_select(p, [out])
    torch.cuda.synchronize()
    idx = out.indices.cpu().numpy()
    for b in range(Bt):
        for h in range(Hkv):
            want = O.select_unit(s[b, h, :N - W].astype(np.float64), Bud - W, N, W)
            np.testing.assert_array_equal(idx[b, h], want)
    assert np.all(out.counts.cpu().numpy() == Bud)
    np.testing.assert_array_equal(out.offsets.cpu().numpy(), np.tile(np.arange(Hkv + 1) * Bud, (Bt, 1)))


def _candidate_list_bytes(n_layers, Bt, Hkv):
    """What the head-adaptive selection asks of a workspace: two 1024-entry lists of 4-byte words per head."""
    return n_layers * Bt * Hkv * 1024 * 4 * 2


# with a workspace every head's best candidates are listed by a workgroup of its own and a small
# kernel splits the pool; without one (or with lists too long for it: the 400-row budget) one
# workgroup per batch item ranks the scores of all heads
@pytest.mark.parametrize("lists", [True, False])
@pytest.mark.parametrize("kind", ["normal", "ties", "constant"])
@pytest.mark.parametrize("N,W,Bud,Hkv,floor", [(512, 8, 64, 4, 14), (3000, 32, 128, 3, 0), (600, 4, 50, 5, 46),
                                               (33000, 32, 128, 4, 24), (3000, 32, 400, 4, 10)])
def test_adaptive_budget_selection_is_bit_exact(kind, N, W, Bud, Hkv, floor, lists):
    print(f"[case] select adaptive kind={kind} N={N} W={W} B={Bud} Hkv={Hkv} floor={floor} lists={lists}", flush=True)
    rng = np.random.default_rng([2, N, Bud])
    Bt = 2
    s = _scores(kind, rng, Bt, Hkv, N, W)
    if kind == "normal":
        s[:, :, :N - W] *= np.linspace(0.5, 2.0, Hkv, dtype=np.float32)[None, :, None]   # heads of unequal weight
    p = B.make_params("bf16", Bt, Hkv, Hkv, 128, N, W, Bud, budget_mode="adaptive", budget_floor=floor)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    out.indices.fill_(-1)
    ws = torch.empty(_candidate_list_bytes(1, Bt, Hkv), dtype=torch.uint8, device="cuda:0") if lists else None
    B.mixkv_select(p, [out], ws)
    torch.cuda.synchronize()
    idx = out.indices.cpu().numpy().reshape(Bt, Hkv * Bud)
    cnt, off = out.counts.cpu().numpy(), out.offsets.cpu().numpy()
    for b in range(Bt):
        bp = O.adaptive_budgets(s[b, :, :N - W].astype(np.float64), Bud, W, floor)
        np.testing.assert_array_equal(cnt[b], bp + W)
        np.testing.assert_array_equal(off[b], np.concatenate([[0], np.cumsum(bp + W)]))
        for h in range(Hkv):
            want = O.select_unit(s[b, h, :N - W].astype(np.float64), int(bp[h]), N, W)
            np.testing.assert_array_equal(idx[b, off[b, h]:off[b, h + 1]], want)
        assert off[b, Hkv] == Hkv * Bud                        # the pool is used up


def test_adaptive_selection_over_several_layers_with_candidate_lists():
    """Layers beyond one launch group, each with its own scores, through the candidate lists."""
    N, W, Bud, Hkv, floor, Bt, L = 2100, 16, 96, 4, 20, 2, 34
    print(f"[case] select adaptive layers={L} N={N} W={W} B={Bud} Hkv={Hkv} floor={floor}", flush=True)
    rng = np.random.default_rng([5, N, Bud])
    p = B.make_params("bf16", Bt, Hkv, Hkv, 128, N, W, Bud, budget_mode="adaptive", budget_floor=floor)
    ss, outs = [], []
    for l in range(L):
        s = _scores("normal" if l % 2 else "ties", rng, Bt, Hkv, N, W)
        out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
        out.scores = torch.from_numpy(s).to("cuda:0")
        ss.append(s)
        outs.append(out)
    ws = torch.empty(_candidate_list_bytes(L, Bt, Hkv), dtype=torch.uint8, device="cuda:0")
    B.mixkv_select(p, outs, ws)
    torch.cuda.synchronize()
    for l in range(L):
        idx = outs[l].indices.cpu().numpy().reshape(Bt, Hkv * Bud)
        cnt, off = outs[l].counts.cpu().numpy(), outs[l].offsets.cpu().numpy()
        for b in range(Bt):
            bp = O.adaptive_budgets(ss[l][b, :, :N - W].astype(np.float64), Bud, W, floor)
            np.testing.assert_array_equal(cnt[b], bp + W)
            for h in range(Hkv):
                want = O.select_unit(ss[l][b, h, :N - W].astype(np.float64), int(bp[h]), N, W)
                np.testing.assert_array_equal(idx[b, off[b, h]:off[b, h + 1]], want)


@pytest.mark.parametrize("kind", ["normal", "ties"])
@pytest.mark.parametrize("N,W,Bud,Hkv,L", [(512, 8, 64, 4, 3), (4099, 32, 300, 2, 34), (33000, 32, 128, 2, 1)])
def test_per_head_budget_selection_is_bit_exact(kind, N, W, Bud, Hkv, L):
    print(f"[case] select per-head kind={kind} N={N} W={W} B={Bud} Hkv={Hkv} L={L}", flush=True)
    rng = np.random.default_rng([3, N, Bud])
    Bt = 2
    # budgets between W and 2B - W per head, then trimmed so that every layer fits its Hkv * B rows
    hb = rng.integers(W, 2 * Bud - W + 1, size=(L, Hkv)).astype(np.int32)
    hb[0, 0] = W                                               # a head that keeps the window only
    for l in range(L):
        while hb[l].sum() > Hkv * Bud:
            hb[l, np.argmax(hb[l])] -= 1
    p = B.make_params("bf16", Bt, Hkv, Hkv, 128, N, W, Bud, budget_mode="per_head", head_budgets=hb)
    ss, outs = [], []
    for l in range(L):
        s = _scores(kind, rng, Bt, Hkv, N, W)
        out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
        out.scores = torch.from_numpy(s).to("cuda:0")
        out.indices.fill_(-1)
        ss.append(s)
        outs.append(out)
    ws = torch.empty((L * Hkv * 4 + 255) // 256 * 256, dtype=torch.uint8, device="cuda:0")   # the table only
    B.mixkv_select(p, outs, ws)
    torch.cuda.synchronize()
    for l in range(L):
        idx = outs[l].indices.cpu().numpy().reshape(Bt, Hkv * Bud)
        off = np.concatenate([[0], np.cumsum(hb[l])])
        np.testing.assert_array_equal(outs[l].counts.cpu().numpy(), np.tile(hb[l], (Bt, 1)))
        np.testing.assert_array_equal(outs[l].offsets.cpu().numpy(), np.tile(off, (Bt, 1)))
        for b in range(Bt):
            for h in range(Hkv):
                want = O.select_unit(ss[l][b, h, :N - W].astype(np.float64), int(hb[l, h]) - W, N, W)
                np.testing.assert_array_equal(idx[b, off[h]:off[h + 1]], want)
            assert np.all(idx[b, off[Hkv]:] == -1)             # unused capacity is left alone


def test_per_head_budget_tables_are_validated_on_the_host():
    N, W, Bud, Hkv = 512, 8, 64, 2
    good = np.array([[8, 120]], dtype=np.int32)
    s = _scores("normal", np.random.default_rng(4), 1, Hkv, N, W)
    ws = torch.empty(256, dtype=torch.uint8, device="cuda:0")

    def call(hb, workspace=ws):
        p = B.make_params("bf16", 1, Hkv, Hkv, 128, N, W, Bud, budget_mode="per_head", head_budgets=hb)
        out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
        out.scores = torch.from_numpy(s).to("cuda:0")
        out.indices.fill_(-7)
        try:
            B.mixkv_select(p, [out], workspace)
            status = B.MIXKV_OK
        except B.MixkvError as e:
            status = e.status
        torch.cuda.synchronize()
        return status, out

    assert call(good)[0] == B.MIXKV_OK
    for bad in ([[7, 64]], [[8, 513]], [[64, 65]]):            # below W, above N, more than Hkv * B in all
        status, out = call(np.array(bad, dtype=np.int32))
        assert status == B.MIXKV_ERR_INVALID_ARG
        assert torch.all(out.indices == -7)                    # nothing was launched
    assert call(None)[0] == B.MIXKV_ERR_INVALID_ARG            # no table
    assert call(good, None)[0] == B.MIXKV_ERR_INVALID_ARG      # no workspace to stage it in


# Rows beyond one workgroup's registers are cut into segments whose lists are merged, and head-adaptive lists may be
# longer than the selection-only workspace holds, if the caller brings a workspace of the full size.  Cases: one
# candidate past a segment, a last segment shorter than the lists, more kept than a segment holds, 8192- and
# 16384-candidate segments, budgets whose split streams its lists from memory, a list that is the whole row, and
# a budget too long for the merge.
@pytest.mark.parametrize("kind", ["normal", "ties"])
@pytest.mark.parametrize("mode,N,W,Bud,Hkv,floor", [
    ("fixed", 32768 + 32 + 1, 32, 128, 2, 0), ("fixed", 9 * 4096 + 5 + 8, 8, 300, 1, 0), ("fixed", 40000, 16, 5000, 1, 0),
    ("fixed", 140001, 32, 96, 2, 0), ("fixed", 300007, 32, 64, 1, 0), ("fixed", 70000, 32, 40000, 1, 0), ("fixed", 33000, 32, 32, 2, 0),
    ("per_head", 50001, 32, 700, 3, 0), ("adaptive", 33000, 32, 128, 4, 24), ("adaptive", 66001, 8, 900, 4, 100),
    ("adaptive", 3000, 32, 600, 4, 100), ("adaptive", 9001, 32, 1200, 8, 3), ("adaptive", 700, 4, 600, 5, 20),
    ("adaptive", 20000, 32, 3000, 3, 2968)])
def test_selection_on_a_full_workspace_is_bit_exact(kind, mode, N, W, Bud, Hkv, floor):
    print(f"[case] select full workspace kind={kind} {mode} N={N} W={W} B={Bud} Hkv={Hkv} floor={floor}", flush=True)
    rng = np.random.default_rng([7, N, Bud])
    Bt = 2
    s = _scores(kind, rng, Bt, Hkv, N, W)
    if kind == "normal" and mode == "adaptive":
        s[:, :, :N - W] *= np.linspace(0.5, 2.0, Hkv, dtype=np.float32)[None, :, None]
    hb = np.array([[2 * Bud - W - (j % 2) * (2 * Bud - 2 * W) if j < Hkv - 1 else W for j in range(Hkv)]], dtype=np.int32)
    p = B.make_params("bf16", Bt, Hkv, Hkv, 128, N, W, Bud, budget_mode=mode, budget_floor=floor,
                      head_budgets=hb if mode == "per_head" else None)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    out.indices.fill_(-1)
    B.mixkv_select(p, [out], B.alloc_workspace(p, 1, "cuda:0"))
    torch.cuda.synchronize()
    idx = out.indices.cpu().numpy().reshape(Bt, Hkv * Bud)
    cnt, off = out.counts.cpu().numpy(), out.offsets.cpu().numpy()
    for b in range(Bt):
        if mode == "adaptive":
            bp = O.adaptive_budgets(s[b, :, :N - W].astype(np.float64), Bud, W, floor)
        else:
            bp = (hb[0] if mode == "per_head" else np.full(Hkv, Bud)) - W
        np.testing.assert_array_equal(cnt[b], bp + W)
        np.testing.assert_array_equal(off[b], np.concatenate([[0], np.cumsum(bp + W)]))
        for h in range(Hkv):
            want = O.select_unit(s[b, h, :N - W].astype(np.float64), int(bp[h]), N, W)
            np.testing.assert_array_equal(idx[b, off[b, h]:off[b, h + 1]], want)


# Lists that one workgroup cannot merge go through rounds of partial merges: one to four rounds, groups and segments that do
# not divide evenly, a last segment of one candidate, heads that keep nothing beside the window, the longest list a round
# takes and the most entries that one merge takes.
@pytest.mark.parametrize("kind", ["normal", "ties", "constant"])
@pytest.mark.parametrize("mode,N,W,Bud,Hkv,floor", [
    ("adaptive", 130688, 32, 1200, 4, 16), ("adaptive", 131072, 8, 2048, 8, 0), ("adaptive", 130688, 32, 960, 4, 0),
    ("fixed", 3 * 16384 + 1 + 32, 32, 16384 + 32, 1, 0), ("fixed", 300007, 32, 9000, 1, 0), ("fixed", 524288 + 32, 32, 16416, 1, 0),
    ("per_head", 90001, 32, 6000, 3, 0)])
def test_long_lists_merged_in_rounds_are_bit_exact(kind, mode, N, W, Bud, Hkv, floor):
    test_selection_on_a_full_workspace_is_bit_exact(kind, mode, N, W, Bud, Hkv, floor)


# Head-adaptive pools of more than 32 and up to 64 entries per thread of the split's one workgroup: lists that end inside a thread's run, the most
# entries that its 16-bit counts admit, one past them, and floors that take everything.
@pytest.mark.parametrize("kind", ["normal", "ties", "constant"])
@pytest.mark.parametrize("N,W,Bud,Hkv,floor", [(9001, 32, 650, 8, 3), (20000, 8, 2631, 5, 2), (20000, 8, 2632, 5, 3), (20000, 32, 12032, 4, 12000),
                                               (4100, 4, 600, 9, 17)])
def test_split_of_long_pools_is_bit_exact(kind, N, W, Bud, Hkv, floor):
    test_selection_on_a_full_workspace_is_bit_exact(kind, "adaptive", N, W, Bud, Hkv, floor)
