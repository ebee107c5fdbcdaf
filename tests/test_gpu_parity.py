"""GPU parity: the HIP path through the C ABI against the float64 oracle on identical seeded inputs."""
import numpy as np
import pytest
import torch

from oracle import mixkv_oracle as O
from paper_2510_20707_amd import binding as B
from paper_2510_20707_amd import synth
from tests import harness as H

pytestmark = pytest.mark.gpu
WL = synth.WORKLOADS


def _say(*a):
    print(*a, flush=True)


def _run_and_check(wl, n_layers=None, units=None, layer_ids=None, **over):
    layer_ids = list(range(n_layers or wl.n_layers)) if layer_ids is None else layer_ids
    layers = [synth.make_layer(wl, l) for l in layer_ids]
    _say(f"[case] {wl.name} dtype={wl.dtype} L={len(layers)} Bt={wl.batch} Hq={wl.n_q_heads} Hkv={wl.n_kv_heads} "
         f"D={wl.head_dim} N={wl.seq_len} W={wl.window} B={over.get('budget', wl.budget)} over={over}")
    rg = [H.given_weights(wl, l) for l in layer_ids] if over.get("mix") == "given_r" else None
    hb = over.pop("head_budgets", None)
    lse = [H.window_lse(wl, lay, over.get("causal_window", True)) for lay in layers] if over.pop("given_lse", False) else None
    p, outs = H.run_compress(wl, layers, r_given=rg, head_budgets=hb, lse=lse, **over)
    tot = dict(max_err=0.0, band=0, exact=0, checked=0)
    for i, (lay, out) in enumerate(zip(layers, outs)):
        st = H.check_layer(wl, lay, p, out, units=units, r_given=None if rg is None else rg[i],
                           head_budgets=None if hb is None else hb[i], lse=None if lse is None else lse[i], **over)
        tot["max_err"] = max(tot["max_err"], st["max_err"])
        for k in ("band", "exact", "checked"):
            tot[k] += st[k]
    _say(f"       checked {tot['checked']} units: max score err {tot['max_err']:.2e}, identical index sets "
         f"{tot['exact']}, near-tie candidates {tot['band']}")
    return tot


def test_c1_tiny_fp32():
    st = _run_and_check(WL["c1"])
    assert st["exact"] == st["checked"] == 2


def test_c2_single_layer_bf16():
    _run_and_check(WL["c2"])


@pytest.mark.parametrize("over", [
    dict(pool="avg"), dict(pool="none"), dict(intrinsic="none"), dict(causal_window=False),
    dict(pool="max", pool_kernel=3, softmax_scale=0.125), dict(budget=8), dict(budget=512),
])
def test_c1_variants(over):
    _run_and_check(WL["c1"], **over)


@pytest.mark.parametrize("over", [dict(pool="avg"), dict(intrinsic="none"), dict(causal_window=False, pool="none")])
def test_c2_variants(over):
    _run_and_check(WL["c2"], **over)


@pytest.mark.parametrize("dtype,D,N,W,Hq,Hkv,B", [
    ("bf16", 64, 1000, 5, 6, 2, 37),       # G*W = 15 rows (one padded tile), ragged key tail
    ("f32", 128, 777, 9, 4, 4, 100),       # G = 1, fp32 with D = 128
    ("bf16", 128, 333, 32, 16, 2, 40),     # G*W = 256 rows = 8 tiles, two chunks
    ("bf16", 128, 2049, 17, 3, 1, 64),     # one key past a chunk boundary, odd window
    ("f32", 64, 64, 31, 2, 1, 40),         # window half of the sequence
    # no spare query tile for the mean key in pass 2 (G*W a whole number of wave slots): its tile is
    # dealt over the waves by contraction chunk, 1, 2 or 4 chunks per wave
    ("bf16", 64, 900, 32, 4, 1, 64),       # G*W = 128: 4 tiles on 4 waves, 4 chunks
    ("f32", 64, 700, 32, 8, 2, 80),        # the same in fp32: 8 chunks
    ("f32", 128, 600, 32, 4, 1, 64),       # fp32, D = 128: 16 chunks
    ("bf16", 128, 1200, 32, 16, 1, 64),    # G*W = 512: 16 tiles on 8 waves x 2
])
def test_ragged_shapes(dtype, D, N, W, Hq, Hkv, B):
    wl = WL["c2"].with_(name="ragged", dtype=dtype, head_dim=D, seq_len=N, window=W, n_q_heads=Hq, n_kv_heads=Hkv,
                        budget=B, batch=2, text_prefix=min(16, N // 4), text_suffix_start=N - max(W, N // 8))
    _run_and_check(wl, n_layers=2)


# Few query rows: every wave takes whole key tiles of its own.  One and two query tiles, full and ragged; fewer tiles
# than waves, a single tile, runs that end inside a tile; key statistics and value norms on and off.
@pytest.mark.parametrize("dtype,D,N,W,Hq,Hkv,over", [
    ("f32", 64, 1003, 16, 4, 2, {}), ("f32", 128, 515, 32, 2, 2, {}), ("f32", 128, 300, 33, 1, 1, {}), ("f32", 64, 90, 31, 4, 2, {}),
    ("bf16", 64, 2049, 32, 4, 2, {}), ("bf16", 64, 40, 8, 8, 2, {}), ("bf16", 128, 1000, 8, 8, 2, dict(intrinsic="knorm")),
    ("bf16", 128, 31, 5, 2, 1, dict(budget=7)), ("bf16", 128, 777, 32, 2, 2, dict(causal_window=False)), ("f32", 64, 130, 8, 2, 1, dict(mix="imp_only", intrinsic="none")),
])
def test_few_query_rows(dtype, D, N, W, Hq, Hkv, over):
    wl = WL["c2"].with_(name="few-rows", dtype=dtype, head_dim=D, seq_len=N, window=W, n_q_heads=Hq, n_kv_heads=Hkv, batch=2,
                        budget=min(N, W + 20), text_prefix=min(8, N // 4), text_suffix_start=N - min(8, N // 4))
    _run_and_check(wl, n_layers=2, **over)


# One and two query tiles of either type, whole tiles and a ragged one, for the two tests below.
FEW_ROWS = [("bf16", 64, 16, 4, 2), ("bf16", 64, 32, 4, 2), ("bf16", 128, 8, 8, 2), ("f32", 64, 16, 4, 2), ("f32", 64, 32, 4, 2),
            ("f32", 128, 9, 4, 2), ("f32", 128, 32, 4, 2)]


# Logits as in the next test, where the waves of a run hold offsets of their own.  A logit of up to 700 in the log2 domain
# carries two roundings of half a unit, 2 * 2^-15, so fp32 weights are only good to 6e-5; bf16 inputs have 1e-4 anyway.
@pytest.mark.parametrize("scale", [30.0, 150.0])
@pytest.mark.parametrize("dtype,D,W,Hq,Hkv", FEW_ROWS)
def test_few_query_rows_with_large_logits(dtype, D, W, Hq, Hkv, scale):
    wl = WL["c2"].with_(name="few-rows-large", dtype=dtype, head_dim=D, seq_len=2048, window=W, n_q_heads=Hq, n_kv_heads=Hkv,
                        text_suffix_start=1984, softmax_scale=scale)
    lay = synth.make_layer(wl, 0)
    _say(f"[case] few rows, large logits {dtype} D={D} W={W} Hq={Hq} scale={scale}")
    p, outs = H.run_compress(wl, [lay])
    sc, G = outs[0].scores.cpu().numpy().astype(np.float64), wl.group
    for h in range(Hkv):
        want = O.score_unit(lay.K[0, h], lay.V[0, h], lay.Q[0, h * G:(h + 1) * G], H.oracle_params(wl))["s_comp"]
        err = np.abs(sc[0, h, :wl.seq_len - W] - want) / np.maximum(np.abs(want), np.abs(want).mean())
        _say(f"       head {h}: max score err {err.max():.2e}")
        assert err.max() <= 1e-4


@pytest.mark.parametrize("dtype,D,W,Hq,Hkv", FEW_ROWS)
def test_few_query_rows_on_a_strided_cache(dtype, D, W, Hq, Hkv):
    # tokens outermost, heads inside, both in larger slabs: every stride differs from the dense ones
    wl = WL["c2"].with_(name="few-rows-strided", dtype=dtype, head_dim=D, seq_len=1001, window=W, n_q_heads=Hq, n_kv_heads=Hkv,
                        batch=2, text_suffix_start=940)
    lay = synth.make_layer(wl, 0)
    dev = "cuda:0"
    _say(f"[case] few rows, strided {dtype} D={D} W={W} Hq={Hq}")
    _, ref = H.run_compress(wl, [lay])
    p = H.gpu_params(wl)

    def strided(x):
        buf = torch.full((2, wl.seq_len + 3, Hkv + 1, D), float("nan"), dtype=B.TORCH_DTYPE[p.dtype], device=dev)
        view = buf[:, :wl.seq_len, :Hkv].permute(0, 2, 1, 3)
        view.copy_(H.to_device(wl, x))
        return view

    out = B.alloc_layer_out(p, dev)
    B.mixkv_compress(p, [strided(lay.K)], [strided(lay.V)], [H.to_device(wl, lay.Q)], [out], B.alloc_workspace(p, 1, dev))
    torch.cuda.synchronize()
    for name in ("scores", "redundancy", "indices", "counts", "offsets", "K_out", "V_out"):
        assert torch.equal(getattr(out, name).view(torch.uint8), getattr(ref[0], name).view(torch.uint8)), name


@pytest.mark.parametrize("scale", [30.0, 150.0])
def test_large_logits_move_the_softmax_offset_mid_run(scale):
    # Logits with a standard deviation of 30 and 150: at 150 a row meets keys far more than 88 above
    # everything its first key tile held, so the running softmax offset of pass 1 has to move in the middle of a
    # run (the terms relative to the old offset overflow a float); at 30 the sums grow far beyond 1
    # without overflowing.  Both must give the oracle's scores.
    wl = WL["c2"].with_(name="large-logits", seq_len=2048, text_suffix_start=1984, batch=1)
    _run_and_check(wl, softmax_scale=scale)


@pytest.mark.parametrize("name,over", [("c1", {}), ("c2", {}), ("c2", dict(intrinsic="knorm")), ("c1", dict(intrinsic="knorm"))])
def test_zero_keys_are_normalised_to_the_zero_vector(name, over):
    # a key of norm zero has no direction: its normalised key is the zero vector (it adds nothing to the mean key,
    # its diversity score is 0, its key-norm score 0), in the window as among the candidates
    wl = WL[name]
    lay = synth.make_layer(wl, 0)
    for i in (0, 5, wl.seq_len // 2, wl.seq_len - wl.window - 1, wl.seq_len - 1):
        lay.K[:, :, i, :] = 0.0
    lay.K[:, 0, 7, :] = 0.0
    _say(f"[case] zero keys {wl.name} over={over}")
    p, outs = H.run_compress(wl, [lay], **over)
    st = H.check_layer(wl, lay, p, outs[0], **over)
    _say(f"       checked {st['checked']} units: max score err {st['max_err']:.2e}, identical index sets {st['exact']}")
    assert st["checked"] == wl.batch * wl.n_kv_heads


def test_budget_edges():
    wl = WL["c1"]
    _run_and_check(wl, budget=wl.window)          # B' = 0: window only
    _run_and_check(wl, budget=wl.seq_len)         # keep everything


@pytest.mark.parametrize("name,kw", [
    ("c1", {}),
    # longer rows: 16 and 32 candidates per thread in the fused mix-and-select kernel
    ("c2", dict(seq_len=12000, batch=1, n_q_heads=4, n_kv_heads=2, text_suffix_start=11900)),
    ("c2", dict(seq_len=20000, batch=1, n_q_heads=4, n_kv_heads=2, text_suffix_start=19900)),
    # beyond the fused kernel's row length: segments, and the merge of their lists
    ("c2", dict(seq_len=33000, batch=1, n_q_heads=4, n_kv_heads=2, text_suffix_start=32900)),
])
def test_identical_keys_degenerate_head(name, kw):
    # r = 1, constant diversity: every mixed score is ~0 and any selection is a valid tie-break.
    # The constant diversity has to cancel exactly against its own minimum, or the 1/eps of the
    # min-max normalisation blows a rounding residue up to the size of the scores.
    wl = WL[name].with_(name="degenerate", **kw) if kw else WL[name]
    lay = synth.make_layer(wl, 0)
    lay.K[:] = lay.K[0, 0, 0]
    p, outs = H.run_compress(wl, [lay])
    red = outs[0].redundancy.cpu().numpy()
    assert np.all(np.abs(red - 1.0) < 1e-5)
    sc = outs[0].scores.cpu().numpy()[:, :, :wl.seq_len - wl.window]
    u = O.score_unit(lay.K[0, 0], lay.V[0, 0], lay.Q[0, :2], H.oracle_params(wl))
    assert np.abs(sc[0, 0]).max() < 1e-4 * np.abs(u["s_imp"]).max()
    idx = outs[0].indices.cpu().numpy()
    for h in range(2):
        assert len(set(idx[0, h].tolist())) == wl.budget
    # every unit through the invariants of a compacted cache: counts and offsets, kept positions
    # unique, ascending and in range, window rows last, gathered rows bit-identical to the source
    H.check_layer(wl, lay, p, outs[0], units=[])


def test_c3_two_layers_all_budgets():
    wl = WL["c3"]
    for budget in (64, 128, 256, 512):
        _run_and_check(wl, layer_ids=[0, 17], units=[(0, 0), (0, 3)], budget=budget)


def _oracle_kwargs(wl, **over):
    op = H.oracle_params(wl, **over)
    return {f: getattr(op, f) for f in op.__dataclass_fields__}


def test_c3_full_cache_bench_configuration():
    # the launch configuration bench.py times: all 28 layers in one call, compared with the oracle on
    # every one of the 112 units (the oracle runs in worker processes while the GPU call is set up)
    from tests import oracle_pool
    wl = WL["c3"]
    layers = [synth.make_layer(wl, l) for l in range(wl.n_layers)]
    _say(f"[case] c3 full cache, {wl.n_layers} layers in one call, oracle on all {wl.n_units} units")
    ora = oracle_pool.score_layers("c3", {}, range(wl.n_layers), _oracle_kwargs(wl))
    p, outs = H.run_compress(wl, layers)
    tot = dict(max_err=0.0, exact=0, checked=0)
    for l, (lay, out) in enumerate(zip(layers, outs)):
        st = H.check_layer(wl, lay, p, out, oracle_units=ora[l])
        tot["max_err"] = max(tot["max_err"], st["max_err"])
        tot["exact"] += st["exact"]
        tot["checked"] += st["checked"]
    _say(f"       {tot}")
    assert tot["checked"] == wl.n_units


def test_c4_llama_shaped_two_layers():
    _run_and_check(WL["c4"], layer_ids=[0, 31], units=[(0, 0), (0, 7)])


def test_c4_llama_shaped_full_depth_one_call():
    # all 32 layers (256 units) in one call; oracle on units of the first, middle and last layers,
    # invariants on every unit
    wl = WL["c4"]
    layers = [synth.make_layer(wl, l) for l in range(wl.n_layers)]
    _say(f"[case] c4 full depth, {wl.n_layers} layers in one call")
    p, outs = H.run_compress(wl, layers, want_scores=True)
    sample = {0: [(0, 0), (0, 5)], 1: [(0, 7)], 15: [(0, 2), (0, 6)], 16: [(0, 3)], 30: [(0, 1)], 31: [(0, 4), (0, 7)]}
    checked = 0
    for l, (lay, out) in enumerate(zip(layers, outs)):
        st = H.check_layer(wl, lay, p, out, units=sample.get(l, []))
        checked += st["checked"]
        if l in sample:
            _say(f"       layer {l}: {st}")
    assert checked == sum(len(v) for v in sample.values()) >= 8


def test_c5_long_video_adaptive_one_layer():
    wl = WL["c5"].with_(batch=2)
    _run_and_check(wl, layer_ids=[3], units=[(0, h) for h in range(4)])


def test_c5_long_video_adaptive_full_depth_one_call():
    # all 28 layers x batch 4 (448 units) in one call, head-adaptive budgets; oracle on complete
    # (layer, batch item) groups of four heads (so the budget split is compared too) of the first,
    # middle and last layers, every batch item covered; invariants on every unit
    wl = WL["c5"]
    layers = [synth.make_layer(wl, l) for l in range(wl.n_layers)]
    _say(f"[case] c5 full depth, {wl.n_layers} layers x batch {wl.batch} in one call")
    p, outs = H.run_compress(wl, layers, want_scores=True)
    sample = {0: [0], 13: [1, 2], 27: [3]}                 # layer -> batch items
    checked = 0
    for l, (lay, out) in enumerate(zip(layers, outs)):
        units = [(b, h) for b in sample.get(l, []) for h in range(wl.n_kv_heads)]
        st = H.check_layer(wl, lay, p, out, units=units)
        checked += st["checked"]
        if l in sample:
            _say(f"       layer {l}: {st}")
    assert checked == 16


def test_adaptive_small_all_units():
    wl = WL["c2"].with_(name="adaptive-small", seq_len=1024, text_suffix_start=960, batch=3, budget=96,
                        budget_mode="adaptive", budget_floor=16, sigma=(0.1, 0.8))
    _run_and_check(wl, n_layers=2)
    _run_and_check(wl, n_layers=1, budget_floor=0)
    _run_and_check(wl, n_layers=1, budget_floor=64)     # floor == B': nothing left to pool
    # a pool that may go to one head whole: the lists hold every candidate
    _run_and_check(wl, n_layers=1, budget=400)


# Lists as long as the pool, kept in the per-key rows the mix has read: 8, 16 and 32 candidates per thread, split from
# registers (up to 16 384 entries per batch item) and from memory.
@pytest.mark.parametrize("N,Hkv,budget,floor", [(7000, 4, 900, 200), (12000, 4, 900, 0), (12000, 2, 5000, 37), (30000, 2, 3000, 0), (30000, 2, 6000, 500)])
def test_adaptive_budgets_with_long_lists(N, Hkv, budget, floor):
    wl = WL["c2"].with_(name="adaptive-lists", seq_len=N, text_suffix_start=N - 100, n_q_heads=Hkv, n_kv_heads=Hkv, budget=budget,
                        budget_mode="adaptive", budget_floor=floor, sigma=(0.1, 0.8))
    _run_and_check(wl, n_layers=1)


def test_more_layers_than_one_launch_group():
    wl = WL["c1"].with_(n_layers=35)
    _run_and_check(wl, n_layers=35)


def test_strided_cache_and_no_optional_outputs():
    wl = WL["c2"].with_(seq_len=1024, text_suffix_start=960)
    lay = synth.make_layer(wl, 0)
    p = H.gpu_params(wl)
    dev = "cuda:0"
    # K and V live in one [Bt, Hkv, 2, N+8, D] buffer: head stride and batch stride differ from the dense ones
    buf = torch.zeros((wl.batch, wl.n_kv_heads, 2, wl.seq_len + 8, wl.head_dim), dtype=torch.bfloat16, device=dev)
    buf[:, :, 0, :wl.seq_len] = H.to_device(wl, lay.K)
    buf[:, :, 1, :wl.seq_len] = H.to_device(wl, lay.V)
    K, V = buf[:, :, 0, :wl.seq_len], buf[:, :, 1, :wl.seq_len]
    out = B.alloc_layer_out(p, dev, scores=False, redundancy=False)
    out.offsets = None
    ws = B.alloc_workspace(p, 1, dev)
    B.mixkv_compress(p, [K], [V], [H.to_device(wl, lay.Q)], [out], ws)
    torch.cuda.synchronize()
    ref_p, ref = H.run_compress(wl, [lay])
    assert torch.equal(out.indices, ref[0].indices)
    assert torch.equal(out.K_out.view(torch.int16), ref[0].K_out.view(torch.int16))
    assert torch.equal(out.V_out.view(torch.int16), ref[0].V_out.view(torch.int16))


def test_two_runs_are_bit_identical():
    wl = WL["c2"]
    lay = synth.make_layer(wl, 0)
    _, a = H.run_compress(wl, [lay])
    _, b = H.run_compress(wl, [lay])
    assert torch.equal(a[0].scores.view(torch.int32), b[0].scores.view(torch.int32))
    assert torch.equal(a[0].indices, b[0].indices)
    assert torch.equal(a[0].redundancy.view(torch.int32), b[0].redundancy.view(torch.int32))


def test_score_entry_point_matches_compress_scores():
    wl = WL["c2"].with_(seq_len=2048, text_suffix_start=1984)
    lay = synth.make_layer(wl, 0)
    p, ref = H.run_compress(wl, [lay])
    dev = "cuda:0"
    out = B.alloc_layer_out(p, dev, select=False, gather=False)
    ws = B.alloc_workspace(p, 1, dev)
    B.mixkv_score(p, [H.to_device(wl, lay.K)], [H.to_device(wl, lay.V)], [H.to_device(wl, lay.Q)], [out], ws)
    torch.cuda.synchronize()
    assert torch.equal(out.scores.view(torch.int32), ref[0].scores.view(torch.int32))
    # ... and mixkv_select on those scores reproduces compress' indices
    sel = B.alloc_layer_out(p, dev, scores=False, redundancy=False, gather=False)
    sel.scores = out.scores
    B.mixkv_select(p, [sel])
    torch.cuda.synchronize()
    assert torch.equal(sel.indices, ref[0].indices) and torch.equal(sel.counts, ref[0].counts)


# Long rows are cut into segments whose length depends on what is kept; the scores may not depend on the cut.  Budgets
# that cut 66 001 tokens into segments of 4096, 8192 and 16 384 candidates, and one too large for the lists; 140 001
# tokens are scored in segments of 8192, 270 001 in segments of 16 384.
@pytest.mark.parametrize("N,Hkv,pool,budgets", [(66001, 2, "max", (64, 1232, 2048, 9032)), (140001, 2, "avg", (64, 1232)),
                                                (270001, 1, "none", (64, 3000))])
def test_scores_of_long_rows_do_not_depend_on_the_budget(N, Hkv, pool, budgets):
    wl = WL["c2"].with_(name="long-bits", seq_len=N, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64 * Hkv, batch=1,
                        text_suffix_start=N - 100, pool=pool)
    lay = synth.make_layer(wl, 0)
    dev = "cuda:0"
    K, V, Q = ([H.to_device(wl, x)] for x in (lay.K, lay.V, lay.Q))
    p = H.gpu_params(wl)
    alone = B.alloc_layer_out(p, dev, select=False, gather=False)
    B.mixkv_score(p, K, V, Q, [alone], B.alloc_workspace(p, 1, dev))
    for mode in ("fixed", "adaptive"):
        for budget in budgets:
            if mode == "adaptive" and budget > N // 20:
                continue
            _say(f"[case] {wl.name} N={N} {mode} B={budget}")
            p = H.gpu_params(wl, budget=budget, budget_mode=mode)
            out = B.alloc_layer_out(p, dev)
            ws = B.alloc_workspace(p, 1, dev)
            B.mixkv_compress(p, K, V, Q, [out], ws)
            # mixkv_select on the scores taken alone reproduces compress' indices
            sel = B.alloc_layer_out(p, dev, scores=False, redundancy=False, gather=False)
            sel.scores = alone.scores
            B.mixkv_select(p, [sel], ws)
            torch.cuda.synchronize()
            assert torch.equal(out.scores.view(torch.int32), alone.scores.view(torch.int32))
            for name in ("indices", "counts", "offsets"):
                assert torch.equal(getattr(sel, name), getattr(out, name)), name


# ------------------------------------------------------------------ ablation variants (Sec. 4.3, Table 4)

VARIANTS = [dict(intrinsic="knorm"), dict(mix="sum"), dict(mix="div_only"), dict(mix="imp_only"), dict(mix="given_r"),
            dict(mix="imp_only", intrinsic="none"), dict(mix="sum", intrinsic="knorm"),
            dict(mix="given_r", intrinsic="knorm", pool="avg")]


@pytest.mark.parametrize("over", VARIANTS)
def test_c1_scoring_variants(over):
    _run_and_check(WL["c1"], **over)


@pytest.mark.parametrize("over", VARIANTS[:5])
def test_c2_scoring_variants(over):
    _run_and_check(WL["c2"], **over)


@pytest.mark.parametrize("name,kw,over", [
    ("c1", {}, dict(mix="imp_only", intrinsic="none")),
    ("c1", {}, dict(mix="imp_only", intrinsic="vnorm", pool="avg")),
    ("c2", {}, dict(mix="imp_only", intrinsic="none")),
    ("c2", dict(seq_len=1000, text_suffix_start=940, budget_mode="adaptive", budget_floor=8), dict(mix="imp_only")),
    # beyond the fused mix kernel's row length: segments
    ("c2", dict(seq_len=33000, batch=1, n_q_heads=2, n_kv_heads=1, text_suffix_start=32900), dict(mix="imp_only", intrinsic="none")),
])
def test_importance_only_without_a_redundancy_output_skips_the_key_statistics(name, kw, over):
    # The importance-only score (Table 4; the SnapKV-style base of Sec. 4.1) reads neither key norms nor
    # the mean key nor r; when the caller does not ask for r either, the first pass does not compute
    # them.  Results must be those of the oracle all the same, and equal to the run that does compute
    # them (same arithmetic for everything that is read).
    wl = WL[name].with_(name="imp-only", **kw) if kw else WL[name]
    lay = synth.make_layer(wl, 0)
    _say(f"[case] {wl.name} importance only, no redundancy output, {over}")
    p, outs = H.run_compress(wl, [lay], want_redundancy=False, **over)
    st = H.check_layer(wl, lay, p, outs[0], **over)
    assert st["checked"] == wl.batch * wl.n_kv_heads
    p2, ref = H.run_compress(wl, [lay], want_redundancy=True, **over)
    assert torch.equal(outs[0].scores.view(torch.int32), ref[0].scores.view(torch.int32))
    assert torch.equal(outs[0].indices, ref[0].indices) and torch.equal(outs[0].counts, ref[0].counts)


def test_scoring_variants_adaptive_budgets_and_long_fallback():
    wl = WL["c2"].with_(name="adaptive-variants", seq_len=1024, text_suffix_start=960, batch=2, budget=96,
                        budget_mode="adaptive", budget_floor=16, sigma=(0.1, 0.8))
    _run_and_check(wl, layer_ids=[1], mix="given_r", intrinsic="knorm")
    # sequences too long for the fused mix kernel are mixed in segments
    wl = WL["c2"].with_(name="long", seq_len=33000, batch=1, n_q_heads=2, n_kv_heads=1, text_suffix_start=32900)
    _run_and_check(wl, n_layers=1, budget=400, mix="sum", intrinsic="knorm")


# Rows cut into segments: pooling windows that reach over the cuts (sliding window and generic loop), a last segment of
# one candidate, key-norm scores, more than one batch item.
@pytest.mark.parametrize("N,over", [(32768 + 32 + 1, dict(pool="avg", pool_kernel=5)), (33100, dict(pool="max", pool_kernel=31)),
                                    (33001, dict(pool="avg", pool_kernel=9, intrinsic="knorm", budget=300)), (36864 + 33, dict(pool="none"))])
def test_long_rows_pool_across_segments(N, over):
    wl = WL["c2"].with_(name="long-pool", seq_len=N, batch=2, n_q_heads=2, n_kv_heads=1, text_suffix_start=N - 100)
    _run_and_check(wl, n_layers=1, **over)


# Segments of 8192 and 16 384 candidates: the last one shorter than the lists or than the pooling window's reach, window and
# generic pooling, key-norm scores, head-adaptive and per-head budgets.
@pytest.mark.parametrize("N,Hkv,over", [
    (66001, 1, dict(budget=1232)), (66001, 1, dict(budget=2048, pool="avg", pool_kernel=9, intrinsic="knorm")),
    (140001, 1, dict(pool="max", pool_kernel=31)), (65536 + 32 + 3, 1, dict(budget=3032)), (73728 + 32 + 2, 1, dict(budget=1300)),
    (66001, 2, dict(budget=700, budget_mode="adaptive", budget_floor=50)), (66001, 2, dict(budget=2048, budget_mode="adaptive", mix="sum")),
    (66001, 2, dict(budget=1000, budget_mode="per_head", head_budgets=np.array([[1900, 64]], dtype=np.int32)))])
def test_long_rows_in_wide_segments(N, Hkv, over):
    wl = WL["c2"].with_(name="long-wide", seq_len=N, n_q_heads=Hkv, n_kv_heads=Hkv, text_suffix_start=N - 100, sigma=(0.1, 0.8))
    _run_and_check(wl, n_layers=1, **over)


# Budgets beyond what the merge holds: the row is mixed in segments, its scores go to the workspace, and the selection
# kernels rank the whole row.
@pytest.mark.parametrize("Hkv,over", [(1, dict(budget=30000)), (2, dict(budget=16000, budget_mode="adaptive", budget_floor=100)),
                                      (2, dict(budget=16000, budget_mode="per_head", head_budgets=np.array([[31000, 64]], dtype=np.int32)))])
def test_long_rows_with_budgets_beyond_the_merge(Hkv, over):
    wl = WL["c2"].with_(name="long-budget", seq_len=33000, n_q_heads=Hkv, n_kv_heads=Hkv, text_suffix_start=32900, sigma=(0.1, 0.8))
    lay = synth.make_layer(wl, 0)
    hb = over.get("head_budgets")
    kw = {k: v for k, v in over.items() if k != "head_budgets"}
    _say(f"[case] {wl.name} Hkv={Hkv} {over}, no scores asked for")
    p, outs = H.run_compress(wl, [lay], want_scores=False, head_budgets=hb, **kw)
    st = H.check_layer(wl, lay, p, outs[0], head_budgets=None if hb is None else hb[0], **kw)
    assert st["checked"] == Hkv


# Rows that no cut into 32 segments reaches: the one-workgroup mix and selection kernels.
def test_rows_beyond_any_cut_take_the_plain_mix_and_selection():
    N = 524288 + 32 + 9
    wl = WL["c2"].with_(name="longest", seq_len=N, head_dim=64, n_q_heads=1, n_kv_heads=1, text_suffix_start=N - 100)
    lay = synth.make_layer(wl, 0)
    for over in (dict(), dict(intrinsic="knorm", mix="sum", pool="avg", pool_kernel=9, budget=700),
                 dict(mix="imp_only", pool="none", budget_mode="adaptive", budget_floor=5)):
        want_scores = over.get("mix") != "imp_only"            # without: the scores go to the workspace, the key statistics are skipped
        _say(f"[case] {wl.name} N={N} {over}")
        p, outs = H.run_compress(wl, [lay], want_scores=want_scores, want_redundancy=want_scores, **over)
        st = H.check_layer(wl, lay, p, outs[0], **over)
        _say(f"       max score err {st['max_err']:.2e}, identical index sets {st['exact']}")
        assert st["checked"] == 1
        if want_scores:
            alone = B.alloc_layer_out(p, "cuda:0", select=False, gather=False)
            B.mixkv_score(p, [H.to_device(wl, lay.K)], [H.to_device(wl, lay.V)], [H.to_device(wl, lay.Q)], [alone], B.alloc_workspace(p, 1, "cuda:0"))
            torch.cuda.synchronize()
            assert torch.equal(alone.scores.view(torch.int32), outs[0].scores.view(torch.int32))


# One value row far longer than the others: the means over the segments must not lose the others' low bits to it (a sum of
# 33 000 ordinary norms taken from that row's was wrong by 3.6e-5 of the score, beyond the 1e-5 of fp32 inputs).
@pytest.mark.parametrize("at", [0, 1, 4095, 20000])
def test_long_rows_with_one_outlying_value_norm(at):
    wl = WL["c2"].with_(name="long-outlier", dtype="f32", seq_len=33000, batch=1, n_q_heads=1, n_kv_heads=1, window=8, text_suffix_start=32900)
    lay = synth.make_layer(wl, 0)
    lay.V[:, :, at, :] *= 300.0
    _say(f"[case] long row, value row {at} times 300")
    p, outs = H.run_compress(wl, [lay])
    st = H.check_layer(wl, lay, p, outs[0])
    _say(f"       max score err {st['max_err']:.2e}")


def test_long_rows_of_equal_keys_and_values_with_an_eps_without_a_reciprocal():
    # the normalised value norm and diversity are 0 / eps = 0 whatever eps > 0, also where 1 / eps is no float
    wl = WL["c2"].with_(name="long-equal", seq_len=33000, batch=1, n_q_heads=2, n_kv_heads=1, text_suffix_start=32900)
    lay = synth.make_layer(wl, 0)
    lay.K[:] = lay.K[0, 0, 0]
    lay.V[:] = lay.V[0, 0, 0]
    _say("[case] long row of equal keys and values, eps 1e-40")
    _, ref = H.run_compress(wl, [lay], mix="sum")
    _, out = H.run_compress(wl, [lay], mix="sum", eps=1e-40)
    assert torch.isfinite(ref[0].scores[:, :, :wl.seq_len - wl.window]).all()
    assert torch.equal(out[0].scores.view(torch.int32), ref[0].scores.view(torch.int32))
    assert torch.equal(out[0].indices, ref[0].indices)


def test_given_r_needs_the_weights():
    wl = WL["c1"]
    with pytest.raises(B.MixkvError) as e:
        H.run_compress(wl, [synth.make_layer(wl, 0)], mix="given_r")      # rejected on the host, nothing launched
    assert e.value.status == B.MIXKV_ERR_INVALID_ARG


def test_given_r_equal_to_own_redundancy_reproduces_the_head_adaptive_mix():
    wl = WL["c2"]
    lay = synth.make_layer(wl, 0)
    p, outs = H.run_compress(wl, [lay])
    red = outs[0].redundancy.cpu().numpy()
    p2, outs2 = H.run_compress(wl, [lay], r_given=[red], mix="given_r")
    assert torch.equal(outs[0].scores, outs2[0].scores) and torch.equal(outs[0].indices, outs2[0].indices)
    assert torch.equal(outs[0].redundancy, outs2[0].redundancy)


# ------------------------------------------------------------------ budgets given per layer and head

def _pyramid(L, Hkv, top, bottom):
    """A layer-wise schedule: `top` rows per head in layer 0 falling linearly to `bottom` in the last."""
    per_layer = np.round(np.linspace(top, bottom, L)).astype(np.int32)
    return np.repeat(per_layer[:, None], Hkv, axis=1)


def test_per_head_budgets_c1_and_c2():
    wl = WL["c1"]
    _run_and_check(wl, budget_mode="per_head", head_budgets=np.array([[wl.window, 120]], dtype=np.int32))
    wl = WL["c2"]
    hb = np.array([[wl.window, 64, 500, wl.seq_len]], dtype=np.int32)        # window only ... keep everything
    _run_and_check(wl, budget_mode="per_head", head_budgets=hb, budget=int(-(-hb.sum() // 4)))


def test_per_layer_pyramid_over_two_launch_groups():
    wl = WL["c1"].with_(n_layers=35)
    hb = _pyramid(35, wl.n_kv_heads, 2 * wl.budget - wl.window, wl.window)   # mean = the fixed budget
    rng = np.random.default_rng(5)
    hb[::2] += rng.integers(-3, 4, size=hb[::2].shape).astype(np.int32)      # and some head-wise spread
    hb = np.clip(hb, wl.window, None)
    _run_and_check(wl, n_layers=35, budget_mode="per_head", head_budgets=hb, budget=int(hb.sum(axis=1).max() + 1) // 2 + 1)


def test_per_head_budgets_ragged_f32_and_long_fallback():
    wl = WL["c2"].with_(name="ragged-ph", dtype="f32", head_dim=64, seq_len=777, window=9, n_q_heads=4, n_kv_heads=4,
                        budget=100, batch=2, text_prefix=16, text_suffix_start=700)
    hb = np.array([[9, 10, 333, 40], [48, 100, 100, 152]], dtype=np.int32)
    _run_and_check(wl, n_layers=2, budget_mode="per_head", head_budgets=hb)
    wl = WL["c2"].with_(name="long-ph", seq_len=33000, batch=1, n_q_heads=4, n_kv_heads=2, text_suffix_start=32900)
    _run_and_check(wl, n_layers=1, budget_mode="per_head", head_budgets=np.array([[300, 64]], dtype=np.int32), budget=200)


def test_equal_per_head_budgets_reproduce_fixed_mode_bit_for_bit():
    wl = WL["c2"]
    lay = synth.make_layer(wl, 0)
    p, outs = H.run_compress(wl, [lay])
    hb = np.full((1, wl.n_kv_heads), wl.budget, dtype=np.int32)
    p2, outs2 = H.run_compress(wl, [lay], budget_mode="per_head", head_budgets=hb)
    for name in ("indices", "counts", "offsets", "K_out", "V_out", "scores"):
        a, b = getattr(outs[0], name), getattr(outs2[0], name)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name


# ------------------------------------------------------------------ softmax normalisers handed over by the caller

def test_given_lse_c1_c2_and_variants():
    _run_and_check(WL["c1"], given_lse=True)
    _run_and_check(WL["c1"], given_lse=True, causal_window=False, pool="avg")
    _run_and_check(WL["c2"], given_lse=True)
    _run_and_check(WL["c2"], given_lse=True, intrinsic="knorm", mix="sum")


@pytest.mark.parametrize("dtype,D,N,W,Hq,Hkv,B", [
    ("bf16", 64, 1000, 5, 6, 2, 37), ("f32", 128, 777, 9, 4, 4, 100), ("bf16", 128, 333, 32, 16, 2, 40),
])
def test_given_lse_ragged_shapes(dtype, D, N, W, Hq, Hkv, B):
    wl = WL["c2"].with_(name="ragged-lse", dtype=dtype, head_dim=D, seq_len=N, window=W, n_q_heads=Hq, n_kv_heads=Hkv,
                        budget=B, batch=2, text_prefix=min(16, N // 4), text_suffix_start=N - max(W, N // 8))
    _run_and_check(wl, n_layers=2, given_lse=True)


def test_given_lse_c3_two_layers_and_adaptive_budgets():
    _run_and_check(WL["c3"], layer_ids=[0, 17], units=[(0, 0), (0, 3)], given_lse=True)
    wl = WL["c2"].with_(name="adaptive-lse", seq_len=1024, text_suffix_start=960, batch=2, budget=96,
                        budget_mode="adaptive", budget_floor=16, sigma=(0.1, 0.8))
    _run_and_check(wl, n_layers=2, given_lse=True)


def test_given_lse_must_cover_every_layer_of_a_call():
    wl = WL["c1"].with_(n_layers=2)
    layers = [synth.make_layer(wl, l) for l in range(2)]
    p = H.gpu_params(wl)
    Ks, Vs, Qs = ([H.to_device(wl, getattr(l, n)) for l in layers] for n in ("K", "V", "Q"))
    outs = [B.alloc_layer_out(p, "cuda:0") for _ in layers]
    ws = B.alloc_workspace(p, 2, "cuda:0")
    lse0 = torch.from_numpy(H.window_lse(wl, layers[0])).to("cuda:0")
    with pytest.raises(B.MixkvError) as e:
        B.mixkv_compress(p, Ks, Vs, Qs, outs, ws, window_lse=[lse0, None])
    assert e.value.status == B.MIXKV_ERR_INVALID_ARG


def test_very_long_video_cache_128k_tokens():
    # 256 frames of 510 tokens: beyond the fused mix kernel (mixed in segments, their lists merged, rows gathered),
    # 1024 chunks per head in the streaming kernels; oracle on one head
    wl = WL["c5"].with_(name="video-128k", batch=1, seq_len=64 + 256 * 510 + 64, text_suffix_start=64 + 256 * 510,
                        n_frames=256, budget_mode="fixed", budget=256)
    _run_and_check(wl, layer_ids=[0], units=[(0, 2)])


def test_calls_on_two_streams_with_their_own_workspaces_match_the_serial_results():
    """The library keeps no state between calls: two calls in flight on two streams of the caller
    (default priority), each with its own workspace and outputs, give bit for bit what the same
    calls give one after the other, and a call's results are complete once its own stream is."""
    wl = WL["c2"].with_(name="two-streams", batch=2)
    dev = "cuda:0"
    sets = []
    for first in (0, 2):
        layers = [synth.make_layer(wl, l) for l in (first, first + 1)]
        p = H.gpu_params(wl)
        Ks = [H.to_device(wl, l.K, dev) for l in layers]
        Vs = [H.to_device(wl, l.V, dev) for l in layers]
        Qs = [H.to_device(wl, l.Q, dev) for l in layers]
        outs = [B.alloc_layer_out(p, dev, scores=True) for _ in layers]
        ws = B.alloc_workspace(p, len(layers), dev)
        sets.append((B.PreparedCall(p, Ks, Vs, Qs, outs, ws), outs))
    _say(f"[case] two streams {wl.name} dtype={wl.dtype} L=2+2 Bt={wl.batch}")

    def snapshot(outs):
        return [[t.clone() for t in (o.scores, o.redundancy, o.indices, o.counts, o.K_out, o.V_out)] for o in outs]

    want = []
    for call, outs in sets:
        call.compress()
        torch.cuda.synchronize()
        want.append(snapshot(outs))
        for o in outs:                                     # so that the concurrent run has to write everything again
            for t in (o.scores, o.redundancy, o.indices, o.counts, o.K_out, o.V_out):
                t.zero_()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(3):
        for (call, _), st in zip(sets, streams):
            call.compress(stream=st)
        for (call, outs), st, w in zip(sets, streams, want):
            st.synchronize()                               # this call's stream only
            for got_l, want_l in zip(snapshot(outs), w):
                for g, x in zip(got_l, want_l):
                    assert torch.equal(g, x), f"repetition {rep}: a call on its own stream differs from the serial run"
    torch.cuda.synchronize()


def test_a_call_captured_in_a_graph_replays_to_the_eager_results():
    """A call allocates nothing, records no memset and never synchronises, so a caller can capture
    it in a graph.  Three replays, with the outputs cleared by ordinary eager work and a
    synchronisation between them, must each reproduce the eager results bit for bit."""
    wl = WL["c2"].with_(name="graph", batch=2)
    dev = "cuda:0"
    layers = [synth.make_layer(wl, l) for l in (0, 1)]
    p = H.gpu_params(wl)
    Ks = [H.to_device(wl, l.K, dev) for l in layers]
    Vs = [H.to_device(wl, l.V, dev) for l in layers]
    Qs = [H.to_device(wl, l.Q, dev) for l in layers]
    outs = [B.alloc_layer_out(p, dev, scores=True) for _ in layers]
    ws = B.alloc_workspace(p, len(layers), dev)
    call = B.PreparedCall(p, Ks, Vs, Qs, outs, ws)
    _say(f"[case] graph capture {wl.name} dtype={wl.dtype} L=2 Bt={wl.batch}")
    fields = lambda o: (o.scores, o.redundancy, o.indices, o.counts, o.K_out, o.V_out)
    call.compress()
    torch.cuda.synchronize()
    want = [[t.clone() for t in fields(o)] for o in outs]
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        call.compress(side)                                # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call.compress(torch.cuda.current_stream())
    torch.cuda.synchronize()
    for rep in range(3):
        for o in outs:
            for t in fields(o):
                t.zero_()                                  # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            for g, x in zip(fields(o), w):
                assert torch.equal(g, x), f"replay {rep} differs from the eager call"


def test_long_rows_few_query_rows_and_lists_replay_from_a_graph():
    """The same for the kernels of long rows (segments, merge, split), of few query rows and of a selection on a full-size
    workspace, captured one after the other in one graph."""
    wl = WL["c2"].with_(name="graph-long", seq_len=33100, n_q_heads=2, n_kv_heads=2, text_suffix_start=33000, window=8)
    dev = "cuda:0"
    lay = synth.make_layer(wl, 0)
    p = H.gpu_params(wl, budget=200, budget_mode="adaptive", budget_floor=20)
    out, sel = B.alloc_layer_out(p, dev), B.alloc_layer_out(p, dev, scores=False, redundancy=False, gather=False)
    sel.scores = out.scores
    ws = B.alloc_workspace(p, 1, dev)
    call = B.PreparedCall(p, [H.to_device(wl, lay.K)], [H.to_device(wl, lay.V)], [H.to_device(wl, lay.Q)], [out], ws)
    _say(f"[case] graph capture {wl.name} N={wl.seq_len}")

    def both(stream):
        call.compress(stream)
        B.mixkv_select(p, [sel], ws, stream)

    fields = (out.scores, out.redundancy, out.indices, out.counts, out.offsets, out.K_out, out.V_out, sel.indices, sel.counts, sel.offsets)
    both(None)
    torch.cuda.synchronize()
    want = [t.clone() for t in fields]
    assert torch.equal(sel.indices, out.indices)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        both(side)                                         # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            both(torch.cuda.current_stream())
    torch.cuda.synchronize()
    for rep in range(3):
        for t in fields:
            t.zero_()                                      # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for g, x in zip(fields, want):
            assert torch.equal(g, x), f"replay {rep} differs from the eager call"
