"""The threshold search of the selection kernels where its steps change over: boundary bins that hold up to, and more
than, the keys that are ranked by counting; keys that only differ in their last bits below a few outliers (several
histograms); both signs; whole bins; both thresholds of a head-adaptive list in one bin.  Whole-number work: bit-exact
against the oracle's selection on the same float32 scores, ties included."""
import numpy as np
import pytest
import torch

from oracle import mixkv_oracle as O
from paper_2510_20707_amd import binding as B

pytestmark = pytest.mark.gpu
W = 8


def _scores(kind, rng, shape):
    if kind.startswith("crowd"):                    # that many scores share the first histogram's bin of the boundary
        m = int(kind[5:])
        s = rng.random(shape)                       # below 1
        flat = s.reshape(-1, shape[-1])
        for row in flat:
            row[rng.choice(shape[-1], m, replace=False)] = 1.5 + 1e-6 * rng.integers(0, 3 * m, m)
        flat[:, 0] = -3e38                          # both signs: the first digit holds the sign and the exponent
        flat[:, -1] = 3e38
    elif kind == "last bits":                       # all in one bin of the first two digits, but for an outlier
        s = (0x3f000000 + rng.integers(0, 40, shape)).astype(np.uint32).view(np.float32).astype(np.float64)
        s[..., 1] = -1e-38
    elif kind == "signed":
        s = rng.standard_normal(shape) * np.exp(rng.standard_normal(shape) * 8)
    elif kind == "two values":
        s = np.where(rng.random(shape) < 0.01, 2.0, 1.0)
    else:
        raise ValueError(kind)
    return s.astype(np.float32)


KINDS = ["crowd127", "crowd128", "crowd129", "crowd700", "last bits", "signed", "two values"]


# candidates: 512 threads of 4 and of 8, 1024 of 8, 16 and 32, and a row in segments
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("Nc,Bp", [(2048, 100), (4096, 129), (8190, 60), (8192, 2000), (16383, 128), (32000, 150), (40000, 65)])
def test_thresholds_of_a_head(kind, Nc, Bp):
    print(f"[case] thresholds kind={kind} Nc={Nc} Bp={Bp}", flush=True)
    rng = np.random.default_rng([61, Nc, Bp])
    Hkv, N = 2, Nc + W
    s = np.concatenate([_scores(kind, rng, (1, Hkv, Nc)), np.full((1, Hkv, W), np.inf, dtype=np.float32)], -1)
    p = B.make_params("bf16", 1, Hkv, Hkv, 128, N, W, Bp + W)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    B.mixkv_select(p, [out], B.alloc_workspace(p, 1, "cuda:0"))
    idx = out.indices.cpu().numpy()
    for h in range(Hkv):
        np.testing.assert_array_equal(idx[0, h], O.select_unit(s[0, h, :Nc].astype(np.float64), Bp, N, W))


# lists of a layer together: 4, 16 and 32 entries per thread of the split's workgroup, 32 in every thread, one list or one entry more (64 per
# thread), lists shorter than a thread's entries, heads that keep all they have
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("Nc,Bp,floor,Hkv", [(1000, 40, 13, 4), (4096, 300, 128, 4), (6000, 700, 512, 8), (3000, 2400, 0, 8), (4096, 1500, 11, 8),
                                             (2979, 2700, 300, 11), (9, 5, 1, 40), (4097, 1500, 11, 8)])
def test_thresholds_of_the_head_adaptive_split(kind, Nc, Bp, floor, Hkv):
    if kind.startswith("crowd") and int(kind[5:]) > Nc:
        kind = "crowd5"
    print(f"[case] split thresholds kind={kind} Nc={Nc} Bp={Bp} floor={floor} Hkv={Hkv}", flush=True)
    rng = np.random.default_rng([62, Nc, Bp])
    N = Nc + W
    s = np.concatenate([_scores(kind, rng, (1, Hkv, Nc)), np.full((1, Hkv, W), np.inf, dtype=np.float32)], -1)
    p = B.make_params("bf16", 1, Hkv, Hkv, 128, N, W, Bp + W, budget_mode="adaptive", budget_floor=floor)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    B.mixkv_select(p, [out], B.alloc_workspace(p, 1, "cuda:0"))
    idx, cnt, off = out.indices.cpu().numpy().reshape(-1), out.counts.cpu().numpy()[0], out.offsets.cpu().numpy()[0]
    bp = O.adaptive_budgets(s[0, :, :Nc].astype(np.float64), Bp + W, W, floor)
    np.testing.assert_array_equal(cnt, bp + W)
    np.testing.assert_array_equal(off, np.concatenate([[0], np.cumsum(bp + W)]))
    for h in range(Hkv):
        np.testing.assert_array_equal(idx[off[h]:off[h + 1]], O.select_unit(s[0, h, :Nc].astype(np.float64), int(bp[h]), N, W))


# Equal scores meet in one bin of a histogram.  Whatever their share of a head, the selection takes no more than twice what it takes on
# scores that are spread (measured: at most 1.45 times; 3.4 to 6.6 times if every one of them is counted by an atomic of its own).
@pytest.mark.parametrize("mode,floor", [("fixed", 0), ("adaptive", 128)])
def test_equal_scores_take_no_longer_than_spread_ones(mode, floor):
    L, Hkv, Nc, Bp = 28, 4, 32000, 480
    N, rng, us = Nc + W, np.random.default_rng(63), {}
    one = np.full((1, Hkv, Nc), 0.25)
    far = one.copy()
    far[..., 3] = 1e30
    kinds = {"spread": rng.standard_normal((1, Hkv, Nc)), "equal": one, "equal but one": far,
             "two values": np.where(rng.random((1, Hkv, Nc)) < 0.01, 2.0, 1.0), "halves": np.where(rng.random((1, Hkv, Nc)) < 0.5, 2.0, 1.0),
             "neighbours": 1.5 + rng.integers(0, 4, (1, Hkv, Nc)) * 2.0 ** -23}
    p = B.make_params("bf16", 1, Hkv, Hkv, 128, N, W, Bp + W, budget_mode=mode, budget_floor=floor)
    for kind, s in kinds.items():
        print(f"[case] tied scores {mode} {kind}", flush=True)
        s = np.concatenate([s.astype(np.float32), np.full((1, Hkv, W), np.inf, dtype=np.float32)], -1)
        outs = []
        for _ in range(L):
            outs.append(B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False))
            outs[-1].scores = torch.from_numpy(s).to("cuda:0")
        ws = B.alloc_workspace(p, L, "cuda:0")
        stream, graph, calls = torch.cuda.Stream(), torch.cuda.CUDAGraph(), 10
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            B.mixkv_select(p, outs, ws)
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(calls):
                B.mixkv_select(p, outs, ws)
        times = []
        for _ in range(7):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 1000 / calls)
        us[kind] = sorted(times)[3]
    print(us, flush=True)
    assert max(us.values()) <= 2 * us["spread"], us


def _infinite(kind, rng, shape):
    s = rng.standard_normal(shape).astype(np.float32)
    if kind == "few finite":                        # the threshold lies among scores of -inf
        s[rng.random(shape) < 0.99] = -np.inf
    elif kind == "both":
        s[rng.random(shape) < 0.3] = -np.inf
        s[rng.random(shape) < 0.002] = np.inf
    elif kind == "many above":                      # ... of +inf
        s[rng.random(shape) < 0.4] = np.inf
    elif kind == "nothing finite":
        s[:] = np.where(rng.random(shape) < 0.1, np.inf, -np.inf)
    else:
        s[:] = -np.inf
    return s


# Candidate scores of -inf and +inf are scores like any other (and no key of theirs is the one that stands for "no candidate")
@pytest.mark.parametrize("kind", ["few finite", "both", "many above", "nothing finite", "all -inf"])
@pytest.mark.parametrize("mode,Nc,Bp,floor,Hkv", [("fixed", 1000, 100, 0, 2), ("fixed", 32000, 1500, 0, 1), ("fixed", 40000, 900, 0, 2),
                                                  ("adaptive", 1001, 60, 13, 3), ("adaptive", 8192, 480, 128, 4)])
def test_infinite_scores(kind, mode, Nc, Bp, floor, Hkv):
    print(f"[case] infinite scores {mode} {kind} Nc={Nc} Bp={Bp} floor={floor} Hkv={Hkv}", flush=True)
    N = Nc + W
    s = np.concatenate([_infinite(kind, np.random.default_rng([64, Nc]), (1, Hkv, Nc)), np.full((1, Hkv, W), np.inf, dtype=np.float32)], -1)
    p = B.make_params("bf16", 1, Hkv, Hkv, 128, N, W, Bp + W, budget_mode=mode, budget_floor=floor)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    B.mixkv_select(p, [out], B.alloc_workspace(p, 1, "cuda:0"))
    ranked = np.nan_to_num(s[0, :, :Nc].astype(np.float64), posinf=1e300, neginf=-1e300)      # (the oracle marks what is taken by -inf)
    bp = O.adaptive_budgets(ranked, Bp + W, W, floor) if mode == "adaptive" else np.full(Hkv, Bp)
    idx, off = out.indices.cpu().numpy().reshape(-1), np.concatenate([[0], np.cumsum(bp + W)])
    np.testing.assert_array_equal(out.counts.cpu().numpy()[0], bp + W)
    for h in range(Hkv):
        np.testing.assert_array_equal(idx[off[h]:off[h + 1]], O.select_unit(ranked[h], int(bp[h]), N, W))


# NaN scores are not supported, but what is kept are still the wanted numbers of distinct positions in ascending order
@pytest.mark.parametrize("word", [0x7fc00000, 0xffffffff])
@pytest.mark.parametrize("mode,Nc,Bp,floor,Hkv", [("fixed", 1000, 100, 0, 2), ("fixed", 8190, 600, 0, 2), ("fixed", 40000, 900, 0, 2), ("adaptive", 8192, 480, 128, 4)])
@pytest.mark.parametrize("share", [0.01, 1.0])
def test_nan_scores_leave_the_output_in_order(word, mode, Nc, Bp, floor, Hkv, share):
    print(f"[case] nan scores {word:x} {mode} Nc={Nc} share={share}", flush=True)
    N, rng = Nc + W, np.random.default_rng([65, Nc])
    s = rng.standard_normal((1, Hkv, N)).astype(np.float32)
    s.view(np.uint32)[rng.random(s.shape) < share] = word
    p = B.make_params("bf16", 1, Hkv, Hkv, 128, N, W, Bp + W, budget_mode=mode, budget_floor=floor)
    out = B.alloc_layer_out(p, "cuda:0", redundancy=False, gather=False)
    out.scores = torch.from_numpy(s).to("cuda:0")
    out.indices.fill_(-1)
    B.mixkv_select(p, [out], B.alloc_workspace(p, 1, "cuda:0"))
    idx, cnt = out.indices.cpu().numpy().reshape(-1), out.counts.cpu().numpy()[0]
    assert cnt.sum() == Hkv * (Bp + W) and cnt.min() >= floor + W
    for rows in np.split(idx, np.cumsum(cnt)[:-1]):
        assert rows[0] >= 0 and np.all(np.diff(rows) > 0)
        np.testing.assert_array_equal(rows[-W:], np.arange(Nc, N))
