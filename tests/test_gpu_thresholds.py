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


# candidates: 256, 512 and 1024 threads of 8, then 16 and 32 per thread, and a row in segments
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


# lists of a layer together: 4 to 32 entries per thread of the split, one entry beyond them (the lists are streamed), lists
# shorter than a thread's entries, heads that keep all they have
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
