"""fp32 attention at the ends of the type's range: keys that score -inf or the lowest values in whole
tiles and key groups, scores far beyond 2^24, probabilities below 2^-126, values near the largest
fp32, and a launch of more workgroups than one grid holds threads for."""

import numpy as np
import pytest
import torch

from gpu_helpers import MASS_TOL, O_TOL, dev, host, max_abs
from oracle import joint_attention

pytestmark = pytest.mark.gpu

# split (subtiles x groups) that the launch takes, head_dim, B, H, n_ref, n_tgt
SHAPES = [
    ("1x4", 64, 1, 2, 100, 130),
    ("1x8", 128, 1, 1, 256, 256),
    ("1x8", 64, 1, 2, 500, 15),
    ("2x2", 128, 1, 24, 33, 545),
    ("4x1", 128, 2, 17, 74, 733),
]


def _run(x, **kw):
    from paper_2609_32415_amd import ops

    t = {k: dev(v, "f32") for k, v in x.items()}
    r = ops.joint_attn(t["q_tgt"], t["k_tgt"], t["v_tgt"], q_ref=t["q_ref"], k_ref=t["k_ref"], v_ref=t["v_ref"],
                       qset="all", kvsrc="fresh", lse=True, ref_mass_refq=True, **kw)
    torch.cuda.synchronize()
    return r


def _keys(n_ref, n_tgt, where):
    """Key numbers (reference first) of a run, or of several, of 16 to 64 aligned keys."""
    n = n_ref + n_tgt
    runs = {"first tile": [(0, 32)], "after the first": [(16, 80)], "reference": [(0, n_ref)], "target": [(n_ref, n)],
            "eighths": [(n * g // 8 // 16 * 16, n * g // 8 // 16 * 16 + 48) for g in range(1, 8)]}[where]
    sel = np.zeros(n, bool)
    for a, b in runs:
        sel[a:b] = True
    return sel[:n_ref], sel[n_ref:]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("where", ["first tile", "after the first", "reference", "target", "eighths"])
@pytest.mark.parametrize("bias", [-3e38, -1e18, -1e9])
def test_masked_keys_add_nothing(shape, where, bias):
    """A reserved query dimension of 1e3 times a low key entry: the products overflow to -inf, or
    are finite scores far below (and spaced far wider than) all others."""
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape} {where} {bias}", flush=True)
    rng = np.random.default_rng(n_ref + n_tgt)
    x = {f"{k}_{s}": rng.standard_normal((B, H, n, D)).astype(np.float32)
         for s, n in (("ref", n_ref), ("tgt", n_tgt)) for k in "qkv"}
    for s, sel in zip(("ref", "tgt"), _keys(n_ref, n_tgt, where)):
        x[f"q_{s}"][..., 0] = 1e3
        x[f"k_{s}"][..., 0] = 0.0
        x[f"k_{s}"][:, :, sel, 0] = bias
    got = _run(x)
    kv = [x[k] for k in ("k_ref", "v_ref", "k_tgt", "v_tgt")]
    want, refq = joint_attention(x["q_tgt"], *kv), joint_attention(x["q_ref"], *kv)
    assert max_abs(host(got.o_tgt), want["o"]) <= O_TOL["f32"]
    assert max_abs(host(got.o_ref), refq["o"]) <= O_TOL["f32"]
    assert max_abs(host(got.ref_mass), want["ref_mass"]) <= MASS_TOL["f32"]
    assert max_abs(host(got.ref_mass_refq), refq["ref_mass"]) <= MASS_TOL["f32"]
    assert max_abs(host(got.lse)[..., 1], want["lse_all"]) <= 1e-5


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("size", [2.0 ** 26, 2.0 ** 34, 2.0 ** 100])
def test_scores_far_beyond_the_mantissa(shape, size):
    """Scores q0 k0 that differ by more than the exponent range: the output is the value of the
    largest, exactly, in whatever order the keys come and also where all scores are negative."""
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape} {size}", flush=True)
    rng = np.random.default_rng(7)
    n = n_ref + n_tgt
    x = {f"{k}_{s}": np.zeros((B, H, m, D), np.float32) for s, m in (("ref", n_ref), ("tgt", n_tgt)) for k in "qk"}
    v = rng.standard_normal((B, H, n, D)).astype(np.float32)
    k0 = np.stack([rng.permutation(n) for _ in range(B * H)]).reshape(B, H, n).astype(np.float32)
    k0 = (k0 + 1.0) * 2.0 ** -10  # 2^-10 apart: 2^16 / sqrt(D) in the score at the smallest size
    sign = np.where(np.arange(n) % 3 == 0, -1.0, 1.0)
    for s, lo, m in (("ref", 0, n_ref), ("tgt", n_ref, n_tgt)):
        x[f"v_{s}"], x[f"k_{s}"][..., 0] = v[:, :, lo:lo + m], k0[:, :, lo:lo + m]
        x[f"q_{s}"][..., 0] = size * sign[lo:lo + m]
    got = _run(x)
    top, low = k0.argmax(2), k0.argmin(2)
    for s, lo, m, o in (("ref", 0, n_ref, got.o_ref), ("tgt", n_ref, n_tgt, got.o_tgt)):
        pick = np.where(sign[lo:lo + m] > 0, top[..., None], low[..., None])
        assert np.array_equal(host(o), np.take_along_axis(v, pick[..., None], 2))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_subnormal_probabilities_reach_the_output(shape):
    """One key at score 0 and value 0, the rest at 2^-130 in probability and 1.5 * 2^127 in value.
    The score scale's and the exponent argument's roundings are 2^-24 of 130 each, a probability's
    2^-150 of 2^-130."""
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape}", flush=True)
    n = n_ref + n_tgt
    x = {}
    for s, lo, m in (("ref", 0, n_ref), ("tgt", n_ref, n_tgt)):
        for k in "qkv":
            x[f"{k}_{s}"] = np.zeros((B, H, m, D), np.float32)
        x[f"q_{s}"][..., 0] = 1.0
        x[f"k_{s}"][..., 0] = -130.0
        x[f"v_{s}"][..., :] = 1.5 * 2.0 ** 127 / n
    x["k_tgt"][:, :, 0, 0] = 0.0
    x["v_tgt"][:, :, 0] = 0.0
    got = _run(x, scale=float(np.log(2.0)))
    want = 1.5 * 2.0 ** -3 * (n - 1) / n
    bar = 4 * 130 * 2.0 ** -24 + 2.0 ** -20 + n * 2.0 ** -24
    for o in (got.o_tgt, got.o_ref):
        assert np.abs(host(o) / want - 1.0).max() <= bar


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("step", [0.0, 4.0, 7.9])
def test_the_largest_values_do_not_overflow(shape, step):
    """A last key `step` above the others in log2, whose value is 0.99 of the largest fp32 and
    theirs a thousandth over the number of keys: no partial sum may exceed the result by much."""
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape} {step}", flush=True)
    n = n_ref + n_tgt
    top = 0.99 * float(np.finfo(np.float32).max)
    x = {}
    for s, m in (("ref", n_ref), ("tgt", n_tgt)):
        for k in "qkv":
            x[f"{k}_{s}"] = np.zeros((B, H, m, D), np.float32)
        x[f"q_{s}"][..., 0] = 1.0
        x[f"v_{s}"][...] = top / n * 1e-3
    x["k_tgt"][:, :, -1, 0] = step
    x["v_tgt"][:, :, -1] = top
    got = _run(x, scale=float(np.log(2.0)))
    w = 2.0 ** step
    want = (w * top + (n - 1) * top / n * 1e-3) / (w + n - 1)
    bar = (n + 4 * 8) * 2.0 ** -24
    for o in (got.o_tgt, got.o_ref):
        assert np.abs(host(o) / want - 1.0).max() <= bar


def test_more_workgroups_than_one_grid_holds():
    """17 million heads of one key: each output row is its value row."""
    from paper_2609_32415_amd import ops

    H = 17_000_000
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1)
    q = torch.ones((1, H, 1, 64), device="cuda:0")
    v = torch.randn((1, H, 1, 64), generator=g, device="cuda:0")
    print("launch", flush=True)
    got = ops.joint_attn(q, q, v, ref_mass=True)
    torch.cuda.synchronize()
    assert torch.equal(got.o_tgt, v)
    assert not got.ref_mass.any()
