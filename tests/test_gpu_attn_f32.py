"""fp32 attention: every split of a launch (query subtiles per workgroup x key groups) at the
sizes where it can go wrong, against the fp64 oracle.

The split follows from (batch, heads, n_ref, n_tgt) on a 256-CU device; the shapes below reach
each one (named in the id, asserted by test_attn_plans.py) with row counts around the 16-row subtiles and key counts around the
16- and 32-key tiles, key groups without keys or without reference keys included."""

import numpy as np
import pytest
import torch

from gpu_helpers import MASS_TOL, O_TOL, dev, host, max_abs
from oracle import joint_attention

pytestmark = pytest.mark.gpu

# split (subtiles x groups), head_dim, B, H, n_ref, n_tgt
SHAPES = [
    ("1x4", 64, 1, 1, 1, 1),
    ("1x4", 128, 1, 2, 15, 17),
    ("1x4", 64, 2, 1, 0, 33),
    ("1x4", 128, 1, 3, 100, 16),
    ("1x8", 128, 1, 1, 16, 497),
    ("1x8", 64, 1, 2, 500, 15),
    ("1x8", 128, 2, 1, 1025, 31),
    ("2x2", 128, 1, 24, 33, 545),
    ("2x2", 64, 2, 48, 31, 129),
    ("2x2", 64, 1, 48, 1, 257),
    ("2x2", 128, 1, 128, 64, 128),
    ("4x1", 128, 2, 17, 74, 733),
    ("4x1", 64, 1, 128, 65, 128),
    ("4x1", 64, 1, 96, 65, 257),
    ("4x1", 128, 1, 80, 31, 320),
]


def _inputs(B, H, n_ref, n_tgt, D, seed):
    rng = np.random.default_rng(seed)
    return {f"{k}_{s}": rng.standard_normal((B, H, n, D)).astype(np.float32)
            for s, n in (("ref", n_ref), ("tgt", n_tgt), ("cache", n_ref)) for k in "qkv"}


def _check(x, qset, kvsrc, layout="bhsd"):
    from paper_2609_32415_amd import ops

    put = (lambda a: dev(a, "f32")) if layout == "bhsd" else (
        lambda a: dev(a.transpose(0, 2, 1, 3), "f32").transpose(1, 2))
    t = {k: put(v) for k, v in x.items()}
    n_ref = x["k_ref"].shape[2]
    cache = kvsrc == "cache"
    got = ops.joint_attn(t["q_tgt"], t["k_tgt"], t["v_tgt"], q_ref=t["q_ref"], k_ref=t["k_ref"], v_ref=t["v_ref"],
                         k_cache=t["k_cache"], v_cache=t["v_cache"], q_cache=t["q_cache"], n_ref=n_ref, qset=qset,
                         kvsrc=kvsrc, lse=True, ref_mass_refq=True)
    torch.cuda.synchronize()
    kv = (x["k_cache"], x["v_cache"]) if cache else (x["k_ref"], x["v_ref"])
    ref = joint_attention(x["q_tgt"], *kv, x["k_tgt"], x["v_tgt"])
    assert max_abs(host(got.o_tgt), ref["o"]) <= O_TOL["f32"]
    assert max_abs(host(got.ref_mass), ref["ref_mass"]) <= MASS_TOL["f32"]
    lse = host(got.lse)
    assert max_abs(lse[..., 1], ref["lse_all"]) <= 1e-5
    if n_ref:
        assert max_abs(lse[..., 0], ref["lse_ref"]) <= 1e-5
    if qset == "all" and n_ref:
        r = joint_attention(x["q_cache"] if cache else x["q_ref"], *kv, x["k_tgt"], x["v_tgt"])
        assert max_abs(host(got.o_ref), r["o"]) <= O_TOL["f32"]
        assert max_abs(host(got.ref_mass_refq), r["ref_mass"]) <= MASS_TOL["f32"]
    return got


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("qset,kvsrc,layout", [("target", "cache", "bhsd"), ("all", "fresh", "bshd")])
def test_every_split_matches_the_oracle(shape, qset, kvsrc, layout):
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape} {qset}/{kvsrc} {layout}", flush=True)
    _check(_inputs(B, H, n_ref, n_tgt, D, n_ref + n_tgt), qset, kvsrc, layout)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[4] > 0 and s[5] > 16][::2], ids=lambda s: "-".join(map(str, s)))
def test_target_rows_are_the_same_with_and_without_reference_queries(shape):
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape}", flush=True)
    x = _inputs(B, H, n_ref, n_tgt, D, 3)
    x["k_cache"], x["v_cache"] = x["k_ref"], x["v_ref"]
    a, b = _check(x, "target", "cache"), _check(x, "all", "fresh")
    assert torch.equal(a.o_tgt, b.o_tgt) and torch.equal(a.ref_mass, b.ref_mass) and torch.equal(a.lse, b.lse)


@pytest.mark.parametrize("shape", [("1x4", 64, 1, 1, 70, 90), ("1x8", 128, 1, 1, 400, 300), ("2x2", 128, 1, 24, 33, 545),
                                   ("4x1", 128, 2, 17, 74, 733)], ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("kind", ["ramp", "spikes"])
def test_running_max_moves(shape, kind):
    """Keys whose scores keep growing from tile to tile (the max moves by less than, and by more
    than, the step that rescales), and single keys far above all earlier ones."""
    _, D, B, H, n_ref, n_tgt = shape
    print(f"shape {shape} {kind}", flush=True)
    x = _inputs(B, H, n_ref, n_tgt, D, 11)
    n = n_ref + n_tgt
    u = np.zeros(D, dtype=np.float32)
    u[0] = 1.0
    gain = np.linspace(0.0, 60.0, n) if kind == "ramp" else np.where(np.arange(n) % 37 == 36, np.arange(n) * 90.0 / n, 0.0)
    for s, lo, m in (("ref", 0, n_ref), ("tgt", n_ref, n_tgt), ("cache", 0, n_ref)):
        x[f"k_{s}"] = x[f"k_{s}"] + (gain[lo:lo + m, None] * np.sqrt(D) * u).astype(np.float32)
        x[f"q_{s}"][..., 0] = np.where(np.arange(m) % 3 == 0, -1.0, 1.5)
    from paper_2609_32415_amd import ops

    t = {k: dev(v, "f32") for k, v in x.items()}
    got = ops.joint_attn(t["q_tgt"], t["k_tgt"], t["v_tgt"], q_ref=t["q_ref"], k_ref=t["k_ref"], v_ref=t["v_ref"],
                         qset="all", kvsrc="fresh", lse=True)
    torch.cuda.synchronize()
    ref = joint_attention(x["q_tgt"], x["k_ref"], x["v_ref"], x["k_tgt"], x["v_tgt"])
    refr = joint_attention(x["q_ref"], x["k_ref"], x["v_ref"], x["k_tgt"], x["v_tgt"])
    # A score of size up to 150 is a sum of D products, whose fp32 rounding is at most |s| 2^-24 per
    # addition where one product dominates, plus four roundings of that size (scaling, exponent
    # argument, the max it is taken against, the logarithm): the bound of an lse, and of the relative
    # error of a probability.
    bar = (D + 4) * 150 * 2.0 ** -24
    assert max_abs(host(got.o_tgt), ref["o"]) <= bar * np.abs(ref["o"]).max()
    assert max_abs(host(got.o_ref), refr["o"]) <= bar * np.abs(refr["o"]).max()
    assert max_abs(host(got.ref_mass), ref["ref_mass"]) <= bar
    assert max_abs(host(got.lse)[..., 1], ref["lse_all"]) <= bar


def test_a_dominant_infinite_or_nan_input_stays_in_its_own_rows():
    """A NaN query row gives a NaN output row and leaves the others as they were; an infinite
    value reaches only its own output column."""
    from paper_2609_32415_amd import ops

    x = _inputs(1, 2, 70, 90, 64, 5)
    run = lambda y: host(ops.joint_attn(dev(y["q_tgt"], "f32"), dev(y["k_tgt"], "f32"), dev(y["v_tgt"], "f32"),
                                        k_ref=dev(y["k_ref"], "f32"), v_ref=dev(y["v_ref"], "f32")).o_tgt)
    base = run(x)
    y = {k: v.copy() for k, v in x.items()}
    y["q_tgt"][0, 1, 17, 3] = np.nan
    got = run(y)
    assert np.isnan(got[0, 1, 17]).all()
    got[0, 1, 17] = base[0, 1, 17]
    assert np.array_equal(got, base)
    y = {k: v.copy() for k, v in x.items()}
    y["v_ref"][0, 0, 69, 5] = np.inf  # the last row of a ragged reference tile
    got = run(y)
    assert np.isposinf(got[0, 0, :, 5]).all()
    got[0, 0, :, 5] = base[0, 0, :, 5]
    assert np.array_equal(got, base)
