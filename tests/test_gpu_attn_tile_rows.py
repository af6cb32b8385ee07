"""The two workgroup sizes of the bf16 attention (256 and 128 query rows). A launch of 128 heads
fills the device with 256-row tiles; the same heads four at a time leave it mostly idle and run
128-row ones (test_attn_plans.py asserts both on the CPU). Without key splits a row is summed in the same order in both, so the outputs are the
same bits; with them they agree with the oracle."""

import numpy as np
import pytest
import torch

from gpu_helpers import MASS_TOL, O_TOL, dev, host, max_abs
from oracle import joint_attention

pytestmark = pytest.mark.gpu


def _tensors(H, D, n_ref, n_tgt, kind, seed=3):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    x = {f"{k}_{s}": torch.randn((1, H, n, D), generator=g, device="cuda:0")
         for s, n in (("ref", n_ref), ("tgt", n_tgt)) for k in "qkv"}
    if kind == "spikes":  # keys that move the running max in later tiles, in either half of a tile
        for s in ("ref", "tgt"):
            x[f"k_{s}"][:, :, 70::97] *= 6.0
            x[f"k_{s}"][:, :, 40::211] *= 9.0
    return {k: v.to(torch.bfloat16) for k, v in x.items()}


def _run(x, h0, h1, qset, **kw):
    from paper_2609_32415_amd import ops

    t = {k: v[:, h0:h1] for k, v in x.items()}
    return ops.joint_attn(t["q_tgt"], t["k_tgt"], t["v_tgt"], q_ref=t["q_ref"], k_ref=t["k_ref"], v_ref=t["v_ref"],
                          qset=qset, kvsrc="fresh", lse=True, ref_mass_refq=True, **kw)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_ref,n_tgt", [(1003, 509), (769, 449), (1024, 512)])
@pytest.mark.parametrize("kind", ["plain", "spikes"])
def test_both_sizes_give_the_same_bits(D, n_ref, n_tgt, kind):
    print(f"D {D} n_ref {n_ref} n_tgt {n_tgt} {kind}", flush=True)
    x = _tensors(128, D, n_ref, n_tgt, kind)
    full = _run(x, 0, 128, "all", workspace=False)
    for h0 in (0, 124):
        part = _run(x, h0, h0 + 4, "all", workspace=False)
        for a, b in ((full.o_tgt, part.o_tgt), (full.o_ref, part.o_ref), (full.ref_mass, part.ref_mass),
                     (full.lse, part.lse), (full.ref_mass_refq, part.ref_mass_refq)):
            assert torch.equal(a[:, h0:h0 + 4], b)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,n_ref,n_tgt", [(1, 700, 1), (1, 640, 127), (2, 1000, 129), (3, 511, 385), (2, 64, 64)])
def test_small_launches_against_the_oracle(D, H, n_ref, n_tgt):
    print(f"D {D} H {H} n_ref {n_ref} n_tgt {n_tgt}", flush=True)
    x = _tensors(H, D, n_ref, n_tgt, "spikes", seed=n_ref)
    got = _run(x, 0, H, "all")
    torch.cuda.synchronize()
    y = {k: host(v) for k, v in x.items()}
    for q, o, m in (("q_tgt", got.o_tgt, got.ref_mass), ("q_ref", got.o_ref, got.ref_mass_refq)):
        ref = joint_attention(y[q], y["k_ref"], y["v_ref"], y["k_tgt"], y["v_tgt"])
        # outputs reach the size of a value where one key dominates: bf16 rounds them by 2^-9 of it
        assert max_abs(host(o), ref["o"]) <= O_TOL["bf16"] + 2.0 ** -8 * np.abs(ref["o"]).max()
        assert max_abs(host(m), ref["ref_mass"]) <= MASS_TOL["bf16"]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,n_ref,n_tgt,split", [(2, 700, 300, False), (2, 700, 300, True), (128, 769, 449, False),
                                                 (5, 300, 15360, True)])
@pytest.mark.parametrize("kind", ["plain", "spikes"])
def test_rows_without_mass_keep_their_outputs(D, H, n_ref, n_tgt, kind, split):
    """Rows that want neither mass nor log-sum-exp take the loop without the fp32 row sums: the same
    bits, on whole and split tiles of 128 rows, whole ones of 256 (128 heads), and both whole and
    split ones of 256 (5 heads)."""
    from paper_2609_32415_amd import ops

    print(f"D {D} H {H} n_ref {n_ref} n_tgt {n_tgt} {kind} split {split}", flush=True)
    x = _tensors(H, D, n_ref, n_tgt, kind)
    ws = ops.attn_workspace(x["q_tgt"], n_ref, "all", "fresh") if split else False
    assert (ws is not False) == split
    kw = dict(q_ref=x["q_ref"], k_ref=x["k_ref"], v_ref=x["v_ref"], qset="all", kvsrc="fresh", workspace=ws)
    run = lambda **f: ops.joint_attn(x["q_tgt"], x["k_tgt"], x["v_tgt"], **kw, **f)
    all_ = run(ref_mass=True, lse=True, ref_mass_refq=True)
    tgt = run(ref_mass=True, lse=True)
    none = run(ref_mass=False)
    lse = run(ref_mass=False, lse=True)
    torch.cuda.synchronize()
    for got in (tgt, none, lse):
        for a, b in ((all_.o_tgt, got.o_tgt), (all_.o_ref, got.o_ref)):
            assert torch.equal(a, b)
    assert torch.equal(all_.ref_mass, tgt.ref_mass)
    assert torch.equal(all_.lse, tgt.lse) and torch.equal(all_.lse, lse.lse)
    assert none.ref_mass is None and none.lse is None


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("decision", [0, 1, 2])
def test_device_decided_rows_without_mass(D, decision):
    from paper_2609_32415_amd import ops

    x = _tensors(24, D, 1100, 700, "plain")
    c = {k: (v.float() * 1.03).to(torch.bfloat16) for k, v in x.items() if k.endswith("ref")}
    print(f"D {D} decision {decision}", flush=True)
    dec = torch.tensor([decision], dtype=torch.int32, device="cuda:0")
    got = ops.joint_attn(x["q_tgt"], x["k_tgt"], x["v_tgt"], q_ref=x["q_ref"], k_ref=x["k_ref"], v_ref=x["v_ref"],
                         k_cache=c["k_ref"], v_cache=c["v_ref"], q_cache=c["q_ref"], kvsrc="device", decision=dec)
    src = x if decision == 2 else c
    want = ops.joint_attn(x["q_tgt"], x["k_tgt"], x["v_tgt"], q_ref=src["q_ref"], k_ref=src["k_ref"],
                          v_ref=src["v_ref"], qset="all", kvsrc="fresh", ref_mass_refq=True, workspace=False)
    torch.cuda.synchronize()
    bar = 2.0 ** -8
    assert max_abs(host(got.o_tgt), host(want.o_tgt)) <= bar * float(want.o_tgt.float().abs().max())
    assert max_abs(host(got.ref_mass), host(want.ref_mass)) <= 1e-5
    if decision:
        assert max_abs(host(got.o_ref), host(want.o_ref)) <= bar * float(want.o_ref.float().abs().max())
