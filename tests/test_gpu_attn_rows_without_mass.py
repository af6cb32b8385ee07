"""bf16 attention outputs are the same bits whether mass and log-sum-exp are asked for or not: rows
that want neither take a key loop without the fp32 row sums, which has to move the running max at
the same tiles. Launches of 128-row tiles in key chunks, of whole 256-row tiles, and of both."""

import pytest
import torch

from gpu_helpers import O_TOL, host, max_abs
from oracle import joint_attention

pytestmark = pytest.mark.gpu

SHAPES = [(2, 64, 700, 300), (2, 128, 700, 300), (5, 64, 300, 15360), (5, 128, 300, 15360), (128, 128, 769, 449)]


def _tensors(H, D, n_ref, n_tgt, kind):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n_ref)
    x = {f"{k}_{s}": torch.randn((1, H, n, D), generator=g, device="cuda:0")
         for s, n in (("ref", n_ref), ("tgt", n_tgt)) for k in "qkv"}
    if kind == "spikes":
        for s in ("ref", "tgt"):
            x[f"k_{s}"][:, :, 70::97] *= 6.0
            x[f"k_{s}"][:, :, 40::211] *= 9.0
    if kind == "ramp":
        # scores that grow by 0.3 to 0.9 in log2 per 64 keys, by a rate of the row's 32-row group: the
        # sums of a tile's probabilities cross their bound over and over, in any part of a tile
        for s, lo, n in (("ref", 0, n_ref), ("tgt", n_ref, n_tgt)):
            rate = 0.5 + torch.arange(n, device="cuda:0") // 32 % 7 / 6.0
            up = 0.6 * torch.arange(lo, lo + n, device="cuda:0") / 64.0
            x[f"q_{s}"][..., 0] = rate
            x[f"k_{s}"][..., 0] = up % 100.0 * D ** 0.5 * 0.6931
    return {k: v.to(torch.bfloat16) for k, v in x.items()}


@pytest.mark.parametrize("H,D,n_ref,n_tgt", SHAPES)
@pytest.mark.parametrize("kind", ["plain", "spikes", "ramp"])
@pytest.mark.parametrize("split", [True, False])
def test_outputs_do_not_depend_on_what_else_is_asked_for(H, D, n_ref, n_tgt, kind, split):
    from paper_2609_32415_amd import ops

    print(f"H {H} D {D} n_ref {n_ref} n_tgt {n_tgt} {kind} split {split}", flush=True)
    x = _tensors(H, D, n_ref, n_tgt, kind)
    ws = ops.attn_workspace(x["q_tgt"], n_ref, "all", "fresh") if split else False
    assert not split or (ws is not False) == (H < 100)  # 128 heads split nothing
    run = lambda **f: ops.joint_attn(x["q_tgt"], x["k_tgt"], x["v_tgt"], q_ref=x["q_ref"], k_ref=x["k_ref"],
                                     v_ref=x["v_ref"], qset="all", kvsrc="fresh", workspace=ws, **f)
    full = run(ref_mass=True, lse=True, ref_mass_refq=True)
    for asked in (dict(ref_mass=False), dict(ref_mass=True), dict(ref_mass=False, lse=True),
                  dict(ref_mass=False, ref_mass_refq=True)):
        got = run(**asked)
        assert torch.equal(got.o_tgt, full.o_tgt) and torch.equal(got.o_ref, full.o_ref), asked
        for name in ("ref_mass", "lse", "ref_mass_refq"):
            t = getattr(got, name)
            assert t is None or torch.equal(t, getattr(full, name)), (asked, name)
    # the last rows of each set against the oracle: 2^-8 of the largest output for a dominant value
    y = {k: host(v[:, :1]) for k, v in x.items()}
    for s, o in (("ref", full.o_ref), ("tgt", full.o_tgt)):
        want = joint_attention(y[f"q_{s}"][:, :, -200:], y["k_ref"], y["v_ref"], y["k_tgt"], y["v_tgt"])["o"]
        assert max_abs(host(o[:, :1, -200:]), want) <= O_TOL["bf16"] + 2.0 ** -8 * abs(want).max()
