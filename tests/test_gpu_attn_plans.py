"""Plans of the bf16 attention across the K/V modes of one shape: a workspace made for one mode
serves the others, and a device-decided launch gives the bits of the explicit one."""

import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(B, H, D, n_ref, n_tgt):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n_ref)
    x = {f"{k}_{s}": torch.randn((B, H, n, D), generator=g, device="cuda:0").to(torch.bfloat16)
         for s, n in (("ref", n_ref), ("tgt", n_tgt), ("cache", n_ref)) for k in "qkv"}
    return x


def _run(x, mode, ws, **kw):
    from paper_2609_32415_amd import ops

    n_ref = x["k_ref"].shape[2]
    ref = dict(q_ref=x["q_ref"], k_ref=x["k_ref"], v_ref=x["v_ref"])
    cache = dict(k_cache=x["k_cache"], v_cache=x["v_cache"], q_cache=x["q_cache"])
    ends = [64, n_ref]
    args = {
        "reuse": dict(qset="target", kvsrc="cache", **cache),
        "fresh": dict(qset="all", kvsrc="fresh", **ref),
        "restore": dict(qset="all", kvsrc="cache", **cache),
        "segments": dict(qset="target", kvsrc="segments", seg_end=ends, seg_cache=[True, False], **ref, **cache),
        "seg_mass": dict(qset="target", kvsrc="segments", seg_end=ends, seg_cache=[True, False], seg_mass=True, **ref,
                         **cache),
        "device": dict(kvsrc="device", **ref, **cache),
    }[mode]
    return ops.joint_attn(x["q_tgt"], x["k_tgt"], x["v_tgt"], workspace=ws, **args, **kw)


def _workspace(x, mode):
    from paper_2609_32415_amd import ops

    qset = "all" if mode in ("fresh", "restore") else "target"
    src = {"reuse": "cache", "fresh": "fresh", "restore": "cache", "seg_mass": "segments"}.get(mode, mode)
    return ops.attn_workspace(x["q_tgt"], x["k_ref"].shape[2], qset, src, n_seg_mass=2 if mode == "seg_mass" else 0)


# Segments run 256-row tiles, the other modes 128-row ones in some of these; all queries whole and
# target queries in key chunks, all in chunks, and both.
SHAPES = [(2, 9, 128, 5339, 151), (1, 5, 128, 300, 3000), (1, 24, 128, 1024, 1024), (1, 8, 64, 2056, 1875),
          (1, 24, 64, 2106, 566), (1, 24, 128, 2378, 259)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("made_for", ["reuse", "segments", "seg_mass", "device"])
def test_a_workspace_of_the_target_queries_serves_every_mode(shape, made_for):
    x = _tensors(*shape)
    ws = _workspace(x, made_for)
    for mode in ("reuse", "segments", "seg_mass"):
        print(f"shape {shape} made for {made_for}, used by {mode}", flush=True)
        got = _run(x, mode, ws)
        # seg_mass alone needs more, and runs whole tiles with less
        want = _run(x, mode, ws if mode == "seg_mass" else _workspace(x, mode))
        assert torch.equal(got.o_tgt, want.o_tgt) and torch.equal(got.ref_mass, want.ref_mass)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_a_workspace_of_a_device_decided_launch_serves_the_explicit_ones(shape):
    x = _tensors(*shape)
    ws = _workspace(x, "device")
    for mode in ("reuse", "fresh", "restore", "segments"):
        print(f"shape {shape} used by {mode}", flush=True)
        got, want = _run(x, mode, ws), _run(x, mode, _workspace(x, mode))
        assert torch.equal(got.o_tgt, want.o_tgt) and torch.equal(got.ref_mass, want.ref_mass)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_a_workspace_that_holds_the_256_row_plan_is_enough(shape):
    """Down to the least size the launch takes it, on the workgroup size whose partials fit; less is
    refused."""
    from paper_2609_32415_amd import _lib as L

    B, H, D, n_ref, n_tgt = shape
    x = _tensors(*shape)
    whole = _run(x, "reuse", False)
    need = None
    try:
        _run(x, "reuse", torch.empty(16, dtype=torch.uint8, device="cuda:0"))
    except L.RefadaptError as e:
        assert e.status == L.RA_EWORKSPACE
        need = int(str(e).split("needs ")[1].split()[0])
    print(f"shape {shape} least workspace {need}", flush=True)
    if need is not None:
        got = _run(x, "reuse", torch.empty(need, dtype=torch.uint8, device="cuda:0"))
        assert (got.o_tgt.float() - whole.o_tgt.float()).abs().max() <= 1e-2
        with pytest.raises(L.RefadaptError):
            _run(x, "reuse", torch.empty(need - 16, dtype=torch.uint8, device="cuda:0"))


# rows per workgroup; tiles of all queries / of the target queries, whole or in key chunks
DEVICE_SHAPES = [
    (1, 24, 128, 882, 1549),   # 128, whole / whole
    (1, 3, 64, 773, 119),      # 128, whole / chunks
    (1, 1, 64, 861, 2114),     # 128, chunks / chunks
    (1, 24, 128, 2378, 259),   # 128, both / chunks
    (1, 16, 64, 118, 1929),    # 256, whole / whole
    (1, 12, 64, 1292, 1231),   # 256, whole / chunks
    (1, 1, 64, 1638, 1947),    # 256, chunks / chunks
    (1, 24, 64, 1847, 705),    # 256, both / chunks
]


@pytest.mark.parametrize("shape", DEVICE_SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("split", [True, False])
def test_a_device_decided_launch_gives_the_explicit_bits(shape, split):
    x = _tensors(*shape)
    ws = _workspace(x, "device") if split else False
    for decision, mode in ((0, "reuse"), (1, "restore"), (2, "fresh")):
        print(f"shape {shape} split {split} decision {decision}", flush=True)
        dec = torch.tensor([decision], dtype=torch.int32, device="cuda:0")
        o_ref = torch.full_like(x["q_ref"], 7.0)
        got = _run(x, "device", ws, decision=dec, o_ref=o_ref)
        want = _run(x, mode, _workspace(x, mode) if split else False)
        assert torch.equal(got.o_tgt, want.o_tgt) and torch.equal(got.ref_mass, want.ref_mass)
        assert torch.equal(got.o_ref, want.o_ref) if decision else bool((o_ref == 7.0).all())
