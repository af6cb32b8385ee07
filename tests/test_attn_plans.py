"""Host check of the attention's work decomposition: compiles tests/plan_check.cpp against the
kernels' plan header and asserts which kernel variant each shape of the GPU tests takes on a
256-CU device, so that a test of one variant cannot come to run another unnoticed."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_32415_amd", "csrc")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    cc = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
    if cc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    src = os.path.join(ROOT, "tests", "plan_check.cpp")
    r = subprocess.run([cc, "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", CSRC, src, "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr

    def ask(lines):
        text = "".join(" ".join(map(str, x)) + "\n" for x in lines)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0
        return r.stdout.splitlines()

    return ask


def _bf16(plans, shapes):
    """Per shape (B, H, D, n_ref, n_tgt): the plan of all queries and that of the target queries."""
    keys = ("bm", "whole", "split", "chunks", "ws", "seg_ws", "bm_whole")
    out = []
    for line in plans([("bf16", *s) for s in shapes]):
        v = list(map(int, line.split()))
        out.append((dict(zip(keys, v[:7])), dict(zip(keys, v[7:]))))
    assert len(out) == len(shapes)
    return out


def test_fp32_shapes_take_the_split_their_name_says(plans):
    import test_gpu_attn_f32
    import test_gpu_attn_f32_range

    shapes = [*test_gpu_attn_f32.SHAPES, *test_gpu_attn_f32_range.SHAPES]
    # the shapes of the moving max carry their split too
    shapes += [("1x4", 64, 1, 1, 70, 90), ("1x8", 128, 1, 1, 400, 300), ("2x2", 128, 1, 24, 33, 545),
               ("4x1", 128, 2, 17, 74, 733)]
    got = plans([("f32", B, H, D, nr, nt) for _, D, B, H, nr, nt in shapes])
    assert got == [s[0] for s in shapes]


def test_tile_row_shapes_take_both_workgroup_sizes(plans):
    """Without key splits 128 heads fill the device with 256-row tiles, four leave it to 128-row ones."""
    for D in (64, 128):
        for nr, nt in ((1003, 509), (769, 449), (1024, 512)):
            full, part = _bf16(plans, [(1, 128, D, nr, nt), (1, 4, D, nr, nt)])
            assert full[0]["bm_whole"] == 256 and part[0]["bm_whole"] == 128
        small = _bf16(plans, [(1, H, D, nr, nt) for H, nr, nt in
                              ((1, 700, 1), (1, 640, 127), (2, 1000, 129), (3, 511, 385), (2, 64, 64))])
        assert all(p[0]["bm"] == 128 for p in small)


def test_bare_row_shapes(plans):
    """Rows without mass: split 128-row tiles, whole 256-row tiles, and 256-row tiles both whole and
    split (the shape of test_gpu_attn_rows_without_mass)."""
    import test_gpu_attn_rows_without_mass as t

    p = _bf16(plans, [(1, *s) for s in t.SHAPES])
    kinds = {(s[1], q["bm"], q["whole"] > 0, q["split"] > 0) for s, (q, _) in zip(t.SHAPES, p)}
    assert {(64, 256, True, True), (128, 256, True, True), (64, 128, False, True), (128, 128, False, True),
            (128, 256, True, False)} <= kinds


def test_device_shapes_take_every_pair_of_plans(plans):
    import test_gpu_attn_plans as t

    p = _bf16(plans, t.DEVICE_SHAPES)
    assert all(a["bm"] == y["bm"] for a, y in p)  # one workgroup size for both query sets
    kinds = [(a["bm"], a["whole"] > 0, a["split"] > 0, y["whole"] > 0, y["split"] > 0) for a, y in p]
    assert kinds == [(bm, *k) for bm in (128, 256) for k in
                     ((True, False, True, False), (True, False, False, True), (False, True, False, True),
                      (True, True, False, True))]


@pytest.mark.parametrize("D", [64, 128])
def test_workspaces_hold_every_plan_and_grow_with_segments(plans, D):
    """Over a spread of shapes: the workspace asked for holds the split items of the chosen plan,
    and per-segment masses ask for more exactly where 256-row tiles are split."""
    shapes = [(B, H, D, nr, nt) for B in (1, 2) for H in (1, 3, 9, 24) for nr in (64, 300, 1003, 5339, 12544)
              for nt in (64, 151, 1024, 4096)]
    for s, sets in zip(shapes, _bf16(plans, shapes)):
        for p in sets:
            items = p["split"] * p["chunks"]
            assert p["ws"] >= (items * p["bm"] * (D + 5) * 4 if p["split"] else 0), s
            assert p["seg_ws"] == 0 or p["seg_ws"] > p["ws"], s
            if p["bm"] == 256 and p["split"]:
                assert p["seg_ws"] == p["ws"] + items * 256 * 3 * 4, s
