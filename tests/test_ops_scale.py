"""The softmax scale of joint_attn: whatever float() takes reaches the C structure as that number
(on CPU tensors posing as device ones, with the C call noted instead of made)."""

from decimal import Decimal
from fractions import Fraction

import numpy as np
import pytest
import torch

from paper_2609_32415_amd import _lib as L
from paper_2609_32415_amd import ops


class _Posing(torch.Tensor):
    is_cuda = True


@pytest.mark.parametrize("scale,want", [
    (None, 0.0), (0, 0.0), (0.125, 0.125), (2, 2.0), ("0.25", 0.25), (Decimal("0.5"), 0.5), (Fraction(3, 4), 0.75),
    (np.float32(0.375), 0.375), (np.array(0.625), 0.625), (torch.tensor(0.875), 0.875), (-1.0, -1.0),
    (1e39, float("inf")),
])
def test_scale_reaches_the_structure(monkeypatch, scale, want):
    seen = []
    monkeypatch.setattr(L, "refadapt_joint_attn_packed", lambda desc, args, stream: seen.append(L.DESC_PACK.unpack(desc)))
    monkeypatch.setattr(ops, "_stream", lambda: 0)
    x = torch.zeros((1, 2, 8, 64), dtype=torch.bfloat16).as_subclass(_Posing)
    ops.joint_attn(x, x, x, scale=scale, o_tgt=x, ref_mass=False, workspace=False)
    assert seen[0][:6] == (1, 2, 64, 0, 8, L.RA_BF16) and seen[0][6] == want
