"""The controller writes its decisions, scores and ages through views of its logs: where a caller
puts slices of larger tensors in their place, each word still goes to its own cell (on the CPU, with
the entry points replaced by ones that note the words they are given)."""

import pytest
import torch

from paper_2609_32415_amd import controller as C


class _Ops:
    """Stands in for ops: marks the words it is given."""

    def q_change_gate_workspace(self, q):
        return None

    def attn_workspace(self, *a, **k):
        return False

    def new_gate_state(self, device, delta_max=0):
        return torch.zeros(4, dtype=torch.int32)

    def q_change_gate(self, q, q_prev, mass, theta, state, b, t, mode, eps, d_out, decision_out, score_out, workspace):
        decision_out.fill_(100 * t + b)
        score_out.copy_(torch.tensor([1.0, 2.0, 3.0]) + 10 * (100 * t + b))
        d_out.fill_(100 * t + b)

    def joint_attn(self, *a, **k):
        pass

    def cache_commit(self, *a, age=None, step=None, **k):
        age.fill_(1000 + step)


@pytest.mark.parametrize("views", ["own", "rows", "strided"])
def test_words_go_to_their_own_cells(monkeypatch, views):
    monkeypatch.setattr(C, "ops", _Ops())
    T, nb, B, H = 3, 4, 1, 2
    ctl = C.Controller(nb, T, B, H, 8, 8, 64, 0.1, dtype=torch.float32, device="cpu")
    big = None
    if views != "own":
        big = [torch.full((5, T + 2, nb + 3), -7, dtype=torch.int32), torch.full((5, T + 2, nb + 3, 3), -7.0),
               torch.full((5, nb + 3), -7, dtype=torch.int32)]
        t0, b0 = (0, 0) if views == "rows" else (1, 2)
        ctl.decisions = big[0][2, t0:t0 + T, b0:b0 + nb]
        ctl.scores = big[1][2, t0:t0 + T, b0:b0 + nb]
        ctl.age = big[2][2, b0:b0 + nb]
    x = [{f"{k}_{s}": torch.zeros((B, H, 8, 64)) for k in "qkv" for s in ("ref", "tgt")} for _ in range(nb)]
    for t in range(T):
        ctl.step(t, x)
    cells = 100 * torch.arange(T)[:, None] + torch.arange(nb)
    assert torch.equal(ctl.decisions.long(), cells)
    assert torch.equal(ctl.scores, 10.0 * cells[..., None] + torch.tensor([1.0, 2.0, 3.0]))
    assert ctl.age.tolist() == [1000 + T - 1] * nb
    assert torch.equal(ctl.d, cells[-1].float()[:, None, None].expand(nb, B, H))
    if big is not None:  # nothing beside them
        assert int((big[0] == -7).sum()) == big[0].numel() - T * nb
        assert int((big[1] == -7).sum()) == big[1].numel() - 3 * T * nb
        assert int((big[2] == -7).sum()) == big[2].numel() - nb


@pytest.mark.parametrize("t,b", [(3, 0), (-1, 0), (0, -1), (0, 4)])
def test_steps_and_blocks_outside_the_trajectory_are_refused(monkeypatch, t, b):
    monkeypatch.setattr(C, "ops", _Ops())
    ctl = C.Controller(4, 3, 1, 2, 8, 8, 64, 0.1, dtype=torch.float32, device="cpu")
    x = {f"{k}_{s}": torch.zeros((1, 2, 8, 64)) for k in "qkv" for s in ("ref", "tgt")}
    with pytest.raises(IndexError):
        ctl.block(t, b, x)
    assert bool((ctl.decisions == -1).all())
