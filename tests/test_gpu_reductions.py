"""Small reductions at the edges of their batches: the adjacent exposure change around the 64 steps
a wavefront takes at once, and the second passes of the pair and Q-change statistics around the
records a thread stages at once and the heads a workgroup takes, against fp64."""

import numpy as np
import pytest
import torch

from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [2, 7, 63, 64, 65, 128, 130])
@pytest.mark.parametrize("nb,bh", [(1, 1), (3, 24), (61, 7), (2, 100)])
def test_adjacent_change(T, nb, bh):
    from paper_2609_32415_amd import ops

    m = np.random.default_rng(T * 1000 + bh).uniform(0.05, 0.65, (T, nb, bh)).astype(np.float32)
    print(f"T {T} nb {nb} bh {bh}", flush=True)
    got = host(ops.adjacent_mass_change(dev(m, "f32")))
    want = 100.0 * np.abs(np.diff(m.astype(np.float64).mean(2), axis=0)).mean(0)
    np.testing.assert_allclose(got, want, rtol=2.0 ** -23)  # fp64 inside, one rounding of the result


# rows -> chunks per head at head_dim 128: 1 -> 1, 48 -> 3, 300 -> 8, 4096 -> 32, 9000 -> 64
@pytest.mark.parametrize("H", [1, 31, 32, 33, 65])
@pytest.mark.parametrize("n", [1, 48, 300, 4096, 9000])
def test_second_passes(H, n):
    from paper_2609_32415_amd import ops

    g = torch.Generator(device="cuda:0")
    g.manual_seed(n + H)
    print(f"H {H} n {n}", flush=True)
    a, b = (torch.randn((1, H, n, 128), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    mass = torch.rand((1, H, n), generator=g, device="cuda:0")
    norm = lambda x: x.double().square().sum((2, 3)).sqrt()
    ab, ba = norm(a.double() - b.double()) / norm(b), norm(b.double() - a.double()) / norm(a)
    theta = torch.full((1,), float("inf"), device="cuda:0")
    d, _, scores = ops.q_change_gate(a, b, mass, theta, ops.new_gate_state("cuda:0"), 0, 1)
    # a term passes at most 128 fp32 additions (9000 rows: 71 in its thread, 10 across threads)
    rtol = 128 * 2.0 ** -24
    np.testing.assert_allclose(host(d), host(ab), rtol=rtol)
    np.testing.assert_allclose(host(ops.q_change(a, b)), host(ab), rtol=rtol)
    m = mass.double().mean(-1)
    np.testing.assert_allclose(host(scores), [float(ab.mean()), float(m.mean()), float((ab * m).mean())], rtol=rtol)
    d_r, d_t, rho = ops.drift_log_ratio(a, b, b, a)
    np.testing.assert_allclose(host(d_r), host(ab), rtol=rtol)
    np.testing.assert_allclose(host(d_t), host(ba), rtol=rtol)
    np.testing.assert_allclose(host(rho), host((ab / ba).log10()), atol=rtol)
    # slices of different lengths share a launch: the shorter one's records are padded
    if n > 1:
        s = n // 2
        d_r, d_t, _ = ops.drift_log_ratio(a, b, b[:, :, :s], a[:, :, :s])
        np.testing.assert_allclose(host(d_r), host(ab), rtol=rtol)
        np.testing.assert_allclose(host(d_t), host(norm(b[:, :, :s].double() - a[:, :, :s].double()) / norm(a[:, :, :s])), rtol=rtol)


@pytest.mark.parametrize("H,n,d", [(8192, 4, 64), (1025, 40, 64), (33, 7000, 128), (2, 256, 64), (3, 9, 128), (5, 145, 128)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_gate_final_rounds(H, n, d, dtype):
    """Heads around the rounds of the gate's one workgroup (as many as its threads or its staged
    records allow, up to the most heads the gate takes), and slices of one to eight small chunks."""
    from paper_2609_32415_amd import ops

    g = torch.Generator(device="cuda:0")
    g.manual_seed(H + n)
    print(f"H {H} n {n} d {d} {dtype}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    a, b = (torch.randn((1, H, n, d), generator=g, device="cuda:0").to(dt) for _ in range(2))
    mass = torch.rand((1, H, n), generator=g, device="cuda:0")
    theta = torch.full((1,), float("inf"), device="cuda:0")
    got, _, scores = ops.q_change_gate(a, b, mass, theta, ops.new_gate_state("cuda:0"), 0, 1)
    norm = lambda x: x.double().square().sum((2, 3)).sqrt()
    want, m = norm(a.double() - b.double()) / norm(b), mass.double().mean(-1)
    rtol = 128 * 2.0 ** -24  # as above
    np.testing.assert_allclose(host(got), host(want), rtol=rtol)
    np.testing.assert_allclose(host(scores), [float(want.mean()), float(m.mean()), float((want * m).mean())], rtol=rtol)
