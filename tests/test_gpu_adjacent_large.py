"""The exposure change over more blocks than one grid holds a wavefront for, and over several
rounds of blocks per workgroup."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,nb", [(2, 67_200_000), (3, (1 << 20) + 1), (66, (1 << 20) + 3)])
def test_adjacent_change_of_many_blocks(T, nb):
    from paper_2609_32415_amd import ops

    print(f"T {T} nb {nb}", flush=True)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(nb)
    m = torch.rand((T, nb, 1), generator=g, device="cuda:0")
    got = ops.adjacent_mass_change(m)
    d = m[..., 0].double()
    want = 100.0 * (d[1:] - d[:-1]).abs().mean(0)
    # fp64 inside, in step order, and one rounding of the result
    assert bool(((got.double() - want).abs() <= want * 2.0 ** -23).all())
