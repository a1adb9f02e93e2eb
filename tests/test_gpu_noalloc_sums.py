"""lks_step_noalloc against lks_step where the library's own array holds the
partial sums of fewer steps than a launch on tiles takes, or of none: the same
bits, sums included."""
import pytest
import torch

from paper_2603_13618_amd import lks

pytestmark = pytest.mark.gpu


# 8 x 8 (nx = 8) and 16 x 16 tiles of up to 7 steps; the array holds the sums of
# 262,140 tile steps: 6, 5, 2, 1 and no steps of these
@pytest.mark.parametrize("nx,tile,tiles", [(8, 8, 40000), (12, 16, 50000), (8, 8, 90000), (8, 8, 200000),
                                           (8, 8, 262200)])
def test_sums_are_those_of_step(nx, tile, tiles):
    ny = tile * tiles - 3
    print("case", nx, ny, flush=True)
    a, b = (lks.Lattice(9, nx, ny, "f32", tau=0.6, max_steps=16, layout="planes") for _ in range(2))
    g = torch.Generator(device=a.device).manual_seed(tiles)
    w = torch.tensor([1 / 36, 1 / 9, 1 / 36, 1 / 9, 4 / 9, 1 / 9, 1 / 36, 1 / 9, 1 / 36], device=a.device)
    state = w[:, None, None] * 0.02 * (torch.rand(9, ny, nx, device=a.device, generator=g) - 0.5)
    for lat in (a, b):
        lat.restore(state)
    a.step(9)
    cur = lks.step_noalloc(b.cfg, b.pop, b.sensors, b.flags, b.sums, 0, 0, 9)
    torch.cuda.synchronize()
    assert cur == a.current()[0]
    assert torch.equal(a.state, b.pop[cur])
    assert torch.equal(a.sensors, b.sensors) and torch.equal(a.flags, b.flags)
    assert torch.equal(a.sums, b.sums)
