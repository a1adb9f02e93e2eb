"""D2Q9 extension sensors on rows of odd length: FP32 computes them with one cell
per thread; FP64 has no such kernel, and the call is refused with the context as
it was, however many steps it asks for."""
import numpy as np
import pytest
import torch

from paper_2603_13618_amd import inputs, lks

pytestmark = pytest.mark.gpu

EXT = ("kn", "alpha", "strain")


def _lattice(nx, ny, dtype, **kw):
    lat = lks.Lattice(9, nx, ny, dtype, tau=0.6, max_steps=9, ext=EXT, **kw)
    lat.init(*inputs.random_state((ny, nx), 5, (0.95, 1.05), 0.05))
    return lat


@pytest.mark.parametrize("nx,ny,vec", [(33, 29, 0), (97, 64, 0), (301, 40, 0), (64, 64, 1)])
def test_fp64_is_refused_before_any_step(nx, ny, vec):
    lat = _lattice(nx, ny, "f64", launch_vec=vec)
    lat.pop[1].fill_(7.0)
    lat.sums.fill_(3.0)
    before = [t.clone() for t in (lat.pop[0], lat.pop[1], lat.sums)]
    lat.step(0)
    for steps in (1, 2, 9):
        with pytest.raises(lks.LksError) as e:
            lat.step(steps)
        assert e.value.status == 3, steps            # LKS_EHIP
        assert lat.current() == (0, 0), steps
        torch.cuda.synchronize()
        for was, now in zip(before, (lat.pop[0], lat.pop[1], lat.sums)):
            assert torch.equal(was, now), steps
    with pytest.raises(lks.LksError):
        lat.step_from(lat.pop[0], lat.pop[1])
    torch.cuda.synchronize()
    assert torch.equal(lat.pop[1], before[1])


@pytest.mark.parametrize("nx,ny", [(33, 29), (97, 64), (563, 517)])
def test_fp32_steps_in_one_call_or_several(nx, ny):
    a, b = _lattice(nx, ny, "f32"), _lattice(nx, ny, "f32")
    a.step(9)
    for _ in range(9):
        b.step(1)
    torch.cuda.synchronize()
    assert a.current() == b.current() and a.check() == b.check()
    assert torch.equal(a.state, b.state) and torch.equal(a.flags, b.flags)
    assert torch.equal(a.sensors.view(torch.int32), b.sensors.view(torch.int32))
