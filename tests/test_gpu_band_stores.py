"""The 64-column bands with non-temporal stores (states beyond the 256 MB
last-level cache whose rows are whole 64-byte pieces), with two and three rows a
wave, against one step per launch: the same arithmetic on the same values, so
the same bits."""
import numpy as np
import pytest
import torch

from paper_2603_13618_amd import inputs, lks

pytestmark = pytest.mark.gpu

THR = np.array([[1e-6, 1e-5], [1e-3, 3e-3], [1e-3, 2e-3], [np.inf, np.inf]])


# 2048 tiles of 64 x 24 cells and more take three rows a wave (4096 x 772, 4096 x 960)
@pytest.mark.parametrize("dtype,nx,ny", [("f32", 1968, 1971), ("f32", 4096, 960), ("f64", 1408, 1411),
                                         ("f64", 4096, 772), ("bf16", 2784, 2787), ("f16", 2784, 2789)])
@pytest.mark.parametrize("layout", ["rows", "planes"])
def test_same_bits_as_one_step_per_launch(dtype, nx, ny, layout):
    fields = inputs.random_state((ny, nx), nx + ny, (0.95, 1.05), 0.05)
    lats = []
    for ls in (0, 1):
        lat = lks.Lattice(9, nx, ny, dtype, tau=0.6, thr=THR, flag_mask=7, max_steps=16, layout=layout,
                          launch_steps=ls)
        lat.init(*fields)
        lats.append(lat)
    a, b = lats
    item = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}
    for steps in (1, 4, 7, 2):
        print("case", dtype, nx, ny, layout, steps, flush=True)
        a.step(steps)
        b.step(steps)
        torch.cuda.synchronize()
        assert a.current() == b.current()
        for x, y in ((a.pop[0], b.pop[0]), (a.pop[1], b.pop[1]), (a.sensors, b.sensors), (a.flags, b.flags)):
            assert torch.equal(x.view(item[x.element_size()]), y.view(item[y.element_size()])), steps
    assert a.check() == b.check()
    sa, sb = a.sums.cpu().numpy()[:14], b.sums.cpu().numpy()[:14]
    # n terms in another order: within n 2^-53 of the sum of magnitudes
    n = nx * ny
    assert np.abs(sa[:, :4] - sb[:, :4]).max() <= n * 2.0 ** -53 * n * 1.5
    assert (np.abs(sa[:, 4:] - sb[:, 4:]) <= n * 2.0 ** -53 * sb[:, 4:]).all()
