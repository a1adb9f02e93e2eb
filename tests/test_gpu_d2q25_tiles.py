"""FP64 single distribution on both of its workgroup tiles (32 x 2 up to 512
tiles of 32 x 4, else 32 x 4), whole and partial, against the FP64 oracle to
the bars of the FP64 parity tests (state 1e-12, sensors 1e-11, sums 1e-12 of
the mass)."""
import numpy as np
import pytest
import torch

from paper_2603_13618_amd import inputs, lks

from gpu_util import deviation, maxnorm, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
@pytest.mark.parametrize("nx,ny", [(256, 256), (257, 250), (256, 260), (288, 256), (290, 303)])
def test_fp64_tiles_match_oracle(orc, nx, ny, bc):
    rho, ux, uy, T, states = inputs.riemann_quadrants(nx, ny, seed=3)
    dx, steps = 1.0 / nx, 3
    dt = inputs.riemann_dt(states, dx)
    lat = lks.Lattice(25, nx, ny, "f64", mu=1e-3, dt=dt, dx=dx, bc=bc, max_steps=steps)
    lat.init(rho, ux, uy, T)
    lat.step(steps)
    torch.cuda.synchronize()
    ref = orc.run(25, orc.equilibrium(25, rho, ux, uy, T), steps, mu=1e-3, dt=dt, dx=dx, bc=bc)
    assert maxnorm(lat.state, deviation(ref["f"], 25)) <= 1e-12
    for k in range(4):
        assert maxnorm(lat.sensors[k], ref["sens"][k]) <= 1e-11, k
    assert np.abs(to_f64(lat.sums)[:, :4] - ref["sums"][:, :4]).max() <= 1e-12 * ref["sums"][0, 0]


@pytest.mark.parametrize("model,dtype", [("bgk", "f32"), ("bgk", "f64"), ("ddf", "f32"), ("ddf", "f64")])
@pytest.mark.parametrize("nx,ny", [(20, 3), (32, 4), (33, 5), (95, 41), (129, 66)])
def test_cells_of_moved_tiles_are_counted_once(model, dtype, nx, ny):
    # the last tile of a row or column is moved inside the grid: its cells'
    # faults, and the mass, must still be counted once
    kw = dict(model="ddf", gamma=1.4, prandtl=0.71) if model == "ddf" else {}
    lat = lks.Lattice(25, nx, ny, dtype, mu=1e-2, dt=1e-6, dx=0.1, **kw)
    rng = np.random.default_rng(nx * ny)
    lat.init(*inputs.random_state((ny, nx), 7, (0.9, 1.1), 0.05, (0.95, 1.05)))
    state = lat.pop[0].clone()
    bad = rng.random((ny, nx)) < 0.3
    bad[-1, -1] = bad[0, 0] = bad[-1, 0] = True
    state[0][torch.from_numpy(bad).to(state.device)] = -0.5      # f_0 = w_0 - 0.5 < 0
    lat.restore(state)
    lat.step(1)
    flags = lat.flags.cpu().numpy()
    assert lat.check() == int((flags >= 128).sum()) and (flags[bad] >= 128).all()
    mass = float(nx * ny + state[:25].double().sum())
    assert abs(float(lat.sums[0, 0]) - mass) <= 1e-6 * nx * ny * (1.0 if dtype == "f32" else 1e-6)
