"""Several D2Q9 steps of a tile per launch (the default) against one step per
launch (launch_steps = 1), through the C ABI.

Every cell's arithmetic is the same function of the same stored values, so
state, the state before the last step, sensors, flags, buffer index and fault
counts must be the same bits.  The per-step sums add each cell's FP64 terms in
another order: n terms of a sum of magnitudes A differ by at most n 2^-53 A;
the bar is 1e-12 of the mass for mass and momentum and 1e-12 relative for the
sensors' totals (n <= 3e5 cells, measured differences are near 1e-16).

Grid sides at the edges of the forms' ranges: a tile of T cells with a halo of
K wraps by at most one period.  8-cell tiles (K = 7) take 8 and 12 cells but not
7 or 9, 16-cell ones 12 and 20, 32-cell ones (K = 5) 19, 64-column bands (K = 3)
34 and 66 but not 33 or 65, 16-row bands 10 and 18 but not 17.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_13618_amd import inputs, lks

pytestmark = pytest.mark.gpu

THR = np.array([[1e-6, 1e-5], [1e-3, 3e-3], [1e-3, 2e-3], [np.inf, np.inf]])
GRIDS = [(7, 9), (8, 8), (9, 12), (12, 12), (16, 15), (20, 37), (37, 22), (66, 18), (129, 128), (257, 255),
         (300, 291), (301, 40), (40, 301), (34, 4100), (33, 4100), (65, 2100), (66, 2100), (4200, 10), (4200, 9),
         (4200, 17), (4200, 18), (19, 4000), (563, 517), (520, 1031), (131100, 20)]


def _pair(nx, ny, dtype, layout, max_steps, far=False, **kw):
    rho, ux, uy = inputs.random_state((ny, nx), nx + ny, (0.7, 1.3) if far else (0.95, 1.05), 0.2 if far else 0.05)
    out = []
    for ls in (0, 1):
        lat = lks.Lattice(9, nx, ny, dtype, tau=0.6, thr=THR, flag_mask=7, max_steps=max_steps, layout=layout,
                          launch_steps=ls, **kw)
        lat.init(rho, ux, uy)
        out.append(lat)
    return out


def _check(a, b):
    torch.cuda.synchronize()
    assert a.current() == b.current()
    cur = a.current()[0]
    for i in (cur, 1 - cur):
        x, y = a.pop[i].contiguous(), b.pop[i].contiguous()
        if x.element_size() == 2:
            x, y = x.view(torch.int16), y.view(torch.int16)
        assert torch.equal(x, y), "state" if i == cur else "state before the last step"
    assert torch.equal(a.sensors, b.sensors)
    assert torch.equal(a.flags, b.flags)
    assert a.check() == b.check()
    sa, sb = a.sums.cpu().numpy(), b.sums.cpu().numpy()
    assert np.abs(sa[:, :4] - sb[:, :4]).max() <= 1e-12 * np.abs(sb[:, 0]).max()
    np.testing.assert_allclose(sa[:, 4:], sb[:, 4:], rtol=1e-12)


@pytest.mark.parametrize("nx,ny", GRIDS)
@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16"])
def test_same_bits_as_one_step_per_launch(dtype, nx, ny):
    layout = "planes" if (nx + ny) % 2 else "rows"
    a, b = _pair(nx, ny, dtype, layout, 32)
    for steps in (1, 2, 10, 3, 7, 5):             # 28 in all; every remainder of 3, 5 and 7
        print("case", dtype, nx, ny, layout, steps, flush=True)
        a.step(steps)
        b.step(steps)
        _check(a, b)


@pytest.mark.parametrize("max_steps", [1, 2, 5])
@pytest.mark.parametrize("nx,ny", [(33, 29), (320, 257), (563, 517)])
def test_sums_ring_shorter_than_the_call(nx, ny, max_steps):
    # sums that a later step of the call overwrites are not kept on the way
    a, b = _pair(nx, ny, "f32", "rows", max_steps, far=True)
    for steps in (11, 4):
        a.step(steps)
        b.step(steps)
        _check(a, b)


@pytest.mark.parametrize("nt", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16"])
def test_states_beyond_the_cache(dtype, nt):
    # above 256 MB of state FP32 and FP64 run their single steps in the row kernel
    n = {"f32": 1900, "f64": 1340, "bf16": 2700}[dtype] + (64 if nt else -70)
    a, b = _pair(n, n + 3, dtype, "rows", 16)
    for steps in (8, 1, 3, 4):
        a.step(steps)
        b.step(steps)
        torch.cuda.synchronize()
        assert torch.equal(a.flags, b.flags) and torch.equal(a.sensors, b.sensors)
    _check(a, b)


def test_splitting_a_run_keeps_the_sums():
    for nx, ny in ((100, 90), (250, 250), (700, 333)):
        a, b = (_pair(nx, ny, "f32", "rows", 40)[0] for _ in range(2))
        a.step(40)
        for steps in (1, 13, 26):
            b.step(steps)
        torch.cuda.synchronize()
        assert torch.equal(a.sums, b.sums) and torch.equal(a.state, b.state)


@pytest.mark.parametrize("nx,ny", [(256, 256), (640, 512)])
def test_scratch_of_the_one_step_kernels_is_enough(nx, ny):
    a, b = _pair(nx, ny, "f32", "rows", 8)
    full = lks.scratch_bytes(a.cfg)
    one = lks.make_config(9, nx, ny, "f32", tau=0.6, max_steps=8, layout=lks.LAYOUT_ROWS, launch_steps=1)
    least = lks.scratch_bytes(one)
    assert least <= full
    buf = lks.Buffers.from_buffer_copy(a.buf)
    for nbytes, status in ((least, 0), (least - 1, 1)):
        buf.scratch_bytes = nbytes
        ctx = ctypes.c_void_p()
        got = lks.lib().lks_create(ctypes.byref(a.cfg), ctypes.byref(buf), lks._stream_handle(a.device),
                                   ctypes.byref(ctx))
        assert got == status
        if status == 0:
            lks._check(lks.lib().lks_restore(ctx, 0, 0), ctx)
            lks._check(lks.lib().lks_step(ctx, 8, 1), ctx)
            b.step(8)
            torch.cuda.synchronize()
            assert torch.equal(a.pop[0], b.pop[0]) and torch.equal(a.flags, b.flags)
            np.testing.assert_allclose(a.sums.cpu().numpy()[:, 4:], b.sums.cpu().numpy()[:, 4:], rtol=1e-12)
            lks.lib().lks_destroy(ctx)


def test_captured_graph_replays():
    nx, ny, steps = 300, 200, 9
    a, b = _pair(nx, ny, "f32", "rows", steps)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            cur = lks.step_noalloc(a.cfg, a.pop, a.sensors, a.flags, a.sums, 0, 0, steps)
    assert cur == steps % 2
    start = b.pop[0].clone()
    for _ in range(3):
        a.pop[0].copy_(start)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        b.restore(start, 0)
        b.step(steps)
        torch.cuda.synchronize()
        assert torch.equal(a.pop[cur], b.state) and torch.equal(a.sensors, b.sensors)
        assert torch.equal(a.flags, b.flags)
        np.testing.assert_allclose(a.sums.cpu().numpy()[:, 4:], b.sums.cpu().numpy()[:, 4:], rtol=1e-12)


def _same_outputs(a, b):
    torch.cuda.synchronize()
    assert a.current() == b.current()
    assert torch.equal(a.state, b.state)
    assert torch.equal(a.sensors.view(torch.int64 if a.sensors.dtype == torch.float64 else torch.int32),
                       b.sensors.view(torch.int64 if b.sensors.dtype == torch.float64 else torch.int32))
    assert torch.equal(a.flags, b.flags)
    assert a.check() == b.check()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny", [(40, 33), (300, 280), (564, 517)])
def test_extension_sensors_of_the_last_step(dtype, nx, ny):
    # computed in a call's last step only: the same bits as calls of one step
    rho, ux, uy = inputs.random_state((ny, nx), 5, (0.95, 1.05), 0.05)
    thr = np.full((lks.MAX_EXT, 2), np.inf)
    thr[lks.EXT_NAMES.index("kn")] = (1e-3, 1e-2)
    a, b = (lks.Lattice(9, nx, ny, dtype, tau=0.6, thr=THR, flag_mask=7 | lks.flag_x("kn"), max_steps=9,
                        ext=("kn", "alpha", "strain"), thr_ext=thr) for _ in range(2))
    for lat in (a, b):
        lat.init(rho, ux, uy)
    a.step(9)
    for _ in range(9):
        b.step(1)
    _same_outputs(a, b)


@pytest.mark.parametrize("ext", [None, ("kn", "qf")])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("model", ["bgk", "ddf"])
def test_d2q25_sensors_of_the_last_step(model, dtype, ext):
    nx, ny = 70, 45
    rho, ux, uy, T, states = inputs.riemann_quadrants(nx, ny, seed=2)
    dx = 1.0 / nx
    kw = dict(model="ddf", gamma=1.4, prandtl=0.71) if model == "ddf" else {}
    a, b = (lks.Lattice(25, nx, ny, dtype, mu=1e-3, dt=inputs.riemann_dt(states, dx), dx=dx, bc=(1, 1),
                        thr=[[1e-6, 1e-4]] + [[1e-4, 1e-3]] * 3, flag_mask=15, max_steps=6, ext=ext, **kw)
            for _ in range(2))
    for lat in (a, b):
        lat.init(rho, ux, uy, T)
    a.step(6)
    for _ in range(6):
        b.step(1)
    _same_outputs(a, b)
    np.testing.assert_allclose(a.sums.cpu().numpy(), b.sums.cpu().numpy(), rtol=1e-12, atol=1e-300)
