"""How a run is split into calls changes no bit of it: one call of nine steps
against calls of one, two, five and one, on D2Q9 states beyond the 256 MB
last-level cache (where single steps have been run by another kernel than
several at a time) and in it."""
import numpy as np
import pytest
import torch

from paper_2603_13618_amd import inputs, lks

pytestmark = pytest.mark.gpu

THR = np.array([[1e-6, 1e-5], [1e-3, 3e-3], [1e-3, 2e-3], [np.inf, np.inf]])
CALLS = (1, 2, 5, 1)


def _pair(nx, ny, dtype, layout, **kw):
    fields = inputs.random_state((ny, nx), nx + ny, (0.95, 1.05), 0.05)
    out = []
    for _ in range(2):
        lat = lks.Lattice(9, nx, ny, dtype, tau=0.6, thr=THR, flag_mask=7, max_steps=sum(CALLS), layout=layout, **kw)
        lat.init(*fields)
        out.append(lat)
    return out


def _bits(t):
    return t.view({1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[t.element_size()])


def _run_and_compare(a, b):
    a.step(sum(CALLS))
    for steps in CALLS:
        b.step(steps)
    torch.cuda.synchronize()
    assert a.current() == b.current() and a.check() == b.check()
    for x, y in ((a.state, b.state), (a.sensors, b.sensors), (a.flags, b.flags), (a.sums, b.sums)):
        assert torch.equal(_bits(x), _bits(y))


# rows that are whole 64-byte pieces (non-temporal stores) and rows that are not
@pytest.mark.parametrize("dtype,nx,ny", [("f32", 1968, 1971), ("f32", 1964, 1971), ("f32", 1967, 1971),
                                         ("f64", 1408, 1411), ("f64", 1404, 1411), ("f64", 1407, 1411),
                                         ("bf16", 2784, 2787), ("f32", 700, 333)])
@pytest.mark.parametrize("layout", ["rows", "planes"])
def test_any_split_gives_the_same_bits(dtype, nx, ny, layout):
    _run_and_compare(*_pair(nx, ny, dtype, layout))


# the tile kernel's forms, the bands with two and three rows a wave, both stores
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("layout", ["rows", "planes"])
@pytest.mark.parametrize("nx,ny", [(40, 33), (150, 130), (300, 280), (700, 334), (1968, 1971), (4096, 772)])
def test_any_split_gives_the_same_bits_with_extension_sensors(dtype, nx, ny, layout):
    thr = np.full((lks.MAX_EXT, 2), np.inf)
    thr[lks.EXT_NAMES.index("kn")] = (1e-3, 1e-2)
    kw = dict(ext=("kn", "alpha", "strain"), thr_ext=thr)
    a, b = _pair(nx, ny, dtype, layout, **kw)
    _run_and_compare(a, b)
    row = _pair(nx, ny, dtype, layout, launch_steps=1, **kw)[0]      # the one-step kernel
    row.step(sum(CALLS))
    torch.cuda.synchronize()
    for x, y in ((a.state, row.state), (a.sensors, row.sensors), (a.flags, row.flags)):
        assert torch.equal(_bits(x), _bits(y))
