"""The grids whose D2Q9 steps run in the tile kernel, by the scratch that the
library asks for: several steps of a tile per launch need more partial sums than
one step per launch (launch_steps = 1) on these shapes, and the same where the
one-step kernels run."""
import pytest

from paper_2603_13618_amd import lks

# elements of the state that 32-bit indexes reach
CELLS = 2 ** 32 // 9


def _extra(nx, ny, dtype):
    """Bytes of scratch for the automatic launch shape beyond launch_steps = 1."""
    auto, one = (lks.scratch_bytes(lks.make_config(9, nx, ny, dtype, max_steps=16, launch_steps=ls))
                 for ls in (0, 1))
    assert auto >= one > 0
    return auto - one


@pytest.mark.parametrize("dtype", ["f32", "f64", "bf16", "f16"])
@pytest.mark.parametrize("nx", [8, 12, 20, 32, 33])
def test_grids_beyond_32_bit_indexes_run_one_step_kernels(dtype, nx):
    # too narrow for the 64-column bands; the tile kernel's indexes have 32 bits
    assert _extra(nx, 1_000_000, dtype) > 0
    for ny in (CELLS // nx + 1, 2 * CELLS // nx, 16 * CELLS // nx):
        assert _extra(nx, ny, dtype) == 0, ny
