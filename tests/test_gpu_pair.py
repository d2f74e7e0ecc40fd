"""The kernels that take two plain steps per launch (pair_step_kernel in strips
and chunks, pair_tile_kernel in tiles) against
one launch per step, through the C ABI: the states bitwise the same."""
import sys

import numpy as np
import pytest

from paper_1412_6238_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbe():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1412_6238_amd import lbe_csf
    return lbe_csf


# grids around the strips of 56 columns and chunks of few rows: one strip, one
# column past it, strips of unequal width, chunks of one row, a last chunk that
# ends next to the top wall, chunks whose cones reach a wall from the rows
# before, a grid narrower than a strip's margin, periodic in y
CASES = [(3, 8, 1, 1), (7, 9, 0, 4), (56, 12, 1, 5), (57, 13, 1, 4), (113, 16, 0, 7),
         (64, 10, 1, 9), (200, 31, 1, 3), (130, 40, 1, 40), (300, 25, 0, 12), (1030, 11, 1, 2)]
# ... and around the tiles of 2, 4 or 8 rows: a last tile of one row, tiles
# whose margin reaches the wall, a periodic grid shorter than tile and margin
TILES = [(3, 8, 1, 4), (7, 9, 0, 4), (40, 100, 1, 2), (56, 12, 1, 8), (57, 13, 1, 4),
         (113, 17, 0, 8), (200, 31, 1, 2), (130, 41, 0, 4), (300, 25, 1, 8)]


@pytest.mark.parametrize("kind,nx,ny,walls,rows",
                         [("1",) + c for c in CASES] + [("2",) + c for c in TILES])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32_dev"])
def test_pair_matches_single_steps(lbe, monkeypatch, kind, nx, ny, walls, rows, form, precision):
    """An odd count and diagnostic steps, so that pairs start at both states,
    with and without diagnostics, and single steps come in between."""
    case = wl.random_case(nx, ny, seed=5 * nx + ny, walls_y=walls, n_drops=2, csf_form=form)
    out = []
    for pair in ("0", kind):
        monkeypatch.setenv("LBE_CSF_PAIR", pair)
        monkeypatch.setenv("LBE_CSF_PAIR_ROWS", str(rows))
        monkeypatch.setenv("LBE_CSF_SMALL", "0")
        print(f"case pair={pair} {nx}x{ny} walls={walls} rows={rows} form={form} {precision}",
              flush=True)
        sim = lbe.Simulation(case["params"], case["phi0"], case["T0"],
                             case["Twall_bot"] if walls else None,
                             case["Twall_top"] if walls else None, precision=precision,
                             diag_every=9)
        sim.step(2)
        sim.step(11)
        out.append((sim.get_state().cpu().numpy(), sim.step_count, sim.diag_history()))
    assert out[0][1] == out[1][1] == 13
    np.testing.assert_array_equal(out[1][0], out[0][0])
    # the diagnostics are FP64 sums over other blocks: equal to rounding (at
    # most nx * ny terms of either sign, each rounded once)
    assert len(out[0][2]) == len(out[1][2]) == 2
    for a, b in zip(out[0][2], out[1][2]):
        assert (a["step"], a["n_nonfinite"]) == (b["step"], b["n_nonfinite"])
        for k in ("mass", "energy", "sum_cy", "sum_cx"):
            assert a[k] == pytest.approx(b[k], rel=1e-11), k
    sys.stdout.flush()


# strips of 58 columns and chunks of few rows: as above, for the step with two
# densities, whose cones are one row and column narrower
DENSITY = [(3, 8, 1, 1), (7, 9, 0, 4), (58, 12, 1, 5), (59, 13, 1, 3), (117, 16, 0, 7),
           (200, 31, 1, 4), (130, 40, 1, 40), (300, 25, 0, 12)]


@pytest.mark.parametrize("nx,ny,walls,rows", DENSITY)
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32_dev"])
def test_one_launch_density_step_matches_two(lbe, monkeypatch, nx, ny, walls, rows, form, precision):
    """Two densities in one launch (density_step_kernel) against the pressure
    pass and the step: the states bitwise the same, the diagnostics to
    rounding."""
    case = wl.random_case(nx, ny, seed=7 * nx + ny, walls_y=walls, n_drops=2, csf_form=form,
                          rho2=2.5)
    out = []
    for pair in ("0", "1"):
        monkeypatch.setenv("LBE_CSF_PAIR", pair)
        monkeypatch.setenv("LBE_CSF_PAIR_ROWS", str(rows))
        print(f"case one launch={pair} {nx}x{ny} walls={walls} rows={rows} form={form} {precision}",
              flush=True)
        sim = lbe.Simulation(case["params"], case["phi0"], case["T0"],
                             case["Twall_bot"] if walls else None,
                             case["Twall_top"] if walls else None, precision=precision,
                             diag_every=3)
        sim.step(5)
        out.append((sim.get_state().cpu().numpy(), sim.diag_history()))
    np.testing.assert_array_equal(out[1][0], out[0][0])
    assert len(out[0][1]) == len(out[1][1]) == 2
    for a, b in zip(out[0][1], out[1][1]):
        for k in ("mass", "energy", "sum_cy", "sum_cx"):
            assert a[k] == pytest.approx(b[k], rel=1e-11), k
