"""Which kernels a handle's steps run: the names that torch's profiler records.

A wrong route gives the right numbers (all kernels give the same bits), so only
the names show that an override, or a rule on the grid, was followed."""
import re

import pytest

from paper_1412_6238_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbe():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1412_6238_amd import lbe_csf
    return lbe_csf


def kernels(lbe, nx, ny, precision, steps, **kw):
    """Short names of the library's kernels of sim.step(steps), in order."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    case = wl.random_case(nx, ny, seed=nx + ny, **kw)
    sim = lbe.Simulation(case["params"], case["phi0"], case["T0"], case["Twall_bot"],
                         case["Twall_top"], precision=precision)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA, ProfilerActivity.CPU]) as prof:
        sim.step(steps)
        torch.cuda.synchronize()
    events = sorted((e for e in prof.events() if "lbe::" in e.name), key=lambda e: e.time_range.start)
    names = [re.search(r"lbe::(\w+)(<[^(]*>)?", e.name) for e in events]
    return [(m[1], [v.strip() for v in (m[2] or "<>")[1:-1].split(",")]) for m in names]


@pytest.mark.parametrize("precision", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("pipe", ["0", "1", "2"])
def test_row_pipeline_override(lbe, monkeypatch, pipe, precision):
    """LBE_CSF_PIPE asks for a row pipeline and gets it (136 x 40, blocks of
    four waves in FP64: the shape that tests/test_gpu_parity.py compares)."""
    monkeypatch.setenv("LBE_CSF_TILE", "0")
    monkeypatch.setenv("LBE_CSF_PIPE", pipe)
    monkeypatch.setenv("LBE_CSF_ROWS", "7")
    ks = kernels(lbe, 136, 40, precision, 2)
    assert [k[0] for k in ks] == ["step_kernel"] * 2, ks
    assert all(k[1][-1] == pipe for k in ks), ks   # the last parameter is the pipeline


@pytest.mark.parametrize("precision,nw,want", [("fp32_dev", "1", "1"), ("fp32_dev", "8", "8"),
                                               ("fp64", "8", "2")])
def test_pair_block_override(lbe, monkeypatch, precision, nw, want):
    """LBE_CSF_PAIR_NW picks the blocks that tests/test_gpu_pair_variants.py
    compares (FP64 has one kind)."""
    monkeypatch.setenv("LBE_CSF_PAIR", "1")
    monkeypatch.setenv("LBE_CSF_PAIR_NW", nw)
    ks = kernels(lbe, 500, 33, precision, 4)
    assert [k[0] for k in ks] == ["pair_step_kernel"] * 2, ks
    assert all(k[1][-1] == want for k in ks), ks   # the last parameter: waves a block


@pytest.mark.parametrize("nx,ny,precision,rho2,want", [
    (16, 16, "fp64", 0, ["small_step_kernel"]),
    (8, 64, "fp64", 0, ["pair_tile_kernel"] * 2), (160, 300, "fp32_dev", 0, ["pair_tile_kernel"] * 2),
    (8, 4096, "fp32_dev", 0, ["tile_step_kernel"] * 4),
    (742, 75, "fp32_dev", 0, ["tile_step_kernel"] * 4),
    (144, 364, "fp32_dev", 0, ["pair_tile_kernel"] * 2),
    (256, 512, "fp32_dev", 0, ["tile_step_kernel"] * 4),
    (728, 728, "fp64", 0, ["tile_step_kernel"] * 4), (743, 790, "fp64", 0, ["pair_step_kernel"] * 2),
    (512, 1030, "fp64", 0, ["pair_step_kernel"] * 2), (130, 4462, "fp64", 0, ["tile_step_kernel"] * 4),
    (130, 5010, "fp64", 0, ["pair_step_kernel"] * 2), (23, 28696, "fp64", 0, ["tile_step_kernel"] * 4),
    (23, 66000, "fp64", 0, ["pair_step_kernel"] * 2), (4000, 126, "fp64", 0, ["pair_step_kernel"] * 2),
    (1160, 1020, "fp32_dev", 0, ["tile_step_kernel"] * 4),
    (1250, 1010, "fp32_dev", 0, ["pair_step_kernel"] * 2),
    (60, 22001, "fp32_dev", 0, ["tile_step_kernel"] * 4),
    (60, 25834, "fp32_dev", 0, ["pair_step_kernel"] * 2),
    (1300, 1100, "fp32_dev", 2.0, ["tile_step_kernel"] * 8),
    (1400, 1100, "fp32_dev", 2.0, ["density_step_kernel"] * 4),
    (60, 26000, "fp32_dev", 2.0, ["step_kernel"] * 8),
    (500, 590, "fp64", 2.0, ["tile_step_kernel"] * 8),
    (500, 610, "fp64", 2.0, ["density_step_kernel"] * 4)])
def test_default_routes(lbe, monkeypatch, nx, ny, precision, rho2, want):
    """Four plain steps on grids at both sides of each rule."""
    for v in ("PAIR", "PAIR_NW", "PAIR_ROWS", "NW", "ROWS", "PIPE", "STREAM", "TILE", "SMALL"):
        monkeypatch.delenv("LBE_CSF_" + v, raising=False)
    ks = kernels(lbe, nx, ny, precision, 4, **(dict(rho2=rho2) if rho2 else {}))
    assert [k[0] for k in ks] == want, ks


@pytest.mark.parametrize("nx,ny,precision,rho2,nw", [
    (52, 58654, "fp32_dev", 0, "1"), (254, 12008, "fp32_dev", 0, "1"), (400, 7626, "fp32_dev", 0, "8"),
    (2000, 1526, "fp32_dev", 0, "8"), (23, 132609, "fp64", 2.0, "1"), (800, 3800, "fp64", 2.0, "4")])
def test_blocks_of_large_grids(lbe, monkeypatch, nx, ny, precision, rho2, nw):
    """Above 3M sites the waves of a block take neighbouring strips, on widths
    that fill such blocks."""
    for v in ("PAIR", "PAIR_NW", "PAIR_ROWS", "NW", "ROWS", "PIPE", "STREAM", "TILE", "SMALL"):
        monkeypatch.delenv("LBE_CSF_" + v, raising=False)
    ks = kernels(lbe, nx, ny, precision, 2, **(dict(rho2=rho2) if rho2 else {}))
    want = "density_step_kernel" if rho2 else "pair_step_kernel"
    assert all(k[0] == want and k[1][-1] == nw for k in ks) and len(ks) == (2 if rho2 else 1), ks
