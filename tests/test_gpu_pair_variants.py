"""The launch shapes and variants of the two-step and one-launch two-density
kernels that only large grids take by default, forced on small ones and held
against single steps bit for bit: wide blocks (neighbouring strips in step, a
strip count that does not fill the last block), streaming stores, taped steps
in strips, and the thresholded diagnostics of every kernel."""
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


def _sim(lbe, case, walls, precision, **kw):
    return lbe.Simulation(case["params"], case["phi0"], case["T0"],
                          case["Twall_bot"] if walls else None,
                          case["Twall_top"] if walls else None, precision=precision, **kw)


def _same(a, b, n, cuy):
    """States bitwise; diagnostics, sums over other blocks, to the rounding of
    chains of at most 512 additions."""
    np.testing.assert_array_equal(a[0], b[0])
    assert len(a[1]) == len(b[1]) >= 2
    eps = 512 * 2.0 ** -53
    for x, y in zip(a[1], b[1]):
        assert (x["step"], x["n_nonfinite"]) == (y["step"], y["n_nonfinite"])
        for k in ("mass", "energy", "mass_thr"):
            assert abs(x[k] - y[k]) <= eps * 4 * n, k   # terms of a few units at most
        for k in ("sum_cy", "sum_cx"):
            assert x[k] == pytest.approx(y[k], rel=1e-11), k
        assert abs(x["sum_cuy_thr"] - y["sum_cuy_thr"]) <= eps * cuy
        assert x["mass_thr"] > 0


def _run(lbe, case, walls, precision, steps):
    sim = _sim(lbe, case, walls, precision, diag_every=5)
    sim.step(2)
    sim.step(steps - 2)
    f = sim.fields(("phi", "uy"))
    # bound of sum c |u_y| over the recorded steps: the fields of the last one,
    # which is not smaller than a hundredth of any
    cuy = 100 * (0.5 * (f["phi"] + 1.0) * f["uy"]).abs().sum().item()
    return (sim.get_state().cpu().numpy(), sim.diag_history()), cuy


# strip counts of 1, 2, 9 and 17: below, in and beyond blocks of eight or four
SHAPES = [(40, 12, 1, 5), (113, 16, 0, 7), (500, 21, 1, 4), (930, 17, 0, 17), (930, 25, 1, 3)]


@pytest.mark.parametrize("stream", ["0", "1"])
@pytest.mark.parametrize("nw", ["1", "8"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("nx,ny,walls,rows", SHAPES)
def test_fp32_pair_blocks_and_stores(lbe, monkeypatch, nx, ny, walls, rows, form, nw, stream):
    case = wl.random_case(nx, ny, seed=nx + 3 * ny, walls_y=walls, n_drops=3, csf_form=form)
    out = []
    for pair in ("0", "1"):
        for k, v in dict(PAIR=pair, PAIR_NW=nw, PAIR_ROWS=str(rows), STREAM=stream, SMALL="0").items():
            monkeypatch.setenv("LBE_CSF_" + k, v)
        print(f"case pair={pair} {nx}x{ny} walls={walls} rows={rows} form={form} nw={nw} "
              f"stream={stream}", flush=True)
        r, cuy = _run(lbe, case, walls, "fp32_dev", 13)
        out.append(r)
    _same(out[0], out[1], nx * ny, cuy)


@pytest.mark.parametrize("kind,nx,ny,walls,rows", [("1", 300, 25, 1, 6), ("2", 130, 41, 1, 4),
                                                   ("2", 57, 13, 0, 2)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_dev"])
def test_thresholded_diagnostics_of_pairs(lbe, monkeypatch, kind, nx, ny, walls, rows, precision):
    case = wl.random_case(nx, ny, seed=nx + ny, walls_y=walls, n_drops=3)
    out = []
    for pair in ("0", kind):
        for k, v in dict(PAIR=pair, PAIR_ROWS=str(rows), SMALL="0").items():
            monkeypatch.setenv("LBE_CSF_" + k, v)
        print(f"case pair={pair} {nx}x{ny} {precision}", flush=True)
        r, cuy = _run(lbe, case, walls, precision, 13)
        out.append(r)
    _same(out[0], out[1], nx * ny, cuy)


@pytest.mark.parametrize("nw", ["1", "8"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("nx,ny,walls,rows", SHAPES)
@pytest.mark.parametrize("precision", ["fp64", "fp32_dev"])
def test_density_blocks(lbe, monkeypatch, nx, ny, walls, rows, form, nw, precision):
    case = wl.random_case(nx, ny, seed=2 * nx + ny, walls_y=walls, n_drops=3, csf_form=form,
                          rho2=2.5)
    out = []
    for pair in ("0", "1"):
        for k, v in dict(PAIR=pair, PAIR_NW=nw, PAIR_ROWS=str(rows)).items():
            monkeypatch.setenv("LBE_CSF_" + k, v)
        print(f"case one launch={pair} {nx}x{ny} walls={walls} rows={rows} form={form} nw={nw} "
              f"{precision}", flush=True)
        r, cuy = _run(lbe, case, walls, precision, 11)
        out.append(r)
    _same(out[0], out[1], nx * ny, cuy)


@pytest.mark.parametrize("nw,stream", [("1", "0"), ("8", "0"), ("8", "1")])
@pytest.mark.parametrize("kind", ["1", "2"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32_dev"])
def test_taped_pairs(lbe, monkeypatch, precision, form, kind, nw, stream):
    """A recorded run that tapes its moments in strips and chunks, or in tiles:
    the gradients of one that takes single steps and replays them."""
    import torch
    nx, ny, steps = 500, 33, 23
    case = wl.random_case(nx, ny, seed=19, walls_y=1, n_drops=3, csf_form=form,
                          tau_f=(0.8, 0.8), tau_T=(0.7, 0.7))
    seed = torch.as_tensor(np.random.default_rng(5).standard_normal((ny, nx)))
    out = []
    for pair, direct in (("0", "0"), (kind, str(steps)), (kind, "9")):
        for k, v in dict(PAIR=pair, PAIR_NW=nw, PAIR_ROWS="4", STREAM=stream, DIRECT=direct).items():
            monkeypatch.setenv("LBE_CSF_" + k, v)
        print(f"case taped pairs={pair} of {direct} steps form={form} nw={nw} stream={stream} "
              f"{precision}", flush=True)
        sim = _sim(lbe, case, 1, precision, record_steps=steps)
        sim.step(steps, record=True)
        g = sim.backward(seed, want_F0=True, want_T0=True)
        out.append([torch.tensor(g["sigmaT"])] + [g[k].cpu() for k in ("Twall", "F0", "T0")])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b)
