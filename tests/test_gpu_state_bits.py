"""The bits of states, diagnostics and gradients, against stored ones.

The droplet velocity u_r = sum c u_y / sum c of a short run is the residue of a
sum that cancels over several orders of magnitude, so it carries the rounding
of every population: two evaluations of one collision that agree to FP32
rounding in the fields differ by up to 1e-2 of u_r.  A kernel that takes over a
grid, or a cheaper form of the collision, must therefore leave every bit of the
state as it was.  tests/golden/state_bits.json holds digests of the states, the
diagnostic sums and the gradients that the library of commit 5897d12 (one
launch a step, moments replayed in the backward pass) gives for the runs below.

    PYTHONPATH=<checkout> python tests/test_gpu_state_bits.py > tests/golden/state_bits.json

writes that file with the library of a checkout.  The inputs use correctly
rounded operations only (no tanh), so that they are the same on every host.
"""
import hashlib
import json
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
GOLDEN = os.path.join(HERE, "golden", "state_bits.json")

CONST = dict(tau_f=(0.9, 0.9), tau_T=(0.8, 0.8))
VARY = dict(tau_f=(0.8, 1.3), tau_T=(0.7, 1.1))
LINEAR = dict(T_shift=3.0, T_grad=0.0078125, force=(1e-6, -2e-6))   # T reference of the FP32 form

# nx, ny, walls, parameters: the small-grid path, tiles (one and two steps a
# launch), strips and chunks (FP64 from 0.5M, FP32 from 1.2M sites), rows
RUNS = [
    (8, 64, 1, VARY), (8, 64, 1, dict(CONST, **LINEAR)),
    (40, 100, 1, CONST), (57, 13, 1, dict(VARY, **LINEAR)), (20, 17, 0, CONST),
    (200, 100, 1, dict(CONST, csf_form=1, **LINEAR)), (256, 128, 1, CONST),
    (300, 200, 0, dict(VARY, csf_form=1)), (64, 40, 1, dict(VARY, rho2=2.5, **LINEAR)),
    (130, 41, 1, dict(CONST, rho2=2.0, csf_form=1)),
    (1200, 1030, 1, dict(CONST, **LINEAR)), (1230, 1003, 1, dict(VARY, csf_form=1)),
    (1200, 1030, 1, dict(CONST, rho2=2.0, **LINEAR)), (2048, 800, 1, dict(CONST, **LINEAR)),
]
GRADS = [
    (130, 40, 1, CONST, 16), (70, 33, 0, VARY, 9), (20, 17, 1, dict(CONST, csf_form=1), 16),
    (300, 200, 1, dict(VARY, csf_form=1), 5), (300, 200, 1, CONST, 12),
    (1200, 1030, 1, dict(CONST, **LINEAR), 4),
]
PRECISIONS = ("fp64", "fp32_dev")


def _case(nx, ny, walls, over):
    """A few droplets with a piecewise cubic profile, a rough temperature and
    rough walls."""
    rng = np.random.default_rng(1000 * nx + ny)
    p = dict(nx=nx, ny=ny, walls_y=walls, rho=1.0, cv=1.0, tau_g=0.9, mobility=0.02, width=2.5,
             beta=0.25, sigma0=1e-2, sigmaT=5e-4, Tref=0.5, force=(0.0, 0.0), p0=0.0, T_shift=0.0,
             T_grad=0.0, csf_form=0)
    p.update(over)
    if not walls:
        p["T_grad"] = 0.0
    x, y = np.arange(nx)[None, :] + 0.5, np.arange(ny)[:, None] + 0.5
    phi = np.full((ny, nx), -1.0)
    for _ in range(3):
        cx, cy = rng.uniform(0, nx), rng.uniform(0, ny)
        R = rng.uniform(2.0, max(2.5, min(nx, ny) / 4))
        dx = np.minimum(np.abs(x - cx), nx - np.abs(x - cx))
        s = np.clip((R - np.sqrt(dx * dx + (y - cy) * (y - cy))) / 4.0, -1.0, 1.0)
        phi = np.maximum(phi, s * (1.5 - 0.5 * s * s))
    phi = phi + 0.01 * (rng.random((ny, nx)) - 0.5)
    T0 = p["T_shift"] + p["T_grad"] * y + (rng.random((ny, nx)) - 0.5)
    tb = p["T_shift"] + (rng.random(nx) - 0.5)
    tt = p["T_shift"] + p["T_grad"] * ny + (rng.random(nx) - 0.5)
    return p, phi, T0, (tb if walls else None), (tt if walls else None)


def _key(nx, ny, walls, over, precision, *rest):
    return " ".join([f"{nx}x{ny}", f"walls={walls}", precision, *map(str, rest),
                     json.dumps(over, sort_keys=True)])


def _digest(t):
    return hashlib.sha256(np.ascontiguousarray(t.cpu().numpy()).tobytes()).hexdigest()[:32]


SUMS = ("mass", "energy", "sum_cy", "sum_cx", "mass_thr", "sum_cuy_thr", "u_r")


def _run(lbe, nx, ny, walls, over, precision):
    """One step, its state and diagnostics, then eleven more (diagnostics along
    the way, so that single steps and pairs alternate)."""
    p, phi, T0, tb, tt = _case(nx, ny, walls, over)
    sim = lbe.Simulation(p, phi, T0, tb, tt, precision=precision, diag_every=6)
    sim.step(1)
    d = sim.diagnostics()
    f = sim.fields(("phi", "uy"))
    out = dict(one=_digest(sim.get_state()), **{k: d[k] for k in SUMS})
    cuy = (0.5 * (f["phi"] + 1.0) * f["uy"]).abs().sum().item()
    sim.step(11)
    out["twelve"] = _digest(sim.get_state())
    out["history"] = [{k: h[k] for k in SUMS} for h in sim.diag_history()]
    return out, cuy


def _grad(lbe, nx, ny, walls, over, steps, precision):
    import torch
    p, phi, T0, tb, tt = _case(nx, ny, walls, over)
    sim = lbe.Simulation(p, phi, T0, tb, tt, precision=precision, record_steps=steps)
    sim.step(steps, record=True)
    seed = np.random.default_rng(steps).random((ny, nx)) - 0.5
    g = sim.backward(torch.as_tensor(seed), want_F0=True, want_T0=True)
    torch.cuda.synchronize()
    return dict(sigmaT=float(g["sigmaT"]).hex(), **{k: _digest(g[k]) for k in ("Twall", "F0", "T0")})


@pytest.fixture(scope="module")
def lbe():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1412_6238_amd import lbe_csf
    return lbe_csf


@pytest.fixture(scope="module")
def golden():
    with open(GOLDEN) as f:
        return json.load(f)


def _close(got, ref, cuy, n, key):
    # FP64 sums over other blocks than the stored ones: no chain of additions
    # is longer than 256 here, each rounded once; terms of either sign in
    # sum_cuy_thr, which u_r divides by mass_thr
    eps = 256 * 2.0 ** -53
    for k in ("mass", "energy", "sum_cy", "sum_cx", "mass_thr"):
        assert abs(got[k] - ref[k]) <= eps * n * max(1.0, abs(ref[k]) / n), (key, k)
    assert abs(got["sum_cuy_thr"] - ref["sum_cuy_thr"]) <= eps * cuy, (key, "sum_cuy_thr")
    tol_u = eps * cuy / ref["mass_thr"] + eps * abs(ref["u_r"])
    assert abs(got["u_r"] - ref["u_r"]) <= 2 * tol_u, (key, "u_r", got["u_r"], ref["u_r"])


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("run", RUNS, ids=lambda r: f"{r[0]}x{r[1]}")
def test_states_and_diagnostics(lbe, golden, run, precision):
    key = _key(*run, precision)
    print(f"case {key}", flush=True)
    got, cuy = _run(lbe, *run, precision)
    ref = golden["runs"][key]
    _close(got, ref, cuy, run[0] * run[1], key)
    assert got["one"] == ref["one"], key
    assert got["twelve"] == ref["twelve"], key


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("case", GRADS, ids=lambda c: f"{c[0]}x{c[1]}-{c[4]}")
def test_gradients(lbe, golden, case, precision):
    key = _key(*case[:4], precision, case[4])
    print(f"case {key}", flush=True)
    assert _grad(lbe, *case, precision) == golden["grads"][key], key


if __name__ == "__main__":
    from paper_1412_6238_amd import lbe_csf as L
    print(f"library: {L.LIB_PATH}", file=sys.stderr, flush=True)
    out = dict(runs={_key(*r, p): _run(L, *r, p)[0] for r in RUNS for p in PRECISIONS},
               grads={_key(*c[:4], p, c[4]): _grad(L, *c, p) for c in GRADS for p in PRECISIONS})
    json.dump(out, sys.stdout, indent=1)
