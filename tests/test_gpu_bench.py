"""bench.py's accounting of the bytes a step moves follows what the handle
does: steps in pairs, single ones where diagnostics or an override ask for
them, one launch or two with two densities."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("args,env,per_pass,stored", [
    ([], {}, 2, 216), (["--diag-every", "1"], {}, 1, 432), ([], {"LBE_CSF_PAIR": "0"}, 1, 432),
    ([], {"LBE_CSF_ROWS": "16"}, 1, 432), (["--rho2", "2.0"], {}, 1, 432),
    (["--rho2", "2.0"], {"LBE_CSF_PAIR": "0"}, 1, 432 + 216 + 16)])
def test_bytes_per_update(args, env, per_pass, stored):
    """512 x 1024 in FP64, where plain steps go in pairs."""
    cmd = [sys.executable, os.path.join(ROOT, "bench.py"), "--workload", "droplet", "--precision",
           "fp64", "--steps", "10", "--warmup", "2", "--no-cpu-baseline", "--no-error-check", *args]
    print("case", args, env, flush=True)
    clean = {k: v for k, v in os.environ.items() if not k.startswith("LBE_CSF_")}
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=100, env={**clean, **env}, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    out = json.loads(r.stdout.strip().splitlines()[-1])
    assert out["config"]["steps_per_pass"] == per_pass
    assert out["config"]["stored_bytes_per_site_update"] == stored
    want = stored * out["config"]["sites"] / (out["ms_per_step"] * 1e-3) / 1e9
    assert out["roofline"]["achieved"] == pytest.approx(want, rel=1e-3)
