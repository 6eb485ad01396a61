"""The level moves of a large cell, drawn by a whole workgroup, against the
oracle's sequential draws: sparse levels (most decrements redrawn), levels
at the top (increments redrawn), fewer and more moves than one batch."""
import numpy as np
import pytest

import oracle
import usp_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,T_tr,T_vib,steps", [(1025, 300.0, 900.0, 3), (2500, 400.0, 700.0, 4),
                                                (120000, 20000.0, 3000.0, 2),
                                                (60000, 9e5, 8e5, 2)])
def test_block_picks_equal_sequential_draws(n, T_tr, T_vib, steps):
    from paper_2508_05642_amd import usp
    prob, parts = W.batch0d([n], T_tr=[T_tr], T_rot=[T_tr], T_vib=[T_vib], dens=[1e23], dt=4e-9,
                            f32=False, seed=n)
    print(f"[block picks] n={n} T_vib={T_vib}", flush=True)
    parts["vib"] = np.minimum(parts["vib"], 255)
    gpu, orc = usp.DeviceState(prob, parts), oracle.Sim(prob, parts)
    assert -(-gpu.cap // gpu.M) > 1024  # the split path
    gpu.step(0, steps)
    orc.step_native(0, steps)
    a, b = gpu.state(), orc.state()
    # FP64 on both sides: the levels, and the counted events, are the same
    assert np.array_equal(a["pid"], b["pid"]) and np.array_equal(a["vib"], b["vib"])
    ca, cb = gpu.cnt(), orc.cnt()
    for k in ("PICK_FAIL", "CONS_SKIP", "VIB_SAT"):
        assert ca[k] == cb[k], (k, ca[k], cb[k])
    # the scalings follow from the levels: round-off of sums over n particles
    v = np.sqrt(prob.gas.R * T_tr)
    for k in ("cx", "cy", "cz"):
        assert np.abs(a[k] - b[k]).max() <= 1e-9 * v, k
