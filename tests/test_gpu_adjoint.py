"""GPU pathwise adjoint (usp_step_taped / usp_adjoint_step through the C
ABI) against the oracle's gradient (oracle/adjoint.py, PyTorch FP64
replay with autograd) on the same seeded 1D runs.

Bar: the outputs agree to 1e-10 (mass flow) and to the fixed-point
rounding of the wall sampling (shear); each gradient entry agrees to 1e-7
of its magnitude (FP64 on both sides; the chains differ in operation order
and in how the secant heat capacity is evaluated near equal temperatures).
"""
import dataclasses
import sys

import numpy as np
import pytest

import usp_workloads as W
from oracle import adjoint as A

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _channel(cells=12, ppc=120, seed=7, shear=200.0):
    prob = W.poiseuille(kn=0.05, cells=cells, ppc=ppc, f32=False, seed=seed)
    parts = W.particles_for(prob)
    n = parts["n"]
    y = parts["y"][:n]
    parts["cx"][:n] += shear * np.sin(np.pi * y / 1e-3)
    parts["cz"][:n] *= 1.2
    return prob, parts


def _compare(J, G, Jo, Go, what):
    assert abs(J[0] - Jo[0]) <= 1e-10 * abs(Jo[0]), (what, J[0], Jo[0])
    assert abs(J[1] - Jo[1]) <= 1e-6 * abs(Jo[1]), (what, J[1], Jo[1])
    rel = np.abs(G - Go) / np.maximum(np.abs(Go), 1e-300)
    _say(f"  {what}: J {J}, worst relative gradient difference {rel.max():.3g}")
    assert np.all(rel <= 1e-7), (what, G, Go)


@pytest.mark.parametrize("K,segment", [(6, 4), (6, 32)])
def test_adjoint_matches_oracle_gradient(K, segment):
    """d(mdot, tau_w)/d(Z_rot, omega, mu_ref) over K steps, checkpointed in
    segments of `segment` steps, against the oracle's autograd gradient."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint
    prob, parts = _channel()
    _say(f"[adjoint] cells={prob.grid.ny} n={parts['n']} K={K} segment={segment}")
    path = A.Path(A.Record(prob, parts, 40, K))
    Jo, Go = path.gradient()
    adj = PathwiseAdjoint(prob, parts, K, segment)
    J = adj.forward(40).cpu().numpy()
    G = adj.backward().cpu().numpy()
    _compare(J, G, Jo, Go, f"K={K} segment={segment}")


def test_adjoint_segments_bit_identical():
    """The re-run of a segment reproduces the forward bit for bit, so the
    gradient does not depend on the checkpoint spacing."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint
    prob, parts = _channel(cells=10, ppc=100, seed=11)
    Gs = []
    for seg in (1, 3, 8):
        adj = PathwiseAdjoint(prob, parts, 8, seg)
        adj.forward(3)
        Gs.append(adj.backward().cpu().numpy())
    assert np.array_equal(Gs[0], Gs[1]) and np.array_equal(Gs[0], Gs[2])


def test_mass_flow_gradient_vanishes_without_boundary_events():
    """No particle meets a boundary: every cell keeps its momentum, so the
    mass flow does not depend on theta along the path."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint
    prob, parts = _channel(cells=10, ppc=150, seed=3, shear=300.0)
    n = parts["n"]
    rng = np.random.default_rng(5)
    L = prob.grid.ny * prob.grid.dy
    parts["y"][:n] = L * (0.3 + 0.4 * rng.random(n))
    prob = dataclasses.replace(prob, dt=2e-10)
    prob.bc = dataclasses.replace(prob.bc, g=(0.0, 0.0, 0.0))
    adj = PathwiseAdjoint(prob, parts, 4, 2)
    J = adj.forward(0).cpu().numpy()
    G = adj.backward().cpu().numpy()
    th = np.array([prob.gas.Z_rot, prob.gas.omega, prob.gas.mu_ref])
    assert np.all(np.abs(G[0] * th) <= 1e-11 * abs(J[0])), G[0]
    assert np.any(G[1] != 0.0) or J[1] == 0.0


def test_autograd_function_contracts_the_jacobian():
    """PathwiseOutputs: backward of w . J gives w^T dJ/dtheta."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint, PathwiseOutputs
    prob, parts = _channel(cells=8, ppc=100, seed=5)
    theta = torch.tensor([prob.gas.Z_rot, prob.gas.omega, prob.gas.mu_ref], dtype=torch.float64,
                         requires_grad=True)
    J = PathwiseOutputs.apply(theta, prob, parts, 2, 5, 2)
    w = torch.tensor([3.0, -0.5], dtype=torch.float64)
    (J * w).sum().backward()
    adj = PathwiseAdjoint(prob, parts, 5, 2)
    adj.forward(2)
    G = adj.backward().cpu()
    assert torch.allclose(theta.grad, w @ G, rtol=1e-12, atol=0.0)


def test_adjoint_full_size_two_segments():
    """The benchmarked case at full size (Poiseuille Kn 0.05, 100 cells x 500
    particles, FP64, a checkpoint every 32 steps) over 40 steps from its
    initial state: two segments, so the reverse pass restores a checkpoint
    and re-runs it.  Outputs and gradient against the oracle's autograd
    gradient of the same path."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint
    prob = W.poiseuille(kn=0.05, cells=100, ppc=500, f32=False, seed=7)
    parts = W.particles_for(prob)
    K = 40
    _say(f"[adjoint-full] cells={prob.grid.ny} n={parts['n']} K={K} segment=32")
    Jo, Go = A.Path(A.Record(prob, parts, 0, K)).gradient()
    adj = PathwiseAdjoint(prob, parts, K, 32)
    J = adj.forward(0).cpu().numpy()
    G = adj.backward().cpu().numpy()
    _compare(J, G, Jo, Go, f"full size K={K}")


def _step_outcomes(prob, parts, K):
    """The discrete outcomes of K GPU steps from the initial state: after
    every step the particle order (ids: the bin order and cell switches),
    cells, levels, offsets and the cumulative event counters (wall hits,
    Cholesky fallbacks, clamps, ...)."""
    from paper_2508_05642_amd import usp
    st = usp.DeviceState(prob, parts)
    out = []
    for k in range(K):
        st.step(k, 1)
        s = st.state()
        out.append((s["pid"], s["cell"], s["vib"], st.offsets.cpu().numpy(),
                    np.array(sorted(st.cnt().items()), dtype=object)))
    return out


def _oracle_run(prob, parts, K):
    """J of K oracle steps (the wall shear in FP64, from the run's own
    record) and the run's discrete outcomes: bin order, offsets, levels,
    cells after the flight and every branch the gradient holds fixed."""
    rec = A.Record(prob, parts, 0, K)
    p = A.Path(rec)
    J = p.run(p.theta0()).detach().numpy()
    out = [(S["binned"]["pid"], S["offsets"], S["cons"]["vib"], S["flight"]["cell"],
            d["event"].numpy(), d["fixed"].numpy(), d["rot"].numpy(), d["vel"].numpy(),
            d["ty"].numpy()) for d, S in zip(p.dec, rec.steps)]
    return J, out


def test_adjoint_equals_central_differences_full_size():
    """The benchmarked case at full size (Poiseuille Kn 0.05, 100 cells x
    500 particles, FP64): the GPU gradient of both outputs over 8 steps
    against central differences of complete runs at theta +- h (h = 1e-6
    relative, same seed), within 1e-3, with no discrete outcome changed
    between the runs (asserted step by step).  The mass flow's differences
    come from GPU runs (FP64 field sums); the wall shear's from the
    oracle's runs, whose shear is summed in FP64 (the GPU's wall sums are
    fixed point at 2^-16 m/s a hit, coarser than an h = 1e-6 change)."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint, with_theta
    prob = W.poiseuille(kn=0.05, cells=100, ppc=500, f32=False, seed=7)
    parts = W.particles_for(prob)
    K, h = 8, 1e-6
    _say(f"[adjoint-fd] cells={prob.grid.ny} n={parts['n']} K={K} h={h}")
    base = _step_outcomes(prob, parts, K)
    _, obase = _oracle_run(prob, parts, K)
    adj = PathwiseAdjoint(prob, parts, K, 32)
    adj.forward(0)
    G = adj.backward().cpu().numpy()
    th0 = np.array([prob.gas.Z_rot, prob.gas.omega, prob.gas.mu_ref])
    for p in range(3):
        Jg, Jo = [], []
        for sg in (1, -1):
            th = th0.copy()
            th[p] += sg * h * th0[p]
            pr = with_theta(prob, th)
            for a, b in zip(base, _step_outcomes(pr, parts, K)):
                for x, y in zip(a, b):
                    assert np.array_equal(x, y), ("gpu", p, sg)
            Jg.append(PathwiseAdjoint(pr, parts, K, 32).forward(0).cpu().numpy())
            J, out = _oracle_run(pr, parts, K)
            for a, b in zip(obase, out):
                for x, y in zip(a, b):
                    assert np.array_equal(x, y), ("oracle", p, sg)
            Jo.append(J)
        fd = np.array([(Jg[0][0] - Jg[1][0]), (Jo[0][1] - Jo[1][1])]) / (2 * h * th0[p])
        rel = np.abs(G[:, p] - fd) / np.abs(fd)
        _say(f"  d/d{('Z_rot', 'omega', 'mu_ref')[p]}: adjoint {G[:, p]}, FD {fd}, rel {rel}")
        assert np.all(rel <= 1e-3), (p, G[:, p], fd)


@pytest.mark.parametrize("cells,ppc", [(140, 150), (257, 90), (300, 90), (1100, 90), (6, 1300)])
def test_adjoint_of_every_particle_phase(cells, ppc):
    """The taped particle phase over tiles (more than 256 cells), with its
    order from buckets of cells (more than 1024) and in cells past the FP64
    stage of 1024 slots; the reverse by a wave a cell (more than 128 cells of
    fewer than 128) and by 8: the step it makes is usp_step's (the large cells
    aside, whose step adds its sums by chunks), and the gradient the
    oracle's.  (No particle's Cholesky test fails on these paths: the oracle's
    autograd has no value where one does.)"""
    from paper_2508_05642_amd import usp
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint
    prob, parts = _channel(cells=cells, ppc=ppc, seed=13)
    _say(f"[adjoint, phases] cells={cells} n={parts['n']}")
    K = 3
    adj = PathwiseAdjoint(prob, parts, K, 2)
    if ppc <= 1024:
        a, b = (usp.DeviceState(prob, parts) for _ in range(2))
        for k in range(K):
            a.step(20 + k)
            b.step_taped(20 + k, adj.tapes[0], adj.aws)
        sa, sb = a.state(), b.state()
        for k in sa:
            if isinstance(sa[k], np.ndarray):
                assert np.array_equal(sa[k], sb[k]), k
        assert torch.equal(a.offsets, b.offsets) and a.cnt() == b.cnt()
    Jo, Go = A.Path(A.Record(prob, parts, 20, K)).gradient()
    J = adj.forward(20).cpu().numpy()
    G = adj.backward().cpu().numpy()
    _compare(J, G, Jo, Go, f"{cells} cells of {ppc}")


@pytest.mark.parametrize("Z_vib", [50.0, 5.0])
def test_adjoint_with_vibrational_exchange(Z_vib):
    """The channel's gas relaxes no vibration (Z_vib 1e14: the exchange factor
    b is below 1e-12, where forward and reverse take the gammas' vibrational
    parts as zero); here a hot gas does, so the reverse goes through the
    relaxed temperature and the secant heat capacity."""
    from paper_2508_05642_amd.adjoint import PathwiseAdjoint
    prob = W.poiseuille(kn=0.05, cells=12, ppc=150, f32=False, seed=17)
    prob.gas = dataclasses.replace(prob.gas, Z_vib=Z_vib)
    parts = W.particles_for(prob)
    n, rng = parts["n"], np.random.default_rng(17)
    s = np.sqrt(prob.gas.R * 6000.0)
    for k in ("cx", "cy", "cz"):
        parts[k][:n] = s * rng.standard_normal(n)
    parts["cx"][:n] += 200.0 * np.sin(np.pi * parts["y"][:n] / 1e-3)
    parts["cz"][:n] *= 1.1
    parts["erot"][:n] = rng.exponential(prob.gas.R * 4000.0, n)
    parts["vib"][:n] = np.floor(rng.exponential(5000.0 / prob.gas.theta_vib, n))
    prob = dataclasses.replace(prob, dt=prob.dt / 8)
    _say(f"[adjoint, vibration] Z_vib={Z_vib} n={n}")
    Jo, Go = A.Path(A.Record(prob, parts, 40, 4)).gradient()
    adj = PathwiseAdjoint(prob, parts, 4, 3)
    J = adj.forward(40).cpu().numpy()
    G = adj.backward().cpu().numpy()
    _compare(J, G, Jo, Go, f"Z_vib={Z_vib}")
