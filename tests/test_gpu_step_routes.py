"""usp_step on the routes of its bin and particle phase that the grid, the
buffer or wall sampling selects, against the other routes."""
import numpy as np
import pytest

import usp_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BIG = 9 << 20  # a capacity past the sorted bin's on grids of more than 1024 cells


def _usp():
    from paper_2508_05642_amd import usp
    return usp


def _same(a, b):
    sa, sb = a.state(), b.state()
    assert sa["n"] == sb["n"] and sa["next_pid"] == sb["next_pid"]
    for k in sa:
        if isinstance(sa[k], np.ndarray):
            assert np.array_equal(sa[k], sb[k]), k
    assert torch.equal(a.offsets, b.offsets) and a.cnt() == b.cnt()


@pytest.mark.parametrize("scale,ppc,f32", [(0.2, 30.0, True), (0.2, 220.0, True), (0.26, 90.0, False)])
def test_step_takes_its_tiles_from_either_bin(scale, ppc, f32):
    """Four steps whose tile index comes from the neighbour-group bin's scan
    against four whose tile index comes from the sorted bin: a small state cut
    evenly (30 a cell) and windows by the mean cell.  (The larger buffer's mean
    slots per cell stay below the stage, past which cells are split.)"""
    usp = _usp()
    prob = W.cylinder(scale=scale, f32=f32, ppc=ppc)
    parts = W.particles_for(prob)
    print(f"[step routes] scale={scale} ppc={ppc} f32={f32} n={parts['n']}", flush=True)
    assert -(-BIG // prob.grid.ncells) <= (2048 if f32 else 1024)
    a = usp.DeviceState(prob, parts, capacity=int(1.6 * parts["n"]))
    b = usp.DeviceState(prob, parts, capacity=BIG)
    for st in (a, b):
        st.step(0, 1)
        st.step(1, 3)
    _same(a, b)
    assert np.array_equal(a.moments(), b.moments())


@pytest.mark.parametrize("f32", [True, False])
def test_unordered_input_of_more_cells_than_the_sort_takes(f32):
    """2^20 + 3 cells, no segments passed: every particle goes through the
    claimed slots of the neighbour-group route, a few cells with more than a
    wave's sort holds among them."""
    usp = _usp()
    M, n = (1 << 20) + 3, 60000
    rng = np.random.default_rng(8)
    grid = W.Grid(dim=0, nx=M, ny=1, fnum=1.0, volume=np.ones(M), flags=np.zeros(M, np.uint8))
    prob = W.Problem("cells", W.Gas(), grid, W.BC(), dt=1e-8, seed=1, f32=f32)
    cell = rng.integers(0, M, n)
    cell[: n // 2] = rng.integers(0, 3, n // 2) * (M - 1) // 2
    cell = rng.permutation(cell)
    cell[rng.random(n) < 0.05] = -1
    dt = np.float32 if f32 else np.float64
    v = {k: rng.standard_normal(n).astype(dt) for k in ("cx", "cy", "cz", "erot")}
    parts = dict(n=n, cap=n, x=None, y=None, vib=rng.integers(0, 200, n), cell=cell,
                 pid=rng.permutation(n).astype(np.uint32), next_pid=n, **v)
    print(f"[step routes] cells={M} f32={f32}", flush=True)
    st = usp.DeviceState(prob, parts)
    st.bin()
    got, keep = st.state(), np.nonzero(cell >= 0)[0]
    order = keep[np.argsort(cell[keep], kind="stable")]
    assert np.array_equal(got["cell"], cell[order])
    for k in ("cx", "cy", "cz", "erot"):
        assert np.array_equal(got[k], parts[k][order].astype(np.float64)), k
    assert np.array_equal(got["pid"], parts["pid"][order])
    assert np.array_equal(got["vib"], parts["vib"][order])
    off = np.concatenate([[0], np.cumsum(np.bincount(cell[keep], minlength=M))])
    assert np.array_equal(st.offsets.cpu().numpy(), off)


@pytest.mark.parametrize("f32", [True, False])
@pytest.mark.parametrize("cells,ppc", [(16, 60), (5, 700), (256, 30)])
def test_wall_sums_of_a_channel(cells, ppc, f32):
    """A workgroup per cell adds its wall hits up in LDS first (8 or 16
    waves): the same integers as the flight kernel's own additions, after
    each of three steps."""
    usp = _usp()
    prob = W.poiseuille(kn=0.05, cells=cells, ppc=ppc, f32=f32)
    parts = W.particles_for(prob)
    n = parts["n"]
    parts["cx"][:n] += 250.0
    print(f"[wall sums] cells={cells} ppc={ppc} f32={f32}", flush=True)
    a, b, c = (usp.DeviceState(prob, parts) for _ in range(3))
    for st in (a, b, c):
        st.enable_sampling(0)
    for k in range(3):
        for st in (a, b):
            st.bin(gather=st is a)
            st.do_moments()
            st.do_reconstruct()
        a.update(k)
        b.collide(k)
        b.conserve(k)
        b.advect(k)
        c.step(k)
        sa, sb = a.surface_sums(), b.surface_sums()
        assert np.array_equal(sa, sb)
        hits = sb[:, usp.SURF_HITS].sum()
        assert hits > 0 and np.count_nonzero(sb) == np.count_nonzero(sb[:2])
        if k == 0:
            # the step forms the cell state in a kernel of its own: a few
            # units of the last place of the stored velocities and, a hit,
            # one of the sums' 2^-16 m/s or 1/16 J/kg steps
            sc = c.surface_sums()
            assert np.array_equal(sc[:, usp.SURF_HITS], sb[:, usp.SURF_HITS])
            assert np.array_equal(sc[:, usp.SURF_QVIB], sb[:, usp.SURF_QVIB])
            v = 6.0 * np.sqrt(prob.gas.R * 300.0) + 500.0
            ulp = 4 * (2.0 ** -23 if f32 else 2.0 ** -50)
            for q in (usp.SURF_PX, usp.SURF_PY, usp.SURF_PZ, usp.SURF_PN, usp.SURF_PT):
                tol = hits * (1 + ulp * v * usp.SURF_P_SCALE)
                assert np.abs(sc[:, q] - sb[:, q]).max() <= tol, q
            for q in (usp.SURF_ETR, usp.SURF_EROT):
                tol = hits * (1 + ulp * 3 * v * v * usp.SURF_E_SCALE)
                assert np.abs(sc[:, q] - sb[:, q]).max() <= tol, q


@pytest.mark.parametrize("f32", [True, False])
def test_step_reads_this_steps_stencils(f32):
    """On a grid of at most 256 cells the particle phase makes its cell's
    stencil word itself.  Half the cells empty out and fill again from step to
    step, and the records hold other words on entry: the particles are those
    of the single phases."""
    usp = _usp()
    cells = 40
    rng = np.random.default_rng(4)
    prob = W.poiseuille(kn=0.05, cells=cells, ppc=30, f32=f32)
    parts = W.particles_for(prob)
    n = parts["n"]
    # clusters of three cells that drift by about a cell a step
    home = rng.integers(0, cells // 5, n) * 5 + rng.integers(0, 3, n)
    parts["y"][:n] = (home + 0.05 + 0.9 * rng.random(n)) * prob.grid.dy
    parts["cy"][:n] = parts["cy"][:n] * 0.2 + prob.grid.dy / prob.dt
    print(f"[step stencils] f32={f32} n={n}", flush=True)
    a, b = (usp.DeviceState(prob, parts) for _ in range(2))
    for k in range(4):
        for st in (a, b):
            st.cs.view(torch.uint8).fill_(0x5A)
        a.step(k)
        b.bin()
        b.do_moments()
        b.do_reconstruct()
        words = b.cs.view(torch.uint8)[usp.NCS * 8 * cells:].view(-1)[: 128 * cells].view(cells, 128)
        got = a.cs.view(torch.uint8)[usp.NCS * 8 * cells:].view(-1)[: 128 * cells].view(cells, 128)
        assert torch.equal(got[:, 60:64], words[:, 60:64])
        assert len(torch.unique(words[:, 60:64].contiguous().view(torch.int32))) > 1
        b.collide(k)
        b.conserve(k)
        b.advect(k)
        sa, sb = a.state(), b.state()
        assert np.array_equal(sa["pid"], sb["pid"]) and np.array_equal(sa["vib"], sb["vib"])
        v = np.sqrt(prob.gas.R * 300.0)
        for q in ("cx", "cy", "cz"):
            assert np.abs(sa[q] - sb[q]).max() <= (1e-5 if f32 else 1e-9) * v, q
        # go on from one state, so that the steps compare the stencils alone
        for q in usp.DeviceState.FIELDS:
            if b.bufs[b.cur][q] is not None:
                b.bufs[b.cur][q].copy_(a.bufs[a.cur][q])
        b.bufs[b.cur]["cell"].copy_(a.bufs[a.cur]["cell"])


def _roomy(M, dim, f32):
    """A periodic box (or independent cells) of M cells of 0 to 9 particles in
    a buffer of more slots a cell than the particle phase's stage."""
    rng = np.random.default_rng(M)
    nx, ny = (M, 1) if dim == 0 else (1, M) if dim == 1 else (M // 31 if M % 31 == 0 else 32, 0)
    if dim == 2:
        ny = M // nx
    M = nx * ny
    h = 1e-4
    gas = W.Gas()
    grid = W.Grid(dim=dim, nx=nx, ny=ny, dx=h, dy=h, fnum=1e22 * h * h / 5, volume=np.full(M, h * h),
                  flags=np.zeros(M, np.uint8))
    s = np.sqrt(gas.R * 300.0)
    prob = W.Problem("roomy", gas, grid, W.BC(kind=(W.BC_PERIODIC,) * 4), dt=0.3 * h / s, seed=3, f32=f32)
    cell = np.repeat(np.arange(M), rng.integers(0, 10, M))
    n = len(cell)
    u = 0.001 + 0.998 * rng.random((2, n))
    parts = dict(n=n, cap=n, x=(cell % nx + u[0]) * h if dim == 2 else None,
                 y=((cell // nx if dim == 2 else cell) + u[1]) * h if dim else None,
                 erot=rng.exponential(gas.R * 300.0, n), vib=rng.integers(0, 3, n),
                 cell=cell.astype(np.int32), pid=np.arange(n, dtype=np.uint32), next_pid=n,
                 **{k: s * rng.standard_normal(n) for k in ("cx", "cy", "cz")})
    return prob, parts, M * ((2048 if f32 else 1024) + 1)


@pytest.mark.parametrize("f32", [True, False])
@pytest.mark.parametrize("M,dim", [(1023, 0), (1023, 1), (1023, 2), (1024, 0), (1024, 1), (1024, 2)])
def test_step_past_the_stage_by_phases_or_chunks(M, dim, f32):
    """Buffers of more slots a cell than the stage: from 1024 cells on a step is
    the single phases (their bits); below, its sums go by chunks of the cells
    (FP64 sums of at most nine terms in another order: a few 1e-16 of the
    velocities, which a FP32 state rounds to 6e-8)."""
    usp = _usp()
    prob, parts, cap = _roomy(M, dim, f32)
    print(f"[step routes] roomy M={M} dim={dim} f32={f32} n={parts['n']}", flush=True)
    a, b = (usp.DeviceState(prob, parts, capacity=cap) for _ in range(2))
    steps = 3 if M >= 1024 else 1
    a.step(5, steps)
    for k in range(steps):
        if dim or k == 0:
            b.bin()
        b.do_moments()
        b.do_reconstruct()
        b.collide(5 + k)
        b.conserve(5 + k)
        if dim:
            b.advect(5 + k)
    if M >= 1024:
        _same(a, b)
        assert np.array_equal(a.moments(), b.moments())
        return
    sa, sb = a.state(), b.state()
    assert sa["n"] == sb["n"] and np.array_equal(sa["pid"], sb["pid"])
    assert np.array_equal(sa["vib"], sb["vib"])
    v = np.sqrt(prob.gas.R * 300.0)
    for k in ("cx", "cy", "cz"):
        assert np.abs(sa[k] - sb[k]).max() <= (1e-5 if f32 else 1e-9) * v, k
