"""Moments of grids of few cells (a workgroup or a wave a cell) against
numpy, at the edges of the lanes' strides and of the rule that picks the
kernel, and the step's fused moments and cell state against the phases."""
import numpy as np
import pytest

import usp_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [0, 1, 2, 63, 64, 65, 255, 256, 257, 1023, 1025, 1300]


def _channel(M, f32, seed):
    """A 1D grid of M cells, the first of the sizes above, the rest small."""
    rng = np.random.default_rng(seed)
    counts = np.array((SIZES + [3] * M)[:M])
    grid = W.Grid(dim=1, nx=1, ny=M, dy=1.0, fnum=1e15, volume=np.ones(M), flags=np.zeros(M, np.uint8))
    bc = W.BC(kind=(W.BC_PERIODIC,) * 4)
    prob = W.Problem("sizes", W.Gas(), grid, bc, dt=1e-9, seed=3, f32=f32)
    cell = np.repeat(np.arange(M), counts)
    n = len(cell)
    dt = np.float32 if f32 else np.float64
    s = np.sqrt(prob.gas.R * 3000.0)
    parts = dict(n=n, cap=n, x=None, y=(cell + 0.1 + 0.8 * rng.random(n)).astype(dt),
                 cx=(900.0 + s * rng.standard_normal(n)).astype(dt),
                 cy=(s * rng.standard_normal(n)).astype(dt),
                 cz=(s * rng.standard_normal(n)).astype(dt),
                 erot=rng.exponential(prob.gas.R * 2000.0, n).astype(dt),
                 vib=rng.integers(0, 9, n), cell=cell, pid=np.arange(n, dtype=np.uint32), next_pid=n)
    return prob, parts, cell


def _numpy_moments(parts, cell, M):
    N = np.bincount(cell, minlength=M).astype(float)

    def mean(v):
        return np.bincount(cell, weights=v, minlength=M) / np.maximum(N, 1)

    c = [parts[k].astype(np.float64) for k in ("cx", "cy", "cz")]
    e, lev = parts["erot"].astype(np.float64), parts["vib"].astype(np.float64)
    U = [mean(v) for v in c]
    d = [v - u[cell] for v, u in zip(c, U)]
    q2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
    out = [N, *U] + [mean(d[i] * d[j]) for i, j in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
    er, lv = mean(e), mean(lev)
    out += [er, lv] + [mean(0.5 * q2 * v) for v in d] + [mean(v * (e - er[cell])) for v in d]
    return np.array(out + [mean(v * (lev - lv[cell])) for v in d])


@pytest.mark.parametrize("f32", [True, False])
@pytest.mark.parametrize("M", [1, 12, 512, 513, 4096, 4097])
def test_moments_of_few_cells(M, f32):
    from paper_2508_05642_amd import usp
    prob, parts, cell = _channel(M, f32, M)
    print(f"[wide moments] M={M} n={parts['n']} f32={f32}", flush=True)
    cap = parts["n"] + 64  # mean slots per cell below the stage: not the split path
    st = usp.DeviceState(prob, parts, capacity=cap)
    st.bin()
    st.do_moments()
    m, ref = st.moments(), _numpy_moments(parts, cell, M)
    c = np.sqrt(prob.gas.R * 3000.0) + 900.0
    e = c * c
    scale = np.array([1.0] + [c] * 3 + [e] * 6 + [e, 9.0] + [e * c] * 6 + [9.0 * c] * 3)
    # FP64 sums of at most 1300 terms of the order of the scale
    assert np.abs(m - ref).max(axis=1).tolist() <= (1e-10 * scale).tolist()
    gathered = usp.DeviceState(prob, parts, capacity=cap)
    gathered.bin(gather=True)
    gathered.do_moments()
    assert np.array_equal(gathered.moments(), m)
    # the step's own moments and cell state
    st.do_reconstruct()
    stepped = usp.DeviceState(prob, parts, capacity=cap)
    stepped.step(0)
    assert np.array_equal(stepped.moments(), m)
    a, b = stepped.cellstate(), st.cellstate()
    # the same chain of some hundred FP64 operations, contracted differently at most
    assert np.all(np.abs(a - b) <= 1e-12 * np.abs(b))
    sa, sb = stepped.cs.view(torch.uint8), st.cs.view(torch.uint8)
    rec = slice(usp.NCS * 8 * M, (usp.NCS * 8 + 128) * M)
    # stencil words of the packed records (byte 60 of 128)
    ra, rb = sa[rec].view(M, 128)[:, 60:64], sb[rec].view(M, 128)[:, 60:64]
    assert torch.equal(ra, rb)


@pytest.mark.parametrize("f32", [True, False])
@pytest.mark.parametrize("M", [500, 4000])
def test_wide_sums_keep_the_order_of_rows(M, f32):
    """A workgroup per cell and a row of 16 lanes per cell add a cell's
    particles in one order: the same cells in a grid past the rule's line
    (empty cells appended) give the same bits."""
    from paper_2508_05642_amd import usp
    out = []
    for cells in (M, 4200):
        prob, parts, cell = _channel(M, f32, 5)
        prob.grid = W.Grid(dim=1, nx=1, ny=cells, dy=1.0, fnum=1e15, volume=np.ones(cells),
                           flags=np.zeros(cells, np.uint8))
        st = usp.DeviceState(prob, parts, capacity=parts["n"] + 64)
        st.bin()
        st.do_moments()
        out.append(st.moments()[:, :M])
    assert np.array_equal(*out)


@pytest.mark.parametrize("f32", [True, False])
@pytest.mark.parametrize("M", [1, 12, 512, 513, 4096, 4097])
def test_every_moment_of_few_cells_against_numpy(M, f32):
    """Each plane by itself against FP64 numpy sums of the stored values: a
    cell's sums have at most 1300 terms of some ten times the plane's scale,
    each off by a few 1e-16 of it (1e-12 of the scale in all)."""
    from paper_2508_05642_amd import usp
    prob, parts, cell = _channel(M, f32, M + 1)
    print(f"[wide moments, planes] M={M} n={parts['n']} f32={f32}", flush=True)
    st = usp.DeviceState(prob, parts, capacity=parts["n"] + 64)
    st.bin()
    st.do_moments()
    m, ref = st.moments(), _numpy_moments(parts, cell, M)
    assert np.array_equal(m[0], ref[0])
    c = np.sqrt(prob.gas.R * 3000.0) + 900.0
    e = c * c
    scale = np.array([c] * 3 + [e] * 6 + [e, 9.0] + [e * c] * 6 + [9.0 * c] * 3)
    err = np.abs(m - ref).max(axis=1)[1:]
    assert np.all(err <= 1e-10 * scale), (err / scale).tolist()


@pytest.mark.parametrize("f32", [True, False])
def test_rows_load_one_by_one_as_ahead(f32):
    """Sparse grids (at most ten slots a cell) take the rows' plain loop: the
    bits of the loop that loads ahead, which a roomier buffer selects, in cells
    of 0 to 90 particles."""
    from paper_2508_05642_amd import usp
    M, rng = 4200, np.random.default_rng(9)
    counts = rng.integers(0, 8, M)
    counts[[3, 4, 77, 78, 4199]] = [90, 0, 16, 17, 64]
    grid = W.Grid(dim=1, nx=1, ny=M, dy=1.0, fnum=1e15, volume=np.ones(M), flags=np.zeros(M, np.uint8))
    prob = W.Problem("sparse", W.Gas(), grid, W.BC(kind=(W.BC_PERIODIC,) * 4), dt=1e-9, seed=3, f32=f32)
    cell = np.repeat(np.arange(M), counts)
    n = len(cell)
    s = np.sqrt(prob.gas.R * 3000.0)
    parts = dict(n=n, cap=n, x=None, y=cell + 0.1 + 0.8 * rng.random(n), cell=cell,
                 erot=rng.exponential(prob.gas.R * 2000.0, n), vib=rng.integers(0, 9, n),
                 pid=np.arange(n, dtype=np.uint32), next_pid=n,
                 **{k: s * rng.standard_normal(n) for k in ("cx", "cy", "cz")})
    out = []
    for cap in (10 * M, 10 * M + 1):
        for gather in (False, True):
            st = usp.DeviceState(prob, parts, capacity=cap)
            st.bin(gather=gather)
            st.do_moments()
            out.append(st.moments())
    print(f"[sparse rows] n={n} f32={f32}", flush=True)
    for m in out[1:]:
        assert np.array_equal(m, out[0])
