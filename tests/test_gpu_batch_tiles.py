"""Batched 0D steps against usp_step, bit for bit, at the edges of the tiles:
cells at the stage's size and one particle past it, cells on either side of
the line between 16 lanes and a wave, tiles whose last cell does not fit
beside the others, and windows without a cell."""
import numpy as np
import pytest

import usp_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = {True: [100, 16, 128, 129, 4352, 1500, 4300, 4353, 0, 1, 2, 30, 2047, 2400, 9000, 17],
         False: [100, 16, 128, 129, 2304, 500, 2250, 2305, 0, 1, 2, 30, 511, 2000, 5000, 17]}


@pytest.mark.parametrize("f32,tile", [(True, 0), (True, 512), (True, 2048), (False, 0)])
@pytest.mark.parametrize("shift", [0, 5])
def test_tiles_equal_step(f32, tile, shift):
    from paper_2508_05642_amd import usp
    counts = np.roll(SIZES[f32], shift)
    M = len(counts)
    rng = np.random.default_rng(shift)
    prob, parts = W.batch0d(counts, T_tr=rng.uniform(2000, 20000, M), T_rot=rng.uniform(200, 1000, M),
                            T_vib=rng.uniform(200, 1000, M), dens=np.full(M, 1e23), dt=2e-8, f32=f32)
    print(f"[batch tiles] f32={f32} tile={tile} shift={shift} n={parts['n']}", flush=True)
    a, b = usp.DeviceState(prob, parts), usp.DeviceState(prob, parts)
    a.step(10, 4)
    b.step(10, 1)
    b.batch(11, 3, tile, 2)
    torch.cuda.synchronize()
    sa, sb = a.state(), b.state()
    for k in sa:
        if isinstance(sa[k], np.ndarray):
            assert np.array_equal(sa[k], sb[k]), k
    assert a.cnt() == b.cnt()
    assert np.array_equal(a.moments(), b.moments())
    assert np.array_equal(a.cellstate(), b.cellstate())


@pytest.mark.parametrize("f32,tile,n", [(True, 0, 1536), (True, 0, 3072), (True, 512, 1024),
                                        (True, 1024, 2048), (True, 2048, 2048), (False, 0, 1024)])
def test_empty_cells_past_the_last_window(f32, tile, n):
    """A full state whose particles end on a window's edge, with empty cells
    behind them: those cells' averages are written and their skips counted."""
    from paper_2508_05642_amd import usp
    counts = np.array([n - 300, 300, 0, 0, 0])
    prob, parts = W.batch0d(np.maximum(counts, 1), T_tr=[9000.0] * 5, T_rot=[300.0] * 5,
                            T_vib=[300.0] * 5, dens=np.full(5, 1e23), dt=2e-8, f32=f32)
    parts = {k: v[:n] if isinstance(v, np.ndarray) else v for k, v in parts.items()}
    parts["n"] = n
    print(f"[batch tiles, empty end] f32={f32} tile={tile} n={n}", flush=True)
    a, b = (usp.DeviceState(prob, parts, capacity=n) for _ in range(2))
    for st in (a, b):
        st.bin()
        st.mom.fill_(-7.0)
        st.cs.fill_(-7.0)
    a.step(0, 3)
    b.batch(0, 3, tile, 2)
    torch.cuda.synchronize()
    assert np.array_equal(a.moments(), b.moments())
    assert np.array_equal(a.cellstate(), b.cellstate())
    assert a.cnt() == b.cnt()


@pytest.mark.parametrize("f32,tile", [(True, 0), (True, 512), (True, 1024), (True, 2048), (False, 0),
                                      (False, 512)])
def test_thousands_of_small_cells_equal_step(f32, tile):
    """The 4-wave shape of the tiles (thousands of cells; FP32 with 2048 slots
    keeps the 8-wave one): small cells, and among them cells at its stage's
    size (2240 FP32, 1200 FP64), one past it and far past it, and empty ones."""
    from paper_2508_05642_amd import usp
    M, rng = 3100, np.random.default_rng(6)
    counts = rng.integers(0, 200, M)
    edge = 2240 if f32 else 1200
    counts[[5, 900, 901, 2000, 2500, M - 2]] = [edge, edge + 1, edge - 1, 3 * edge, 1025, 6000]
    counts[[0, 902, M - 1]] = 0
    prob, parts = W.batch0d(np.maximum(counts, 1), T_tr=rng.uniform(2000, 20000, M),
                            T_rot=rng.uniform(200, 1000, M), T_vib=rng.uniform(200, 1000, M),
                            dens=np.full(M, 1e23), dt=2e-8, f32=f32)
    n = parts["n"]
    keep = np.nonzero(counts[parts["cell"][:n]] > 0)[0]  # batch0d puts one in every cell
    parts = {k: v[keep] if isinstance(v, np.ndarray) else v for k, v in parts.items()}
    parts["n"] = n = len(keep)
    assert 300000 <= n <= 400 * M
    print(f"[batch tiles, small cells] f32={f32} tile={tile} n={n}", flush=True)
    a, b = (usp.DeviceState(prob, parts, capacity=n) for _ in range(2))
    for st in (a, b):
        st.bin()
        st.mom.fill_(-7.0)
        st.cs.fill_(-7.0)
    a.step(10, 3)
    b.batch(10, 3, tile, 2)
    torch.cuda.synchronize()
    sa, sb = a.state(), b.state()
    for k in sa:
        if isinstance(sa[k], np.ndarray):
            assert np.array_equal(sa[k], sb[k]), k
    assert a.cnt() == b.cnt()
    assert np.array_equal(a.moments(), b.moments())
    assert np.array_equal(a.cellstate(), b.cellstate())
