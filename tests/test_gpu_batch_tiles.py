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
