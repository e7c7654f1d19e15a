"""The block reduction of the per-step sums and the small boxes' work split:
the sums of a step's history against the FP64 sums of the stored state."""
import numpy as np
import pytest

import synth


@pytest.mark.gpu
@pytest.mark.parametrize("method", ["bgk", "mrt", "dugks"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [4, 5, 31, 32, 33, 53, 54, 80, 82])
def test_history_sums_equal_stored_state(method, precision, n):
    """Sizes on both sides of each work split (LBE: blocks of 128 threads up
    to 32^3 in FP32 and 53^3 in FP64, one BGK cell per thread above 80^3),
    with last blocks partly filled.  Every population carries a gradient
    along x, y and z beside the noise, so that a lane, row, wavefront or
    block left out or counted twice shows.  FP64: 1e-13 of sum |f| (the
    reduction tree adds ~20 roundings of 1.1e-16); FP32: 1e-7 (each cell's
    moments rounded to 6e-8)."""
    import paper_1601_03815_amd as dhit
    i = np.arange(n) / n
    f0 = synth.random_populations(n, seed=n, amplitude=0.005)
    f0 += 0.003 * i[None, None, None, :] + 0.002 * i[None, None, :, None] - 0.004 * i[None, :, None, None]
    if precision == "fp32":
        f0 = f0.astype(np.float32).astype(np.float64)
    with dhit.Box(n, method, precision, 0.02) as b:
        b.set_populations(f0)
        b.step(2)
        got = b.sums_history(2)[1]
        f = b.get_populations()
        m = b.moments(want_fields=False)[2]
    c = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, 1, 0),
                  (1, -1, 0), (-1, -1, 0), (1, 0, 1), (-1, 0, 1), (1, 0, -1), (-1, 0, -1), (0, 1, 1), (0, -1, 1),
                  (0, 1, -1), (0, -1, -1)])
    j = np.tensordot(c.T.astype(float), f, axes=1)
    want = np.array([f.sum(), *j.sum(axis=(1, 2, 3)), 0.5 * (j * j).sum()])
    tol = (1e-13 if precision == "fp64" else 1e-7) * np.abs(f).sum()
    assert np.abs(got - want).max() <= tol and np.abs(m - want).max() <= tol
