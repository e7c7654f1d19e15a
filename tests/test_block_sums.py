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


@pytest.mark.gpu
@pytest.mark.parametrize("method,sizes", [("bgk", (5, 32, 50, 51, 64, 80, 82)), ("mrt", (17, 33, 50, 51)),
                                          ("dugks", (5, 33, 64, 96))])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_run_of_steps_equals_single_steps(method, sizes, precision):
    """In a run of steps the next step's launch adds a step's block sums up
    (up to 1024 of them: LBE FP64 50^3, 80^3, FP32 64^3; one size above each is
    here too); a step called alone adds up its own.  Same history and
    populations bit for bit, also with event timing on (which keeps the
    launches apart) and across calls of odd and even lengths."""
    import paper_1601_03815_amd as dhit
    for n in sizes:
        f0 = synth.random_populations(n, seed=n, amplitude=0.005)
        out = []
        for calls, timing in (((1,) * 9, False), ((9,), False), ((4, 5), False), ((3, 1, 5), False), ((9,), True)):
            with dhit.Box(n, method, precision, 0.02) as b:
                b.set_populations(f0)
                if timing:
                    dhit.set_kernel_timing(b.handle, True)
                for k in calls:
                    b.step(k)
                if timing:
                    t = dhit.read_kernel_timings(b.handle)
                    assert t["finalize"][1] == 9
                out.append((b.sums_history(9), b.get_populations()))
        for h, f in out[1:]:
            np.testing.assert_array_equal(h, out[0][0])
            np.testing.assert_array_equal(f, out[0][1])
