"""The order in which a step's sums are added up does not depend on how the
step was called: alone, in a run of steps (whose launches carry one block more,
for the sums of the step before) or with event timing on."""
import numpy as np
import pytest

import synth


def _cancelling_field(n, seed):
    """Populations whose momentum nearly cancels inside every column tile (6
    rows of y) and over the box, beside noise: the sums are small beside the
    wavefront totals they are made of, so that another order of those totals
    shows in the last bits."""
    f = synth.random_populations(n, seed=seed, amplitude=1e-4)
    wave = 0.02 * np.cos(2.0 * np.pi * np.arange(n) / 6.0)[None, :, None]
    for plus, minus in ((1, 2), (3, 4), (5, 6)):
        f[plus] += wave
        f[minus] -= wave
    return f


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("tile,chunk", [(32, 9), (32, 6), (32, 3), (16, 9)])
def test_runs_equal_single_steps_on_a_mesh(precision, tile, chunk):
    """DUGKS on a stretched mesh, 66^3: tiles of 30 (14) x 6 columns, 264, 363,
    726 and 440 work items, so that the launches hold blocks on both sides of
    number 256 (and 512), the last padded to a multiple of 8, and all of
    them defer their sums (at most 1024).  Histories and populations bit for
    bit."""
    import paper_1601_03815_amd as dhit
    n = 66
    w = synth.stretched_widths(n, (0.2, 0.3, 0.25))
    f0 = _cancelling_field(n, 11)
    out = []
    for calls, timing in (((1,) * 9, False), ((9,), False), ((4, 5), False), ((9,), True)):
        with dhit.Box(n, "dugks", precision, 0.02, dt=0.4, tile_width=tile, z_chunk=chunk) as b:
            b.set_mesh(w)
            b.set_populations(f0)
            if timing:
                dhit.set_kernel_timing(b.handle, True)
            for k in calls:
                b.step(k)
            out.append((b.sums_history(9), b.get_populations()))
    for h, f in out[1:]:
        np.testing.assert_array_equal(h, out[0][0])
        np.testing.assert_array_equal(f, out[0][1])
