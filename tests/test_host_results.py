"""Results on the host: large copies split into chunks over threads, and the
ring of per-step sums read in one or two copies."""
import ctypes
import threading

import numpy as np
import pytest

import synth


@pytest.mark.gpu
@pytest.mark.parametrize("n", [30, 31, 48, 73])
def test_populations_come_back_whole(n):
    """get_populations(set_populations(f)) is f, bit for bit (FP64), for
    totals below and above the size from which copies are split (4 MiB),
    ragged sizes, and a destination at every 8-byte phase of a cache line
    (chunks end on fixed host addresses)."""
    import paper_1601_03815_amd as dhit
    f = synth.random_populations(n, seed=n)
    with dhit.Box(n, "mrt", "fp64", 0.02) as b:
        b.set_populations(f)
        for phase in range(0, 9, 2):
            out = np.full(19 * n ** 3 + 16, np.nan)
            view = out[phase:phase + 19 * n ** 3]
            assert dhit._binding._lib.get_populations(b.handle, ctypes.c_void_p(view.ctypes.data)) == 0
            np.testing.assert_array_equal(view, f.ravel())
            assert np.isnan(out[:phase]).all() and np.isnan(out[phase + 19 * n ** 3:]).all()


@pytest.mark.gpu
def test_copies_of_several_threads():
    """Two host threads reading two boxes at once (each copy has pinned
    buffers of its own) get their own box's fields."""
    import paper_1601_03815_amd as dhit
    n = 64
    fs = [synth.random_populations(n, seed=s) for s in (1, 2)]
    bad = []

    def work(f):
        with dhit.Box(n, "bgk", "fp64", 0.02) as b:
            b.set_populations(f)
            for _ in range(5):
                drho = b.moments()[0]
                if np.abs(drho - f.sum(0)).max() > 1e-15 * 19:
                    bad.append("moments")
                if not np.array_equal(b.get_populations(), f):
                    bad.append("populations")

    ts = [threading.Thread(target=work, args=(f,)) for f in fs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


@pytest.mark.gpu
def test_history_across_the_ring():
    """The history keeps 4096 steps; a range that wraps around its end comes
    back in order (each step's sums read once by a count of one as it was
    taken)."""
    import paper_1601_03815_amd as dhit
    with dhit.Box(4, "bgk", "fp64", 0.05) as b:
        b.set_populations(synth.random_populations(4, seed=3))
        b.step(4090)
        seen = list(b.sums_history(4090))
        for _ in range(12):
            b.step(1)
            seen.append(b.sums_history(1)[0])
        for count in (0, 1, 5, 6, 7, 12, 4095, 4096):
            got = b.sums_history(count)
            np.testing.assert_array_equal(got, np.array(seen[len(seen) - count:]).reshape(count, 5))
        with pytest.raises(dhit.DhitError):
            b.sums_history(4097)
