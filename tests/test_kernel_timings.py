"""Event timing of the launches outside the runs of steps."""
import pytest

import synth


@pytest.mark.gpu
@pytest.mark.parametrize("method", ["bgk", "mrt"])
def test_start_and_spectrum_are_timed(method):
    """Every pass of the LBE initial-state iteration is an LBE launch, and the
    totals of a spectrum's derivative sums a finalisation."""
    import paper_1601_03815_amd as dhit
    n = 16
    u = synth.dhit_field(n, seed=1, k0=2, u_rms=0.05)
    with dhit.Box(n, method, "fp64", 0.02) as b:
        dhit.set_kernel_timing(b.handle, True)
        b.init_consistent(u, None, 7)
        t = dhit.read_kernel_timings(b.handle)
        assert t["lbe"][1] == 7 and t["lbe"][0] > 0
        b.energy_spectrum(n // 2)
        t = dhit.read_kernel_timings(b.handle)
        assert t["finalize"][1] >= 1 and t["lbe"][1] == 0
