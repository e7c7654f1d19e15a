"""The transforms' plans and work space of a box, shared by everything that
works in spectral space."""
import time

import numpy as np
import pytest

import synth


@pytest.mark.gpu
@pytest.mark.parametrize("n", [12, 31, 64, 97, 131, 300, 509])
def test_work_space_bytes(n):
    """Seven half spectra (three fields, their transforms, one more) and one
    work area, which hipFFT asks for up to four times three half spectra of
    (odd sizes): at most 19 half spectra (n odd: 152 bytes per cell and a
    little)."""
    import paper_1601_03815_amd as dhit
    got = dhit.spectrum_bytes(dhit.default_params(n, "mrt", "fp64", 0.01))
    half = 16 * n * n * (n // 2 + 1)
    small = 8 * (20 * int(3 ** 0.5 * (n // 2 + 1) + 2) + 16 + 15 * 1024)
    assert 7 * half <= got <= 19 * half + small


@pytest.mark.gpu
def test_first_spectrum_after_a_start_makes_no_plan():
    """initial_pressure and energy_spectrum use the same two plans: the first
    spectrum of a box that has had its pressure takes about as long as a later
    one (a plan takes some 15 times as long).  Best of five boxes."""
    import torch

    import paper_1601_03815_amd as dhit
    n = 32
    u = synth.dhit_field(n, seed=1, k0=4, u_rms=0.05)
    first, later = [], []
    for _ in range(5):
        with dhit.Box(n, "mrt", "fp64", 0.01) as b:
            b.init_consistent(u, b.initial_pressure(u), 2)
            for out in (first, later):
                b.synchronize()
                t = time.perf_counter()
                b.energy_spectrum(n // 2)
                out.append(time.perf_counter() - t)
    torch.cuda.synchronize()
    assert min(first) <= 5 * min(later), (first, later)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 16, 33])
def test_order_of_calls_does_not_matter(n):
    """Spectrum, vorticity and pressure in any order on one box give the bits
    that each gives alone on a new box, and leave the state as it is."""
    import paper_1601_03815_amd as dhit
    u = synth.dhit_field(n, seed=2, k0=2, u_rms=0.05)

    def box(method):
        b = dhit.Box(n, method, "fp64", 0.01)
        b.init_velocity_field(u)
        b.step(2)
        return b

    calls = {"E": lambda b: np.concatenate([np.ravel(x) for x in _spectrum(b, n)]),
             "w": lambda b: b.vorticity(), "p": lambda b: b.initial_pressure(u)}
    for method in ("mrt", "dugks"):
        alone = {}
        for k, f in calls.items():
            with box(method) as b:
                alone[k] = f(b)
        for order in ("Ewp", "pwE", "wpE", "pEpw"):
            with box(method) as b:
                for k in order:
                    np.testing.assert_array_equal(calls[k](b), alone[k], err_msg=order + " " + k)


def _spectrum(b, n):
    E, st = b.energy_spectrum(n // 2)[:2]
    return E, [st[k] for k in ("K", "eps", "S", "F")]
