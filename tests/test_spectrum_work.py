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


@pytest.mark.gpu
@pytest.mark.parametrize("n", [405, 512])
def test_large_transforms(n):
    """Batched transforms of large boxes (an odd size with a work area among
    them) on the Taylor-Green field u = U (sin x cos y cos z, -cos x sin y cos z,
    0): K = U^2/8 in shell 2 (|k|^2 = 3), S = 0, F = 27/8, and the vorticity
    -U k (cos x sin y sin z, sin x cos y sin z, -2 sin x sin y cos z), k = 2 pi/n,
    on planes of each axis.  1e-11: rounding of transforms of 1e8 points (about
    1e-15 log2 n^3 relative) with margin; F of fourth powers 1e-9."""
    import torch

    import paper_1601_03815_amd as dhit
    U = 0.05
    print("large transforms: n=%d" % n, flush=True)
    torch.cuda.empty_cache()
    x = 2.0 * np.pi * torch.arange(n, dtype=torch.float64, device="cuda") / n
    s, c = torch.sin(x), torch.cos(x)
    zyx = lambda fz, fy, fx: fz[:, None, None] * fy[None, :, None] * fx[None, None, :]
    u = torch.zeros((3, n, n, n), dtype=torch.float64, device="cuda")
    u[0] = U * zyx(c, c, s)
    u[1] = -U * zyx(c, s, c)
    with dhit.Box(n, "mrt", "fp64", 0.01) as b:
        b.init_velocity_field_device(u)
        E, st = b.energy_spectrum(4)[:2]
        w = b.vorticity()
    k = 2.0 * np.pi / n
    assert abs(st["K"] - U * U / 8) <= 1e-11 * U * U and abs(E[2] - U * U / 8) <= 1e-11 * U * U
    assert abs(st["eps"] - 2 * 0.01 * 3 * k * k * U * U / 8) <= 1e-11 * k * k * U * U
    assert abs(st["S"]) <= 1e-9 and abs(st["F"] - 27.0 / 8.0) <= 1e-9
    sn, cn = s.cpu().numpy(), c.cpu().numpy()
    for i in (0, n // 3, n - 1):
        plane = lambda fz, fy, fx: {0: fz[i] * np.outer(fy, fx), 1: fy[i] * np.outer(fz, fx), 2: fx[i] * np.outer(fz, fy)}
        want = [plane(sn, sn, cn), plane(sn, cn, sn), plane(cn, sn, sn)]
        for axis in range(3):
            for a, f in enumerate((-1.0, -1.0, 2.0)):
                got = np.take(w[a], i, axis=axis)
                assert np.abs(got - f * U * k * want[a][axis]).max() <= 1e-11 * U, (i, axis, a)
    del u
    torch.cuda.empty_cache()
