"""The finalisation of a step's sums for boxes of many blocks."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_slices_of_every_box(tmp_path):
    """The rule that splits the block partials over the finalisation's blocks
    (runtime.hpp), for one cell per thread in blocks of 256 at every n."""
    exe = str(tmp_path / "finalize")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    os.path.join(HERE, "finalize_cases.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("method,precision,n", [("bgk", "fp64", 400), ("bgk", "fp64", 406), ("bgk", "fp64", 408),
                                                ("mrt", "fp32", 407), ("mrt", "fp32", 515)])
def test_sums_of_many_blocks(method, precision, n):
    """On both sides of 64 x 4096 partials (407^3 cells, one per thread), and
    where the last slice is short: the sums of a step against double sums of
    the stored state, whose populations carry an offset that makes every
    slice count.  FP64: 1e-13 of sum |f|; FP32: 1e-7 (each cell's moments
    rounded to 6e-8)."""
    import torch

    import paper_1601_03815_amd as dhit
    print("many blocks: %s %s n=%d" % (method, precision, n), flush=True)
    torch.cuda.empty_cache()
    box = dhit.Box(n, method, precision, 0.02)
    try:
        cur = box.populations_tensor()
        g = torch.Generator(device="cuda").manual_seed(n)
        for q in range(19):
            cur[q].copy_(0.002 + 0.001 * q / 19 + 0.01 * (torch.rand(n ** 3, device="cuda", generator=g) - 0.5))
        torch.cuda.synchronize()
        box.step(1)
        got = box.sums_history(1)[0]
        f = box.populations_tensor()
        c = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, 1, 0),
             (1, -1, 0), (-1, -1, 0), (1, 0, 1), (-1, 0, 1), (1, 0, -1), (-1, 0, -1), (0, 1, 1), (0, -1, 1),
             (0, 1, -1), (0, -1, -1)]
        j = torch.zeros((3, n ** 3), dtype=torch.float64, device="cuda")
        mass = total = 0.0
        for q in range(19):
            x = f[q].double()
            mass += float(x.sum())
            total += float(x.abs().sum())
            for a in range(3):
                if c[q][a]:
                    j[a] += c[q][a] * x
        want = np.array([mass, *(float(j[a].sum()) for a in range(3)), 0.5 * float((j * j).sum())])
    finally:
        box.close()
        torch.cuda.empty_cache()
    assert np.abs(got - want).max() <= (1e-13 if precision == "fp64" else 1e-7) * total
