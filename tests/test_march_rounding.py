"""The DUGKS march gives the same populations bit for bit whatever its work
split: z-chunk, column-tile width and width of the address offsets."""
import numpy as np
import pytest

import synth


@pytest.mark.gpu
@pytest.mark.parametrize("mesh", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [5, 31, 40])
def test_tile_widths_and_chunks_same_bits(n, precision, mesh):
    """Both tile widths, which share the faces of a tile differently between
    their wavefronts, and chunks that start on even and odd planes (the FP32
    march takes two planes per turn), five steps."""
    import paper_1601_03815_amd as dhit
    f0 = synth.random_populations(n, seed=900 + n, amplitude=0.01)
    want = None
    for tile in (32, 16):
        for chunk in (0, 1, 2, 3, n // 2, n):
            with dhit.Box(n, "dugks", precision, 0.02, dt=0.37, rho0=1.1, tile_width=tile, z_chunk=chunk) as b:
                if mesh:
                    b.set_mesh(synth.stretched_widths(n))
                b.set_populations(f0)
                b.step(5)
                got = b.get_populations()
            want = got if want is None else want
            np.testing.assert_array_equal(got, want, err_msg="tile %d chunk %d" % (tile, chunk))


@pytest.mark.gpu
@pytest.mark.parametrize("mesh", [False, True])
@pytest.mark.parametrize("tile,chunk", [(32, 21), (16, 37)])
@pytest.mark.parametrize("precision,n", [("fp32", 1024), ("fp64", 816)])
def test_largest_boxes_same_bits_as_small_ones(precision, n, tile, chunk, mesh):
    """Boxes whose population arrays pass 4 GB (64-bit offsets) and repeat a
    16^3 box along each axis, widths too: one step equals the small box's, every
    cell, bit for bit.  Odd chunks put the images on even and odd planes."""
    import torch

    import paper_1601_03815_amd as dhit
    P = 16
    reps = n // P
    dt = torch.float64 if precision == "fp64" else torch.float32
    f16 = synth.random_populations(P, seed=n, amplitude=0.01)
    if precision == "fp32":
        f16 = f16.astype(np.float32).astype(np.float64)
    w16 = synth.stretched_widths(P)
    with dhit.Box(P, "dugks", precision, 0.0025, dt=0.4) as b:
        if mesh:
            b.set_mesh(w16)
        b.set_populations(f16)
        b.step(1)
        want = b.get_populations()
    print("largest: %s n=%d tile %d mesh %s" % (precision, n, tile, mesh), flush=True)
    torch.cuda.empty_cache()   # the box takes 150-170 GB: return what earlier tests cached
    box = dhit.Box(n, "dugks", precision, 0.0025, dt=0.4, tile_width=tile, z_chunk=chunk)
    try:
        if mesh:
            box.set_mesh(np.tile(w16, (1, reps)))
        cur = box.populations_tensor()
        with torch.cuda.stream(box.stream):
            for q in range(19):
                t = torch.from_numpy(f16[q]).to("cuda", dt)
                cur[q].view(n, n, n).copy_(t.repeat(reps, reps, reps))
        box.stream.synchronize()
        box.step(1)
        got = box.populations_tensor()
        bad = 0
        with torch.cuda.stream(box.stream):
            for q in range(19):
                r = torch.from_numpy(want[q]).to("cuda", dt)[:, None, :, None, :]
                g = got[q].view(reps, P, reps, P, reps, P)
                bad += sum(int((g[k] != r).sum()) for k in range(reps))
        assert bad == 0
    finally:
        box.close()
        torch.cuda.empty_cache()
