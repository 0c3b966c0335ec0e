"""The B-spline gather from the potential box staged in LDS (wholly, its centre, or not at all)
against the gather from memory, through the C ABI: the same arithmetic on the same nodes, and an exact
deposit, so the same bits.
"""
import numpy as np
import pytest

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu


# a beam inside the grid; one over the whole domain, to its edge (particles
# leave); boxes that fit beside the charge tile, in part, or not (256^2)
@pytest.mark.parametrize("nx,ny,sigma", [(64, 32, 1e-3), (36, 24, 4e-3), (132, 100, 3e-3),
                                         (180, 152, 2.5e-3), (256, 256, 3e-3), (16, 256, 2e-3)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("thick", [False, True])
def test_staged_potential_gives_the_same_bits(gpu, nx, ny, sigma, precision, thick):
    n = 60_001
    print(f"[case] staged B-spline gather grid={nx}x{ny} {precision} thick={thick}", flush=True)
    g = inputs.make_grid(nx, ny, 6e-3, 6e-3)
    if thick:
        p = inputs.gaussian_beam6d(n, 31, sigma, 1e-4, sigma, 1e-4)
        lat = inputs.fodo_thick(4, 4.2 / 25, 2e-8)
    else:
        p = inputs.gaussian_beam(n, 31, sigma, 1e-3, sigma, 1e-3)
        lat = inputs.ring(4.2 / 4, 4.3 / 4, 4, 2e-8, four_by_four=True)
    outs = []
    # 60 particles and more per lane (the staged form), then 1 (the whole grid as the tile wherever
    # that fits)
    for blocks, threads in ((2, 512), (0, 0)):
        with gpu.Context(g, precision) as ctx:
            ctx.set_option(gpu.OPT_GATHER, gpu.GATHER_BSPLINE)
            if blocks:
                ctx.set_option(gpu.OPT_PASS_BLOCKS, blocks)
                ctx.set_option(gpu.OPT_PASS_THREADS, threads)
            d = gpu.to_device(p)
            ctx.track(d, lat, 3)
            outs.append({k: v.cpu().numpy() for k, v in d.items()})
    assert np.abs(outs[0]["px"] - p["px"]).max() > 0
    for k in p:
        np.testing.assert_array_equal(outs[0][k], outs[1][k], err_msg=k)
