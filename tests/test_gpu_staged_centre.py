"""Field boxes of which only the centre, or nothing, fits in LDS beside the charge tile, through the C ABI:
the streamed pass (arrays above 128 MiB) against the per-element calls, whose kick on a context without a
previous deposit knows no box and gathers from memory; the B-spline gather against the oracle.
"""
import numpy as np
import pytest
import torch

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu


# FP64 (16-byte nodes) and mixed (8): the box fits whole (64^2, 128^2 narrow); its centre does, a third of it
# (128^2 wide), a quarter (160x128), in FP64 an eighth or less (180x152); nothing fits (200^2).
@pytest.mark.parametrize("nx,ny,sigma", [(64, 64, 1e-3), (128, 128, 1e-3), (128, 128, 2.5e-3),
                                         (160, 128, 2.5e-3), (180, 152, 2.5e-3), (200, 200, 2.5e-3)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("weights", [False, True])
def test_streamed_kicks_equal_the_calls(gpu, nx, ny, sigma, precision, weights):
    n, kappa = 4_300_001, 2e-8
    print(f"[case] streamed centre grid={nx}x{ny} sigma={sigma} {precision} weights={weights}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx + ny)
    p = {k: torch.randn(n, generator=gen, dtype=torch.float64, device="cuda") * s
         for k, s in (("x", sigma), ("px", 1e-3), ("y", sigma), ("py", 1e-3))}
    p["lost"] = torch.zeros(n, dtype=torch.uint8, device="cuda")
    if weights:
        p["w"] = torch.rand(n, generator=gen, dtype=torch.float32, device="cuda")
    q = {k: v.clone() for k, v in p.items()}
    g = inputs.make_grid(nx, ny, 6e-3, 6e-3)
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 1, kappa, four_by_four=True)

    def fresh():
        return gpu.Context(g, precision)

    with fresh() as ctx:
        ctx.track(p, lat, 3)
    for _ in range(3):
        with fresh() as ctx:
            ctx.push(q, lat[:1])
            rho, _ = ctx.deposit(q)
            ex, ey = ctx.solve(rho, 1.0 / (2.0 ** 24 * n))
        with fresh() as ctx:
            ctx.kick(q, ex, ey, kappa)
    torch.cuda.synchronize()
    for k in p:
        assert torch.equal(p[k], q[k]), k


def _bar(orc, p, grid, kappa, kicks, ref):
    """An FP32 potential within 1e-5 of max|phi| moves the gradient by at most 1e-5 max|phi| times 2 (the sum
    of |B'| over the stencil) per spacing and axis; over the kicks, relative to the rms momenta, times 2."""
    q, _ = orc.deposit(inputs.copy_parts(p), grid)
    phi = orc.potential(q, 1.0 / ((1 << 24) * len(p["x"])), grid)
    de = 1e-5 * np.abs(phi).max() * 2.0 / min(grid["dx"], grid["dy"])
    return 2 * kicks * kappa * de / min(ref["px"].std(), ref["py"].std())


# FP64 (8-byte nodes): centre (128^2), nothing (180x152, 256^2); mixed (4): whole, centre (180x140), nothing
@pytest.mark.parametrize("nx,ny", [(128, 128), (180, 140), (180, 152), (256, 256)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_bspline_centre_matches_oracle(gpu, orc, nx, ny, precision):
    n, kappa = 60_001, 4e-7
    print(f"[case] B-spline centre grid={nx}x{ny} {precision}", flush=True)
    g = inputs.make_grid(nx, ny, 6e-3, 6e-3)
    p = inputs.gaussian_beam(n, 17, 2.5e-3, 1e-3, 2.5e-3, 1e-3)
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 2, kappa, four_by_four=True)
    ref = inputs.copy_parts(p)
    orc.track(ref, g, lat, 1, gather="bspline")
    with gpu.Context(g, precision) as ctx:
        ctx.set_option(gpu.OPT_GATHER, gpu.GATHER_BSPLINE)
        ctx.set_option(gpu.OPT_PASS_BLOCKS, 2)  # many particles per lane: the staged form
        d = gpu.to_device(p)
        ctx.track(d, lat, 1)
        got = gpu.to_host(d)
    bar = 1e-10 if precision == "fp64" else _bar(orc, p, g, kappa, 2, ref)
    alive = ref["lost"] == 0
    if precision == "fp64":
        np.testing.assert_array_equal(got["lost"], ref["lost"])
    else:
        alive &= got["lost"] == 0
        assert alive.sum() >= 0.999 * (ref["lost"] == 0).sum()
    err = max(np.abs(got[k] - ref[k])[alive].max() / ref[k].std() for k in ("x", "px", "y", "py"))
    print(f"[centre] {nx}x{ny} {precision}: {err:.3e} (bar {bar:.3e})", flush=True)
    assert err <= bar
