"""The grid phase at every FFT length (16 to 512 points along each axis).

Each length has its own kernels (lanes and elements per lane differ), and a
workgroup holds one column or row at the long lengths and several at the
short ones, the last workgroup some spare ones.  Bars as in the parity tests:
max|E - E_ref| / max|E_ref| <= 1e-12 (FP64), 1e-5 (FP32) against the direct-sum
oracle; batched beams bit-exact to the single-beam path.
"""
import numpy as np
import pytest

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu

# full and ragged sides of every length: 16, 32, 64, 128, 256 and 512 points
SIDES = [(8, 8), (16, 12), (9, 256), (32, 20), (20, 32), (33, 64), (64, 128), (64, 40), (100, 100),
         (128, 16), (129, 68), (256, 132), (255, 256), (12, 24)]


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("nx,ny", SIDES)
def test_field_at_every_fft_length(gpu, orc, nx, ny, precision, bar):
    import torch
    print(f"[case] solve {nx}x{ny} {precision}", flush=True)
    g = inputs.make_grid(nx, ny, 6e-3, 5e-3)
    rng = np.random.Generator(np.random.PCG64(nx * 1000 + ny))
    q = np.zeros(nx * ny, dtype=np.int64)
    # 60 charged nodes, the grid's corners among them
    at = np.unique(np.concatenate([[0, ny - 1, nx * ny - ny, nx * ny - 1],
                                   rng.integers(0, nx * ny, 60)]))
    q[at] = rng.integers(1, 1 << 24, at.size)
    scale = 1.0 / (float(1 << 24) * at.size)
    want = orc.solve(q, scale, g)
    with gpu.Context(g, precision) as ctx:
        ex, ey = ctx.solve(torch.from_numpy(q).cuda(), scale)
        for got, ref in zip((ex, ey), want):
            err = np.abs(got.cpu().numpy() - ref.reshape(-1)).max() / np.abs(ref).max()
            assert err <= bar, err


@pytest.mark.parametrize("sides", [SIDES, [s for s in SIDES if max(s) <= 128]],
                         ids=["up_to_512", "up_to_256"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batched_lengths_bit_exact_to_single_beams(gpu, sides, precision):
    import torch
    print(f"[case] batch of {len(sides)} grids {precision}", flush=True)
    kappa = inputs.kappa_for_tune_shift(-0.2, 1e-6, 16)
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 4, kappa)
    grids = [inputs.make_grid(nx, ny, 6e-3, 6e-3) for nx, ny in sides]
    beams = [inputs.gaussian_beam(500 + 321 * k, 40 + k) for k in range(len(sides))]
    parts, offsets = inputs.concat_parts(beams)
    d = gpu.to_device(parts)
    with gpu.Batch(grids, offsets, precision) as b:
        b.track(d, [lat] * len(sides), 2)
        fields = [b.get_field(k) for k in range(len(sides))]
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in d.items()}
    for k, g in enumerate(grids):
        one = gpu.to_device(beams[k])
        with gpu.Context(g, precision) as ctx:
            ctx.track(one, lat, 2)
            ex, ey = ctx.get_field()
            assert torch.equal(ex, fields[k][0]) and torch.equal(ey, fields[k][1]), sides[k]
            for key, v in one.items():
                np.testing.assert_array_equal(v.cpu().numpy(),
                                              got[key][offsets[k]:offsets[k + 1]])
