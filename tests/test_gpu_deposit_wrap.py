"""Deposits whose 32-bit LDS cells wrap (256 particles of one workgroup on a node), through the C ABI,
at the particle counts where a wave's or a workgroup's last round is full, ragged or missing: each
call must give the oracle's exact charge whatever the previous one left.
"""
import numpy as np
import pytest

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu


def _on_nodes(n, grid, nodes, spread, seed):
    """n particles spread over `nodes` random nodes, off them by up to `spread` cells."""
    rng = np.random.Generator(np.random.PCG64(seed))
    i = rng.integers(2, grid["nx"] - 2, nodes)[rng.integers(0, nodes, n)]
    j = rng.integers(2, grid["ny"] - 2, nodes)[rng.integers(0, nodes, n)]
    return {"x": grid["x_min"] + (i + spread * rng.random(n)) * grid["dx"],
            "px": rng.standard_normal(n) * 1e-3,
            "y": grid["y_min"] + (j + spread * rng.random(n)) * grid["dy"],
            "py": rng.standard_normal(n) * 1e-3, "lost": np.zeros(n, dtype=np.uint8)}


@pytest.mark.parametrize("n", [255, 256, 257, 512, 131_072, 131_073, 600_001])
@pytest.mark.parametrize("nx,ny", [(32, 32), (256, 256)])
def test_wraps_come_and_go_bit_exact(gpu, orc, n, nx, ny):
    print(f"[case] deposit wraps n={n} grid={nx}x{ny}", flush=True)
    g = inputs.make_grid(nx, ny)
    # wraps on one node, beside it, nowhere (twice), on two nodes
    beams = [_on_nodes(n, g, 1, 0.0, 1), _on_nodes(n, g, 1, 1e-3, 2), _on_nodes(n, g, 40_000, 1.0, 3),
             _on_nodes(n, g, 3000, 1.0, 4), _on_nodes(n, g, 2, 1e-3, 5)]
    with gpu.Context(g) as ctx:
        for k, p in enumerate(beams):
            q_ref, n_ref = orc.deposit(inputs.copy_parts(p), g)
            for lost in (True, False):
                d = gpu.to_device({key: v for key, v in p.items() if lost or key != "lost"})
                rho, n_in = ctx.deposit(d)
                np.testing.assert_array_equal(rho.cpu().numpy(), q_ref, err_msg=f"beam {k}")
                assert int(n_in.item()) == n_ref == n


@pytest.mark.parametrize("n,ring", [(1, "maps"), (63, "maps"), (65, "sext"), (4096, "maps"),
                                    (131_073, "sext"), (262_145, "maps"), (700_001, "sext")])
def test_track_of_a_dense_beam(gpu, orc, n, ring):
    """A beam a tenth of a cell wide on a coarse grid, every depositing pass of
    the track wrapping cells; the elements are one resident map, or a map and
    a sextupole.  No space charge (kappa = 0): the
    coordinates are the maps' own, bit for bit; the field is the oracle's."""
    print(f"[case] dense track n={n} {ring}", flush=True)
    g = inputs.make_grid(16, 16, 6e-3, 6e-3)
    p = inputs.gaussian_beam(n, 77, 5e-5, 5e-5, 5e-5, 5e-5)
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 4, 0.0, four_by_four=ring == "sext",
                      k2l=5.0 if ring == "sext" else 0.0, sext_every=1 if ring == "sext" else 0)
    ref = inputs.copy_parts(p)
    for _ in range(2):
        orc.push(ref, lat)
    q_ref, _ = orc.deposit(inputs.copy_parts(ref), g)
    ex, ey = orc.solve(q_ref, 1.0 / (float(1 << 24) * n), g)
    with gpu.Context(g) as ctx:
        d = gpu.to_device(p)
        ctx.track(d, lat, 2)
        got = ctx.get_field()
        for key in ("x", "px", "y", "py", "lost"):
            np.testing.assert_array_equal(d[key].cpu().numpy(), ref[key], err_msg=key)
        for u, v in zip(got, (ex, ey)):
            assert np.abs(u.cpu().numpy() - v.reshape(-1)).max() <= 1e-12 * np.abs(v).max()
