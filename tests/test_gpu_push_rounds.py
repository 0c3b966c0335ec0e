"""Push-only calls at the particle counts where a lane's rounds begin and end (512 workgroups of 1024
lanes; arrays above 128 MiB are streamed, two rounds ahead), through the C ABI, against the oracle: the
linear maps are exact, so the same bits.
"""
import numpy as np
import pytest

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu

LANES = 512 * 1024


@pytest.mark.parametrize("n", [1, 65, LANES - 1, LANES, LANES + 1, 2 * LANES, 2 * LANES + 63,
                               8 * LANES + 1, 9 * LANES - 64])
def test_push_rounds_bit_exact(gpu, orc, n):
    print(f"[case] push n={n}", flush=True)
    p = inputs.gaussian_beam(n, 5, 1e-3, 1e-3, 1e-3, 1e-3)
    p["lost"][::7] = 1  # frozen particles keep their coordinates
    e = inputs.ring(4.2 / 4, 4.3 / 4, 4, 0.0, four_by_four=True)
    e = e[e["kind"] != inputs.SC][:2]
    ref = inputs.copy_parts(p)
    orc.push(ref, e)
    with gpu.Context(inputs.make_grid(32, 32, 6e-3, 6e-3)) as ctx:
        d = gpu.to_device(p)
        ctx.push(d, e)
        for k in p:
            np.testing.assert_array_equal(d[k].cpu().numpy(), ref[k], err_msg=k)
