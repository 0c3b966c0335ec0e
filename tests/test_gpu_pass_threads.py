"""The workgroup size option through the C ABI: every size gives the same bits, zero returns a context to the
automatic choice, and other values are refused."""
import numpy as np
import pytest

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu


# the edges of the automatic choice on a small and on a large grid
@pytest.mark.parametrize("n", [65_536, 65_537, 131_072, 131_073])
@pytest.mark.parametrize("nx", [64, 128])
def test_back_to_the_automatic_size(gpu, n, nx):
    print(f"[case] pass threads n={n} grid={nx}", flush=True)
    p = inputs.gaussian_beam(n, 3, 1e-3, 1e-3, 1e-3, 1e-3)
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 4, 2e-8)

    def track(ctx):
        d = gpu.to_device(p)
        ctx.track(d, lat, 2)
        return gpu.to_host(d)

    with gpu.Context(inputs.make_grid(nx)) as ctx:
        ref = track(ctx)
        for threads in (256, 1024, 0, 512, 0):
            ctx.set_option(gpu.OPT_PASS_THREADS, threads)
            got = track(ctx)
            for k in p:
                np.testing.assert_array_equal(got[k], ref[k], err_msg=f"{threads} {k}")
        for threads in (-1, 1, 64, 128, 768, 2048):
            with pytest.raises(gpu.ScpicError) as e:
                ctx.set_option(gpu.OPT_PASS_THREADS, threads)
            assert e.value.code == gpu.EINVAL
