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


# arrays above 128 MiB: the streamed form, in step with 1024 threads and ordered below
@pytest.mark.parametrize("four_by_four", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_streamed_sizes_give_the_same_bits(gpu, four_by_four, precision):
    print(f"[case] streamed pass threads 4x4={four_by_four} {precision}", flush=True)
    p = inputs.gaussian_beam(4_300_001, 3, 2e-3, 1e-3, 2e-3, 1e-3)
    p["lost"][1000:70_000] = 1
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 2, 2e-8, four_by_four=four_by_four, k2l=5.0, sext_every=2)
    ref = None
    for threads in (0, 256, 512, 1024):
        with gpu.Context(inputs.make_grid(128), precision) as ctx:
            ctx.set_option(gpu.OPT_PASS_THREADS, threads)
            d = gpu.to_device(p)
            ctx.track(d, lat, 2)
            got = gpu.to_host(d)
        ref = ref or got
        for k in p:
            np.testing.assert_array_equal(got[k], ref[k], err_msg=f"{threads} {k}")
