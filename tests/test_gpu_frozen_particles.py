"""Frozen (lost) particles, through the C ABI: no pass stores a wave of them, none changes one, and none
treats a moving particle beside them differently.
"""
import numpy as np
import pytest
import torch

from paper_2010_11540_amd import inputs

pytestmark = pytest.mark.gpu

WAVE, GROUP = 64, 512


def _frozen(n, seed):
    """Whole workgroups, whole waves, half a wave, single lanes, and the last particles."""
    lost = np.zeros(n, dtype=np.uint8)
    lost[:3 * GROUP] = 1
    lost[5 * GROUP:5 * GROUP + 7 * WAVE] = 1
    lost[7 * GROUP + WAVE // 2:8 * GROUP] = 1
    rng = np.random.Generator(np.random.PCG64(seed))
    lost[rng.integers(0, n, n // 50)] = 1
    lost[-70:] = 1
    return lost


def _run(gpu, form, parts, graph):
    n = len(parts["x"])
    if form == "batch":
        cut = n // 3
        grids = [inputs.make_grid(64), inputs.make_grid(128)]
        lat = inputs.ring(4.2 / 4, 4.3 / 4, 4, 0.0, four_by_four=True)
        d = gpu.to_device(parts)
        with gpu.Batch(grids, [0, cut, n]) as b:
            b.track(d, [lat, lat], 2)
            torch.cuda.synchronize()
        return gpu.to_host(d)
    six = form in ("thick", "line")
    lat = (inputs.fodo_thick(4, 4.2 / 25, 0.0) if six else
           inputs.ring(4.2 / 4, 4.3 / 4, 4, 0.0, four_by_four=form != "two", k2l=5.0, sext_every=2))
    with gpu.Context(inputs.make_grid(64, 64) if form == "line" else inputs.make_grid(128, 100),
                     "mixed" if form == "mixed" else "fp64") as ctx:
        ctx.set_option(gpu.OPT_USE_GRAPH, int(graph))
        if form == "bspline":
            ctx.set_option(gpu.OPT_GATHER, gpu.GATHER_BSPLINE)
        if form == "line":
            ctx.set_option(gpu.OPT_SOLVER, gpu.SOLVER_PIPE)
            ctx.set_line_density(inputs.make_line(4.0, 64))
        d = gpu.to_device(parts)
        if form == "push":
            ctx.push(d, lat[lat["kind"] != inputs.SC][:2])
        else:
            ctx.track(d, lat, 2)
        torch.cuda.synchronize()
    return gpu.to_host(d)


# one round per lane or fewer (the whole grid as the tile, where that is a form), several (the staged
# box), and arrays above 128 MiB (streamed); without charge (kappa = 0) a particle's motion does not
# depend on the others'
@pytest.mark.parametrize("form,n", [(f, n) for f in ("four", "two", "mixed", "push", "batch", "thick",
                                                     "line", "bspline") for n in (30_011, 700_001)]
                         + [(f, 4_300_001) for f in ("four", "two", "push", "batch")])
def test_frozen_particles_stay_and_the_others_move(gpu, form, n):
    print(f"[case] frozen particles {form} n={n}", flush=True)
    # a wide beam: particles leave the grid during the track
    make = inputs.gaussian_beam6d if form in ("thick", "line") else inputs.gaussian_beam
    p = make(n, 13, 2.5e-3, 1e-3, 2.5e-3, 1e-3)
    free = _run(gpu, form, p, True)
    lost = _frozen(n, 3)
    q = inputs.copy_parts(p)
    q["lost"][:] = lost
    got = _run(gpu, form, q, n < 100_000)
    on = lost == 0
    if form != "push":
        assert free["lost"].any() and not free["lost"].all()
    np.testing.assert_array_equal(got["lost"], np.where(on, free["lost"], 1))
    for k in p:
        if k != "lost":
            np.testing.assert_array_equal(got[k][on], free[k][on], err_msg=k)
            np.testing.assert_array_equal(got[k][~on], p[k][~on], err_msg=k)


# A particle that moves is read and written (65 bytes in four dimensions), a frozen one only read (33):
# half the traffic.  The bound leaves the rest of a step (grid phase, launches), the same for both, its share.
@pytest.mark.parametrize("op,n", [("push", 8_000_000), ("track", 8_000_000), ("track", 3_000_000)])
def test_a_lost_beam_is_not_written_again(gpu, op, n):
    print(f"[case] lost beam {op} n={n}", flush=True)
    p = gpu.to_device(inputs.gaussian_beam(n, 7, 1e-3, 1e-3, 1e-3, 1e-3))
    lat = inputs.ring(4.2 / 4, 4.3 / 4, 4, 0.0)
    best = {}
    with gpu.Context(inputs.make_grid(64, 64)) as ctx:
        def call():
            if op == "push":
                ctx.push(p, lat[:1])
            else:
                ctx.track(p, lat, 2)
        for lost in (0, 1):
            p["lost"].fill_(lost)
            times = []
            for _ in range(8):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                for _ in range(4):
                    call()
                b.record()
                b.synchronize()
                times.append(a.elapsed_time(b))
            best[lost] = min(times)
    print(f"[lost beam] {op} n={n}: moving {best[0]:.3f} ms, lost {best[1]:.3f} ms", flush=True)
    assert best[1] <= 0.75 * best[0]
