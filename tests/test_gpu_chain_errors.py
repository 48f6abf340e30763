"""Errors of the resident DROP chain, forced from the host: a workgroup missing
at the barrier leaves counters that no longer match the launches queued behind
it.  Those end at once, also after the error flag was cleared by a new image;
the error is reported, and the context goes on with per-block launches."""
import time

import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(64, 64, 2), (200, 200, 8)])   # shared tiles, whole ones
def scan(request):
    grid = synth.centered_grid(*request.param, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * request.param[0])
    return grid, synth.generate(grid, ph, 80_000, 60, 5), synth.initial_image(grid, ph)


def context(scan, **kw):
    ctx = tvs.Context(scan[0], block_size=800, path_mode="f32", **kw)
    ctx.load_histories(scan[1])
    ctx.set_image(scan[2])
    return ctx


def cycle(ctx):
    ctx.iterate(1, 0.02, 2, 0.75, seed=11)


@pytest.mark.parametrize("new_image_before_the_check", [False, True])
def test_sweeps_after_a_time_out_end_at_once(scan, new_image_before_the_check):
    with context(scan, sweep_kernel=1) as ctx:
        assert not ctx.debug_sweep()[0]
        cycle(ctx)
        want = ctx.get_image()
    with context(scan) as ctx:
        assert ctx.debug_sweep()[0]
        cycle(ctx)
        np.testing.assert_array_equal(ctx.get_image(), want)
        print(f"time-out state, {scan[0]}", flush=True)
        assert ctx.debug_sweep(1)[0]
        t = time.monotonic()
        for _ in range(3):
            cycle(ctx)
            if new_image_before_the_check:
                ctx.set_image(scan[2])
        cycle(ctx)
        with pytest.raises(tvs.TvsError) as e:
            ctx.get_image()
        assert time.monotonic() - t < 5.0
        assert e.value.status == tvs.TVS_EDEVICE
        assert not ctx.debug_sweep()[0]
        ctx.set_image(scan[2])                  # goes on, block by block
        cycle(ctx)
        np.testing.assert_array_equal(ctx.get_image(), want)
        ctx.load_histories(scan[1])             # and with the chain again
        ctx.set_image(scan[2])
        assert ctx.debug_sweep()[0]
        cycle(ctx)
        np.testing.assert_array_equal(ctx.get_image(), want)


def test_debug_sweep_refuses_other_requests(scan):
    with tvs.Context(scan[0]) as ctx:
        with pytest.raises(tvs.TvsError) as e:
            ctx.debug_sweep()
        assert e.value.status == tvs.TVS_ESTATE
        ctx.load_histories(scan[1])
        for what in (-1, 7):
            with pytest.raises(tvs.TvsError) as e:
                ctx.debug_sweep(what)
            assert e.value.status == tvs.TVS_EINVAL
