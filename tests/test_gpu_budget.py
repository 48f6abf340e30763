"""The resident DROP chain under a short budget: its workspace gives way only to
a call that then fits, and comes back when the call has given its memory back.

Whether a sweep took the chain is read from the statistics: with a time sample
longer than the sweep only launches of many blocks are timed, and they count
every block."""
import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu

N, B = 60_000, 3200
BLOCKS = -(-N // B)
HULL = dict(wepl_in_mm=10.0, wepl_out_mm=1.0, min_in=1, max_out=3)
BATCH = [dict(lam=0.02, N=1, alpha=0.75, seed=q) for q in range(32)]


@pytest.fixture(scope="module")
def scan():
    grid = synth.centered_grid(64, 64, 4, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 48.0)
    return grid, synth.generate(grid, ph, N, 60, 5), synth.initial_image(grid, ph)


def context(scan, budget=0, mode="f32"):
    ctx = tvs.Context(scan[0], block_size=B, path_mode=mode, time_sample=1_000_000,
                      hbm_budget_bytes=budget)
    ctx.load_histories(scan[1])
    return ctx


def cycle(ctx, scan):
    """One cycle's image, and the blocks that the chain ran."""
    ctx.set_image(scan[2])
    ctx.iterate(1, 0.02, 2, 0.75, seed=11)
    return ctx.get_image(), ctx.stats()["k_samples"]


@pytest.fixture(scope="module")
def plain(scan):
    with context(scan) as ctx:
        held = ctx.stats()["device_bytes"]
        image, blocks = cycle(ctx, scan)
        assert blocks == BLOCKS
        return held, image, ctx.hull_detect(**HULL)


@pytest.mark.parametrize("call", [
    lambda c: c.initial_fbp(7200, median_radius=0),     # 28 B for each of 2.8 M bins
    lambda c: c.iterate_batch(1, BATCH),                # 32 images and subgradients
])
def test_refused_call_leaves_the_chain(scan, plain, call):
    held, want, _ = plain
    with context(scan, held + 1024) as ctx:
        with pytest.raises(tvs.TvsError) as e:
            call(ctx)
        assert e.value.status == tvs.TVS_ENOMEM
        image, blocks = cycle(ctx, scan)
        assert blocks == BLOCKS
        np.testing.assert_array_equal(image, want)


@pytest.mark.parametrize("mode", ["f32", "otf"])
def test_chain_comes_back_after_a_call_that_took_its_room(scan, plain, mode):
    with context(scan, mode=mode) as ctx:
        held = ctx.stats()["device_bytes"]
    with context(scan, held + 1024, mode) as ctx:
        for _ in range(2):
            np.testing.assert_array_equal(ctx.hull_detect(**HULL), plain[2])
            assert ctx.stats()["device_bytes"] == held
            image, blocks = cycle(ctx, scan)
            assert blocks == BLOCKS
            np.testing.assert_array_equal(image, plain[1])


def test_launches_while_a_batch_holds_the_room(scan, plain):
    """Images of a batch that stay: per-block launches, the same image; a load
    whose histories leave room brings the chain back."""
    with context(scan) as ctx:
        ctx.iterate_batch(1, BATCH[:4])
        held = ctx.stats()["device_bytes"]
    with context(scan, held - 1024) as ctx:
        ctx.iterate_batch(1, BATCH[:4])
        image, blocks = cycle(ctx, scan)
        assert blocks == 0
        np.testing.assert_array_equal(image, plain[1])
        half = {k: v[: N // 2] for k, v in scan[1].items()}
        ctx.load_histories(half)
        cycle(ctx, scan)
        assert ctx.stats()["k_samples"] == -(-N // 2 // B)
        assert ctx.stats()["device_bytes"] <= held - 1024
