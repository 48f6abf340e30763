"""A refused launch of the resident chain (another process held the device's
cooperative queue), forced from the host: the sweep goes on by per-block
launches, the next ones by launches beside the row formation, and then the
chain is tried again.  The images are the same all along.

With a time sample longer than the sweep, the statistics count the blocks that
the chain ran."""
import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu

N, B, CHUNK = 40_000, 640, 3200        # 13 chunks in groups of three, the last one of one
BLOCKS = -(-N // B)
GROUP = 3 * CHUNK // B


@pytest.fixture(scope="module")
def scan():
    grid = synth.centered_grid(48, 40, 2, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 30.0)
    return grid, synth.generate(grid, ph, N, 60, 5), synth.initial_image(grid, ph)


def cycles(scan, n, refuse_before, chunk, **kw):
    images, blocks = [], []
    with tvs.Context(scan[0], block_size=B, chunk_histories=chunk, time_sample=1_000_000,
                     **kw) as ctx:
        ctx.load_histories(scan[1])
        ctx.set_image(scan[2])
        for q in range(n):
            if q == refuse_before:
                ctx.debug_sweep(2)
            ctx.iterate(1, 0.02, 1, 0.75, seed=11)
            images.append(ctx.get_image())
            blocks.append(ctx.stats()["k_samples"])
    return images, blocks


def test_chain_is_tried_again_after_a_refused_launch(scan):
    want, none = cycles(scan, 20, None, CHUNK, sweep_kernel=1)
    assert none == [0] * 20
    got, blocks = cycles(scan, 20, 1, CHUNK)
    assert blocks == [BLOCKS, BLOCKS - GROUP] + [0] * 15 + [BLOCKS] * 3
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


def test_one_chunk_is_tried_every_sweep(scan):
    got, blocks = cycles(scan, 4, 1, N)
    assert blocks == [BLOCKS, 0, BLOCKS, BLOCKS]
    want, _ = cycles(scan, 4, None, N, sweep_kernel=1)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)
