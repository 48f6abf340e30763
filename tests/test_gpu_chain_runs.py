"""The resident DROP chain where it is known to run: with a time sample longer
than the sweep, the statistics count the blocks of the chain's launches, and
they must be all of them.  Images as with launches per block, bit for bit.

Cases: regions of several tiles with lists of more entries than the lanes hold
(4,096, taken in several rounds), full row tables on them, blocks past what one
launch takes (1,024), rows of several chunks formed as one; and corrections
summed in float64 on regions of several tiles (held to a few float32
roundings: their order of addition is not fixed)."""
import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


def both(grid, h, x0, B, lam, **kw):
    out = []
    n = len(h["ex"])
    for kernel in (0, 1):
        print(f"chain runs: {tuple(grid[:3])} n {n} B {B} {kw} sweep_kernel {kernel}", flush=True)
        with tvs.Context(grid, block_size=B, sweep_kernel=kernel, time_sample=10_000_000,
                         **kw) as ctx:
            ctx.load_histories(h)
            ctx.set_image(x0)
            ctx.iterate(2, lam, 2, 0.75, seed=11)
            out.append(ctx.get_image())
            assert ctx.stats()["k_samples"] == (2 * -(-n // B) if kernel == 0 else 0)
    return out


@pytest.mark.parametrize("dims,n,B,mode,chunk", [
    ((200, 200, 16), 160_000, 6400, "f32", 0),          # 5.5 tiles per CU, two rounds
    ((256, 256, 32), 256_001, 12_800, "q16", 0),        # 17 tiles per CU, three rounds
    ((160, 160, 12), 204_700, 25_600, "f16", 0),        # 2.8 tiles per CU, four rounds
    ((160, 160, 12), 153_600, 25_600, "otf", 25_600),   # the same, chunks formed as one
    ((128, 128, 8), 250_000, 102_400, "f32", 0),        # up to five tiles, full row tables
    ((150, 150, 5), 300_000, 102_400, "q16", 0),        # about one tile, 20 rounds
    ((64, 64, 1), 220_000, 200, "f32", 0),              # 1,100 blocks: two launches
    ((128, 128, 4), 440_001, 400, "otf", 0),            # 1,101 of them, the last one ragged
])
def test_chain_runs_and_equals_launches(dims, n, B, mode, chunk):
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * min(dims[0], dims[1]))
    h = synth.generate(grid, ph, n, 90, 77)
    x0 = synth.initial_image(grid, ph)
    a, b = both(grid, h, x0, B, 0.02, path_mode=mode, chunk_histories=chunk)
    assert np.max(np.abs(a - x0)) > 1e-3
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("dims,n,B", [((200, 200, 16), 153_600, 6400),
                                      ((160, 160, 12), 204_800, 25_600),
                                      ((256, 256, 32), 256_000, 12_800)])
def test_chain_runs_with_large_corrections(dims, n, B):
    """Rows that clip a corner of every slice by a short chord, from a zero image:
    corrections past 2^21 / B."""
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    h = synth.generate(grid, synth.catphan_like(grid, 0.75 * min(dims[0], dims[1])), n, 90, 3)
    rng = np.random.default_rng(1)
    k = rng.choice(n, 400, replace=False)
    cut = rng.uniform(0.002, 0.2, 400)
    cx, cy = 0.5 * dims[0], 0.5 * dims[1]
    for key, v in dict(ex=cx - cut - 5, ey=cy + 5, qx=cx + 5, qy=cy - cut - 5, eth=0, eps=0, qth=0,
                       qps=0, ux=2 ** -0.5, uy=-2 ** -0.5, wepl=150.0).items():
        h[key][k] = v
    h["qz"][k] = h["ez"][k]
    a, b = both(grid, h, np.zeros(grid.nvox, np.float32), B, 0.02, path_mode="f32")
    assert np.max(np.abs(a)) > 1.0
    assert np.max(np.abs(a.astype(np.float64) - b) / np.maximum(np.abs(b), 0.1)) <= 1e-6
