"""Which launches a sweep takes by the library's own choice, on both sides of
the rules' lines."""
import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


def scan(dims, n):
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * min(dims[0], dims[1]))
    return grid, ph, synth.generate(grid, ph, n, 90, 5)


@pytest.mark.parametrize("dims,n,B,mode,chunk,threads", [
    ((64, 64, 1), 10_000, 3200, "f32", 0, 256),
    ((256, 256, 32), 51_200, 25_600, "q16", 0, 256),       # 17 tiles per CU, lists of 1,200
    ((256, 256, 32), 12_800, 3200, "q16", 0, 128),         # of 150
    ((320, 320, 64), 25_600, 12_800, "f32", 0, 128),       # 52 tiles per CU, lists of 240
    ((512, 512, 100), 25_600, 12_800, "q16", 0, 128),      # 208 tiles per CU, lists of 90
    ((64, 64, 2), 10_000, 640, "otf", 0, 256),             # one chunk
    ((64, 64, 2), 10_000, 640, "otf", 3200, 128),          # several: rows beside the launches
])
def test_lanes_of_a_tile(dims, n, B, mode, chunk, threads):
    grid, ph, h = scan(dims, n)
    print(f"lanes {dims} B {B} {mode}", flush=True)
    with tvs.Context(grid, block_size=B, path_mode=mode, chunk_histories=chunk) as ctx:
        ctx.load_histories(h)
        assert ctx.debug_sweep()[1] == threads
    with tvs.Context(grid, block_size=B, path_mode=mode, chunk_histories=chunk,
                     tile_threads=64) as ctx:
        ctx.load_histories(h)
        assert ctx.debug_sweep() == (False, 64)


@pytest.mark.parametrize("dims,n,B,mode,chain", [
    ((64, 64, 1), 400_000, 204_800, "f32", True),          # few tiles: always
    ((64, 64, 2), 3200, 3200, "q16", True),
    ((128, 128, 8), 204_800, 102_400, "f32", True),        # 1.3 tiles per CU
    ((160, 160, 12), 204_800, 25_600, "q16", True),        # 2.8
    ((160, 160, 12), 204_800, 102_400, "q16", False),
    ((200, 200, 10), 256_000, 12_800, "f32", True),        # 3.4
    ((200, 200, 10), 102_400, 51_200, "f32", False),
    ((200, 200, 10), 102_400, 51_200, "otf", False),
    ((200, 200, 16), 160_000, 6400, "f32", True),          # 5.5
    ((200, 200, 16), 51_200, 25_600, "f32", False),
    ((256, 256, 32), 320_000, 12_800, "q16", True),        # 16.7
    ((256, 256, 32), 102_400, 51_200, "q16", False),
    ((200, 200, 16), 100_000, 3200, "f32", True),          # 32 blocks of it
    ((200, 200, 16), 12_800, 3200, "f32", False),          # four
    ((256, 256, 32), 3200, 3200, "otf", False),            # one
    ((320, 320, 64), 6400, 3200, "f32", False),            # more tiles than the LDS holds
])
def test_chain_or_launches(dims, n, B, mode, chain):
    grid, ph, h = scan(dims, n)
    x0 = synth.initial_image(grid, ph)
    out = []
    for kernel in (0, 1):
        print(f"chain or launches: {dims} B {B} {mode} sweep_kernel {kernel}", flush=True)
        with tvs.Context(grid, block_size=B, path_mode=mode, sweep_kernel=kernel,
                         time_sample=1_000_000) as ctx:
            ctx.load_histories(h)
            assert ctx.debug_sweep()[0] == (chain and kernel == 0)
            ctx.set_image(x0)
            ctx.iterate(1, 0.02, 1, 0.75, seed=11)
            out.append(ctx.get_image())
            blocks = -(-n // B)
            assert ctx.stats()["k_samples"] == (blocks if chain and kernel == 0 else 0)
    np.testing.assert_array_equal(out[0], out[1])


def test_few_blocks_in_several_chunks():
    """On the fly with several chunks the rows decide: formed as one, then the
    chain, also where each group holds a few blocks."""
    grid, ph, h = scan((200, 200, 16), 19_200)
    with tvs.Context(grid, block_size=3200, chunk_histories=3200) as ctx:
        ctx.load_histories(h)
        assert ctx.debug_sweep()[0]
