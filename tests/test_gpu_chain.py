"""The resident DROP chain against one launch per block, through the C ABI.

Both sum the same rounded integers, so their images are equal bit for bit;
only the float64 side sums of very large corrections depend on the order of
additions (held to a few float32 roundings).  Cases: several workgroups per
tile (few tiles), one tile and several tiles per workgroup, ragged last
blocks and lists, lists longer than the lanes hold, more rows in a tile than
its table has slots, every entry form, an empty scan, and grids or blocks
past the chain's limits (which take the launches)."""
import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


def images(grid, h, x0, cycles, lam, **cfg):
    out = []
    for kernel in (0, 1):
        print(f"chain case {tuple(grid[:3])} {cfg} sweep_kernel {kernel}", flush=True)
        with tvs.Context(grid, sweep_kernel=kernel, **cfg) as ctx:
            ctx.load_histories(h)
            ctx.set_image(x0)
            ctx.iterate(cycles, lam, 2, 0.75, seed=11)
            out.append(ctx.get_image())
            ctx.iterate(1, lam, 2, 0.75, seed=11)      # goes on from the chain's image
            out.append(ctx.get_image())
    return out[0], out[1], out[2], out[3]


@pytest.mark.parametrize("dims,n,angles,B,mode,chunk", [
    ((16, 16, 1), 3000, 20, 3200, "f32", 0),        # one tile, one block, 32 workgroups at most
    ((17, 33, 2), 20_011, 30, 997, "otf", 3000),    # rows of tiles one voxel wide, ragged blocks
    ((64, 64, 1), 60_000, 90, 3200, "f32", 0),      # 16 workgroups per tile
    ((64, 64, 1), 60_000, 90, 64, "q16", 0),        # short lists
    ((64, 64, 1), 60_000, 90, 30_000, "f16", 0),    # lists longer than the lanes hold, full tables
    ((128, 128, 3), 150_000, 60, 3200, "q16", 0),   # about half a tile per CU
    ((131, 97, 7), 120_000, 90, 1009, "f16", 0),    # about one tile per CU
    ((200, 200, 16), 200_000, 180, 3200, "otf", 64_000),
    ((200, 200, 16), 200_000, 180, 25_600, "f32", 0),
    ((256, 256, 32), 250_000, 360, 25_600, "q16", 0),   # about 17 tiles per CU
    ((256, 256, 32), 100_000, 360, 3200, "otf", 0),
])
def test_chain_equals_launches(dims, n, angles, B, mode, chunk):
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * min(dims[0], dims[1]))
    h = synth.generate(grid, ph, n, angles, 77)
    x0 = synth.initial_image(grid, ph)
    a, a2, b, b2 = images(grid, h, x0, 2, 0.02, block_size=B, path_mode=mode,
                          chunk_histories=chunk)
    assert np.max(np.abs(a - x0)) > 1e-3
    np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(a2, b2)


@pytest.mark.parametrize("dims,B", [((64, 64, 1), 8000), ((131, 97, 7), 50_000),
                                    ((200, 200, 16), 200_000)])
def test_chain_large_corrections(dims, B):
    """From a zero image with rows that clip the grid's corner by a short chord:
    corrections past 2^21 / B, which are summed in float64."""
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    h = synth.generate(grid, synth.catphan_like(grid, 0.75 * min(dims[0], dims[1])), 200_000, 90, 3)
    rng = np.random.default_rng(1)
    k = rng.choice(200_000, 400, replace=False)
    cut = rng.uniform(0.002, 0.2, 400)                 # lines across one corner
    cx, cy = 0.5 * dims[0], 0.5 * dims[1]
    for key, v in dict(ex=cx - cut - 5, ey=cy + 5, qx=cx + 5, qy=cy - cut - 5, eth=0, eps=0, qth=0,
                       qps=0, ux=2 ** -0.5, uy=-2 ** -0.5, wepl=150.0).items():
        h[key][k] = v
    h["qz"][k] = h["ez"][k]
    x0 = np.zeros(grid.nvox, np.float32)
    a, a2, b, b2 = images(grid, h, x0, 2, 0.02, block_size=B, path_mode="f32")
    assert np.max(np.abs(a)) > 1.0                     # a corner voxel took large corrections
    for x, ref in ((a, b), (a2, b2)):
        assert np.max(np.abs(x.astype(np.float64) - ref) / np.maximum(np.abs(ref), 0.1)) <= 1e-6


def test_chain_of_no_rows():
    """Histories that all miss the grid, and none at all."""
    grid = synth.centered_grid(48, 48, 2, 1.0, 1.0, 2.5)
    h = synth.miss_histories(grid, 80.0, 5000, 5)
    x0 = np.linspace(0, 1, grid.nvox).astype(np.float32)
    for hist in (h, {k: v[:0] for k, v in h.items()}):
        with tvs.Context(grid, block_size=640, path_mode="f32") as ctx:
            ctx.load_histories(hist)
            ctx.set_image(x0)
            ctx.iterate(2, 0.02, 0, 0.75)
            np.testing.assert_array_equal(ctx.get_image(), x0)


def test_chain_contexts_on_threads():
    """Chains of several contexts on threads and streams of their own."""
    import threading
    grid = synth.centered_grid(128, 128, 4, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 96.0)
    h = synth.generate(grid, ph, 100_000, 90, 9)
    x0 = synth.initial_image(grid, ph)

    def one(out, q):
        with tvs.Context(grid, block_size=800, path_mode="q16") as ctx:
            ctx.load_histories(h)
            ctx.set_image(x0)
            ctx.iterate(3, 0.02, 1, 0.75, seed=q)
            out[q] = ctx.get_image()
    single, many = {}, {}
    for q in range(3):
        one(single, q)
    th = [threading.Thread(target=one, args=(many, q)) for q in range(3)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for q in range(3):
        np.testing.assert_array_equal(single[q], many[q])


@pytest.mark.parametrize("n,chunk,dims", [
    (450_000, 150_000, (24, 24, 2)),      # the buffers hold all chunks
    (700_001, 70_400, (24, 24, 2)),       # four groups of three chunks, the last one of one
    (400_000, 66_000, (40, 9, 1)),        # regions of several workgroups
])
def test_chunks_formed_together_equal_launches(n, chunk, dims):
    """On the fly with several chunks: the chain runs over all the buffers'
    chunks at once, per-block launches over one after the other; the images
    are the same bits, also when a batch takes the buffers in between."""
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * min(dims[0], dims[1]))
    h = synth.generate(grid, ph, n, 90, 77)
    x0 = synth.initial_image(grid, ph)
    settings = [dict(lam=0.02, N=2, alpha=0.75), dict(lam=0.01, N=1, alpha=0.5)]
    got = []
    for kernel in (0, 1):
        print(f"joined chunks: {dims} {n} histories, chunk {chunk}, sweep_kernel {kernel}",
              flush=True)
        with tvs.Context(grid, block_size=1600, sweep_kernel=kernel, chunk_histories=chunk) as ctx:
            ctx.load_histories(h)
            ctx.set_image(x0)
            ctx.iterate(2, 0.02, 2, 0.75, seed=11)
            a = ctx.get_image()
            ctx.iterate_batch(1, settings)
            b = ctx.get_batch_image(1)
            ctx.iterate(1, 0.02, 2, 0.75, seed=11)
            got.append((a, b, ctx.get_image()))
    assert np.max(np.abs(got[0][0] - x0)) > 1e-3
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
