"""The tuner's choice between the resident chain and launches per block: what it
reports is its fastest candidate, what the context's sweeps run (read from the
statistics: with a time sample longer than the sweep only the chain's launches
are counted), and what a configuration takes to run the same; from the cache
too.  A cache file that knows launches only is measured anew where there is a
chain, and taken where there is none."""
import os

import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu

LONG = 1_000_000


def scan(dims, n):
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * min(dims[0], dims[1]))
    return grid, synth.generate(grid, ph, n, 90, 5), synth.initial_image(grid, ph)


def context(s, **kw):
    ctx = tvs.Context(s[0], time_sample=LONG, **kw)
    ctx.load_histories(s[1])
    ctx.set_image(s[2])
    return ctx


def cycle(ctx, x0):
    ctx.set_image(x0)
    ctx.iterate(1, 0.02, 1, 0.75, seed=11)
    return ctx.get_image(), ctx.stats()["k_samples"]


@pytest.mark.parametrize("dims,n,B,mode,chunk", [
    ((64, 64, 1), 30_000, 3200, "f32", 0),           # few tiles: the chain by far
    ((128, 128, 4), 60_000, 3200, "otf", 0),
    ((128, 128, 4), 60_000, 3200, "otf", 6400),      # several chunks: whole sweeps
    ((200, 200, 16), 160_000, 6400, "q16", 0),
])
def test_reported_choice_is_what_runs(tmp_path, dims, n, B, mode, chunk):
    s = scan(dims, n)
    kw = dict(block_size=B, path_mode=mode, chunk_histories=chunk)
    blocks = -(-n // B)
    cache = os.path.join(tmp_path, "tune.txt")
    with context(s, sweep_kernel=1, **kw) as ctx:
        want, none = cycle(ctx, s[2])
        assert none == 0
        r = ctx.autotune(0.02, cache)                # no chain here: launches only
        assert r["sweep_kernel"] in (1, 2) and {c["sweep"] for c in r["candidates"]} == {1, 2}
        assert cycle(ctx, s[2])[1] == 0
    assert len(open(cache).read().split()) == 5
    for again in (False, True):
        print(f"tuned choice: {dims} {mode} chunk {chunk} cache {again}", flush=True)
        with context(s, **kw) as ctx:
            r = ctx.autotune(0.02, cache)
            assert r["from_cache"] == again
            assert (r["tile_threads"] == 0) == (r["sweep_kernel"] == 0)
            if not again:
                first = r
                assert 0 in {c["sweep"] for c in r["candidates"]}
                if not chunk:
                    best = min(r["candidates"], key=lambda c: c["ms"])
                    assert (r["tile_threads"], r["sweep_kernel"], r["ms_per_block"]) == (
                        best["threads"], best["sweep"], best["ms"])
            assert r["sweep_kernel"] == first["sweep_kernel"]
            assert r["ms_per_block"] == pytest.approx(first["ms_per_block"], abs=1e-6)
            image, ran = cycle(ctx, s[2])
            assert ran == (blocks if r["sweep_kernel"] == 0 else 0)
            np.testing.assert_array_equal(image, want)
            ctx.load_histories(s[1])                 # and after another load
            assert cycle(ctx, s[2])[1] == ran
    with context(s, sweep_kernel=first["sweep_kernel"], tile_threads=first["tile_threads"],
                 **kw) as ctx:
        assert cycle(ctx, s[2])[1] == ran
    if dims == (64, 64, 1):
        assert first["sweep_kernel"] == 0            # 10 us a block against 109


def test_cached_choice_of_launches_leaves_the_chain(tmp_path):
    """A line whose chain was the slower: launches, until the tuner is asked again."""
    s = scan((64, 64, 1), 30_000)
    cache = os.path.join(tmp_path, "tune.txt")
    with context(s, path_mode="f32") as ctx:
        assert ctx.autotune(0.02, cache)["sweep_kernel"] == 0
        key = open(cache).read().split()[0]
    with open(cache, "a") as fh:
        fh.write(f"{key} 128 2 0.100000 40 0 0.200000\n")
    with context(s, path_mode="f32") as ctx:
        r = ctx.autotune(0.02, cache)
        assert (r["from_cache"], r["tile_threads"], r["sweep_kernel"], r["ms_per_block"]) == (
            True, 128, 2, 0.1)
        assert ctx.debug_sweep() == (False, 128)
        assert cycle(ctx, s[2])[1] == 0
        assert ctx.autotune(0.02)["sweep_kernel"] == 0
        assert cycle(ctx, s[2])[1] == 10


def test_choice_that_outlives_its_scan(tmp_path):
    """Tuned on a scan without a chain (few blocks), then a scan that has one;
    and a chain that was refused while it was timed."""
    s = scan((200, 200, 10), 128_000)
    few = {k: v[:6400] for k, v in s[1].items()}
    with context((s[0], few, s[2]), path_mode="f32") as ctx:
        r = ctx.autotune(0.02)
        assert r["sweep_kernel"] in (1, 2) and cycle(ctx, s[2])[1] == 0
        ctx.load_histories(s[1])
        assert cycle(ctx, s[2])[1] == 40
    s = scan((64, 64, 1), 30_000)
    cache = os.path.join(tmp_path, "tune.txt")
    with context(s, path_mode="f32") as ctx:
        ctx.debug_sweep(2)
        r = ctx.autotune(0.02, cache)
        assert r["sweep_kernel"] in (1, 2) and cycle(ctx, s[2])[1] == 0
        r = ctx.autotune(0.02, cache)            # the file holds no time of the chain
        assert not r["from_cache"] and r["sweep_kernel"] == 0
        assert cycle(ctx, s[2])[1] == 10
