"""A sweep captured by the caller into a HIP graph: per-block launches whose
arguments live until the next load.  Every replay gives the image of a plain
call, bit for bit, with the library's own work between the replays and after
a call that was short of memory (the budget leaves no room for the counters of
the hull detection beside what the context holds)."""
import numpy as np
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,mode", [((64, 64, 4), "f32"), ((131, 97, 7), "q16")])
def test_captured_sweep(dims, mode):
    import torch
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 0.75 * min(dims[0], dims[1]))
    h = synth.generate(grid, ph, 60_000, 60, 5)
    x0 = synth.initial_image(grid, ph)
    kw = dict(block_size=3200, path_mode=mode)
    cycle = dict(K=1, lam=0.02, N=2, alpha=0.75, seed=11)
    with tvs.Context(grid, **kw) as ctx:
        ctx.load_histories(h)
        held = ctx.stats()["device_bytes"]
        ctx.set_image(x0)
        ctx.iterate(**cycle)
        want = ctx.get_image()
    with tvs.Context(grid, hbm_budget_bytes=held + 4096, **kw) as ctx:
        ctx.load_histories(h)
        ctx.set_image(x0)
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
            ctx.iterate(stream=stream, **cycle)
        for replay in range(3):
            print(f"captured sweep {dims} {mode}: replay {replay}", flush=True)
            graph.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(ctx.get_image(), want)
            ctx.set_image(x0)
            ctx.iterate(**cycle)                       # the library's own sweep in between
            np.testing.assert_array_equal(ctx.get_image(), want)
            try:
                ctx.hull_detect(wepl_in_mm=10.0, wepl_out_mm=1.0, min_in=1, max_out=3)
            except tvs.TvsError as e:
                assert e.status == tvs.TVS_ENOMEM
            fill = [torch.full((1 << 16,), -1, dtype=torch.int32, device="cuda:0") for _ in range(64)]
            ctx.set_image(x0)
            torch.cuda.synchronize()
            del fill
