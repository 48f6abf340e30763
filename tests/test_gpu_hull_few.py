"""Hull detection on both sides of the line between few lines (each voxel's count
read as the line enters it) and many: masks equal to the oracle's, with counts
low enough to fill and too high."""
import numpy as np
import pytest

import oracle
from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,n", [((33, 40, 1), 64), ((64, 64, 1), 40_000), ((64, 64, 1), 40_001),
                                    ((31, 17, 5), 39_999)])
def test_hull_of_few_lines(dims, n):
    grid = synth.centered_grid(*dims, 1.0, 1.0, 2.5)
    h = synth.generate(grid, synth.catphan_like(grid, 0.75 * min(dims[0], dims[1])), n, 45, 7)
    with tvs.Context(grid, block_size=3200) as ctx:
        ctx.load_histories(h)
        for min_in, max_out in ((1, 0), (n // 40, 3), (n // 10, n)):
            kw = dict(wepl_in=5.0, wepl_out=8.0, min_in=min_in, max_out=max_out)
            print(f"hull {dims} {n} lines {min_in} {max_out}", flush=True)
            got = ctx.hull_detect(wepl_in_mm=5.0, wepl_out_mm=8.0, min_in=min_in, max_out=max_out)
            np.testing.assert_array_equal(got, oracle.hull(grid, h, **kw))
