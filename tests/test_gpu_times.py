"""What the device times of a sweep cover: the DROP launches without the wait
for rows that are formed before them.  With the resident chain the rows of a
group of chunks are formed first (the first group's beside the TV steps), so
rows and DROP together take no longer than the cycles; with either kernel the
launches take at least the time of their own work, and one chain a sweep is
counted."""
import pytest

from paper_1803_01112_amd import synth, tvs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [0, 160_000])             # one group; four groups of three
@pytest.mark.parametrize("kernel", [0, 1])
def test_drop_time_leaves_out_the_rows(chunk, kernel):
    grid = synth.centered_grid(128, 128, 8, 1.0, 1.0, 2.5)
    ph = synth.catphan_like(grid, 96.0)
    h = synth.generate(grid, ph, 1_600_000 if chunk else 800_000, 90, 5)
    with tvs.Context(grid, block_size=3200, chunk_histories=chunk, sweep_kernel=kernel,
                     time_sample=1_000_000 if kernel == 0 else 1) as ctx:
        ctx.load_histories(h)
        ctx.set_image(synth.initial_image(grid, ph))
        ctx.iterate(2, 0.02, 1, 0.75, seed=11)
        ctx.iterate(3, 0.02, 1, 0.75, seed=11)
        st = ctx.stats()
    print({k: st[k] for k in ("tv_ms_total", "sweep_ms_total", "rows_ms_total", "drop_ms_total",
                              "k1_ms_total", "k_samples", "drop_launches")}, flush=True)
    cycles = st["tv_ms_total"] + st["sweep_ms_total"]
    assert st["drop_launches"] == 3 == st["cycles_timed"]
    assert 0.9 * st["k1_ms_total"] <= st["drop_ms_total"] <= st["sweep_ms_total"] * 1.02
    if kernel == 0:
        assert st["k_samples"] > 0
        assert st["drop_ms_total"] + st["rows_ms_total"] <= 1.05 * cycles
        assert st["drop_ms_total"] <= 1.3 * st["k1_ms_total"]
