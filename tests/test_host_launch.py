"""Launch shapes the library chooses where the caller sets none, read off the
launches it makes against a stand-in for the HIP runtime."""
import pytest

from fakehip import run

WIDTHS = {"fp32_shifted": {(3000, 2000): 512, (1345, 2000): 512, (900, 4500): 512, (1000, 1500): 512, (700, 2000): 256,
                           (1153, 1100): 256, (770, 1700): 128, (1100, 1800): 128, (515, 3000): 64, (300, 6000): 64},
          "fp64": {(3000, 2000): 256, (900, 4500): 256, (770, 1700): 128, (515, 3000): 64, (300, 6000): 64}}


@pytest.mark.parametrize("precision", sorted(WIDTHS))
def test_2d_rows_as_wide_as_a_tenth_more_columns_allows(tmp_path, precision):
    """A row much wider than the grid leaves lanes idle, one that pads the columns
    a little more stages fewer halo cells: the widest within a tenth is taken, for
    one run and for a batch of two."""
    run(tmp_path, f"""
for (nx, ny), width in {WIDTHS[precision]!r}.items():
    cfg = lbw.RunConfig(nx=nx, ny=ny, precision={precision!r})
    h = handle(cfg)
    lbw.check(lib.lbw_step(h, 1))
    got = launches("k_stage_tiled")
    assert len(got) == 3 and all(b == width for _, b, _ in got), (nx, ny, got)
    h = handle([cfg, cfg])
    lbw.check(lib.lbw_step(h, 1))
    assert [b for _, b, _ in launches("k_stage_batched")] == [width] * 3, (nx, ny)
""")
