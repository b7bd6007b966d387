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


FUSED = {"fp32_shifted": {(64, 128): True, (20000, 8): True, (100000, 8): False, (100000, 6): False, (73728, 16): True,
                          (73728, 17): False, (3, 300000): True, (1024, 1152): True, (1024, 1153): False},
         "fp64": {(64, 128): True, (20000, 8): True, (50000, 8): False, (512, 1024): True, (512, 1025): False,
                  (600, 1200): False, (20000, 33): False, (600, 1200, "weno3"): False,
                  (768, 1024, "upwind1"): True, (768, 1025, "upwind1"): False}}


@pytest.mark.parametrize("precision", sorted(FUSED))
def test_one_launch_transport_counts_rows_in_whole_tiles(tmp_path, precision):
    """Grids of few rows leave most of a one-launch tile outside the grid, so they
    take the march from the size on at which their tiles, not their cells, fill the
    chip."""
    run(tmp_path, f"""
for (nx, ny, *scheme), fused in {FUSED[precision]!r}.items():
    h = handle(lbw.RunConfig(nx=nx, ny=ny, precision={precision!r}, scheme_c=(scheme or ["weno5"])[0]))
    lbw.check(lib.lbw_step(h, 4))
    lines = log()
    count = lambda part: sum(l.startswith("launch") and part in l for l in lines)
    assert (count("k_rk3_2d"), count("k_stage_tiled")) == ((2, 6) if fused else (0, 12)), (nx, ny, lines)
""")


@pytest.mark.parametrize("precision,full,sizes", [("fp32_shifted", 3 * 256, [(300, 100, 150), (128, 96, 160), (128, 128, 192)]),
                                                  ("fp64", 2 * 256, [(300, 100, 150), (100, 100, 400), (97, 63, 130)])])
def test_3d_chunks_leave_no_block_for_a_second_round(tmp_path, precision, full, sizes):
    """The vertical chunk is the shortest whose blocks fit the chip together, a last
    chunk cut short counted."""
    run(tmp_path, f"""
for nx, ny, nz in {sizes!r}:
    h = handle(lbw.RunConfig(lattice=19, nx=nx, ny=ny, nz=nz, precision={precision!r}))
    lbw.check(lib.lbw_step(h, 1))
    got = launches("k_stage_tiled")
    assert len(got) == 3 and all(b == 512 and {full} * 3 // 4 < g[0] <= {full} for g, b, _ in got), (nx, ny, nz, got)
""")


@pytest.mark.parametrize("grid", ["lattice=19, nx=256, ny=256, nz=512", "nx=4096, ny=2048"])
def test_streamed_even_half_keeps_16_or_20_waves_or_all(tmp_path, grid):
    """The LDS the even half reserves lets blocks of 16 or 20 waves stay on a CU, the
    same number on each of its four SIMDs; where no number of blocks does, for blocks
    of fewer than four waves and in the odd half, nothing is reserved."""
    run(tmp_path, f"""
for block in range(64, 1025, 64):
    h = handle(lbw.RunConfig({grid}, precision="fp32_shifted"), lbm_block=block)
    lbw.check(lib.lbw_step(h, 2))
    (_, even_block, even), (_, odd_block, odd) = launches("k_collide_stream")
    assert even_block == odd_block == block and odd == 0
    waves, fits = block // 64, (160 << 10) // even if even else 0
    want = [n for n in range(2, 6) if n * waves in (16, 20)]
    assert fits == (max(want) if want else 0), (block, even, fits)
    assert even <= 64 << 10
""")
