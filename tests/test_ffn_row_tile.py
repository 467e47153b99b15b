"""Which row-tile height the bf16 forward takes (laep_ffn_fwd_row_tile): short
tiles only where no load of the experts makes them slower than the 256-row
kernels.  The rows marked 256 are sizes at which short tiles measured slower, by
up to twice with all rows in one expert."""
import pytest

from paper_2601_14327_amd import laep_ffn_fwd_row_tile as row_tile


@pytest.mark.parametrize("R,E,d,f,want", [
    (4096, 128, 2048, 2048, 256),    # one expert: 110 us in 256-row tiles, 218 in 32
    (8192, 128, 2048, 2048, 256),    # one expert 181 / 298 (64), even loads 588 / 676
    (8192, 128, 2048, 1024, 256),    # normal(0, 2) router bias 168 / 202 (64)
    (16384, 256, 1024, 2048, 256),   # the same 278 / 365 (64)
    (11520, 45, 1024, 1024, 256),    # even loads 108 / 134 (128)
    (4096, 16, 2048, 2048, 256),     # even loads 165 / 201 (128)
    (65536, 64, 2048, 1024, 256),
    (32768, 16, 4096, 2048, 256),
    (64, 64, 2048, 1024, 32),        # even loads 163 us in 256-row tiles, 105 in 32
    (512, 64, 2048, 1024, 32),
    (2048, 64, 2048, 1024, 64),      # 189 / 149 (64)
    (2000, 64, 1024, 2048, 64),
    (4096, 16, 1024, 1024, 128),     # 55 / 48 (128)
    (68104, 13, 64, 64, 128),
    (100, 4, 60, 64, 0),             # refused: no multiple of 64
    (-1, 4, 64, 64, 0),
])
def test_row_tile(R, E, d, f, want):
    assert row_tile(R, E, d, f) == want


@pytest.mark.parametrize("d,f", [(64, 64), (192, 320), (1024, 2048), (4096, 1024)])
@pytest.mark.parametrize("E", [1, 16, 256])
def test_more_rows_never_take_shorter_tiles(E, d, f):
    heights = [row_tile(int(1.2 ** i), E, d, f) for i in range(80)]
    assert heights == sorted(heights) and heights[0] == 32 and heights[-1] == 256


@pytest.mark.parametrize("R,E,d,f", [
    (32744, 32, 64, 512), (32744, 32, 1024, 64),   # test_ffn_fwd_parity, one-step k-loops
    (60000, 40, 64, 256),                          # test_ffn_fwd_many_tiles
    (16000, 16, 512, 512),                         # the two concurrent calls
])
def test_sizes_of_the_persistent_kernels_tests(R, E, d, f):
    """GPU tests written for the 256-row kernels run them."""
    assert row_tile(R, E, d, f) == 256
