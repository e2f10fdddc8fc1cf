"""The rule by which batched products choose 64 or 128 right-hand sides per workgroup, at sizes where
both were measured (us on MI355X): it takes the faster one.  No GPU."""
import pytest

from paper_2005_05758_amd import load_library


# (rows, rows per tile, batch, 16-bit right-hand sides, us at 64, us at 128)
@pytest.mark.parametrize("rows,br,batch,bits16,us64,us128", [
    (8192, 32, 68, 0, 71.1, 63.5), (8192, 32, 128, 0, 71.7, 63.4), (8192, 32, 132, 0, 105.8, 123.0), (8192, 32, 192, 0, 105.9, 123.2),
    (8192, 32, 196, 0, 140.3, 123.7), (8192, 32, 260, 0, 174.3, 183.5), (8192, 32, 320, 0, 173.9, 182.9), (8192, 32, 512, 0, 276.0, 244.3),
    (8224, 32, 68, 0, 55.6, 61.3), (8224, 32, 132, 0, 73.9, 93.2), (8224, 32, 260, 0, 110.1, 124.1), (8224, 32, 452, 0, 164.9, 157.0),
    (12000, 32, 128, 0, 36.0, 38.1), (12000, 32, 256, 0, 69.9, 58.0), (4096, 32, 132, 0, 23.8, 20.0), (4096, 32, 260, 0, 34.8, 37.5),
    (4096, 32, 452, 0, 46.6, 39.3), (8192, 16, 128, 0, 42.7, 33.5), (8192, 16, 260, 0, 105.0, 97.4), (4300, 16, 132, 0, 42.4, 46.7),
    (4300, 16, 196, 0, 53.6, 47.7), (8192, 32, 132, 1, 64.9, 61.2), (8192, 32, 260, 1, 106.2, 90.8), (12000, 32, 68, 1, 23.8, 20.6),
    (4096, 32, 260, 1, 23.1, 20.1), (8192, 16, 68, 1, 29.8, 25.2), (8192, 16, 132, 1, 42.3, 43.6), (8192, 16, 260, 1, 67.1, 62.9),
    (4300, 16, 68, 1, 23.1, 24.5), (4300, 16, 132, 1, 29.1, 33.2), (4300, 16, 452, 1, 60.9, 53.3)])
def test_the_faster_width(rows, br, batch, bits16, us64, us128):
    got = load_library().csb_debug_spmm_columns(-(-rows // br), br, batch, bits16)
    assert got == (64 if us64 < us128 else 128)


@pytest.mark.parametrize("tiles,batch", [(1, 512), (100, 128), (300, 64), (300, 4), (255, 128)])
def test_128_needs_a_workgroup_for_every_cu(tiles, batch):
    assert load_library().csb_debug_spmm_columns(tiles, 32, batch, 0) == 64
