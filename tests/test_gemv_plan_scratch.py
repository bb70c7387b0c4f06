"""wh_gemv_noalloc's scratch array holds 64 MiB of slab partials.  About 2048
workgroups of 3 to 16 blocks a lane give these tall matrices two slabs of 48 to
50 MB: a plan of more slabs would have the call refused."""
import pytest

from paper_1902_08018_amd import wh


@pytest.mark.parametrize("rows,cols,rate", [(2856193, 671, 2), (3105866, 655, 4), (2923643, 662, 10), (3132070, 670, 14),
                                            (3223482, 662, 32)])
def test_plan_fits_the_scratch_array(rows, cols, rate):
    p = wh.wh_gemv_plan_info(rows, cols, 0, rows, rate=rate)
    part_rows = 4 * (p["bi_end"] - p["bi_begin"])
    assert p["nslab"] == 1 or p["nslab"] * part_rows * 8 <= 64 << 20
