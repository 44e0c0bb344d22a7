"""GPU parity of Snappy pages on both sides of the size from which the block
decoder takes its large shape (16 KiB of output), in scans of enough blocks (8,192)
for the small one and of fewer: columns whose every page is below or at it, columns
with a page above, both in one scan, and sub-ranges of the row groups.  Every output
buffer is compared with the oracle byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dist", ["uniform", "runs"])
@pytest.mark.parametrize("rows,groups", [(1, 5), (1, 2100), (40, 2040), (40, 2100), (2047, 2100), (2048, 2100),
                                         (2049, 3100), (4096, 5), (4097, 5), (20_000, 5)])
def test_page_sizes(rows, groups, dist):
    # one page per row group: INT32 pages of 4 bytes a row, INT64 pages of 8
    d = {"uniform": dg.UNIFORM, "runs": dg.RUNS}[dist]
    cols = [dg.Col(dg.INT32, dg.PLAIN, False, d, lo=0, hi=900, run_len=9),
            dg.Col(dg.INT64, dg.PLAIN, False, d, lo=0, hi=1 << 40, run_len=30),
            dg.Col(dg.INT32, dg.RLE_DICTIONARY, True, dg.DICTVALS, 0.2, hi=500),
            dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.2, hi=50, str_min=0, str_max=9)]
    data = dg.write(dg.FileSpec(cols=cols, num_rows=groups * rows - rows // 2, rg_rows=rows, page_bytes=1 << 30, codec=dg.SNAPPY,
                                seed=81))
    check_file(data, label=f"{groups} x {rows} rows {dist}")
    check_file(data, columns=[0], rg_begin=groups - 1, rg_end=groups, label=f"{rows} rows {dist}, the last row group")
