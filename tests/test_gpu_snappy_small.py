"""GPU parity of Snappy pages on both sides of the size from which the block
decoder takes its large shape (16 KiB of output): columns whose every page is below
or at it, columns with a page above, both in one scan, and sub-ranges of the row
groups.  Every output buffer is compared with the oracle byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dist", ["uniform", "runs"])
@pytest.mark.parametrize("rows", [1, 40, 2048, 4095, 4096, 4097, 20_000])
def test_page_sizes(rows, dist):
    # one page per row group: INT32 pages of 4 bytes a row, INT64 pages of 8
    d = {"uniform": dg.UNIFORM, "runs": dg.RUNS}[dist]
    cols = [dg.Col(dg.INT32, dg.PLAIN, False, d, lo=0, hi=900, run_len=9),
            dg.Col(dg.INT64, dg.PLAIN, False, d, lo=0, hi=1 << 40, run_len=30),
            dg.Col(dg.INT32, dg.RLE_DICTIONARY, True, dg.DICTVALS, 0.2, hi=500),
            dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.2, hi=50, str_min=0, str_max=9)]
    data = dg.write(dg.FileSpec(cols=cols, num_rows=5 * rows - rows // 2, rg_rows=rows, page_bytes=1 << 30, codec=dg.SNAPPY,
                                seed=81))
    check_file(data, label=f"{rows} rows {dist}")
    check_file(data, columns=[0], rg_begin=4, rg_end=5, label=f"{rows} rows {dist}, the last row group")
