"""GPU parity of DELTA values and strings where the prefix sum over a file's
tiles meets an edge of it: one workgroup sums 4,096 tiles, so files of one tile
below, at and one above that count, and of more than one workgroup's; with scans
of the whole file and from a later row group.  Every output buffer is compared with
the oracle byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("version", [1, 2])
@pytest.mark.parametrize("tiles", [1, 63, 4094, 4095, 4096, 4097, 9000])
def test_tiles_of_a_file(tiles, version):
    cols = [dg.Col(dg.INT64, dg.DELTA_BINARY_PACKED, True, dg.UNIFORM, 0.1, lo=-(1 << 62), hi=1 << 62),
            dg.Col(dg.BYTE_ARRAY, dg.DELTA_LENGTH_BYTE_ARRAY, False, dg.STRINGS, hi=100, str_min=0, str_max=9),
            dg.Col(dg.BYTE_ARRAY, dg.RLE_DICTIONARY, True, dg.STRINGS, 0.1, hi=50, str_min=0, str_max=5)]
    cols = cols[:1] if tiles % 3 else cols
    n, rg = tiles // len(cols), 10  # row groups of one tile per column
    data = dg.write(dg.FileSpec(cols=cols, num_rows=n * rg - 3, rg_rows=rg, page_bytes=1 << 20, seed=31, page_version=version))
    check_file(data, label=f"{tiles} tiles v{version}")
    if n > 2:
        check_file(data, rg_begin=n // 2, rg_end=n, label=f"{tiles} tiles v{version}, second half")
