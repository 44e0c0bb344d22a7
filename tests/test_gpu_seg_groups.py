"""GPU parity of files whose long streams make more 32 KiB segments than one group of
an open holds (4,096): string dictionaries of tens of MB, dictionary-index pages and
DELTA pages of tens of MB, each in several row groups.  Every output buffer is compared
with the oracle byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

COLS = {"strings": (dg.Col(dg.BYTE_ARRAY, dg.RLE_DICTIONARY, False, dg.STRINGS, hi=1 << 30, str_min=24, str_max=44), 900_000, 5),
        "indices": (dg.Col(dg.INT32, dg.RLE_DICTIONARY, True, dg.DICTVALS, 0.01, hi=1 << 20), 14_000_000, 4),
        "deltas": (dg.Col(dg.INT64, dg.DELTA_BINARY_PACKED, False, dg.UNIFORM, lo=-(1 << 62), hi=1 << 62), 4_500_000, 4)}


@pytest.mark.parametrize("kind", sorted(COLS))
def test_groups(kind):
    col, rows, groups = COLS[kind]
    data = dg.write(dg.FileSpec(cols=[col], num_rows=rows * groups, rg_rows=rows, page_bytes=1 << 30, seed=61))
    assert len(data) > 136 << 20  # 4,096 segments and more
    check_file(data, label=f"long {kind}")
