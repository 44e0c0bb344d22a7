"""GPU parity of the open's links between the segments of a long value stream:
string pages and dictionaries of 63 to 65 and 127 to 130 segments of 32 KiB (64 are
linked together), of values of one size, whose chain enters every segment within its
first bytes, and of values of two very different ranges, whose chain now and then
enters a segment far behind them.  Every output buffer is compared with the
oracle byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

SEGMENT = 32 * dg.KiB


@pytest.mark.parametrize("encoding", [dg.PLAIN, dg.RLE_DICTIONARY])
@pytest.mark.parametrize("lens", [(28, 28), (60, 60), (5, 1000)], ids=str)
@pytest.mark.parametrize("segments", [8, 63, 64, 65, 127, 128, 130])
def test_segments(segments, lens, encoding):
    mean = 4 + sum(lens) / 2
    for k in (segments - 0.002, float(segments)):
        n = int(k * SEGMENT / mean)
        rows = n if encoding == dg.PLAIN else 2 * n
        col = dg.Col(dg.BYTE_ARRAY, encoding, False, dg.STRINGS, hi=n if encoding != dg.PLAIN else 300, str_min=lens[0],
                     str_max=lens[1])
        spec = dg.FileSpec(cols=[col], num_rows=rows, rg_rows=rows, page_bytes=1 << 30, seed=61, dict_cap=1 << 30)
        check_file(dg.write(spec), label=f"{segments} segments {lens} {n} values")
