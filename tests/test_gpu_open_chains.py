"""GPU parity of the open's chain index where a stream's length meets an edge of
it: streams just below, at and just above a short segment (8 KiB), a long one
(32 KiB) and the length from which a string page's segments are done side by
side (2 MiB), for PLAIN strings and string dictionaries (values of a few bytes,
ordinary ones, values longer than the candidates of a segment and longer than
a segment), definition levels (dense short runs, long runs), dictionary
indices and DELTA blocks.  Every output buffer is compared with the oracle
byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

SEG = [8 * dg.KiB, 32 * dg.KiB, 64 * dg.KiB, 2 * dg.MiB]


def _check(cols, rows, page, label, **kw):
    check_file(dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=rows, page_bytes=page, seed=11, **kw)), label=label)


@pytest.mark.parametrize("lens", [(0, 3), (8, 44), (1100, 2500), (30_000, 70_000)], ids=str)
def test_plain_strings(lens):
    mean = 4 + sum(lens) / 2
    for seg in SEG[:3] if lens[0] < 1000 else SEG:
        for k in (0.98, 1.0, 1.02, 2.5):
            rows = max(1, int(k * seg / mean))
            _check([dg.Col(dg.BYTE_ARRAY, dg.PLAIN, False, dg.STRINGS, hi=200, str_min=lens[0], str_max=lens[1])], rows,
                   1 << 30, f"strings {lens} {rows} rows")
    if lens[0] < 1000:
        for rows in (int(0.99 * SEG[3] / mean), int(2.2 * SEG[3] / mean)):
            _check([dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.03, hi=200, str_min=lens[0], str_max=lens[1])], rows,
                   1 << 30, f"strings {lens} {rows} rows, one page")


@pytest.mark.parametrize("lens", [(8, 44), (1100, 2500)], ids=str)
def test_string_dictionaries(lens):
    mean = 4 + sum(lens) / 2
    for size in (7_000, 33_000, 2 * dg.MiB + 40_000, 5 * dg.MiB):
        n = max(2, int(size / mean))
        _check([dg.Col(dg.BYTE_ARRAY, dg.RLE_DICTIONARY, True, dg.STRINGS, 0.1, hi=n, str_min=lens[0], str_max=lens[1])],
               2 * n + 100, 64 * dg.KiB, f"string dictionary {lens} {n} entries")


@pytest.mark.parametrize("nulls", [0.0, 0.0005, 0.1, 0.5, 1.0])
@pytest.mark.parametrize("version", [1, 2])
def test_levels_indices_blocks(nulls, version):
    for rows in (1, 1023, 1025, 60_001, 262_145, 700_003):
        cols = [dg.Col(dg.INT32, dg.PLAIN, True, dg.UNIFORM, nulls, lo=0, hi=1 << 30),
                dg.Col(dg.INT32, dg.RLE_DICTIONARY, True, dg.DICTVALS, nulls, hi=2),
                dg.Col(dg.INT64, dg.RLE_DICTIONARY, True, dg.DICTVALS, nulls, hi=5000),
                dg.Col(dg.INT32, dg.RLE_DICTIONARY, True, dg.RUNS, nulls, lo=0, hi=300, run_len=40),
                dg.Col(dg.INT64, dg.DELTA_BINARY_PACKED, True, dg.UNIFORM, nulls, lo=-(1 << 62), hi=1 << 62),
                dg.Col(dg.INT32, dg.DELTA_BINARY_PACKED, True, dg.CONST, nulls, lo=3, hi=4),
                dg.Col(dg.BYTE_ARRAY, dg.DELTA_LENGTH_BYTE_ARRAY, True, dg.STRINGS, nulls, hi=100, str_min=0, str_max=9)]
        _check(cols, rows, 1 << 30, f"levels {nulls} v{version} {rows} rows", page_version=version)
