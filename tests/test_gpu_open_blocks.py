"""GPU parity of files opened and closed again and again, in one thread and in
several at once, in memory that earlier opens of other files have used: files
whose index, dictionaries and decompressed pages are below, at and far above the
size from which an open's memory is kept for the next.  Every output buffer is
compared with the oracle byte for byte."""
from concurrent.futures import ThreadPoolExecutor

import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


def _file(rows, codec):
    cols = [dg.Col(dg.INT64, dg.DELTA_BINARY_PACKED, True, dg.UNIFORM, 0.1, lo=-(1 << 62), hi=1 << 62),
            dg.Col(dg.BYTE_ARRAY, dg.RLE_DICTIONARY, True, dg.STRINGS, 0.1, hi=max(2, rows // 9), str_min=4, str_max=20),
            dg.Col(dg.INT32, dg.RLE_DICTIONARY, False, dg.DICTVALS, hi=max(2, rows // 20))]
    return dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=max(1, rows // 2), page_bytes=256 * dg.KiB, codec=codec,
                                seed=41 + rows))


SIZES = [(rows, codec) for rows in (50, 30_000, 180_000, 1_200_000) for codec in (dg.UNCOMPRESSED, dg.SNAPPY)]


def test_files_in_turn():
    files = [_file(*k) for k in SIZES]
    for k in list(range(len(SIZES))) + list(reversed(range(len(SIZES)))):
        check_file(files[k], label=f"file {SIZES[k]}")


@pytest.mark.parametrize("threads", [2, 4])
def test_files_in_threads(threads):
    files = [_file(*k) for k in SIZES]
    with ThreadPoolExecutor(threads) as ex:
        for fut in [ex.submit(check_file, files[k], label=f"file {SIZES[k]}") for k in list(range(len(SIZES))) * 2]:
            fut.result()
