"""DELTA_BYTE_ARRAY pages whose streams hold more values than the page has rows
(the row counts of the page header and of the footer lowered, the streams left):
refused as corrupt when the file is opened, by the check that comes before the
page's values are expanded and its units written.  The oracle refuses the same
bytes when it reads the column.  A file opened afterwards is scanned and compared
with the oracle byte for byte."""
import numpy as np
import pytest

import datagen as dg
import oracle

ROWS = 8000  # its zigzag varint, as those of all smaller counts written here, takes two bytes


def _varint2(n):
    z = 2 * n
    return bytes([0x80 | (z & 0x7f), z >> 7])


def _file(optional, version, codec, rows=ROWS, null=0.1):
    cols = [dg.Col(dg.BYTE_ARRAY, dg.DELTA_BYTE_ARRAY, optional, dg.STRINGS, null if optional else 0.0, hi=2000, str_min=4,
                   str_max=40)]
    return dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=rows, page_bytes=1 << 24, page_version=version,
                                codec=codec, seed=77))


def _lowered(data, rows):
    """`data`, a file of one page, with its row counts set to `rows`."""
    b = bytearray(np.asarray(data, dtype=np.uint8).tobytes())
    old, new = _varint2(ROWS), _varint2(rows)
    flen = int.from_bytes(b[-8:-4], "little")
    n = 0
    for lo, hi, mark in ((4, 64, b"\x15"), (len(b) - 8 - flen, len(b) - 8, b"\x16")):  # i32 fields, i64 fields
        for at in range(lo, hi - 2):
            if b[at:at + 3] == mark + old:
                b[at + 1:at + 3] = new
                n += 1
    # page header: num_values (V2: num_rows too); footer: rows of the file and of the row group, values of the chunk
    assert n in (4, 5), n
    return np.frombuffer(bytes(b), dtype=np.uint8).copy()


CASES = [(optional, version, codec) for optional in (False, True) for version in (1, 2)
         for codec in (dg.UNCOMPRESSED, dg.SNAPPY)]


@pytest.mark.parametrize("rows", [1, 255, 256, 257, 4000, 7000])
def test_oracle_refuses(rows):
    for case in CASES:
        with pytest.raises(oracle.OracleError):
            oracle.File(_lowered(_file(*case), rows)).read(0)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [0, 1, 255, 256, 257, 4000, 7000])
def test_more_values_than_rows(rows):
    import paper_2602_17335_amd as pqs
    from tests.gpu_util import check_file
    for case in CASES:
        print(f"[gpu] {rows} rows, optional/version/codec {case}", flush=True)
        buf, n = pqs.to_device(_lowered(_file(*case), rows))
        with pytest.raises(pqs.PqError) as e:
            pqs.DeviceFile(buf, n)
        assert e.value.code == pqs.PQ_ECORRUPT
        check_file(_file(*case, rows=700), label=f"after {rows} rows {case}")
