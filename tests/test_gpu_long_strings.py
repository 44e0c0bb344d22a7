"""GPU parity of strings of a few KiB and more, PLAIN and in dictionaries, whose
lengths lie on both sides of 4 KiB a value, from which an open follows a stream value
by value: all of one length, lengths mixed with empty ones, many and few values; and
the same pages with a length that leaves the page, refused as corrupt.  Every output
buffer is compared with the oracle byte for byte."""
import numpy as np
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(4090, 4090), (4092, 4092), (4096, 4096), (0, 9000), (30_000, 70_000)])
@pytest.mark.parametrize("codec", [dg.UNCOMPRESSED, dg.SNAPPY])
def test_lengths(lo, hi, codec):
    for rows, distinct in ((1, 1), (33, 7), (900, 300)):
        cols = [dg.Col(dg.BYTE_ARRAY, dg.RLE_DICTIONARY, True, dg.STRINGS, 0.1, hi=distinct, str_min=lo, str_max=hi),
                dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.3, hi=distinct, str_min=lo, str_max=hi),
                dg.Col(dg.BYTE_ARRAY, dg.PLAIN, False, dg.STRINGS, hi=distinct, str_min=lo, str_max=hi)]
        for page in (1 << 16, 1 << 24):
            check_file(dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=max(1, rows // 2), page_bytes=page, codec=codec,
                                            seed=21)), label=f"strings of {lo} to {hi} bytes, {rows} rows, page {page}")


@pytest.mark.parametrize("encoding", [dg.PLAIN, dg.RLE_DICTIONARY])
@pytest.mark.parametrize("at", [0, 17, -1])
def test_length_past_the_page(encoding, at):
    import paper_2602_17335_amd as pqs
    n = 5000
    data = bytearray(dg.write(dg.FileSpec(cols=[dg.Col(dg.BYTE_ARRAY, encoding, False, dg.STRINGS, hi=1 << 30, str_min=n, str_max=n)],
                                          num_rows=40, rg_rows=40, page_bytes=1 << 24, seed=5)))
    first = data.index(n.to_bytes(4, "little"))
    at = first + (at % 40) * (n + 4)
    assert data[at:at + 4] == n.to_bytes(4, "little")
    data[at:at + 4] = (1 << 20).to_bytes(4, "little")
    bad = np.frombuffer(bytes(data), dtype=np.uint8).copy()
    print(f"[gpu] length past the page, encoding {encoding}", flush=True)
    with pytest.raises(pqs.PqError) as e:
        pqs.DeviceFile(*pqs.to_device(bad))
    assert e.value.code == pqs.PQ_ECORRUPT
