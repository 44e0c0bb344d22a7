"""GPU parity of batches under the default schedule (one wave per tile, the work
described by the tile runs) where its tables meet an edge: one run, as many
as fit the kernel's arguments (64) and one more, more than 64 string columns
(their totals take a launch of their own), requests of one row, of a tile and of a tile
and a row, of no rows; and the same batches from eight work queues.  Every output
buffer is compared with the oracle byte for byte."""
import pytest

import datagen as dg
from tests.test_gpu_batch import _batch, _check_batch, _open

pytestmark = pytest.mark.gpu


def _cols(kind):
    if kind == "string":
        return [dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.1, hi=20, str_min=0, str_max=9)]
    return [dg.Col(dg.INT32, dg.RLE_DICTIONARY, False, dg.DICTVALS, hi=30), dg.Col(dg.INT64, dg.PLAIN, False, dg.UNIFORM)]


@pytest.mark.parametrize("kind", ["string", "fixed"])
@pytest.mark.parametrize("requests", [1, 32, 33, 64, 65, 129])
def test_requests(requests, kind):
    import paper_2602_17335_amd as pqs
    datas = [dg.write(dg.FileSpec(cols=_cols(kind), num_rows=r, rg_rows=2000, page_bytes=1 << 20, seed=51))
             for r in (1, 1024, 1025, 4700)]
    files = _open(datas)
    cols = list(range(len(_cols(kind))))
    # every fourth request of the largest file is of no rows
    reqs = [(files[i % 4], cols, 0, 0 if i % 16 == 7 else None) for i in range(requests)]
    queues = pqs.tuning_default()
    queues.waves_per_cu = 12
    for t, label in ((None, "default"), (queues, "queues")):
        b = _batch(files, reqs)
        b.scan(t)
        b.check()
        _check_batch(b, datas, f"{label} {requests} {kind}")
    b = _batch(files, [(files[3], cols, 1, 1)] * requests)
    b.scan()
    b.check()
    _check_batch(b, datas, f"no rows {requests} {kind}")
