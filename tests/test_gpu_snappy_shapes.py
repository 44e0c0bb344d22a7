"""GPU parity of Snappy pages in scans of enough blocks (8,192) for each of the
block decoder's small shapes, in the batched form over more columns than a launch's
inline table holds (64) and in the streamed form: columns of pages of up to 8 KiB, of
up to 16 KiB and above, all in one batch and by themselves, and a batch in which only
one small shape has enough blocks.  Every output buffer is compared with the oracle
byte for byte."""
import pytest

import datagen as dg
import oracle
from tests.gpu_util import GUARD, POISON, compare_column

pytestmark = pytest.mark.gpu

ROWS = 1030  # a page: 4,120 bytes of INT32, 8,240 of INT64, about 27,000 of strings


def _file(groups, seed):
    return dg.write(dg.FileSpec(
        cols=[dg.Col(dg.INT32, dg.PLAIN, False, dg.UNIFORM, lo=0, hi=900),
              dg.Col(dg.INT64, dg.PLAIN, False, dg.SORTED, lo=0, hi=1 << 40),
              dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.1, hi=300, str_min=20, str_max=30)],
        num_rows=groups * ROWS - 17, rg_rows=ROWS, page_bytes=1 << 30, codec=dg.SNAPPY, seed=seed))


@pytest.mark.parametrize("files,groups", [(70, 120), (70, 60), (9, 920)])
def test_batched(files, groups):
    import paper_2602_17335_amd as pqs
    datas = [_file(groups, 500 + i) for i in range(files)]
    handles = [pqs.DeviceFile(*pqs.to_device(d)) for d in datas]
    oracles = [oracle.File(d) for d in datas]
    for cols in ([0, 1, 2], [0], [0, 1], [1, 2]):
        print(f"[gpu] batch of {files} files of {groups} pages a column, columns {cols}", flush=True)
        b = pqs.Batch([(f, cols, 0, None) for f in handles], poison=POISON, guard=GUARD)
        b.scan()
        b.check()
        for i, o in enumerate(oracles):
            for c in cols:
                compare_column(o.read(c), b.outputs[i][c], f"file {i} col {c}")


# a row group of 8,200 pages or more in each column
@pytest.mark.parametrize("page", [4 * dg.KiB, 10 * dg.KiB])
def test_streamed(page):
    import paper_2602_17335_amd as pqs
    rows = 8300 * page // 4
    data = dg.write(dg.FileSpec(
        cols=[dg.Col(dg.INT32, dg.PLAIN, False, dg.UNIFORM, lo=0, hi=900),
              dg.Col(dg.INT64, dg.PLAIN, True, dg.SORTED, 0.05, lo=0, hi=1 << 40)],
        num_rows=2 * rows - 1, rg_rows=rows, page_bytes=page, codec=dg.SNAPPY, seed=91))
    print(f"[gpu] streamed, pages of {page} bytes", flush=True)
    out = pqs.HostFile(data).scan([0, 1], poison=POISON, guard=GUARD)
    o = oracle.File(data)
    for c in (0, 1):
        compare_column(o.read(c), out[c], f"page {page} col {c}")
