"""A scan that has both a chars buffer too small and a column that it does not
decode reports the buffer, however its kernels are launched; with room enough it
reports the column."""
import ctypes

import pytest

import datagen as dg

pytestmark = pytest.mark.gpu


def _file(rows):
    cols = [dg.Col(dg.BYTE_ARRAY, dg.DELTA_BYTE_ARRAY, False, dg.STRINGS, hi=50, str_min=17_000, str_max=17_000),
            dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.1, hi=300, str_min=3, str_max=30),
            dg.Col(dg.INT32, dg.PLAIN, False, dg.UNIFORM, lo=0, hi=9)]
    return dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=rows, page_bytes=1 << 20, seed=13))


# one launch for every kind of tile, and one per kind
@pytest.mark.parametrize("rows,columns", [(3000, [0, 1, 2]), (3000, [0, 1])])
@pytest.mark.parametrize("short", [False, True])
def test_scan(rows, columns, short):
    import paper_2602_17335_amd as pqs
    f = pqs.DeviceFile(*pqs.to_device(_file(rows)))
    for _ in range(5):
        mask, rg_end, ws, outs, tens = f.allocate(columns)
        if short:
            outs[1].chars_capacity -= 1
        f.scan_into(mask, 0, rg_end, outs, ws)
        with pytest.raises(pqs.PqError) as e:
            f.check(ws)
        assert e.value.code == (pqs.PQ_ECAPACITY if short else pqs.PQ_EUNSUPPORTED)


@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("form", [0, 1])
def test_batch(form, short):
    import paper_2602_17335_amd as pqs
    files = [pqs.DeviceFile(*pqs.to_device(_file(2000 + 100 * i))) for i in range(3)]
    b = pqs.Batch([(f, [0, 1, 2], 0, None) for f in files])
    t = pqs.tuning_default()
    t.form = form
    if short:
        outs = ctypes.cast(b._reqs[2].outs, ctypes.POINTER(pqs.ColumnOut))
        outs[1].chars_capacity -= 1
    for _ in range(3):
        b.scan(t)
        with pytest.raises(pqs.PqError) as e:
            b.check()
        assert e.value.code == (pqs.PQ_ECAPACITY if short else pqs.PQ_EUNSUPPORTED)
