"""GPU parity on both sides of the choice between one decode launch for all
kinds of tiles and one launch per kind (6,000 tiles of one kind): one tile, a few,
the last count decoded in one launch and the first decoded per kind, with a
REQUIRED and an OPTIONAL column, fixed-width values and strings; and scans of no
rows.  Every output buffer is compared with the oracle byte for byte."""
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


def _file(cols, rows, rg_rows):
    return dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=rg_rows, page_bytes=1 << 20, seed=21))


@pytest.mark.parametrize("tiles", [1, 3, 3000, 3001])
@pytest.mark.parametrize("kind", ["plain", "dict", "bss", "string"])
def test_tiles_per_kind(kind, tiles):
    # two columns of one kind: the choice falls at 3,000 tiles each
    rows = tiles * 1024 - 7
    enc = {"plain": dg.PLAIN, "dict": dg.RLE_DICTIONARY, "bss": dg.BYTE_STREAM_SPLIT, "string": dg.RLE_DICTIONARY}[kind]
    if kind == "string":
        cols = [dg.Col(dg.BYTE_ARRAY, enc, o, dg.STRINGS, 0.1 if o else 0.0, hi=50, str_min=0, str_max=5) for o in (False, True)]
    else:
        dist = dg.DICTVALS if kind == "dict" else dg.UNIFORM
        cols = [dg.Col(dg.INT32, enc, o, dist, 0.1 if o else 0.0, lo=0, hi=1000) for o in (False, True)]
    # (one page per column: a page boundary would add a tile)
    data = dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=rows, page_bytes=1 << 30, seed=21))
    check_file(data, label=f"{kind} {tiles} tiles")


def test_no_rows():
    cols = [dg.Col(dg.INT32, dg.PLAIN, False, dg.UNIFORM), dg.Col(dg.BYTE_ARRAY, dg.PLAIN, True, dg.STRINGS, 0.1, hi=10)]
    data = _file(cols, 3000, 1000)
    check_file(data, rg_begin=1, rg_end=1, label="no row groups")
