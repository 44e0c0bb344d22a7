"""GPU parity of columns whose row groups need different decoders (dictionaries with
slots, dictionaries of long entries, PLAIN values after a dictionary, DELTA_BYTE_ARRAY pages
of short and of long values), for every range of row groups and in a batch: a scan launches
the decoders of its own row groups.  Every output buffer is compared with the oracle
byte for byte."""
import io

import numpy as np
import pyarrow as pa
import pyarrow.parquet as pq
import pytest

import oracle
from tests.gpu_util import GUARD, POISON, check_file, compare_column

pytestmark = pytest.mark.gpu

GROUPS, ROWS = 4, 3000


def _group(g, rng):
    """Row group g of the three columns."""
    few = [b"%d" % v for v in rng.integers(0, 40, ROWS)]
    long = [b"%d" % v * 30 for v in rng.integers(100, 140, ROWS)]
    unique = [b"%d/%d" % (i, v) for i, v in enumerate(rng.integers(0, 10**9, ROWS))]
    strings = (few, long, unique, few)[g]
    ints = rng.integers(0, (30, 10**12, 10**12, 30)[g], ROWS)
    times = (1, 400, 1, 3)[g]
    keys = [b"k%d" % v * (times if i % 700 == 5 else 1) for i, v in enumerate(rng.integers(0, 900, ROWS))]
    return strings, ints, keys


def _file(version, compression):
    rng = np.random.default_rng(11)
    bio = io.BytesIO()
    schema = pa.schema([("s", pa.binary()), ("i", pa.int64()), ("k", pa.binary())])
    with pq.ParquetWriter(bio, schema, compression=compression, use_dictionary=["s", "i"], data_page_version=version,
                          dictionary_pagesize_limit=8192, data_page_size=4096, write_batch_size=64,
                          column_encoding={"k": "DELTA_BYTE_ARRAY"}) as w:
        for g in range(GROUPS):
            cols = [pa.array(v, f.type, mask=rng.random(ROWS) < 0.1) for v, f in zip(_group(g, rng), schema)]
            w.write_table(pa.table(cols, schema=schema), row_group_size=ROWS)
    return np.frombuffer(bio.getvalue(), dtype=np.uint8).copy()


@pytest.mark.parametrize("version,compression", [("1.0", "none"), ("2.0", "snappy")])
def test_ranges(version, compression):
    import paper_2602_17335_amd as pqs
    data = _file(version, compression)
    for a in range(GROUPS):
        for b in range(a + 1, GROUPS + 1):
            check_file(data, rg_begin=a, rg_end=b, label=f"row groups {a}..{b} {version} {compression}")
    o = oracle.File(data)
    f = pqs.DeviceFile(*pqs.to_device(data))
    for form in (0, 1):
        print(f"[gpu] batch form {form} {version} {compression}", flush=True)
        ranges = [(g, g + 1) for g in range(GROUPS)] + [(0, GROUPS)]
        b = pqs.Batch([(f, [0, 1, 2], r0, r1) for r0, r1 in ranges], poison=POISON, guard=GUARD)
        t = pqs.tuning_default()
        t.form = form
        b.scan(t)
        b.check()
        for n, (r0, r1) in enumerate(ranges):
            for c in range(3):
                compare_column(o.read(c, r0, r1), b.outputs[n][c], f"form {form} row groups {r0}..{r1} column {c}")
