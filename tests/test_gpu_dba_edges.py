"""GPU parity of DELTA_BYTE_ARRAY pages around a unit of 256 values and around the
longest value (1,024 bytes) of the kernel for pages of short values: value counts
next to a unit's end, longest values of 1,023, 1,024 and 1,025 bytes whose prefixes
reach over the start of a unit, values and prefixes next to the lengths from which
values are copied by all lanes and in pieces, and columns that hold pages of both kernels, in
single scans, in batches of both forms and streamed.  Every output buffer is compared
with the oracle byte for byte."""
import io

import numpy as np
import pyarrow as pa
import pyarrow.parquet as pq
import pytest

import oracle
from tests.gpu_util import GUARD, POISON, check_file, compare_column

pytestmark = pytest.mark.gpu


def _values(n, longest, rng):
    """n values of up to `longest` bytes, one of which has all: prefixes of one base
    of changing length, so that most of a value comes from values before it."""
    base = rng.integers(0, 256, longest, dtype=np.uint8).tobytes()
    cuts = rng.integers(max(0, longest - 40), longest, n)
    cuts[rng.random(n) < 0.02] = 0
    vals = [base[:int(c)] + b"%d" % i for i, c in enumerate(cuts)]
    vals = [v[:longest] for v in vals]
    vals[n // 2] = base
    return vals


def _file(vals, nulls, rng, page=1 << 24, compression="none", groups=1):
    arr = pa.array(vals, mask=rng.random(len(vals)) < 0.1 if nulls else None, type=pa.binary())
    bio = io.BytesIO()
    pq.write_table(pa.table({"k": arr}), bio, use_dictionary=False, compression=compression, data_page_size=page,
                   row_group_size=-(-len(vals) // groups), write_batch_size=64, column_encoding={"k": "DELTA_BYTE_ARRAY"})
    return np.frombuffer(bio.getvalue(), dtype=np.uint8).copy()


@pytest.mark.parametrize("longest", [30, 1023, 1024, 1025, 1500])
@pytest.mark.parametrize("n", [255, 256, 257, 511, 512, 513, 770])
def test_unit_and_length_edges(n, longest):
    rng = np.random.default_rng(n + longest)
    vals = _values(n, longest, rng)
    for nulls in (False, True):
        check_file(_file(vals, nulls, rng), label=f"dba {n} values, longest {longest}, nulls {nulls}")


@pytest.mark.parametrize("near", [160, 1020, 2040, 4092, 8188, 16_380])
def test_lengths_and_prefixes_near(near):
    """Values and prefixes that end a few bytes from a length at which the expansion
    changes its way: copied by a lane or by all, in one piece or in several."""
    rng = np.random.default_rng(near)
    base = rng.integers(0, 256, 16_384, dtype=np.uint8).tobytes()
    vals = []
    for i in range(400):
        cut = max(0, min(near + int(rng.integers(-9, 10)), 16_384)) if rng.random() < 0.8 else int(rng.integers(0, near))
        tail = rng.integers(0, 256, int(rng.choice([0, 1, 3, 5, 300])), dtype=np.uint8).tobytes()
        vals.append((base[:cut] + tail)[:16_384])
    for nulls in (False, True):
        check_file(_file(vals, nulls, rng, page=300_000 if nulls else 1 << 24), label=f"dba near {near}, nulls {nulls}")


def _mixed(rng, compression):
    # stretches of short and of long values: pages of both kernels in one column
    vals = []
    for k in range(12):
        vals += _values(300 + 17 * k, (40, 1024, 1025, 9000)[k % 4], rng)
    return _file(vals, True, rng, page=20_000, compression=compression, groups=3)


@pytest.mark.parametrize("compression", ["none", "snappy"])
def test_pages_of_both_kernels(compression):
    import paper_2602_17335_amd as pqs
    rng = np.random.default_rng(7)
    datas = [_mixed(rng, compression) for _ in range(3)]
    for i, d in enumerate(datas):
        check_file(d, label=f"both kernels {compression} {i}")
    check_file(datas[0], rg_begin=1, rg_end=2, label="the second row group")
    oracles = [oracle.File(d) for d in datas]
    files = [pqs.DeviceFile(*pqs.to_device(d)) for d in datas]
    for form in (0, 1):
        print(f"[gpu] batch form {form} {compression}", flush=True)
        b = pqs.Batch([(f, [0], 0, None) for f in files], poison=POISON, guard=GUARD)
        t = pqs.tuning_default()
        t.form = form
        b.scan(t)
        b.check()
        for i, o in enumerate(oracles):
            compare_column(o.read(0), b.outputs[i][0], f"form {form} file {i}")
    out = pqs.HostFile(datas[1]).scan([0], poison=POISON, guard=GUARD)
    compare_column(oracles[1].read(0), out[0], "streamed")
