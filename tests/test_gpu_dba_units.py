"""GPU parity of DELTA_BYTE_ARRAY pages at the edges of their expansion: value
counts around a group of 64 values and around several units of 256; prefix chains that
reach before the group and before the unit (sorted keys, growing and shrinking
values, one value repeated); empty values; groups over the LDS buffer (4 KiB, 2 KiB
for pages of short values) and single values over it.  Every output buffer is compared with the oracle byte
for byte, with one page and with many."""
import io

import numpy as np
import pyarrow as pa
import pyarrow.parquet as pq
import pytest

from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 63, 64, 65, 1023, 1024, 1025, 2049, 5000]


def _values(kind, n, rng):
    if kind == "sorted":
        return sorted(b"customer/%05d/order/%07d" % (int(a), int(b)) for a, b in
                      zip(rng.integers(0, 300, n), rng.integers(0, 10**7, n)))
    if kind == "random":
        return [rng.integers(97, 100, int(k), dtype=np.uint8).tobytes() for k in rng.integers(0, 40, n)]
    if kind == "sawtooth":  # grows by a byte, then shrinks by one: chains of every length
        base = rng.integers(97, 123, 90, dtype=np.uint8).tobytes()
        return [base[:(k % 180 if k % 180 < 90 else 179 - k % 180)] for k in range(n)]
    if kind == "equal":
        return [b"the same value all along"] * n
    if kind == "empty":
        return [b""] * n
    long = rng.integers(0, 256, 16000, dtype=np.uint8).tobytes()  # up to 16000 bytes, long shared prefixes
    return [long[:int(k)] + b"%d" % i for i, k in enumerate(rng.choice([0, 10, 300, 1500, 4090, 4097, 15000], n))]


@pytest.mark.parametrize("kind", ["sorted", "random", "sawtooth", "equal", "empty", "long"])
@pytest.mark.parametrize("compression", ["none", "snappy"])
def test_unit_edges(kind, compression):
    rng = np.random.default_rng(len(kind))
    for n in COUNTS[:7] if kind == "long" else COUNTS:
        vals = _values(kind, n, rng)
        for page, nulls in ((1 << 24, False), (2048, True)):
            arr = pa.array(vals, mask=rng.random(n) < 0.1 if nulls else None, type=pa.binary())
            bio = io.BytesIO()
            pq.write_table(pa.table({"k": arr}), bio, use_dictionary=False, compression=compression, data_page_size=page,
                           write_batch_size=64, column_encoding={"k": "DELTA_BYTE_ARRAY"})
            check_file(np.frombuffer(bio.getvalue(), dtype=np.uint8).copy(), label=f"dba {kind} {n} page {page}")
