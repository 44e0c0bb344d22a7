"""GPU parity of the Snappy block decoder where a block's stream or output
ends at an edge: pages just below, at and just above one pass of the decoder's
stream (8 KiB), one output block (64 KiB) and two, holding long literals,
runs (copies that repeat their own output with periods of 1 to 70 bytes, of
one thread's stream bytes and across threads), copies of copies, and all of
them mixed.  Every output buffer is compared with the oracle byte for byte."""
import io

import numpy as np
import pyarrow as pa
import pyarrow.parquet as pq
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 8191, 8192, 8193, 16384, 65535, 65536, 65537, 131072, 131077, 196613]


def _text(kind, n, rng):
    """n bytes that compress to the elements `kind` names."""
    if kind == "literal":
        return rng.integers(0, 256, n, dtype=np.uint8).tobytes()
    if kind == "runs":
        out = bytearray()
        period = 1
        while len(out) < n:
            out += rng.integers(0, 256, period, dtype=np.uint8).tobytes() * int(rng.integers(2, 9) * 200 // period + 2)
            period = period % 70 + 1
        return bytes(out[:n])
    if kind == "chains":  # few distinct words in random order: copies of copies
        words = [rng.integers(97, 123, int(k), dtype=np.uint8).tobytes() for k in rng.integers(3, 9, 40)]
        out = bytearray()
        while len(out) < n:
            out += words[int(rng.integers(0, 40))]
        return bytes(out[:n])
    out = bytearray()
    while len(out) < n:
        out += _text(("literal", "runs", "chains")[int(rng.integers(0, 3))], int(rng.integers(1, 6000)), rng)
    return bytes(out[:n])


@pytest.mark.parametrize("kind", ["literal", "runs", "chains", "mixed"])
def test_block_edges(kind):
    rng = np.random.default_rng(len(kind))
    # one value a page, so that a page holds exactly the bytes of one text
    # (and 4 of its length)
    vals = [_text(kind, max(n - 4, 0), rng) for n in EDGES]
    bio = io.BytesIO()
    pq.write_table(pa.table({"s": pa.array(vals, type=pa.binary())}, schema=pa.schema([pa.field("s", pa.binary(), nullable=False)])),
                   bio, use_dictionary=False, compression="snappy", data_page_size=1, write_batch_size=1)
    check_file(np.frombuffer(bio.getvalue(), dtype=np.uint8).copy(), label=f"snappy blocks {kind}")


@pytest.mark.parametrize("dist", ["const", "runs", "sorted"])
@pytest.mark.parametrize("page", [8 * dg.KiB, 64 * dg.KiB, 200_000])
def test_runs_of_values(dist, page):
    d = {"const": dg.CONST, "runs": dg.RUNS, "sorted": dg.SORTED}[dist]
    cols = [dg.Col(t, dg.PLAIN, o, d, 0.02 if o else 0.0, lo=5, hi=1 << 30, run_len=300)
            for t in (dg.INT32, dg.INT64) for o in (False, True)]
    check_file(dg.write(dg.FileSpec(cols=cols, num_rows=70_001, rg_rows=50_000, page_bytes=page, codec=dg.SNAPPY, seed=9)),
               label=f"snappy {dist} page {page}")
