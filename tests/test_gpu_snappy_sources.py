"""GPU parity of Snappy pages whose copies take bytes of earlier copies: from the
whole of the copy before them and from a part of it, from across its start and its
end, from a copy a few elements back, from copies that repeat with a period, and in
chains of values that each copy most bytes of the value before (at offsets of 4, 8
and 16 bytes), with elements at every place of a thread's 16 stream bytes.  The
streams are made by hand, in the place of pages of literals, for pages of every
shape of the block decoder.  Every output buffer is compared with the oracle byte for
byte."""
import random

import numpy as np
import pyarrow as pa
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu


def _varint(n):
    out = bytearray()
    while n > 127:
        out.append(n & 127 | 128)
        n >>= 7
    return bytes(out + bytes([n]))


def _copy(off, n, rng):
    if 4 <= n <= 11 and off < 2048 and rng.random() < 0.5:
        return bytes([(off >> 8) << 5 | (n - 4) << 2 | 1, off & 255])
    if rng.random() < 0.1:
        return bytes([(n - 1) << 2 | 3]) + off.to_bytes(4, "little")
    return bytes([(n - 1) << 2 | 2]) + off.to_bytes(2, "little")


def _literal(n, rng):
    b = rng.randbytes(n)
    if n <= 60 and n:
        return bytes([(n - 1) << 2]) + b
    return bytes([61 << 2]) + (n - 1).to_bytes(2, "little") + b


def _elements(kind, n, rng):
    """Elements of at most n output bytes, and how many these are."""
    out, o, last, w = bytearray(_literal(16, rng)), 16, [(0, 16)], 8
    while o + 64 <= n:
        if kind == "values":  # values of 4, 8 or 16 bytes that differ in their first one or two
            if rng.random() < 0.02:
                w = rng.choice([4, 8, 16])
            k = 2 if rng.random() < 0.05 else 1
            out += _literal(k, rng) + _copy(w, w - k, rng)
            o += w
            continue
        how = rng.randrange(8)
        po, pn = last[-1] if how != 6 else rng.choice(last[-6:])
        if how == 0:
            k = rng.randint(1, 3)
            out += _literal(k, rng)
            o += k
            continue
        if how in (1, 6):    # within the copy (6: one a few copies back)
            a = rng.randrange(pn)
            s, k = po + a, rng.randint(1, pn - a)
        elif how == 2:       # all of it
            s, k = po, pn
        elif how == 3:       # across its start
            s = max(po - rng.randint(1, 9), 0)
            k = rng.randint(1, min(64, pn + po - s))
        elif how == 4:       # across its end
            s, k = po + pn - rng.randint(1, pn), rng.randint(1, 64)
        elif how == 5:       # a period
            s, k = o - rng.randint(1, min(o, 70)), rng.randint(1, 64)
        else:                # eight bytes back
            s, k = o - 8, rng.randint(1, 8)
        out += _copy(o - s, k, rng)
        last.append((o, k))
        o += k
    return out, o


def _stream(kind, n, size, rng):
    """A stream of n output bytes and `size` bytes: elements as `kind` names, literals
    of one byte, and a long one."""
    head = _varint(n)
    body, o = _elements(kind, int(n * 0.45), rng)
    rest = n - o
    ones = size - len(head) - len(body) - 3 - rest  # each a byte longer than in the long literal
    assert 0 <= ones < rest - 60
    for _ in range(ones):
        body += _literal(1, rng)
    long = rest - ones
    body += bytes([61 << 2]) + (long - 1).to_bytes(2, "little") + rng.randbytes(long)
    s = head + bytes(body)
    assert len(s) == size and len(pa.decompress(s, n, codec="snappy")) == n
    return s


# 4-byte values: pages of 4 KiB, 8,160 and 16,000 bytes in scans of enough pages for the small shapes, and of fewer;
# the last of several passes of every shape
@pytest.mark.parametrize("rows,groups", [(1024, 8200), (2040, 8200), (4000, 8200), (2040, 3), (16_000, 9)])
def test_sources(rows, groups):
    rng = random.Random(rows + groups)
    n = 4 * rows
    col = dg.Col(dg.INT32, dg.PLAIN, False, dg.UNIFORM, lo=0, hi=1 << 30)
    data = bytearray(dg.write(dg.FileSpec(cols=[col], num_rows=rows * groups, rg_rows=rows, page_bytes=1 << 30,
                                          codec=dg.SNAPPY, snappy_literal_only=True, seed=71)))
    head, streams, at = _varint(n), [], 4
    size = len(head) + 3 + n  # one literal
    for g in range(groups):
        at = next(i for i in range(at, at + 200) if data[i:i + len(head)] == head and data[i + len(head)] & 3 == 0)
        if not streams:
            assert len(pa.decompress(bytes(data[at:at + size]), n, codec="snappy")) == n
            streams = [_stream(("values", "mixed")[k % 2], n, size, rng) for k in range(min(groups, 24))]
        data[at:at + size] = streams[g % len(streams)]
        at += size
    check_file(np.frombuffer(bytes(data), dtype=np.uint8).copy(), label=f"{groups} pages of {n} bytes")
