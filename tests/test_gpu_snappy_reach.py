"""GPU parity of Snappy pages whose copies reach just up to, at and past the start
of their 64 KiB output block, from a few bytes to many behind it, at the first
block and at later ones: pages with a copy past it are left to the page-sequential
decoder.  The streams are made by hand, in the place of a page of literals.  Every
output buffer is compared with the oracle byte for byte."""
import pyarrow as pa
import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

BLOCK = 65536
ROWS = 60_000  # 240,000 bytes: three blocks and a part of one


def _varint(n):
    out = bytearray()
    while n > 127:
        out.append(n & 127 | 128)
        n >>= 7
    return bytes(out + bytes([n]))


def _stream(old, n, at, off, length=60):
    """A stream of n output bytes and len(old) bytes with the copy (off, length) at
    output byte `at`: literals of `old`'s bytes elsewhere, none past a block."""
    out, pos = bytearray(_varint(n)), 0
    cuts = sorted({at, at + length, n} | set(range(BLOCK, n, BLOCK)))

    def long_literals():
        p, size = 0, 0
        for c in cuts:
            size += 3 if not (p == at) else 3 + length - (c - p)
            size += c - p - (length if p == at else 0)
            p = c
        return size
    ones = len(old) - len(out) - long_literals()  # literals of one byte, each a byte longer than in a long one
    assert 0 <= ones < 30_000
    for _ in range(ones):
        out += bytes([0, old[pos % len(old)]])
        pos += 1
    for c in cuts:
        if pos == at:
            out += bytes([(length - 1) << 2 | 2]) + off.to_bytes(2, "little")
        elif c > pos:
            m = c - pos
            out += bytes([61 << 2]) + (m - 1).to_bytes(2, "little") + bytes(old[(pos + i) % len(old)] for i in range(m))
        pos = max(pos, c)
    return bytes(out)


@pytest.mark.parametrize("block", [0, 1, 3])
@pytest.mark.parametrize("behind", [61, 100, 5000, 30_000])
def test_reach(block, behind):
    n = 4 * ROWS
    col = dg.Col(dg.INT32, dg.PLAIN, False, dg.UNIFORM, lo=0, hi=1 << 30)
    data = bytearray(dg.write(dg.FileSpec(cols=[col], num_rows=ROWS, rg_rows=ROWS, page_bytes=1 << 30, codec=dg.SNAPPY,
                                          snappy_literal_only=True, seed=71)))
    head = _varint(n)
    start = next(i for i in range(4, 200) if data[i:i + len(head)] == head and data[i + len(head)] & 3 == 0)
    size = next(e for e in range(start + n, len(data)) if _is_stream(bytes(data[start:e]), n)) - start
    for extra in (-1, 0, 1, 500):
        off = behind + extra
        if block == 0 and extra > 0:
            continue  # before the page: no valid stream
        new = _stream(bytes(data[start:start + size]), n, block * BLOCK + behind, off)
        assert len(new) == size and len(pa.decompress(new, n, codec="snappy")) == n
        data[start:start + size] = new
        check_file(bytes(data), label=f"block {block}, {behind} bytes behind, offset {off}")


def _is_stream(s, n):
    try:
        return len(pa.decompress(s, n, codec="snappy")) == n
    except Exception:
        return False
