"""Device memory that a closed file leaves for the next open is given back when no
open takes it, without a further call into the library: after a few seconds the
device has as much free memory as before the file was opened (but for the 64 MiB of
freed memory that the runtime itself may hold), also where another thread is in the
middle of a stream capture when that happens, whose graph replays as the same work
done eagerly.  A handle's device_bytes count the whole of the memory it took over."""
import gc
import time

import pytest

import datagen as dg
from tests.gpu_util import check_file

pytestmark = pytest.mark.gpu

MiB = 1 << 20
RUNTIME = 66 * MiB  # freed memory the runtime may hold, and page-sized remainders


def _file(rows=22_000_000):
    # 16 columns of runs: a small file with 344,000 tiles (143 MB of index)
    cols = [dg.Col(dg.INT32, dg.RLE_DICTIONARY, True, dg.CONST, 0.0, lo=7, hi=8) for _ in range(16)]
    return dg.write(dg.FileSpec(cols=cols, num_rows=rows, rg_rows=rows, page_bytes=1 << 20, seed=3))


def _free():
    import torch
    return torch.cuda.mem_get_info()[0]


def _settled():
    """Free memory with nothing kept."""
    import torch
    gc.collect()
    torch.cuda.synchronize()
    time.sleep(5)
    return _free()


def _opened_and_closed():
    """Free memory before the open of a file and after its close."""
    import paper_2602_17335_amd as pqs
    buf, n = pqs.to_device(_file())
    f = pqs.DeviceFile(buf, n)
    f.close()
    before = _settled()
    f = pqs.DeviceFile(buf, n)
    held = before - _free()
    f.close()
    assert held > 130 * MiB, held
    return before, buf


def _wait_free(level, seconds):
    t = time.monotonic()
    while _free() < level and time.monotonic() - t < seconds:
        time.sleep(0.1)
    return _free()


def test_given_back():
    before, _ = _opened_and_closed()
    assert before - _free() > RUNTIME  # kept
    assert _wait_free(before - RUNTIME, 8) >= before - RUNTIME
    check_file(dg.write(dg.small_table(rows=200_000, page_bytes=64 * dg.KiB)), label="after the blocks went")


def test_given_back_during_a_capture():
    import torch
    x = torch.arange(1 << 16, dtype=torch.int64, device="cuda")
    y = x.clone()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        y.mul_(3).add_(x)
    torch.cuda.synchronize()
    y.copy_(x)
    before, _ = _opened_and_closed()
    assert before - _free() > RUNTIME  # kept
    with torch.cuda.graph(g, stream=s):
        y.mul_(3)
        time.sleep(4)  # the blocks go meanwhile
        y.add_(x)
    assert _free() >= before - RUNTIME
    want = x.clone()
    for _ in range(4):
        g.replay()
        want = want * 3 + x
        torch.cuda.synchronize()
        assert torch.equal(y, want)


def test_device_bytes():
    import paper_2602_17335_amd as pqs
    bufs = [pqs.to_device(_file(rows)) for rows in (10_000_000, 13_000_000)]

    def opened(k):
        f = pqs.DeviceFile(*bufs[k])
        n = f.stats().device_bytes
        f.close()
        return n

    opened(0)
    _settled()
    own = opened(0)
    _settled()
    larger = opened(1)
    after = opened(0)  # in the larger file's blocks
    assert own < larger
    assert 1.1 * own < after <= larger
