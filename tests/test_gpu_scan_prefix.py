"""Scans whose downsweep adds up what lies before its tiles itself: template
lengths on both sides of where a block goes from the input to the tile sums and
from those to the spine, jobs of every length around a tile's edge in them, in
every way a job is launched.  Sums are exact."""
import sys

import numpy as np
import pytest

from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu

TILE = 2048
WAYS = {
    "direct": dict(mode="set", callback="event_poll", copy="async_in"),
    "words, poisoned": dict(mode="set", callback="host_flag", flags=A.SET_TF_POISON),
    "captured": dict(mode="set", callback="event_poll", flags=A.SET_TF_CAPTURE),
    "memcpy nodes": dict(mode="set", callback="event_poll", copy="nodes"),
    "sync": dict(mode="sync"),
    "batch": dict(mode="batch", batch_size=4),
}


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("low32", [False, True])
@pytest.mark.parametrize("max_n", [1, TILE, 9 * TILE - 5, 64 * TILE, 64 * TILE + 1, 1024 * TILE, 1024 * TILE + 1])
def test_prefix_sources(torch_gpu, max_n, low32):
    ns = sorted({n for n in (1, 7, TILE - 1, TILE, TILE + 1, 2 * TILE, 5 * TILE + 3, 8 * TILE, 8 * TILE + 1, 9 * TILE, 17 * TILE, 63 * TILE + 1,
                             300 * TILE + 9,
                             max_n - 1, max_n) if 1 <= n <= max_n})
    rng = np.random.default_rng(max_n)
    x = rng.integers(-2**31, 2**31, max_n, dtype=np.int64).astype(np.int32)
    x[: max_n // 2] = np.abs(x[: max_n // 2] | 1)  # sums beyond 32 bits
    istride = -(-4 * max_n // 64) * 64
    tin, nin = pinned(istride)
    nin[:4 * max_n].view(np.int32)[:] = x
    size = 4 if low32 else 8
    ostride = -(-(64 + size * max_n) // 64) * 64
    want = np.cumsum(x.astype(np.int64))
    for way, kw in WAYS.items():
        print("scan prefix", max_n, low32, way)
        sys.stdout.flush()
        kw = dict(kw)
        t = {k: kw.pop(k) for k in ("copy", "flags") if k in kw}
        t["flags"] = t.get("flags", 0) | (A.SET_TF_SCAN_LOW32 if low32 else 0)
        tout, nout = pinned(ostride * len(ns))
        nout[:] = 0xEE
        with Context(workers=2, slots=2, **kw) as ctx:
            tid = ctx.define("scan", max_n=max_n, **t)
            arr = ctx.job_array(len(ns))
            arr["host_in"] = tin.data_ptr()
            arr["in_bytes"] = 4 * np.array(ns)
            arr["host_out"] = tout.data_ptr() + np.arange(len(ns), dtype=np.uint64) * ostride
            arr["out_bytes"] = 64 + size * np.array(ns)
            arr["n"] = ns
            first = ctx.submit_many(tid, arr)
            ctx.drain()
        for i, n in enumerate(ns):
            o = nout[i * ostride:(i + 1) * ostride]
            hd = o[:64].view(A.OUT_HEADER_DTYPE)[0]
            assert hd["job_id"] == first + i and hd["magic"] == A.SET_OUT_MAGIC and hd["canary_ok"] == 1
            got = o[64:64 + size * n]
            assert np.array_equal(got.view(np.int64), want[:n]) if not low32 else \
                np.array_equal(got.view(np.uint32), want[:n].astype(np.uint32)), (way, n)
