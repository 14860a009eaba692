"""Scans whose output is copied by a memcpy node: template lengths on both sides of
where one kernel gives way to two, jobs of every length around a tile's edge.  Sums
are exact."""
import sys

import numpy as np
import pytest

from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu

TILE = 2048


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("mode", ["sync", "set"])
@pytest.mark.parametrize("max_n", [16 * TILE - 1, 16 * TILE, 16 * TILE + 1, 64 * TILE])
def test_lengths(torch_gpu, max_n, mode):
    print("scan, memcpy nodes", max_n, mode)
    sys.stdout.flush()
    ns = np.array(sorted({1, TILE, TILE + 1, 15 * TILE + 7, 16 * TILE - 1, min(max_n, 33 * TILE), max_n - 1, max_n}))
    x = np.random.default_rng(max_n).integers(-2**31, 2**31, max_n, dtype=np.int64).astype(np.int32)
    x[: max_n // 2] |= 1 << 30  # sums beyond 32 bits
    tin, nin = pinned(4 * max_n)
    nin[:4 * max_n].view(np.int32)[:] = x
    stride = -(-(64 + 8 * max_n) // 64) * 64
    tout, nout = pinned(stride * len(ns))
    with Context(mode=mode, workers=2, slots=2 if mode == "set" else 1) as ctx:
        tid = ctx.define("scan", max_n=max_n, copy="nodes")
        arr = ctx.job_array(len(ns))
        arr["host_in"], arr["in_bytes"], arr["n"] = tin.data_ptr(), 4 * ns, ns
        arr["host_out"] = tout.data_ptr() + np.arange(len(ns), dtype=np.uint64) * stride
        arr["out_bytes"] = 64 + 8 * ns
        ctx.submit_many(tid, arr)
        ctx.drain()
    want = np.cumsum(x.astype(np.int64))
    for i, n in enumerate(ns):
        assert np.array_equal(nout[i * stride + 64:i * stride + 64 + 8 * n].view(np.int64), want[:n]), int(n)
