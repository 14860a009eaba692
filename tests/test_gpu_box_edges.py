"""The one-kernel box/histogram at the edges of its tiles: ragged widths and heights,
images of a row or a column, rows at every alignment, blocks that take several
tiles, and more partial rows than the combining kernel reads at once.  Whole numbers,
so equal to the oracle's to the last one."""
import sys

import numpy as np
import pytest

import oracle
from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu

WAYS = {
    "sync": (dict(mode="sync"), {}),
    "direct, poisoned": (dict(mode="set", callback="host_flag"), dict(flags=A.SET_TF_POISON)),
    "memcpy nodes": (dict(mode="set", callback="event_poll"), dict(copy="nodes")),
}
SHAPES = [(1, 1), (1, 7), (7, 1), (2, 2), (3, 5), (16, 64), (17, 33), (17, 65), (63, 63), (64, 65), (65, 64), (65, 1), (1, 65),
          (300, 513), (333, 250), (640, 639), (16, 640), (640, 16), (1, 4099), (4099, 1), (2, 9001), (9001, 3), (70001, 5),
          (5, 70001), (1100, 1027)]


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("way", WAYS)
@pytest.mark.parametrize("shape", SHAPES)
def test_histogram(torch_gpu, shape, way):
    print("box edges", shape, way)
    sys.stdout.flush()
    h, w = shape
    rng = np.random.default_rng(h * 1000 + w)
    imgs = [rng.integers(0, 256, shape, dtype=np.uint8), np.full(shape, 255, np.uint8),
            rng.choice(np.array([0, 255], np.uint8), shape)]
    ib, ob = h * w, 64 + 1024
    stride = -(-ib // 64) * 64
    tin, nin = pinned(3 * stride)
    tout, nout = pinned(6 * ob)
    nin[:] = 0xFF  # what lies behind an image is none of its own
    nout[:] = 0xEE
    for i, im in enumerate(imgs):
        nin[i * stride:i * stride + ib] = im.ravel()
    kw, t = WAYS[way]
    with Context(workers=2, slots=1, **kw) as ctx:
        tid = ctx.define("box_hist", width=w, height=h, **t)
        arr = ctx.job_array(6)
        arr["host_in"] = tin.data_ptr() + np.arange(6, dtype=np.uint64) % 3 * stride
        arr["in_bytes"], arr["out_bytes"] = ib, ob
        arr["host_out"] = tout.data_ptr() + np.arange(6, dtype=np.uint64) * ob
        ctx.submit_many(tid, arr)
        ctx.drain()
    want = [oracle.box_hist(im)[2] for im in imgs]
    for i in range(6):
        assert np.array_equal(nout[i * ob + 64:(i + 1) * ob].view(np.uint32), want[i % 3]), i
