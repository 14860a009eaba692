"""One-kernel images of more tiles than the last block reads at once (2048): tile
counts on both sides of one and two rounds.  The count is that of the template that
returns the images, and the sum is the oracle's."""
import sys

import numpy as np
import pytest

import oracle
from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd import synth
from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _run(torch, img, **kw):
    h, w = img.shape
    tin, nin = pinned(img.nbytes)
    nin[:img.nbytes] = img.ravel().view(np.uint8)
    with Context(mode="sync", workers=1, slots=1) as ctx:
        tid = ctx.define("gauss_sobel", width=w, height=h, threshold=2.0, **kw)
        ob = ctx.out_bytes(tid)
        tout, nout = pinned(ob)
        ctx.submit(tid, host_in=tin.data_ptr(), in_bytes=img.nbytes, host_out=tout.data_ptr(), out_bytes=ob)
        ctx.drain()
    return int(nout[64:68].view(np.uint32)[0]), float(nout[68:72].view(np.float32)[0])


# 2047, 2048, 2049, 4095, 4096, 4356 and 4098 tiles of 16 x 64
@pytest.mark.parametrize("tiles", [(89, 23), (128, 16), (683, 3), (195, 21), (4096, 1), (132, 33), (3, 1366)])
def test_rounds(torch_gpu, tiles):
    print("image tiles", tiles)
    sys.stdout.flush()
    h, w = tiles[0] * 16 - 3, tiles[1] * 64 - 1
    img = synth.normal_image(11, tiles[0] * tiles[1], h, w)
    count, total = _run(torch_gpu, img)
    assert count == _run(torch_gpu, img, flags=A.SET_TF_DEBUG)[0]
    S = oracle.gauss_sobel(img, want_images=False)["sum"]
    assert abs(total - S) <= 1e-5 * abs(S)
