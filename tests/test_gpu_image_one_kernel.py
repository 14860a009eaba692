"""Images whose Gaussian and Sobel run as one kernel: the count is that of the
template that returns the images (the kernels it replaces, same arithmetic),
and the sum the oracle's, at tile edges, tiny sizes and both width classes."""
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


@pytest.mark.parametrize("shape", [(1, 1), (1, 4), (5, 1), (2, 3), (3, 8), (16, 64), (15, 63), (17, 65), (16, 68), (33, 130),
                                   (47, 128), (250, 333), (511, 512), (1020, 1024), (1100, 1025)])
def test_count_and_sum(torch_gpu, shape):
    h, w = shape
    print("one-kernel image", shape)
    sys.stdout.flush()
    imgs = [synth.normal_image(7, k, h, w) for k in range(2)]
    imgs.append(np.full((h, w), 2.5, np.float32))
    got = {}
    for flags in (0, A.SET_TF_DEBUG):
        with Context(mode="sync", workers=1, slots=1) as ctx:
            tid = ctx.define("gauss_sobel", width=w, height=h, threshold=2.0, flags=flags)
            ib, ob = ctx.in_bytes(tid), ctx.out_bytes(tid)
            tin, nin = pinned(ib)
            tout, nout = pinned(ob)
            got[flags] = []
            for im in imgs:
                nin.view(np.float32)[:] = im.ravel()
                nout[:] = 0
                ctx.submit(tid, host_in=tin.data_ptr(), in_bytes=ib, host_out=tout.data_ptr(), out_bytes=ob)
                ctx.drain()
                got[flags].append((int(nout[64:68].view(np.uint32)[0]), float(nout[68:72].view(np.float32)[0])))
    for im, (cnt, s), (cnt_d, s_d) in zip(imgs, got[0], got[A.SET_TF_DEBUG]):
        ref = oracle.gauss_sobel(im, want_images=False)
        assert cnt == cnt_d
        assert abs(s - ref["sum"]) <= 1e-5 * abs(ref["sum"]) + 1e-5 * h * w * (abs(float(im.flat[0])) if im.std() == 0 else 0.0)
