"""One-kernel images, whose last block to arrive ends the job: tile counts at the
edges of the arrival groups, several jobs through each slot, whatever the slot
holds between them (nothing, or poison), in every way a job is launched.  The
count is that of the template that returns the images, to the last one, and the
same image's sum the same bits in every job and every way."""
import sys

import numpy as np
import pytest

import oracle
from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd import synth
from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu

TILE_H, TILE_W = 16, 64  # pixels of a block
WAYS = {
    "direct": dict(mode="set", callback="host_flag"),
    "direct, poisoned": dict(mode="set", callback="host_flag", flags=A.SET_TF_POISON),
    "captured": dict(mode="set", callback="event_poll", flags=A.SET_TF_CAPTURE),
    "memcpy nodes": dict(mode="set", callback="host_flag", copy="nodes"),
    "sync": dict(mode="sync"),
    "batch": dict(mode="batch", batch_size=4),
}


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _context(way):
    kw = dict(WAYS[way])
    t = {k: kw.pop(k) for k in ("copy", "flags") if k in kw}
    return Context(workers=2, slots=2, **kw), t


def _run(ctx, tid, ob, fill):
    k = len(fill)
    stride = -(-ob // 64) * 64
    tout, nout = pinned(stride * k)
    nout[:] = 0xEE
    arr = ctx.job_array(k)
    arr["host_out"] = tout.data_ptr() + np.arange(k, dtype=np.uint64) * stride
    arr["out_bytes"] = ob
    for i, f in enumerate(fill):
        for name, v in f.items():
            arr[name][i] = v
    first = ctx.submit_many(tid, arr)
    ctx.drain()
    outs = nout[:stride * k].reshape(k, stride)
    for i in range(k):
        hd = outs[i][:64].view(A.OUT_HEADER_DTYPE)[0]
        assert hd["job_id"] == first + i and hd["magic"] == A.SET_OUT_MAGIC and hd["canary_ok"] == 1
    return outs


@pytest.mark.parametrize("tiles", [(1, 1), (127, 1), (1, 128), (43, 3), (16, 16), (257, 1), (61, 17)])
def test_images(torch_gpu, tiles):
    h, w = tiles[0] * TILE_H - 1, tiles[1] * TILE_W - 1
    imgs = [synth.normal_image(7, k, h, w) for k in range(3)]
    stride = -(-4 * h * w // 64) * 64
    tin, nin = pinned(stride * 3)
    for i, im in enumerate(imgs):
        nin[i * stride:i * stride + 4 * h * w] = im.ravel().view(np.uint8)
    jobs = [dict(host_in=tin.data_ptr() + (i % 3) * stride, in_bytes=4 * h * w) for i in range(12)]
    with Context(mode="sync", workers=1, slots=1) as ctx:
        tid = ctx.define("gauss_sobel", width=w, height=h, threshold=2.0, flags=A.SET_TF_DEBUG)
        counts = [int(o[64:68].view(np.uint32)[0]) for o in _run(ctx, tid, ctx.out_bytes(tid), jobs[:3])]
    sums = None
    for way in WAYS:
        print("arrivals: images", tiles, way)
        sys.stdout.flush()
        ctx, t = _context(way)
        with ctx:
            tid = ctx.define("gauss_sobel", width=w, height=h, threshold=2.0, **t)
            outs = _run(ctx, tid, 72, jobs)
        if sums is None:
            sums = [outs[i][68:72].tobytes() for i in range(3)]
            for im, s in zip(imgs, sums):
                S = oracle.gauss_sobel(im, want_images=False)["sum"]
                assert abs(float(np.frombuffer(s, np.float32)[0]) - S) <= 1e-5 * abs(S)
        for i, out in enumerate(outs):
            assert int(out[64:68].view(np.uint32)[0]) == counts[i % 3], (way, i)
            assert out[68:72].tobytes() == sums[i % 3], (way, i)


@pytest.mark.parametrize("way", ["direct", "direct, poisoned", "captured", "memcpy nodes"])
@pytest.mark.parametrize("room", [1, 5, 1024, 1025])
def test_vector_batches(torch_gpu, room, way):
    """Batches of one job to a full table, above and below the size up to which
    the last block writes the results itself, several through each slot.  The
    vectors' values are 0 and +-1 and tanh(16) is one in float32, so every sum is
    a whole number and exact."""
    rng = np.random.default_rng(room)
    x = rng.integers(-1, 2, 1 << 22).astype(np.float32)
    xd = torch_gpu.from_numpy(x).cuda()
    yd = torch_gpu.zeros_like(xd)
    ctx, t = _context(way)
    with ctx:
        tid = ctx.define("saxpy_batch", max_n=1 << 16, x_pool=xd, y_pool=yd, batch_max=room, tiles_max=4 * room + 64, **t)
        for count in sorted({1, 4, 5, 511, 513, room - 1, room, 5 * room + 1} - {0}):
            if count > 8 * room:
                continue
            print("arrivals: vector batches of up to", room, way, count)
            sys.stdout.flush()
            v = np.zeros(count, A.VEC_JOB_DTYPE)
            v["n"] = rng.integers(1024, 2048, count)
            v["x_off"] = rng.integers(0, len(x) - 2048, count)
            v["a"] = 16.0
            got, batches = ctx.run_vector_jobs(tid, v)
            want = [x[o:o + n].astype(np.int64).sum() for o, n in zip(v["x_off"].tolist(), v["n"].tolist())]
            assert batches == -(-count // room) and np.array_equal(got, np.array(want, np.float32)), count
