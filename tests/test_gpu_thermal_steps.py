"""Thermal jobs whose steps are taken several to a launch: grids smaller than a
tile's halo, a cell either side of a tile's edge, and step counts around those
where the launches and the halo change."""
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


@pytest.mark.parametrize("shape", [(1, 1), (1, 40), (40, 1), (2, 3), (15, 16), (17, 15), (32, 32), (33, 31), (47, 49),
                                   (49, 65), (57, 112), (64, 113), (512, 512), (511, 514), (700, 771)])
def test_steps_per_launch(torch_gpu, shape):
    """Against the float64 oracle within the bound its docstring derives."""
    h, w = shape
    print("steps per launch", shape)
    sys.stdout.flush()
    t0, p = synth.hotspot_input(6, h * 1000 + w, h, w)
    ib, ob = 8 * h * w, 64 + 4 * h * w
    tin, nin = pinned(ib)
    tout, nout = pinned(ob)
    nin[:].view(np.float32)[:] = np.concatenate([t0.ravel(), p.ravel()])
    for steps in (2, 4, 5, 8, 9, 12, 13, 16, 17, 31, 32):
        with Context(mode="sync", workers=1, slots=1) as ctx:
            tid = ctx.define("hotspot", width=w, height=h, max_n=steps)
            nout[:] = 0
            ctx.submit(tid, host_in=tin.data_ptr(), in_bytes=ib, host_out=tout.data_ptr(), out_bytes=ob)
            ctx.drain()
        got = nout[64:].view(np.float32).reshape(h, w)
        ref = oracle.hotspot(t0, p, steps)
        assert np.max(np.abs(got - ref)) <= oracle.hotspot_tolerance(ref, steps), (shape, steps)


@pytest.mark.parametrize("case", [(256, 256, 16), (250, 333, 1), (260, 516, 1), (2048, 2048, 1), (700, 771, 9)])
def test_rounding_is_below_the_formula_as_it_stands(torch_gpu, case):
    """The steps' rounding error, root mean square against float64, is below that
    of the update formula evaluated term by term in float32: it rounds the
    temperature once a step, the formula four times."""
    h, w, steps = case
    print("thermal rounding", case)
    sys.stdout.flush()
    t0, p = synth.hotspot_input(8, h * 1000 + w, h, w)
    ib, ob = 8 * h * w, 64 + 4 * h * w
    tin, nin = pinned(ib)
    tout, nout = pinned(ob)
    nin[:ib].view(np.float32)[:] = np.concatenate([t0.ravel(), p.ravel()])
    with Context(mode="sync", workers=1, slots=1) as ctx:
        tid = ctx.define("hotspot", width=w, height=h, max_n=steps)
        ctx.submit(tid, host_in=tin.data_ptr(), in_bytes=ib, host_out=tout.data_ptr(), out_bytes=ob)
        ctx.drain()
    got = nout[64:ob].view(np.float32).reshape(h, w)
    f = np.float32
    t, p = t0.astype(f).reshape(h, w), p.astype(f).reshape(h, w)
    for _ in range(steps):
        e = np.pad(t, 1, mode="edge")
        lap_y, lap_x = (e[:-2, 1:-1] + e[2:, 1:-1]) - 2 * t, (e[1:-1, :-2] + e[1:-1, 2:]) - 2 * t
        t = t + f(0.5) * p + f(0.1) * lap_y + f(0.1) * lap_x + f(1 / 640) * (f(300) - t)
    ref = oracle.hotspot(t0, p, steps)
    rms = lambda v: float(np.sqrt(np.mean((v.astype(np.float64) - ref) ** 2)))
    assert t.dtype == np.float32 and rms(got) < rms(t)


@pytest.mark.parametrize("shape", [(1, 1), (9, 260), (362, 362), (363, 362), (64, 2048), (64, 2052)])
def test_output_in_every_way(torch_gpu, shape):
    """Grids on both sides of the size up to which the last launch writes the
    output to host memory: the same bits, with their own header, in every way a
    job is launched, several jobs through each slot."""
    h, w = shape
    t0, p = synth.hotspot_input(9, h * 1000 + w, h, w)
    ib, ob = 8 * h * w, 64 + 4 * h * w
    tin, nin = pinned(ib)
    nin[:ib].view(np.float32)[:] = np.concatenate([t0.ravel(), p.ravel()])
    ways = {"direct": (dict(mode="set", callback="event_poll"), dict(copy="async_in")),
            "words, poisoned": (dict(mode="set", callback="host_flag"), dict(flags=A.SET_TF_POISON)),
            "captured": (dict(mode="set", callback="host_flag"), dict(flags=A.SET_TF_CAPTURE)),
            "memcpy nodes": (dict(mode="set", callback="event_poll"), dict(copy="nodes")),
            "batch": (dict(mode="batch", batch_size=4), {})}
    stride = -(-ob // 64) * 64
    for steps in (1, 16, 17):
        ref = oracle.hotspot(t0, p, steps)
        bits = None
        for way, (kw, t) in ways.items():
            print("thermal output", shape, steps, way)
            sys.stdout.flush()
            tout, nout = pinned(stride * 6)
            nout[:] = 0xEE
            with Context(workers=2, slots=2, **kw) as ctx:
                tid = ctx.define("hotspot", width=w, height=h, max_n=steps, **t)
                arr = ctx.job_array(6)
                arr["host_in"], arr["in_bytes"], arr["out_bytes"] = tin.data_ptr(), ib, ob
                arr["host_out"] = tout.data_ptr() + np.arange(6, dtype=np.uint64) * stride
                first = ctx.submit_many(tid, arr)
                ctx.drain()
            for i in range(6):
                o = nout[i * stride:i * stride + ob]
                hd = o[:64].view(A.OUT_HEADER_DTYPE)[0]
                assert hd["job_id"] == first + i and hd["magic"] == A.SET_OUT_MAGIC and hd["canary_ok"] == 1
                if bits is None:
                    bits = o[64:].tobytes()
                    got = o[64:].view(np.float32).reshape(h, w)
                    assert np.max(np.abs(got - ref)) <= oracle.hotspot_tolerance(ref, steps)
                assert o[64:].tobytes() == bits, (way, i)
