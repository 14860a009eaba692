"""Thermal grids around zero, where the source and not the temperature sets the
size of a step: coefficients that are rounded for grids of 300 K show here."""
import sys

import numpy as np
import pytest

import oracle
from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# the one-cell, register-window and row-band kernels take a single step, the tile kernel several
@pytest.mark.parametrize("shape", [(33, 31), (64, 260), (2048, 2048)])
@pytest.mark.parametrize("kind", ["zero", "cold", "both signs"])
def test_grids_around_zero(torch_gpu, kind, shape):
    """Against the float64 oracle within the bound its docstring derives."""
    h, w = shape
    print("thermal around zero", kind, shape)
    sys.stdout.flush()
    rng = np.random.default_rng(h + w)
    t0 = {"zero": np.zeros(shape), "cold": rng.random(shape), "both signs": rng.standard_normal(shape)}[kind].astype(np.float32)
    p = (np.zeros(shape) if kind == "zero" else 0.01 * rng.random(shape)).astype(np.float32)
    ib, ob = 8 * h * w, 64 + 4 * h * w
    tin, nin = pinned(ib)
    tout, nout = pinned(ob)
    nin[:ib].view(np.float32)[:] = np.concatenate([t0.ravel(), p.ravel()])
    for steps in (1, 2, 9):
        with Context(mode="sync", workers=1, slots=1) as ctx:
            tid = ctx.define("hotspot", width=w, height=h, max_n=steps)
            ctx.submit(tid, host_in=tin.data_ptr(), in_bytes=ib, host_out=tout.data_ptr(), out_bytes=ob)
            ctx.drain()
        got = nout[64:ob].view(np.float32).reshape(shape)
        ref = oracle.hotspot(t0, p, steps)
        assert np.max(np.abs(got - ref)) <= oracle.hotspot_tolerance(ref, steps), (kind, shape, steps)
