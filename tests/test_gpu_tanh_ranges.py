"""The float32 tanh of the vector kernels, range by range: jobs of one element return
it by itself.  In no range is its largest error above that of the device library's
tanhf (through torch) on the same arguments, and it is odd to the bit."""
import sys

import numpy as np
import pytest

from paper_2606_05495_amd import _abi as A

pytestmark = pytest.mark.gpu

EDGES = [1e-3, 0.1, 0.25, 0.5, 0.8, 1.0, 1.5, 2.0, 2.5, 3.0, 5.0, 9.0]


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _tanh(torch, z):
    """One job an element: a = 1, y = 0."""
    out = torch.empty_like(z)
    y = torch.zeros_like(z)
    st = torch.cuda.current_stream().cuda_stream
    for k in range(0, z.numel(), 16384):
        m = min(16384, z.numel() - k)
        v = np.zeros(m, A.VEC_JOB_DTYPE)
        v["n"], v["a"] = 1, 1.0
        v["x_off"] = v["y_off"] = np.arange(k, k + m)
        jobs = torch.from_numpy(v.view(np.uint8)).cuda()
        A.set_run_vector_jobs_noalloc(0, st, z.data_ptr(), y.data_ptr(), z.numel(), 1, jobs.data_ptr(), m,
                                      out[k:].data_ptr(), None, 0)
    return out


@pytest.mark.parametrize("lo,hi", list(zip(EDGES, EDGES[1:])))
def test_no_range_is_worse_than_the_library(torch_gpu, lo, hi):
    print("tanh from", lo, "to", hi)
    sys.stdout.flush()
    torch = torch_gpu
    z = np.unique(np.linspace(lo, hi, 1 << 19, endpoint=False).astype(np.float32))
    zd = torch.from_numpy(z).cuda()
    got, lib = _tanh(torch, zd).cpu().numpy(), torch.tanh(zd).cpu().numpy()
    ref = np.tanh(z.astype(np.float64))
    ulp = np.spacing(ref.astype(np.float32)).astype(np.float64)
    worst = lambda v: float(np.max(np.abs(v.astype(np.float64) - ref) / ulp))
    assert worst(got) <= worst(lib), (worst(got), worst(lib))
    assert np.array_equal(_tanh(torch, -zd).cpu().numpy(), -got)
