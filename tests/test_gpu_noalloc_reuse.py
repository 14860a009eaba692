"""No-allocation calls whose results replace what the call reads, the job array or a
pool: every job's result is that of a call with a place of its own for them."""
import sys

import numpy as np
import pytest

from paper_2606_05495_amd import _abi as A

pytestmark = pytest.mark.gpu

POOL = 1 << 20


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("where", ["jobs", "x", "y"])
@pytest.mark.parametrize("count,n_max", [(2, 9), (200, 4000), (3000, 4000), (200, 70000), (3000, 70000)])
def test_results_in_the_inputs(torch_gpu, count, n_max, where):
    print("results in", where, count, n_max)
    sys.stdout.flush()
    torch = torch_gpu
    rng = np.random.default_rng(count + n_max)
    pools = [torch.from_numpy((2 * rng.random(POOL) - 1).astype(np.float32)).cuda() for _ in range(2)]
    v = np.zeros(count, A.VEC_JOB_DTYPE)
    v["n"] = rng.integers(1, n_max + 1, count)
    v["x_off"], v["y_off"] = (rng.integers(0, POOL - v["n"].astype(np.int64)) for _ in range(2))
    v["a"] = 1.5

    def call(reuse):
        x, y = (p.clone() for p in pools)
        jobs = torch.from_numpy(v.view(np.uint8).copy()).cuda()
        out = {None: torch.zeros(count, dtype=torch.float32, device="cuda"), "jobs": jobs.view(torch.float32),
               "x": x[POOL // 2:], "y": y[POOL // 2:]}[reuse]
        A.set_run_vector_jobs_noalloc(0, torch.cuda.current_stream().cuda_stream, x.data_ptr(), y.data_ptr(), POOL, n_max,
                                      jobs.data_ptr(), count, out.data_ptr(), None, 0)
        return out[:count].cpu().numpy()

    assert call(where).tobytes() == call(None).tobytes()
