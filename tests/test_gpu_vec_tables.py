"""Vector batches whose descriptor table is submitted by hand, with set_submit:
only the words that describe the jobs and their work items count, whatever the
table's padding holds."""
import sys

import numpy as np
import pytest

import oracle
from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd.runtime import Context, pinned

pytestmark = pytest.mark.gpu

HDR = np.dtype([("count", "<u4"), ("total_tiles", "<u4"), ("pad", "<u4", 14)])
DESC = np.dtype([("x_off", "<u8"), ("y_off", "<u8"), ("n", "<u4"), ("a", "<f4"), ("tile_start", "<u4"),
                 ("ntiles", "<u4"), ("tile_elems", "<u4"), ("pad", "<u4", 3)])
POOL = 1 << 21


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def pools(torch_gpu):
    rng = np.random.default_rng(17)
    x = (2 * rng.random(POOL) - 1).astype(np.float32)
    y = (2 * rng.random(POOL) - 1).astype(np.float32)
    return x, y, torch_gpu.from_numpy(x).cuda(), torch_gpu.from_numpy(y).cuda()


def _table(buf, jobs, items, padding, past_end):
    count = len(jobs)
    h, d = buf[:64].view(HDR), buf[64:64 + 48 * count].view(DESC)
    buf[:64 + 48 * count] = padding
    d["x_off"], d["y_off"], d["n"], d["a"], d["tile_elems"] = jobs["x_off"], jobs["y_off"], jobs["n"], jobs["a"], items
    d["ntiles"] = -(-jobs["n"].astype(np.int64) // items) + past_end
    d["tile_start"] = np.concatenate([[0], np.cumsum(d["ntiles"][:-1])])
    h["count"], h["total_tiles"] = count, d["ntiles"].sum()


@pytest.mark.parametrize("block", [128, 256, 1024])
@pytest.mark.parametrize("room", [8, 1025])  # the last kernel writes the results, or a copy does
def test_tables_by_hand(torch_gpu, pools, room, block):
    """The bits of set_run_vector_jobs at the same item size; sizes it does not
    take, and items past a job's end, against the oracle."""
    x, y, xd, yd = pools
    rng = np.random.default_rng(block + room)
    count = 8
    jobs = np.zeros(count, A.VEC_JOB_DTYPE)
    jobs["n"] = [1, 3, 1023, 1024, 65537, 200001, 262144, 300000]
    jobs["x_off"] = rng.integers(0, POOL - jobs["n"].astype(np.int64))
    jobs["y_off"] = rng.integers(0, POOL - jobs["n"].astype(np.int64))
    jobs["a"] = rng.uniform(0.5, 2, count)
    tin, nin = pinned(64 + 48 * count)
    tout, nout = pinned(64 + 4 * count)
    with Context(mode="set", workers=2, slots=2) as ctx:
        tid = ctx.define("saxpy_batch", max_n=POOL, x_pool=xd, y_pool=yd, batch_max=room, tiles_max=2048, block=block)
        for item in (1024, 65536, 262144, 5001, 131076, 300000):
            want = None
            if item % 1024 == 0:
                tune = A.set_vec_tuning()
                for b in range(64):
                    tune.tile_elems[b] = item
                want, _ = ctx.run_vector_jobs(tid, jobs, tuning=tune)
            for padding in (0, 0xFF, rng.integers(0, 256, 64 + 48 * count)):
                for grid, past_end in ((0, 0), (3, 0), (3, 1)):
                    print("table by hand", room, block, item, grid, past_end)
                    sys.stdout.flush()
                    _table(nin, jobs, item, padding, past_end)
                    nout[:] = 0xEE
                    args = A.set_job_args(tin.data_ptr(), 64 + 48 * count, tout.data_ptr(), 64 + 4 * count, count, 0.0, -1)
                    args.grid = grid
                    A.set_submit(ctx.h, tid, args, 0)
                    ctx.drain()
                    got = nout[64:64 + 4 * count].view(np.float32).copy()
                    if want is not None:
                        assert got.tobytes() == want.tobytes(), (item, got, want)
                    for j, s in zip(jobs, got):
                        S, E = oracle.saxpy_tanh_sum(x[j["x_off"]:j["x_off"] + j["n"]], y[j["y_off"]:j["y_off"] + j["n"]], j["a"])
                        assert abs(float(s) - S) <= oracle.vec_tolerance(S, E), (item, int(j["n"]), s, S)
