"""Vector batches whose descriptor table is submitted by hand, with set_submit:
only the words that describe the jobs and their work items count, whatever the
table's padding holds."""
import ctypes
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


@pytest.mark.parametrize("room", [64, 4096])  # tiles_max: a block takes whole items, or their units
@pytest.mark.parametrize("item", [1000, 65539, 131079, 200003])
def test_serving_with_items_of_any_size(torch_gpu, pools, item, room):
    """set_serve takes its tuning's item sizes as they are: one that has no four equal
    parts is summed whole, with the bits of the same request in a batch by hand."""
    print("serving, items of", item, room)
    sys.stdout.flush()
    x, y, xd, yd = pools
    rng = np.random.default_rng(item)
    n = np.array([1, 999, 1001, 60000])[:, None].repeat(4, 1).ravel() if item == 1000 else rng.integers(1, 800000, 16)
    req = np.zeros(len(n), A.REQUEST_DTYPE)
    req["n"], req["a"], req["worker_hint"] = n, rng.uniform(0.5, 2, len(n)), -1
    req["x_off"], req["y_off"] = rng.integers(0, POOL - n), rng.integers(0, POOL - n)
    tune = A.set_vec_tuning()
    for b in range(64):
        tune.tile_elems[b] = item
    cfg = A.set_serve_config()
    cfg.tuning = ctypes.pointer(tune)
    got = np.zeros(len(n), np.float32)
    with Context(mode="set", workers=2, slots=2, callback="host_flag") as ctx:
        tid = ctx.define("saxpy_batch", max_n=POOL, x_pool=xd, y_pool=yd, batch_max=8, tiles_max=room, copy="async_in")
        req["template_id"] = tid
        _, st = A.set_serve(ctx.h, req, cfg, got)
        assert st.completed == len(n) and st.failed == 0
        tin, nin = pinned(64 + 48)
        tout, nout = pinned(64 + 4)
        for j, s in zip(req, got):
            _table(nin, np.array([j]), item, 0, 0)
            ctx.submit(tid, host_in=tin.data_ptr(), in_bytes=64 + 48, host_out=tout.data_ptr(), out_bytes=68, n=1)
            ctx.drain()
            assert nout[64:68].tobytes() == s.tobytes(), (item, int(j["n"]))
            S, E = oracle.saxpy_tanh_sum(x[j["x_off"]:j["x_off"] + j["n"]], y[j["y_off"]:j["y_off"] + j["n"]], j["a"])
            assert abs(float(s) - S) <= oracle.vec_tolerance(S, E), (item, int(j["n"]), s, S)
