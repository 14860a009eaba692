"""Vector jobs at the edges of their units: the float32 tanh by itself, lengths
around a unit's and a row's end, tables long enough for every round of the job
search, and claims of several units."""
import sys

import numpy as np
import pytest

import oracle
from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd.runtime import Context

pytestmark = pytest.mark.gpu

POOL = 1 << 22


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def pools(torch_gpu):
    rng = np.random.default_rng(3)
    x = (2 * rng.random(POOL) - 1).astype(np.float32)
    y = (2 * rng.random(POOL) - 1).astype(np.float32)
    return x, y, torch_gpu.from_numpy(x).cuda(), torch_gpu.from_numpy(y).cuda()


def _noalloc(torch, xd, yd, jobs, max_n, tuning=None, grid=0):
    jd = torch.from_numpy(jobs.view(np.uint8).copy()).cuda()
    rd = torch.full((len(jobs),), -7.0, dtype=torch.float32, device="cuda")
    st = torch.cuda.current_stream()
    A.set_run_vector_jobs_noalloc(0, st.cuda_stream, xd.data_ptr(), yd.data_ptr(), xd.numel(), max_n, jd.data_ptr(),
                                  len(jobs), rd.data_ptr(), tuning, grid)
    return rd.cpu().numpy()


def _jobs(n, xo, yo, a):
    v = np.zeros(len(n), A.VEC_JOB_DTYPE)
    v["n"], v["x_off"], v["y_off"], v["a"] = n, xo, yo, a
    return v


def test_tanh_of_one_element(torch_gpu):
    """Jobs of one element return the float32 tanh itself: within 1.5 ulp of
    float64 (the reciprocal's and the exponential's ulp each count for at most
    0.4 of the result's at the branch, the last rounding for half), odd, and
    exact at zero, infinity and where the result rounds to one."""
    print("tanh of one element")
    sys.stdout.flush()
    mag = np.concatenate([np.geomspace(1e-38, 1e-3, 500), np.linspace(1e-3, 9.5, 15000), [0.8, np.nextafter(0.8, 0)]])
    z = np.concatenate([mag, -mag]).astype(np.float32)
    special = np.array([0.0, np.inf, -np.inf, np.nan, 10.0, -10.0, 3e38, -3e38], np.float32)
    xd = torch_gpu.from_numpy(np.concatenate([z, special])).cuda()
    yd = torch_gpu.zeros_like(xd)
    k = np.arange(xd.numel())
    for part in (k[:16000], k[16000:]):
        got = _noalloc(torch_gpu, xd, yd, _jobs(np.ones(len(part), np.int64), part, part, 1.0), 1)
        for i, t in zip(part, got):
            v = float(xd[i]) if i >= len(z) else None
            if v is not None:
                assert (np.isnan(t) and np.isnan(v)) or t == np.float32(np.tanh(v)), (v, t)
        ok = part < len(z)
        ref = np.tanh(z[part[ok]].astype(np.float64))
        ulp = np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
        err = np.abs(got[ok].astype(np.float64) - ref) / ulp
        assert err.max() <= 1.5, (z[part[ok]][err.argmax()], err.max())


@pytest.mark.parametrize("block", [128, 256, 512, 1024])
def test_lengths_around_rows_and_units(torch_gpu, pools, block):
    """One element either side of a row of groups, of a round of loads and of a
    unit, for each block size, at offsets of every alignment; the same bits
    where the template's room lets blocks take units and where they take items."""
    print("unit edges, block", block)
    sys.stdout.flush()
    x, y, xd, yd = pools
    tile = 65536
    edges = sorted({4 * block, 16 * block, 64 * block, tile // 4, tile // 2, tile, 2 * tile})
    n = np.array([max(1, e + k) for e in edges for k in (-5, -1, 0, 1, 3)])
    jobs = _jobs(n, np.arange(len(n)) % 7, np.arange(len(n)) % 5, 1.25)
    tune = A.set_vec_tuning()
    for b in range(64):
        tune.tile_elems[b] = tile
    with Context(mode="set", workers=2, slots=2) as ctx:
        units = ctx.define("saxpy_batch", max_n=POOL, x_pool=xd, y_pool=yd, batch_max=64, tiles_max=256, block=block)
        items = ctx.define("saxpy_batch", max_n=POOL, x_pool=xd, y_pool=yd, batch_max=8, tiles_max=8, block=block)
        res, _ = ctx.run_vector_jobs(units, jobs, tuning=tune)
        whole, _ = ctx.run_vector_jobs(items, jobs, tuning=tune)
    assert np.array_equal(res.view(np.uint32), whole.view(np.uint32))
    for i, j in enumerate(jobs):
        S, E = oracle.saxpy_tanh_sum(x[j["x_off"]:j["x_off"] + j["n"]], y[j["y_off"]:j["y_off"] + j["n"]], j["a"])
        assert abs(float(res[i]) - S) <= oracle.vec_tolerance(S, E), (block, int(j["n"]), res[i], S)


@pytest.mark.parametrize("count,n_max,grid", [(1, 5, 0), (64, 70000, 0), (65, 300, 3), (256, 9000, 2), (257, 20000, 1), (4097, 3000, 0),
                                              (16384, 1500, 5)])
def test_job_search_and_claims(torch_gpu, pools, count, n_max, grid):
    """Tables of one to three rounds of the job search, rejected jobs among
    them, on few blocks (many claims, runs of several units) and on many; up to 256
    jobs each block plans for itself."""
    print("job search", count, n_max, grid)
    sys.stdout.flush()
    x, y, xd, yd = pools
    rng = np.random.default_rng(count)
    n = rng.integers(1, n_max + 1, count)
    jobs = _jobs(n, rng.integers(0, POOL - n_max, count), rng.integers(0, POOL - n_max, count), 0.75)
    drop = np.arange(count) % 11 == 10
    jobs["n"][drop] = 0
    got = _noalloc(torch_gpu, xd, yd, jobs, n_max, None, grid)
    again = _noalloc(torch_gpu, xd, yd, jobs, n_max, None, 0 if grid else 7)
    assert np.array_equal(got.view(np.uint32), again.view(np.uint32))  # the grid changes no result
    assert np.isnan(got[drop]).all()
    for i in np.flatnonzero(~drop)[::max(1, count // 300)]:
        j = jobs[i]
        S, E = oracle.saxpy_tanh_sum(x[j["x_off"]:j["x_off"] + j["n"]], y[j["y_off"]:j["y_off"] + j["n"]], j["a"])
        assert abs(float(got[i]) - S) <= oracle.vec_tolerance(S, E), (i, int(j["n"]), got[i], S)


@pytest.mark.parametrize("n_max", [1, 3, 4, 257, 1023, 1024, 1025, 8192, 16383, 16384, 32767])
@pytest.mark.parametrize("count", [1, 2, 255, 300, 3000])
def test_short_jobs_match_the_general_path(torch_gpu, pools, count, n_max):
    """A call of short jobs (a block to a job) gives the bits of the same call with
    a grid, which takes the planned path: any alignment, lengths around items and
    rows, rejected jobs, NaN and infinities, and items of 2048 elements."""
    print("short jobs", count, n_max)
    sys.stdout.flush()
    rng = np.random.default_rng(count * 40000 + n_max)
    xd, yd = pools[2].clone(), pools[3]
    at = torch_gpu.from_numpy(rng.integers(0, POOL, 64)).cuda()
    xd[at[:32]] = float("inf")
    xd[at[32:48]] = float("nan")
    edges = [v for v in (1, 2, 3, 4, 5, 255, 256, 1023, 1024, 1025, 2047, 2048, 2049, n_max - 1, n_max) if 1 <= v <= n_max]
    n = np.where(rng.random(count) < 0.5, rng.choice(edges, count), rng.integers(1, n_max + 1, count))
    jobs = _jobs(n, rng.integers(0, POOL - n), rng.integers(0, POOL - n), rng.uniform(0.5, 2, count).astype(np.float32))
    bad = rng.random(count) < 0.05
    jobs["n"][bad & (jobs["n"] % 2 == 0)] = 0
    jobs["n"][bad & (jobs["n"] % 2 == 1)] = n_max + 1
    jobs["x_off"][rng.random(count) < 0.02] = POOL
    tuning = A.set_vec_tuning()
    for b in range(64):
        tuning.tile_elems[b] = 2048
    for t in (None, tuning):
        got = _noalloc(torch_gpu, xd, yd, jobs, n_max, t)
        want = _noalloc(torch_gpu, xd, yd, jobs, n_max, t, grid=7)
        same = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
        assert same.all(), (n[~same], got[~same], want[~same])
        assert np.isnan(got[jobs["n"] == 0]).all() and np.isnan(got[jobs["n"] > n_max]).all()
