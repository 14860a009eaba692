"""Limits of a vector request that set_serve checks, on the CPU fake backend."""
import numpy as np
import pytest

from paper_2606_05495_amd import _abi as A
from paper_2606_05495_amd.runtime import Context

POOLS = (0x1000, 0x2000, 1 << 30)


@pytest.mark.parametrize("tile", [1024, 4096, 1000])
def test_a_request_of_more_items_than_the_batch_holds_is_refused(tile):
    """A batch's partial sums have room for tiles_max work items: a request that needs
    that many is served, one that needs one more is refused like the same job in
    set_run_vector_jobs, and nothing of the schedule runs."""
    tune = A.set_vec_tuning()
    for b in range(64):
        tune.tile_elems[b] = tile
    cfg = A.set_serve_config()
    cfg.tuning = A.ctypes.pointer(tune)
    with Context(backend="fake", workers=2, slots=2) as ctx:
        tid = ctx.define("saxpy_batch", max_n=1 << 20, pool_ptrs=POOLS, batch_max=8, tiles_max=64)
        req = np.zeros(3, A.REQUEST_DTYPE)
        req["template_id"] = tid
        req["a"] = 1.0
        req["n"] = 5, 64 * tile, 64 * tile
        done, st = A.set_serve(ctx.h, req, cfg, np.zeros(3, np.float32))
        assert st.completed == 3 and np.all(done > 0)
        req["n"] = 5, 64 * tile, 64 * tile + 1
        with pytest.raises(A.SetError) as e:
            A.set_serve(ctx.h, req, cfg, np.zeros(3, np.float32))
        assert e.value.code == A.SET_EINVAL and "tiles_max" in str(e.value)
        assert ctx.stats().completed == st.vec_batches
