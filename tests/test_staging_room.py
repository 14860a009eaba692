"""Callers that wait for room in the staging ring, on the CPU fake backend: rings
on both sides of the size from which they are woken at half room, one and several
submitting threads, streams several times the ring."""
import threading

import numpy as np
import pytest

from paper_2606_05495_amd.runtime import Context


@pytest.mark.parametrize("threads", [1, 3])
@pytest.mark.parametrize("ring", [1, 2, 127, 128, 129, 300])
def test_streams_longer_than_the_ring(ring, threads):
    per = 3 * ring + 5
    with Context(backend="fake", workers=4, slots=4, dispatchers=2, staging=ring) as ctx:
        tid = ctx.define("saxpy_tanh_sum", max_n=1 << 20, pool_ptrs=(0x1000, 0x2000, 1 << 30))
        outs = np.zeros((threads * per, 128), np.uint8)
        errors = []

        def stream(k):
            arr = ctx.job_array(per)
            arr["host_out"] = outs.ctypes.data + (k * per + np.arange(per, dtype=np.uint64)) * 128
            arr["out_bytes"], arr["n"], arr["a"] = 68, 5, 1.0
            try:
                ctx.submit_many(tid, arr)
            except Exception as e:  # reported by the main thread
                errors.append(e)

        ts = [threading.Thread(target=stream, args=(k,)) for k in range(threads)]
        for t in ts:
            t.start()
        for t in ts:
            t.join(60)
        assert not errors and not any(t.is_alive() for t in ts)
        ctx.drain(timeout_ns=60_000_000_000)
        st = ctx.stats()
        assert st.completed == st.submitted == threads * per and st.failed == 0
