"""Host threads that enqueue products on the same stream of one context: a split product is two kernels that hand partial sums
over in the stream's workspace, a stream-K launch carries a number, and neither may get mixed up with another thread's.

Bound: single bf16 products, as in the other projection tests.
"""
import threading

import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import NAN_BYTE, TOL_STEP, dev, f64, h64, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [(7 << 8) | (3 << 17), (7 << 8) | (6 << 17) | (3 << 21), 6 << 8])
def test_products_of_two_threads_on_one_stream(flags):
    dt, reps = "bf16", 40
    sizes = [(200, 520, 1024), (96, 1032, 2048)]
    ops = []
    for i, (M, N, K) in enumerate(sizes):
        a = iso_inputs.randn((M, K), seed=61 + i, dtype=dt)
        w = iso_inputs.randn((N, K), seed=71 + i, dtype=dt, scale=K ** -0.5)
        ops.append((dev(a, dt), dev(w, dt), [iso.DeviceArray((M, N), dt, fill_byte=NAN_BYTE) for _ in range(reps)],
                    orc.linear(h64(a, dt), h64(w, dt))))
    with make_ctx(256, 4, 4, 64, 64, dt, 256) as ctx:
        ctx.set_flags(flags)
        start, errors = threading.Barrier(len(sizes)), []

        def enqueue(i):
            try:
                start.wait()
                for c in ops[i][2]:
                    ctx.gemm_rowpar(ops[i][0], ops[i][1], c, *sizes[i], ctx.stream0)
            except Exception as e:
                errors.append(e)

        threads = [threading.Thread(target=enqueue, args=(i,)) for i in range(len(sizes))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        ctx.sync()
        assert not errors, errors
        for _, _, outs, ref in ops:
            for rep, c in enumerate(outs):
                assert orc.max_rel_err(f64(c), ref) <= TOL_STEP[dt], rep
