"""Prompts without transfers: whichever of one or two chunks the library takes, rows and caches are those of the cut that a
kernel-choice flag pins (lengths on both sides of the limit, and longer ones that the estimate decides).

Bound: both results are bf16 layers within TOL_LAYER of the exact one, so they are within twice that of each other.
"""
import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import TOL_LAYER, f64, make_ctx, run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,split", [(2816, 1408), (2817, 1500), (4096, 2458), (4609, 2304)])
def test_whole_or_cut(T, split):
    hidden, nq, nkv, d, ffn = 512, 4, 1, 128, 768
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=47, dtype="bf16")
    x = iso_inputs.make_hidden(T, hidden, seed=47, dtype="bf16")
    with make_ctx(hidden, nq, nkv, d, ffn, "bf16", T) as ctx:
        got = []
        for flags in (0, iso.ISO_FLAG_NO_STREAMK):
            ctx.set_flags(flags)
            got.append([f64(a) for a in run_layer(ctx, iso.upload_weights(w, "bf16"), x, "bf16", T, split, nkv, d, T,
                                                  iso.ISO_COMM_NONE, poison=True)])
    for a, b in zip(*got):
        assert np.isfinite(a).all()
        assert orc.max_rel_err(a, b) <= 2 * TOL_LAYER["bf16"]


@pytest.mark.parametrize("dt,d,comm,fp8", [("f32", 64, iso.ISO_COMM_D2H, 0), ("bf16", 128, iso.ISO_COMM_NONE, 0),
                                           ("bf16", 64, iso.ISO_COMM_D2H_INT8, 0),
                                           ("bf16", 128, iso.ISO_COMM_D2H, iso.ISO_FLAG_FP8_GEMM)])
def test_keep_cut_runs_every_chunk_that_was_asked_for(dt, d, comm, fp8):
    """By default a short prompt is one chunk; with the flag there are as many launches as chunks, on every schedule, and rows
    and caches agree.  Bounds beside the one above: FP8, the roundings that another order of sums moves shift codes by a step (see
    test_gpu_fp8); int8 payload, a neighbouring code at each of the two points, row maximum (at most 6 rms) / 127 apiece."""
    hidden, nq, nkv, ffn, T, bounds = 512, 4, 2, 768, 300, [70, 130, 131, 280]
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=49, dtype=dt)
    x = iso_inputs.make_hidden(T, hidden, seed=49, dtype=dt)
    with make_ctx(hidden, nq, nkv, d, ffn, dt, T) as ctx:
        wd = iso.upload_weights(w, dt)
        if fp8:
            wd = ctx.add_fp8_weights(wd)
        got = []
        for flags, chunks in ((0, 1), (iso.ISO_FLAG_KEEP_CUT, 5)):
            for sched in (iso.ISO_SCHED_OVERLAP, iso.ISO_SCHED_SERIAL, iso.ISO_SCHED_STREAM_PER_CHUNK):
                ctx.set_flags(flags | fp8)
                xd = iso.DeviceArray.from_numpy(x, dt)
                kc, vc = (iso.DeviceArray((1, T, nkv, d), dt, fill_byte=0xFF) for _ in range(2))
                ctx.timing_enable(True)
                ctx.stack_prefill_chunks([wd], xd, kc, vc, T, bounds, comm, sched)
                ctx.sync()
                n = ctx.timing_read()
                ctx.timing_enable(False)
                assert n["attn"][1] == chunks and n["gemm_down"][1] == chunks
                assert n["comm"][1] == (0 if comm == iso.ISO_COMM_NONE else 2 * chunks)
                got.append([f64(a) for a in (xd, kc, vc)])
    tol = 0.2 if fp8 else 2 * TOL_LAYER[dt] + (2 / 127.0 * 6 if comm == iso.ISO_COMM_D2H_INT8 else 0)
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.isfinite(b).all() and orc.max_rel_err(b, a) <= tol


@pytest.mark.parametrize("fp8", [0, iso.ISO_FLAG_FP8_GEMM])
@pytest.mark.parametrize("T,bounds,sched", [(76000, [38000], iso.ISO_SCHED_SERIAL),
                                            (150000, [30000, 70000, 140000], iso.ISO_SCHED_OVERLAP)])
def test_chunks_are_not_put_together_beyond_the_limits_of_their_kernels(T, bounds, sched, fp8):
    """28672 MLP columns: the down projection's operand reaches 2^31 elements at 74899 rows, where its kernel ends.  All of the
    prompt (76000 rows), or the better of its halves (80000), lies beyond, every chunk below: the cut stays, with the same
    kernels and therefore the same bits as with the cut pinned."""
    hidden, nq, nkv, d, ffn, dt = 128, 1, 1, 128, 28672, "bf16"
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=50, dtype=dt)
    x = iso_inputs.make_hidden(T, hidden, seed=50, dtype=dt)
    with make_ctx(hidden, nq, nkv, d, ffn, dt, T) as ctx:
        wd = iso.upload_weights(w, dt)
        if fp8:
            wd = ctx.add_fp8_weights(wd)
        got = []
        for flags in (0, iso.ISO_FLAG_KEEP_CUT):
            ctx.set_flags(flags | fp8)
            xd = iso.DeviceArray.from_numpy(x, dt)
            kc, vc = (iso.DeviceArray((1, T, nkv, d), dt, fill_byte=0xFF) for _ in range(2))
            ctx.timing_enable(True)
            ctx.stack_prefill_chunks([wd], xd, kc, vc, T, bounds, iso.ISO_COMM_NONE, sched)
            ctx.sync()
            n = ctx.timing_read()
            ctx.timing_enable(False)
            assert n["gemm_down"][1] == len(bounds) + 1
            got.append([a.numpy() for a in (xd, kc, vc)] + [n["quant"][1]])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
