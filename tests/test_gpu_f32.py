"""fp32 projections on the fp32 matrix instructions against the CPU oracle, at the edges of their two tile shapes.

Bound: fp32 sums of K products of N(0, 1) and N(0, 1/K) values, relative to the rms of a result (1): K rounding errors of at
most 2^-24 |partial sum| each, of random sign -- 2e-5 covers K = 1664 in the other projection tests as well.
"""
import ctypes

import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import NAN_BYTE, TOL_LAYER, TOL_STEP, dev, f64, h64, make_ctx, run_layer, oracle_weights, shape_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 1, 4), (5, 16, 12), (17, 33, 68),     # less than a tile, one row and column past it, less than a k-step
    (16, 16, 16), (31, 47, 252),              # exactly one k-step for four waves; a last k-step of 12
    (1030, 1100, 36),                         # 17 x 18 tiles of 64 x 64: the larger shape, ragged both ways
])
def test_gemm_rowpar_f32(M, N, K):
    a = iso_inputs.randn((M, K), seed=M + N, dtype="f32")
    w = iso_inputs.randn((N, K), seed=M + K, dtype="f32", scale=K ** -0.5)
    with make_ctx(256, 4, 4, 64, 64, "f32", 256) as ctx:
        c = iso.DeviceArray((M, N), "f32", fill_byte=NAN_BYTE)
        ctx.gemm_rowpar(dev(a, "f32"), dev(w, "f32"), c, M, N, K, ctx.stream0)
        ctx.sync()
        assert orc.max_rel_err(f64(c), orc.linear(h64(a, "f32"), h64(w, "f32"))) <= TOL_STEP["f32"]


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,T,split", [
    (256, 4, 4, 64, 688, 33, 0), (264, 2, 1, 128, 200, 150, 61), (128, 2, 2, 64, 1032, 1100, 0)])
def test_layer_f32_fused_swiglu(hidden, nq, nkv, d, ffn, T, split):
    """SwiGLU in the gate/up projection's epilogue (both tile shapes), attention of both head sizes over several key tiles
    per wave."""
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=41, dtype="f32")
    x = iso_inputs.make_hidden(T, hidden, seed=41, dtype="f32")
    ref = orc.layer_unsplit(h64(x, "f32"), oracle_weights(w, "f32"), shape_of(hidden, nq, nkv, d, ffn))
    with make_ctx(hidden, nq, nkv, d, ffn, "f32", T + 3) as ctx:
        out, kc, vc = run_layer(ctx, iso.upload_weights(w, "f32"), x, "f32", T, split, nkv, d, T + 3, iso.ISO_COMM_D2H,
                                poison=True)
        assert orc.max_rel_err(f64(out), ref["x_out"]) <= TOL_LAYER["f32"]
        assert orc.max_rel_err(f64(kc)[:T], ref["k_cache"]) <= TOL_LAYER["f32"]
        assert np.isnan(f64(kc)[T:]).all()


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,T,split", [
    (64, 4, 2, 64, 200, 17, 5), (264, 2, 1, 128, 520, 150, 61), (264, 4, 4, 64, 688, 129, 128), (256, 4, 1, 64, 688, 300, 31)])
def test_rotary_step_and_cache_write_in_the_qkv_epilogue_f32(hidden, nq, nkv, d, ffn, T, split):
    """Against the separate rotary kernel, which rotates with the same operations: same bits; key counts at the edge of the two
    attention shapes."""
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=43, dtype="f32")
    x = iso_inputs.make_hidden(T, hidden, seed=43, dtype="f32")
    ref = orc.layer_unsplit(h64(x, "f32"), oracle_weights(w, "f32"), shape_of(hidden, nq, nkv, d, ffn))
    with make_ctx(hidden, nq, nkv, d, ffn, "f32", T + 3) as ctx:
        got = []
        for flags in (0, iso.ISO_FLAG_NO_FUSE):
            ctx.set_flags(flags | iso.ISO_FLAG_KEEP_CUT)        # the second chunk rotates from q_offset = split on
            out, kc, vc = run_layer(ctx, iso.upload_weights(w, "f32"), x, "f32", T, split, nkv, d, T + 3, iso.ISO_COMM_D2H,
                                    poison=True)
            assert orc.max_rel_err(f64(out), ref["x_out"]) <= TOL_LAYER["f32"]
            assert np.isnan(f64(kc)[T:]).all() and np.isnan(f64(vc)[T:]).all()
            got.append((kc.numpy()[:T], vc.numpy()[:T]))
        np.testing.assert_array_equal(got[0][0], got[1][0])
        np.testing.assert_array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("hidden,T,split,in_qkv,in_gate_up", [
    (8, 1, 0, 1, 1), (64, 17, 0, 1, 1), (256, 37, 16, 1, 1), (264, 150, 61, 1, 0), (768, 33, 0, 1, 0), (776, 33, 0, 0, 0)])
def test_norms_and_copies_of_a_short_layer_in_its_projections_f32(hidden, T, split, in_qkv, in_gate_up):
    """Norms computed by the projections behind them (up to the longest row that each takes and one piece past it) and partials stored
    to the host by the projections in front of the copies, against the kernels one by one: sums of squares in the same order, so
    everything is the same bits.  Timed, a layer keeps its copies as launches; its records say which norms were launches."""
    nq, nkv, d, ffn = 2, 1, 64, 72
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=47, dtype="f32")
    x = iso_inputs.make_hidden(T, hidden, seed=47, dtype="f32")
    ref = orc.layer_unsplit(h64(x, "f32"), oracle_weights(w, "f32"), shape_of(hidden, nq, nkv, d, ffn))
    with make_ctx(hidden, nq, nkv, d, ffn, "f32", T + 3) as ctx:
        wd = iso.upload_weights(w, "f32")
        sink = np.frombuffer((ctypes.c_char * (2 * (T + 3) * hidden * 4)).from_address(ctx.host_sink()), dtype=np.float32)
        sink = sink.reshape(2, T + 3, hidden)
        got = []
        for flags, timed in ((0, False), (0, True), (iso.ISO_FLAG_NO_FUSE, False)):
            ctx.set_flags(flags | iso.ISO_FLAG_KEEP_CUT)
            sink[:] = np.nan
            ctx.timing_enable(timed)
            out, kc, vc = run_layer(ctx, wd, x, "f32", T, split, nkv, d, T + 3, iso.ISO_COMM_D2H, poison=True)
            if timed:
                launches, chunks = ctx.timing_read(), 2 if split else 1
                assert launches["rmsnorm"][1] == (0 if in_qkv else chunks)
                assert launches["resid_norm"][1] == (0 if in_gate_up else chunks)
                assert launches["comm"][1] == 2 * chunks
                ctx.timing_enable(False)
            assert orc.max_rel_err(f64(out), ref["x_out"]) <= TOL_LAYER["f32"]
            assert np.isnan(sink[:, T:]).all()
            got.append((out.numpy().copy(), kc.numpy()[:T].copy(), vc.numpy()[:T].copy(), sink[:, :T].copy()))
        for other in got[1:]:
            for a, b in zip(got[0], other):
                np.testing.assert_array_equal(a, b)
        # what the host holds is what the layer added to its input
        out, sunk = got[0][0].astype(np.float64), got[0][3].astype(np.float64)
        np.testing.assert_allclose(out, h64(x, "f32") + sunk[0] + sunk[1], rtol=0, atol=1e-5)
