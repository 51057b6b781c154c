"""The 256-column projection tiles with 256, 192 and 128 rows, whole and in shares, at the edges of tiles and of the two-slice
pipeline, with every epilogue.

Bounds as in the other projection tests: one bf16 rounding (2^-8 relative) and fp32 sums, 1e-2; FP8 against another kernel:
exact products, fp32 sums in another order, at most one bf16 unit in the last place.
"""
import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_fp8 import TOL_LAYER_FP8
from test_gpu_parity import NAN_BYTE, TOL_LAYER, TOL_STEP, dev, f64, h64, make_ctx, oracle_weights, run_layer, shape_of

pytestmark = pytest.mark.gpu

WHOLE = {256: 1 << 8, 192: 5 << 8, 128: 4 << 8}
SHARE_TILE = {256: 4, 192: 5, 128: 6}


def shares(bm, n):
    return (7 << 8) | (n << 17) | (SHARE_TILE[bm] << 21)


# one to five slices (prologue alone, both stages, the unrolled pair and its odd end), one row more and less than the tiles and
# their halves, a last column block of 8
@pytest.mark.parametrize("bm", [256, 192, 128])
@pytest.mark.parametrize("M,N,K,S", [(1, 8, 64, 1), (63, 256, 128, 1), (65, 264, 192, 1), (129, 504, 256, 1), (255, 40, 320, 1),
                                     (257, 520, 704, 1), (97, 264, 256, 2), (300, 520, 704, 5)])
def test_gemm(bm, M, N, K, S):
    a = iso_inputs.randn((M, K), seed=M + N, dtype="bf16")
    w = iso_inputs.randn((N, K), seed=M + K, dtype="bf16", scale=K ** -0.5)
    with make_ctx(256, 4, 4, 64, 64, "bf16", 512) as ctx:
        ctx.set_flags(WHOLE[bm] if S == 1 else shares(bm, S))
        c = iso.DeviceArray((M, N), "bf16", fill_byte=NAN_BYTE)
        ctx.gemm_rowpar(dev(a, "bf16"), dev(w, "bf16"), c, M, N, K, ctx.stream0)
        ctx.sync()
        assert orc.max_rel_err(f64(c), orc.linear(h64(a, "bf16"), h64(w, "bf16"))) <= TOL_STEP["bf16"]


@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (129, 264, 128), (300, 520, 704)])
def test_plain_main_loop_of_the_128_x_256_tile(M, N, K):
    a = iso_inputs.randn((M, K), seed=M + N, dtype="bf16")
    w = iso_inputs.randn((N, K), seed=M + K, dtype="bf16", scale=K ** -0.5)
    with make_ctx(256, 4, 4, 64, 64, "bf16", 512) as ctx:
        ctx.set_flags(12 << 8)
        c = iso.DeviceArray((M, N), "bf16", fill_byte=NAN_BYTE)
        ctx.gemm_rowpar(dev(a, "bf16"), dev(w, "bf16"), c, M, N, K, ctx.stream0)
        ctx.sync()
        assert orc.max_rel_err(f64(c), orc.linear(h64(a, "bf16"), h64(w, "bf16"))) <= TOL_STEP["bf16"]


@pytest.mark.parametrize("bm", [256, 192, 128])
@pytest.mark.parametrize("M,N,K,S", [(1, 8, 128, 1), (97, 264, 256, 1), (129, 504, 384, 1), (257, 520, 640, 1), (300, 264, 1408, 3)])
def test_gemm_fp8(bm, M, N, K, S):
    with make_ctx(256, 4, 4, 64, 64, "bf16", 512) as ctx:
        q = []
        for rows, seed in ((M, 1), (N, 2)):
            codes, scale = iso.DeviceArray((rows, K), "u8"), iso.DeviceArray((rows,), "f32")
            x = dev(iso_inputs.randn((rows, K), seed=seed + K, dtype="bf16"), "bf16")
            ctx.quantize_rows_fp8(x, rows, K, codes, scale, ctx.stream0)
            q += [codes, scale]
        outs = []
        for f in (WHOLE[bm] if S == 1 else shares(bm, S), 3 << 8):
            ctx.set_flags(f)
            outs.append(iso.DeviceArray((M, N), "bf16", fill_byte=NAN_BYTE))
            ctx.gemm_fp8(q[0], q[1], q[2], q[3], outs[-1], M, N, K, ctx.stream0)
        ctx.sync()
        assert orc.max_rel_err(f64(outs[0]), f64(outs[1])) <= 2.0 ** -7


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("bm", [256, 192, 128])
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,T,split", [(512, 4, 1, 128, 776, 300, 130), (640, 6, 2, 64, 648, 259, 0),
                                                         (384, 3, 3, 128, 512, 97, 50)])
def test_layer(bm, fp8, hidden, nq, nkv, d, ffn, T, split):
    """SwiGLU and the rotary step + cache write in the epilogue, both head sizes, head counts that leave a tile half empty, against
    the separate kernels: same projection outputs, so V rows are the same bits and K rows too (same rotation)."""
    ffn = ffn // 128 * 128 if fp8 else ffn                          # every projection in FP8, as in the oracle
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=41, dtype="bf16")
    x = iso_inputs.make_hidden(T, hidden, seed=41, dtype="bf16")
    ref = orc.layer_unsplit(h64(x, "bf16"), oracle_weights(w, "bf16"), shape_of(hidden, nq, nkv, d, ffn), fp8=fp8)
    max_seq = T + 5                                                 # rows past the prompt must stay untouched
    with make_ctx(hidden, nq, nkv, d, ffn, "bf16", max_seq) as ctx:
        wd = iso.upload_weights(w, "bf16")
        base = iso.ISO_FLAG_KEEP_CUT
        if fp8:
            wd = ctx.add_fp8_weights(wd)
            base |= iso.ISO_FLAG_FP8_GEMM
        got = []
        for flags in (WHOLE[bm], WHOLE[bm] | iso.ISO_FLAG_NO_FUSE):
            ctx.set_flags(flags | base)
            ctx.timing_enable(True)
            out, kc, vc = run_layer(ctx, wd, x, "bf16", T, split, nkv, d, max_seq, iso.ISO_COMM_D2H, poison=True)
            got.append((f64(out), kc.numpy(), vc.numpy(), ctx.timing_read()["rope_kv"][1]))
            ctx.timing_enable(False)
            assert np.isnan(f64(kc)[T:]).all() and np.isnan(f64(vc)[T:]).all()
            err = orc.max_rel_err(got[-1][0], ref["x_out"])
            assert err <= (TOL_LAYER_FP8 if fp8 else TOL_LAYER["bf16"])
        assert got[0][3] == 0 and got[1][3] == (2 if split else 1)
        np.testing.assert_array_equal(got[0][1][:T], got[1][1][:T])
        np.testing.assert_array_equal(got[0][2][:T], got[1][2][:T])


@pytest.mark.parametrize("hidden,nq,nkv,ffn,T,split", [(640, 6, 2, 648, 259, 0), (256, 3, 3, 520, 127, 63), (128, 1, 1, 264, 129, 1),
                                                       (512, 5, 1, 520, 400, 128)])
def test_heads_of_64_in_the_128_x_128_tile(hidden, nq, nkv, ffn, T, split):
    """A wave of the 128 x 128 tile owns one head of 64: rotary step and cache write in its epilogue, at odd head counts (half of
    the last tile empty) and row remainders, against the separate kernel.  The projection is the same and the rotation is written
    with the same operations: V and K rows are the same bits."""
    w = iso_inputs.make_layer(hidden, nq, nkv, 64, ffn, seed=43, dtype="bf16")
    x = iso_inputs.make_hidden(T, hidden, seed=43, dtype="bf16")
    ref = orc.layer_unsplit(h64(x, "bf16"), oracle_weights(w, "bf16"), shape_of(hidden, nq, nkv, 64, ffn))
    max_seq = T + 5
    with make_ctx(hidden, nq, nkv, 64, ffn, "bf16", max_seq) as ctx:
        wd = iso.upload_weights(w, "bf16")
        got = []
        for flags in (3 << 8, 3 << 8 | iso.ISO_FLAG_NO_FUSE):
            ctx.set_flags(flags | iso.ISO_FLAG_KEEP_CUT)
            ctx.timing_enable(True)
            out, kc, vc = run_layer(ctx, wd, x, "bf16", T, split, nkv, 64, max_seq, iso.ISO_COMM_D2H, poison=True)
            got.append((kc.numpy(), vc.numpy(), ctx.timing_read()["rope_kv"][1]))
            ctx.timing_enable(False)
            assert np.isnan(f64(kc)[T:]).all() and np.isnan(f64(vc)[T:]).all()
            assert orc.max_rel_err(f64(out), ref["x_out"]) <= TOL_LAYER["bf16"]
        assert got[0][2] == 0 and got[1][2] == (2 if split else 1)
        np.testing.assert_array_equal(got[0][0][:T], got[1][0][:T])
        np.testing.assert_array_equal(got[0][1][:T], got[1][1][:T])
