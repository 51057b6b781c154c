"""Narrow tiles and split k ranges of the projection GEMM against the CPU oracle, at the edges of tiles, slices and shares.

Bound of a single product: the bf16 rounding of the result alone is 2^-8 relative (3.9e-3); the fp32 partial sums add
K * 2^-24 at most.  1e-2 is the bound the other projection tests use.
"""
import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import NAN_BYTE, TOL_LAYER, TOL_STEP, dev, f64, h64, make_ctx, run_layer, oracle_weights, shape_of

pytestmark = pytest.mark.gpu

TILES = [0, 1, 2, 3, 4]


def forced(tile, shares):
    return (7 << 8) | (shares << 17) | (tile << 21)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K,shares", [
    (1, 8, 64, 1),          # one row, one piece of columns, one slice
    (31, 72, 128, 2),       # one slice per share
    (33, 136, 704, 3),      # eleven slices in three shares: 3 + 4 + 4
    (129, 264, 1024, 15),   # sixteen slices in fifteen shares
    (257, 520, 448, 2),     # a row past the largest tile, fewer slices than the deepest pipeline has stages
    (300, 64, 4096, 4),     # a single tile column
])
def test_split_gemm(tile, M, N, K, shares):
    dt = "bf16"
    a = iso_inputs.randn((M, K), seed=M + N, dtype=dt)
    w = iso_inputs.randn((N, K), seed=M + K, dtype=dt, scale=K ** -0.5)
    ref = orc.linear(h64(a, dt), h64(w, dt))
    with make_ctx(256, 4, 4, 64, 64, dt, 256) as ctx:
        ctx.set_flags(forced(tile, shares))
        ad, wd = dev(a, dt), dev(w, dt)
        outs = []
        for stream in (ctx.stream0, ctx.stream1, ctx.stream0):      # each stream has a workspace of its own
            c = iso.DeviceArray((M, N), dt, fill_byte=NAN_BYTE)
            ctx.gemm_rowpar(ad, wd, c, M, N, K, stream)
            outs.append(c)
        ctx.sync()
        assert orc.max_rel_err(f64(outs[0]), ref) <= TOL_STEP[dt]
        for c in outs[1:]:                                          # the shares are added in a fixed order
            np.testing.assert_array_equal(c.numpy(), outs[0].numpy())


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K,shares", [(1, 8, 128, 1), (65, 136, 1408, 3), (257, 264, 512, 2)])
def test_split_gemm_fp8(tile, M, N, K, shares):
    dt = "bf16"
    with make_ctx(256, 4, 4, 64, 64, dt, 256) as ctx:
        q = []
        for rows, seed in ((M, 1), (N, 2)):
            x = iso_inputs.randn((rows, K), seed=seed + K, dtype=dt)
            codes, scale = iso.DeviceArray((rows, K), "u8"), iso.DeviceArray((rows,), "f32")
            ctx.quantize_rows_fp8(dev(x, dt), rows, K, codes, scale, ctx.stream0)
            q.append((codes, scale, x))
        ctx.set_flags(forced(tile, shares))
        c = iso.DeviceArray((M, N), dt, fill_byte=NAN_BYTE)
        ctx.gemm_fp8(q[0][0], q[0][1], q[1][0], q[1][1], c, M, N, K, ctx.stream0)
        ctx.set_flags(iso.ISO_FLAG_NO_STREAMK)                      # the whole-tile kernel, itself checked in test_gpu_fp8
        whole = iso.DeviceArray((M, N), dt, fill_byte=NAN_BYTE)
        ctx.gemm_fp8(q[0][0], q[0][1], q[1][0], q[1][1], whole, M, N, K, ctx.stream0)
        ctx.sync()
        # exact products, fp32 sums in another order, one bf16 rounding each: at most one unit in the last place (2^-7)
        assert orc.max_rel_err(f64(c), f64(whole)) <= 2.0 ** -7


@pytest.mark.parametrize("tile,shares", [(0, 1), (1, 3), (2, 1), (3, 2), (4, 2)])
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,T,split", [(512, 4, 1, 128, 776, 300, 130), (512, 8, 2, 64, 640, 97, 0)])
def test_layer_through_split_products(tile, shares, hidden, nq, nkv, d, ffn, T, split):
    """SwiGLU and the rotary step + cache write in the epilogue or the second kernel, for both head sizes, ragged rows and
    MLP columns, against the oracle; V rows equal those of the separate kernels bit for bit."""
    dt = "bf16"
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=31, dtype=dt)
    x = iso_inputs.make_hidden(T, hidden, seed=31, dtype=dt)
    ref = orc.layer_unsplit(h64(x, dt), oracle_weights(w, dt), shape_of(hidden, nq, nkv, d, ffn))
    w_dev = iso.upload_weights(w, dt)
    max_seq = T + 5                                                 # rows past the prompt must stay untouched
    with make_ctx(hidden, nq, nkv, d, ffn, dt, max_seq) as ctx:
        v_rows = []
        for flags in (forced(tile, shares), forced(tile, shares) | iso.ISO_FLAG_NO_FUSE):
            ctx.set_flags(flags)
            out, kc, vc = run_layer(ctx, w_dev, x, dt, T, split, nkv, d, max_seq, iso.ISO_COMM_D2H, poison=True)
            assert orc.max_rel_err(f64(out), ref["x_out"]) <= TOL_LAYER[dt]
            assert orc.max_rel_err(f64(kc)[:T], ref["k_cache"]) <= TOL_LAYER[dt]
            assert np.isnan(f64(kc)[T:]).all() and np.isnan(f64(vc)[T:]).all()
            v_rows.append(vc.numpy()[:T])
        np.testing.assert_array_equal(v_rows[0], v_rows[1])


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("flags", [forced(0, 1), forced(1, 3), forced(2, 1), forced(2, 2), forced(3, 2), forced(4, 2), forced(5, 3),
                                   forced(6, 2), 1 << 8, 4 << 8, 5 << 8])          # the last three: whole 256-column tiles
@pytest.mark.parametrize("T,split,n_layers", [(97, 0, 1), (300, 130, 2)])
def test_residual_in_the_last_down_projection(flags, fp8, T, split, n_layers):
    """With nothing to send the last layer's down projection adds the residual itself: same arithmetic in the same order as the
    kernel that adds it where the partials are sent, so the hidden states are the same bits."""
    hidden, nq, nkv, d, ffn, dt = 640, 4, 1, 128, 768, "bf16"        # 640: two column tiles and a half
    x = iso_inputs.make_hidden(T, hidden, seed=71, dtype=dt)
    with make_ctx(hidden, nq, nkv, d, ffn, dt, T) as ctx:
        layers = [iso.upload_weights(iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=71 + l, dtype=dt), dt) for l in range(n_layers)]
        if fp8:
            layers = [ctx.add_fp8_weights(w) for w in layers]
        ctx.set_flags(flags | iso.ISO_FLAG_KEEP_CUT | (iso.ISO_FLAG_FP8_GEMM if fp8 else 0))
        got = []
        for comm, launches in ((iso.ISO_COMM_NONE, 0), (iso.ISO_COMM_D2H, 2 if split else 1)):
            xd = dev(x, dt)
            kc, vc = (iso.DeviceArray((n_layers, T, nkv, d), dt, fill_byte=NAN_BYTE) for _ in range(2))
            ctx.timing_enable(True)
            ctx.stack_prefill(layers, xd, kc, vc, T, split, comm)
            ctx.sync()
            assert ctx.timing_read()["residual"][1] == launches
            ctx.timing_enable(False)
            got.append(xd.numpy())
        np.testing.assert_array_equal(got[0], got[1])
