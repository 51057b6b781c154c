"""The 192 x 256 projection tile (eight waves of 96 x 64), whole and with its k range in shares, at the edges of the tile.

Bounds: a single product rounds once to bf16 (2^-8 relative) and its fp32 sums add K * 2^-24 at most; 1e-2 is the bound of
the other projection tests.  FP8: exact products, fp32 sums in another order, so at most one bf16 unit in the last place.
"""
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import NAN_BYTE, TOL_LAYER, TOL_STEP, dev, f64, h64, make_ctx, oracle_weights, run_layer, shape_of

pytestmark = pytest.mark.gpu

WHOLE = 5 << 8
SIZES = [(1, 8, 128), (191, 256, 128), (192, 264, 256), (193, 520, 704), (385, 248, 1408)]


def shares(n):
    return (7 << 8) | (n << 17) | (5 << 21)


@pytest.mark.parametrize("flags", [WHOLE, shares(2), shares(4)])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_gemm(flags, M, N, K):
    a = iso_inputs.randn((M, K), seed=M + N, dtype="bf16")
    w = iso_inputs.randn((N, K), seed=M + K, dtype="bf16", scale=K ** -0.5)
    with make_ctx(256, 4, 4, 64, 64, "bf16", 512) as ctx:
        ctx.set_flags(flags)
        c = iso.DeviceArray((M, N), "bf16", fill_byte=NAN_BYTE)
        ctx.gemm_rowpar(dev(a, "bf16"), dev(w, "bf16"), c, M, N, K, ctx.stream0)
        ctx.sync()
        assert orc.max_rel_err(f64(c), orc.linear(h64(a, "bf16"), h64(w, "bf16"))) <= TOL_STEP["bf16"]


@pytest.mark.parametrize("flags", [WHOLE, shares(2)])
@pytest.mark.parametrize("M,N,K", [s for s in SIZES if s[2] % 128 == 0])
def test_gemm_fp8(flags, M, N, K):
    with make_ctx(256, 4, 4, 64, 64, "bf16", 512) as ctx:
        q = []
        for rows, seed in ((M, 1), (N, 2)):
            codes, scale = iso.DeviceArray((rows, K), "u8"), iso.DeviceArray((rows,), "f32")
            x = dev(iso_inputs.randn((rows, K), seed=seed + K, dtype="bf16"), "bf16")
            ctx.quantize_rows_fp8(x, rows, K, codes, scale, ctx.stream0)
            q += [codes, scale]
        outs = []
        for f in (flags, 3 << 8):
            ctx.set_flags(f)
            outs.append(iso.DeviceArray((M, N), "bf16", fill_byte=NAN_BYTE))
            ctx.gemm_fp8(q[0], q[1], q[2], q[3], outs[-1], M, N, K, ctx.stream0)
        ctx.sync()
        assert orc.max_rel_err(f64(outs[0]), f64(outs[1])) <= 2.0 ** -7


@pytest.mark.parametrize("flags", [WHOLE, shares(2), shares(2) | iso.ISO_FLAG_NO_FUSE])
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn,T,split", [(512, 4, 1, 128, 776, 400, 193), (512, 8, 2, 64, 640, 191, 0)])
def test_layer(flags, hidden, nq, nkv, d, ffn, T, split):
    """SwiGLU in the epilogue and in the second kernel, rotary step behind or beside it, ragged rows and MLP columns."""
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=37, dtype="bf16")
    x = iso_inputs.make_hidden(T, hidden, seed=37, dtype="bf16")
    ref = orc.layer_unsplit(h64(x, "bf16"), oracle_weights(w, "bf16"), shape_of(hidden, nq, nkv, d, ffn))
    with make_ctx(hidden, nq, nkv, d, ffn, "bf16", T) as ctx:
        ctx.set_flags(flags)
        out, kc, vc = run_layer(ctx, iso.upload_weights(w, "bf16"), x, "bf16", T, split, nkv, d, T, iso.ISO_COMM_D2H, poison=True)
        assert orc.max_rel_err(f64(out), ref["x_out"]) <= TOL_LAYER["bf16"]
        assert orc.max_rel_err(f64(kc), ref["k_cache"]) <= TOL_LAYER["bf16"]
