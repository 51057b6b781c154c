"""Attention of few rows: the keys of a 32-row block dealt to eight waves, at the edges of its tiles and rounds of tiles.

Bounds as in the attention parity tests: the probabilities (heads of 64: two bf16 terms) and the output round to bf16.
"""
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
import test_gpu_attn_invisible as invisible
from oracle import iso_oracle as orc
from test_gpu_parity import dev, f64, h64, make_ctx

pytestmark = pytest.mark.gpu

WAVE = 7 << 14


# less than a wave's first tile, one key either side of a tile and of a round of eight tiles, ragged last row blocks, a cache that
# ends before the causal reach, one row, heads that do not divide over the eight L2s
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Tc,q_offset,kv_len,nq,nkv", [
    (1, 0, 1, 3, 3), (31, 0, 31, 2, 1), (33, 0, 33, 4, 2), (64, 191, 255, 5, 5), (32, 224, 256, 4, 1), (65, 192, 257, 2, 2),
    (100, 500, 555, 8, 2), (257, 13, 270, 13, 13), (40, 1500, 1540, 3, 1)])
def test_against_the_oracle(d, Tc, q_offset, kv_len, nq, nkv):
    q, k, v = iso_inputs.make_qkv_cache(Tc, kv_len, nq, nkv, d, seed=Tc + q_offset, dtype="bf16")
    ref = orc.attention_chunk(h64(q, "bf16"), h64(k, "bf16"), h64(v, "bf16"), q_offset, kv_len).reshape(Tc, nq * d)
    with make_ctx(256, nq, nkv, d, 64, "bf16", kv_len) as ctx:
        ctx.set_flags(WAVE)
        err = orc.max_rel_err(invisible.attend(ctx, q, k, v, "bf16", nq, d, Tc, q_offset, kv_len), ref)
    tol = invisible.bound("bf16", h64(v, "bf16"), ref)
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("d", [64, 128])
def test_query_rows_inside_a_wider_row(d):
    """The layer hands in the q columns of the fused projection: as the whole layer, with and without the kernel."""
    hidden, nq, nkv, ffn, T = 256, 4, 1, 256, 300
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=61, dtype="bf16")
    x = iso_inputs.make_hidden(T, hidden, seed=61, dtype="bf16")
    with make_ctx(hidden, nq, nkv, d, ffn, "bf16", T) as ctx:
        wd, got = iso.upload_weights(w, "bf16"), []
        for flags in (WAVE, 1 << 14):
            ctx.set_flags(flags | iso.ISO_FLAG_KEEP_CUT)
            xd = dev(x, "bf16")
            kc, vc = (iso.DeviceArray((T, nkv, d), "bf16") for _ in range(2))
            ctx.layer_prefill(wd, xd, kc, vc, T, 130, iso.ISO_COMM_NONE)
            ctx.sync()
            got.append(f64(xd))
        assert orc.max_rel_err(got[0], got[1]) <= 2e-2


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Tc,q_offset,kv_len", [(32, 0, 64), (1, 0, 300), (130, 77, 260), (64, 64, 192)])
def test_rows_behind_the_last_visible_one(d, Tc, q_offset, kv_len):
    invisible.test_cache_rows_behind_the_last_visible_one_may_hold_anything("bf16", d, WAVE, Tc, q_offset, kv_len)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Tc,q_offset,bad", [(40, 0, 17), (200, 77, 150), (130, 500, 628), (70, 2000, 2001)])
def test_a_later_tokens_non_finite_value(d, Tc, q_offset, bad):
    invisible.test_a_later_tokens_non_finite_value_stays_out_of_the_earlier_rows("bf16", d, WAVE, Tc, q_offset, bad)


@pytest.mark.parametrize("dt,d,flags", [("bf16", 64, WAVE), ("bf16", 128, WAVE), ("bf16", 128, 1 << 14), ("bf16", 128, 3 << 12),
                                        ("f32", 64, 0), ("f32", 128, 0)])
def test_a_chunk_that_begins_far_behind_the_cache(dt, d, flags):
    """Every row sees the whole cache: the same bits as from the offset where that begins."""
    Tc, kv, nq = 70, 90, 4
    q, k, v = iso_inputs.make_qkv_cache(Tc, kv, nq, 2, d, seed=5, dtype=dt)
    with make_ctx(256, nq, 2, d, 64, dt, kv) as ctx:
        ctx.set_flags(flags)
        near, far = (invisible.attend(ctx, q, k, v, dt, nq, d, Tc, off, kv) for off in (kv - 1, 2 ** 31 - 1))
    assert (near == far).all()


@pytest.mark.parametrize("d", [64, 128])
def test_scores_far_below_zero(d):
    invisible.test_scores_far_below_zero("bf16", d, WAVE)
