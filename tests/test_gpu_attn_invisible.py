"""Key j is visible to query row i iff j <= q_offset + i and j < kv_len: nothing that a cache holds in a row that a query does
not see may reach that query's output, whatever it is.

Bounds: those of the attention parity tests (bf16: the probabilities and the output round to bf16; heads of 64 and fp32 keep
more bits of the probabilities).
"""
import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import NAN_BYTE, TOL_STEP, dev, f64, h64, make_ctx

pytestmark = pytest.mark.gpu

# bits 12..13: launch shape, 14..16: key shares of the direct-to-LDS kernel
KERNELS = [("bf16", 64, f) for f in (0, 1 << 12, 2 << 12, 3 << 12, (1 << 12) | (3 << 14))] + \
          [("bf16", 128, f) for f in (0, 1 << 12, 2 << 12, 3 << 12, (1 << 12) | (3 << 14))] + [("f32", 64, 0), ("f32", 128, 0)]


def bound(dt, v, ref):
    rms = float(np.sqrt(np.mean(ref * ref)))
    return TOL_STEP["f32"] if dt == "f32" else 2.0 ** -9 * float(np.abs(v).max()) / rms + 2.0 ** -8 + 1e-4


def attend(ctx, q, k, v, dt, nq, d, Tc, q_offset, kv_len):
    out = iso.DeviceArray((Tc, nq * d), dt, fill_byte=NAN_BYTE)
    ctx.attn_chunk(dev(q, dt), dev(k, dt), dev(v, dt), out, Tc, q_offset, kv_len, ctx.stream0)
    ctx.sync()
    return f64(out)


@pytest.mark.parametrize("dt,d,flags", KERNELS)
@pytest.mark.parametrize("Tc,q_offset,kv_len", [(32, 0, 64), (1, 0, 300), (130, 77, 260), (200, 130, 331), (64, 64, 192)])
def test_cache_rows_behind_the_last_visible_one_may_hold_anything(dt, d, flags, Tc, q_offset, kv_len):
    """kv_len > q_offset + Tc over a cache whose later rows were never written (NaN bits)."""
    nq, nkv, seen = 4, 2, q_offset + Tc
    q, k, v = iso_inputs.make_qkv_cache(Tc, kv_len, nq, nkv, d, seed=Tc + q_offset, dtype=dt)
    ref = orc.attention_chunk(h64(q, dt), h64(k, dt), h64(v, dt), q_offset, kv_len).reshape(Tc, nq * d)
    tol = bound(dt, h64(v, dt)[:seen], ref)
    for a in (k, v):
        a[seen:] = np.nan if dt == "f32" else 0xFFFF
    with make_ctx(256, nq, nkv, d, 64, dt, kv_len) as ctx:
        ctx.set_flags(flags)
        err = orc.max_rel_err(attend(ctx, q, k, v, dt, nq, d, Tc, q_offset, kv_len), ref)
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("dt,d,flags", KERNELS)
@pytest.mark.parametrize("Tc,q_offset,bad", [(40, 0, 17), (200, 77, 150), (130, 500, 628), (70, 2000, 2001)])
def test_a_later_tokens_non_finite_value_stays_out_of_the_earlier_rows(dt, d, flags, Tc, q_offset, bad):
    """Key `bad` holds an infinity, a NaN and a finite value per head in V: rows that see it become inf / NaN in those two
    dims and stay right in the others, rows before it stay right everywhere."""
    nq, nkv, kv_len = 4, 2, q_offset + Tc
    q, k, v = iso_inputs.make_qkv_cache(Tc, kv_len, nq, nkv, d, seed=Tc + q_offset, dtype=dt)
    ref = orc.attention_chunk(h64(q, dt), h64(k, dt), h64(v, dt), q_offset, kv_len).reshape(Tc, nq, d)
    tol = bound(dt, h64(v, dt), ref)
    v[bad, :, 3] = np.inf if dt == "f32" else 0x7F80
    v[bad, :, d - 1] = np.nan if dt == "f32" else 0xFFFF
    with make_ctx(256, nq, nkv, d, 64, dt, kv_len) as ctx:
        ctx.set_flags(flags)
        got = attend(ctx, q, k, v, dt, nq, d, Tc, q_offset, kv_len).reshape(Tc, nq, d)
    sees = bad - q_offset
    assert np.isposinf(got[sees:, :, 3]).all() and np.isnan(got[sees:, :, d - 1]).all()
    got[sees:, :, 3], got[sees:, :, d - 1] = ref[sees:, :, 3], ref[sees:, :, d - 1]
    err = orc.max_rel_err(got, ref)
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("dt,d,flags", KERNELS)
def test_scores_far_below_zero(dt, d, flags):
    """Every raw score of a row is -1.6e31 * d: softmax over equal scores, so each row is the mean of the V rows it sees."""
    nq, nkv, Tc, q_offset = 4, 2, 100, 300
    kv_len = q_offset + Tc
    q, k, v = iso_inputs.make_qkv_cache(Tc, kv_len, nq, nkv, d, seed=5, dtype=dt)
    big = lambda shape, x: iso_inputs.store(np.full(shape, x, dtype=np.float32), dt)
    q, k = big(q.shape, 2.0 ** 52), big(k.shape, -(2.0 ** 52))
    v64 = h64(v, dt)
    ref = (np.cumsum(v64, axis=0) / np.arange(1, kv_len + 1)[:, None, None])[q_offset:].repeat(nq // nkv, axis=1)
    tol = bound(dt, v64, ref)
    with make_ctx(256, nq, nkv, d, 64, dt, kv_len) as ctx:
        ctx.set_flags(flags)
        err = orc.max_rel_err(attend(ctx, q, k, v, dt, nq, d, Tc, q_offset, kv_len), ref.reshape(Tc, nq * d))
    assert err <= tol, (err, tol)
