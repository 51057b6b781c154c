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
