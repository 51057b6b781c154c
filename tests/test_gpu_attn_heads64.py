"""Matrix-core attention with heads of 64 against the CPU oracle, in every launch shape, at the edges of row blocks and key
tiles.

The probabilities enter the second product as two bf16 terms (16 mantissa bits): |d out| <= 2^-17 max|v| from them, next to
the 2^-8 rounding of the bf16 output and 2^-9 from the half unit by which a value near it may fall on the other side.
"""
import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import ATTN_CASES, NAN_BYTE, dev, f64, h64, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, 1 << 12, 2 << 12, 3 << 12, (1 << 12) | (3 << 14), (2 << 12) | (2 << 14),
                                   (3 << 12) | (4 << 14)])
@pytest.mark.parametrize("Tc,q_offset,kv_len,nq,nkv", ATTN_CASES + [(777, 0, 777, 8, 2), (129, 1023, 1152, 4, 4)])
def test_attn_chunk_heads_of_64(flags, Tc, q_offset, kv_len, nq, nkv):
    dt, d = "bf16", 64
    q, k, v = iso_inputs.make_qkv_cache(Tc, kv_len, nq, nkv, d, seed=Tc + q_offset, dtype=dt)
    ref = orc.attention_chunk(h64(q, dt), h64(k, dt), h64(v, dt), q_offset, kv_len).reshape(Tc, nq * d)
    rms = float(np.sqrt(np.mean(ref * ref)))
    tol = 2.0 ** -8 + 2.0 ** -9 + 2.0 ** -17 * float(np.abs(h64(v, dt)).max()) / rms
    with make_ctx(256, nq, nkv, d, 64, dt, 1152) as ctx:
        ctx.set_flags(flags)
        qd, kd, vd = dev(q, dt), dev(k, dt), dev(v, dt)
        outs = [iso.DeviceArray((Tc, nq * d), dt, fill_byte=NAN_BYTE) for _ in range(2)]
        for out in outs:
            ctx.attn_chunk(qd, kd, vd, out, Tc, q_offset, kv_len, ctx.stream0)
        ctx.sync()
        err = orc.max_rel_err(f64(outs[0]), ref)
        assert err <= tol, (err, tol)
        np.testing.assert_array_equal(outs[0].numpy(), outs[1].numpy())
