"""Few rows over a long cache: more than four key shares (chosen from the sizes), against one share.

Bound: both are bf16 results of the same fp32 sums in another order, each within TOL_STEP of the exact one.
"""
import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc
from test_gpu_parity import NAN_BYTE, TOL_STEP, dev, f64, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Tc,q_offset,nq,nkv,d", [
    (1, 16383, 2, 1, 128), (40, 6001, 2, 2, 128), (130, 9000, 8, 1, 128), (33, 4095, 4, 2, 64), (200, 8000, 2, 1, 64)])
def test_many_key_shares(Tc, q_offset, nq, nkv, d):
    kv = q_offset + Tc
    q = iso_inputs.randn((Tc, nq, d), seed=51, dtype="bf16")
    k, v = (iso_inputs.randn((kv, nkv, d), seed=s, dtype="bf16") for s in (52, 53))
    with make_ctx(256, nq, nkv, d, 64, "bf16", kv) as ctx:
        qd, kd, vd = dev(q, "bf16"), dev(k, "bf16"), dev(v, "bf16")
        got = []
        for flags in (0, 0, 1 << 14):                    # chosen, chosen again (counters are back at zero), one share
            ctx.set_flags(flags)
            out = iso.DeviceArray((Tc, nq * d), "bf16", fill_byte=NAN_BYTE)
            ctx.attn_chunk(qd, kd, vd, out, Tc, q_offset, kv, ctx.stream0)
            ctx.sync()
            got.append(out)
        np.testing.assert_array_equal(got[0].numpy(), got[1].numpy())
        assert orc.max_rel_err(f64(got[0]), f64(got[2])) <= 2 * TOL_STEP["bf16"]
