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
