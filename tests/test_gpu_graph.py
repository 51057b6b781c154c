"""Entry points recorded into a HIP graph and replayed: every replay must give what the eager call gives.

The graph calls go straight to the HIP runtime that libiso is linked against (the C ABI has no graph functions: a
caller that captures brings its own).  Between replays the test does eager work and synchronises, as a program would.
"""
import ctypes

import numpy as np
import pytest

import paper_2409_11155_amd as iso      # first: binds libiso to the HIP runtime it was built against
import iso_inputs
from oracle import iso_oracle as orc

pytestmark = pytest.mark.gpu

CAPTURE_RELAXED = 2      # hipStreamCaptureModeRelaxed


def hip_runtime():
    """The HIP runtime object already mapped into this process (the one libiso uses)."""
    iso.load()
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert len(paths) == 1, paths
    rt = ctypes.CDLL(paths.pop())
    rt.hipStreamBeginCapture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    rt.hipStreamEndCapture.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    rt.hipGraphInstantiate.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_void_p, ctypes.c_void_p, ctypes.c_char_p,
                                       ctypes.c_size_t]
    rt.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    rt.hipGraphLaunch.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    rt.hipGraphExecDestroy.argtypes = [ctypes.c_void_p]
    rt.hipGraphDestroy.argtypes = [ctypes.c_void_p]
    return rt


class Captured:
    """Records what `enqueue()` puts on `stream` (and on the streams it forks to) into an executable graph."""

    def __init__(self, rt, stream, enqueue, mode=CAPTURE_RELAXED):
        self.rt, self.stream = rt, stream
        assert rt.hipStreamBeginCapture(stream, mode) == 0
        try:
            enqueue()
        finally:
            graph = ctypes.c_void_p()
            rc = rt.hipStreamEndCapture(stream, ctypes.byref(graph))
        assert rc == 0 and graph.value, rc
        self.graph = graph
        self.exe = ctypes.c_void_p()
        assert rt.hipGraphInstantiate(ctypes.byref(self.exe), graph, None, None, 0) == 0

    def nodes(self):
        n = ctypes.c_size_t()
        assert self.rt.hipGraphGetNodes(self.graph, None, ctypes.byref(n)) == 0
        return n.value

    def launch(self, stream=None):
        assert self.rt.hipGraphLaunch(self.exe, self.stream if stream is None else stream) == 0

    def destroy(self):
        self.rt.hipGraphExecDestroy(self.exe)
        self.rt.hipGraphDestroy(self.graph)


def dev(a, dt):
    return iso.DeviceArray.from_numpy(a, dt)


def test_captured_gemm_of_stream_k_size_replays_correctly():
    """512 x 5120 x 8192 is a shape the whole-tile rule gives to the stream-K kernel (20 k-slices per team on 256
    compute units), whose launches are numbered; the eager launches here are forced to it.  Recorded into a graph the
    product must take a launch that can be replayed: three replays, the output cleared and the same stream-K workspace
    used by eager launches in between."""
    dt, (M, N, K) = "bf16", (512, 5120, 8192)
    assert iso.gemm_launch_plan(M, N, K, 256)[0] == 6
    a = iso_inputs.randn((M, K), seed=5, dtype=dt)
    w = iso_inputs.randn((N, K), seed=6, dtype=dt, scale=K ** -0.5)
    ref = orc.linear(iso_inputs.to_f64(a, dt), iso_inputs.to_f64(w, dt))
    rt = hip_runtime()
    cfg = iso.make_cfg(256, 4, 4, 64, 64, dt, 256)
    with iso.Context(cfg) as ctx:
        s0 = ctx.stream0.handle
        ad, wd = dev(a, dt), dev(w, dt)
        other = dev(iso_inputs.randn((M, K), seed=7, dtype=dt), dt)      # a different product for the same workspace
        eager = iso.DeviceArray((M, N), dt, fill_byte=0)
        ctx.set_flags(6 << 8)
        ctx.gemm_rowpar(ad, wd, eager, M, N, K, ctx.stream0)
        ctx.sync()
        ctx.set_flags(0)                                               # recording: the rule's choice for a stream that records
        assert orc.max_rel_err(iso_inputs.to_f64(eager.numpy(), dt), ref) <= 1e-2
        out = iso.DeviceArray((M, N), dt, fill_byte=0xFF)
        g = Captured(rt, s0, lambda: ctx.gemm_rowpar(ad, wd, out, M, N, K, ctx.stream0))
        ctx.sync()
        ctx.set_flags(6 << 8)
        first = None
        for rep in range(3):
            out.fill(0xFF)                                             # NaN pattern: a replay must write every element
            ctx.gemm_rowpar(other, wd, eager, M, N, K, ctx.stream0)    # eager stream-K launch between the replays:
                                                                       # other partial tiles, a newer launch number
            g.launch()
            ctx.sync()
            got = out.numpy().copy()
            assert orc.max_rel_err(iso_inputs.to_f64(got, dt), ref) <= 1e-2, rep
            if first is None:
                first = got
            np.testing.assert_array_equal(got, first)
        g.destroy()


@pytest.mark.parametrize("mode", [0, 1, CAPTURE_RELAXED])              # global, per thread, relaxed
def test_captured_iso_layer_replays_bit_identically_to_the_eager_step(mode):
    """A two-chunk ISO step with both transfers (fork to the second stream, K/V event, two copies per chunk, join)
    recorded from stream0 and replayed three times on fresh inputs and NaN-filled caches."""
    dt, d = "bf16", 128
    hidden, nq, nkv, ffn, T, split = 512, 4, 1, 768, 300, 130
    w = iso_inputs.make_layer(hidden, nq, nkv, d, ffn, seed=21, dtype=dt)
    x = iso_inputs.make_hidden(T, hidden, seed=21, dtype=dt)
    sh = orc.LayerShape(hidden, nq, nkv, d, ffn, 1e-6, 10000.0)
    ref = orc.layer_unsplit(iso_inputs.to_f64(x, dt), {k: iso_inputs.to_f64(v, dt) for k, v in w.items()}, sh)["x_out"]
    rt = hip_runtime()
    cfg = iso.make_cfg(hidden, nq, nkv, d, ffn, dt, 320)
    with iso.Context(cfg) as ctx:
        ctx.set_flags(iso.ISO_FLAG_KEEP_CUT)                           # 300 tokens would be one chunk otherwise
        w_dev = iso.upload_weights(w, dt)
        xd = dev(x, dt)
        kc = iso.DeviceArray((320, nkv, d), dt, fill_byte=0xFF)
        vc = iso.DeviceArray((320, nkv, d), dt, fill_byte=0xFF)
        ctx.layer_prefill(w_dev, xd, kc, vc, T, split, iso.ISO_COMM_D2H, iso.ISO_SCHED_OVERLAP)   # eager: also the warm-up
        ctx.sync()
        eager = xd.numpy().copy()
        assert orc.max_rel_err(iso_inputs.to_f64(eager, dt), ref) <= 2e-2
        g = Captured(rt, ctx.stream0.handle,
                     lambda: ctx.layer_prefill(w_dev, xd, kc, vc, T, split, iso.ISO_COMM_D2H, iso.ISO_SCHED_OVERLAP), mode)
        ctx.sync()
        assert g.nodes() >= 2 * 9                                      # two chunks of seven kernels and two copies at least
        for rep in range(3):
            xd.upload(x)
            kc.fill(0xFF)
            vc.fill(0xFF)
            g.launch()
            ctx.sync()
            np.testing.assert_array_equal(xd.numpy(), eager)
        g.destroy()


@pytest.mark.parametrize("flags", [0, (7 << 8) | (6 << 17) | (4 << 21), 6 << 8])
@pytest.mark.parametrize("fp8", [False, True])
def test_captured_products_hold_no_partial_sums_of_the_context(fp8, flags):
    """Recorded on stream 0 and replayed on another stream beside eager products on stream 0 (by the launch rule, in six shares
    of the k range, by stream-K): one kernel, the caller's buffers only, so every replay and every eager product is right."""
    dt, (M, N, K) = "bf16", (512, 5120, 8192)
    a, b = (iso_inputs.randn((M, K), seed=s, dtype=dt) for s in (81, 82))
    w = iso_inputs.randn((N, K), seed=83, dtype=dt, scale=K ** -0.5)
    linear = orc.linear_fp8 if fp8 else orc.linear
    ref_a, ref_b = (linear(iso_inputs.to_f64(x, dt), iso_inputs.to_f64(w, dt)) for x in (a, b))
    rt = hip_runtime()
    with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, dt, 256)) as ctx:
        other = iso.Stream()

        def operands(x):
            if not fp8:
                return [dev(x, dt), dev(w, dt)]
            out = []
            for m in (x, w):
                q, s = iso.DeviceArray(m.shape, "u8"), iso.DeviceArray((m.shape[0],), "f32")
                ctx.quantize_rows_fp8(dev(m, dt), m.shape[0], K, q, s, ctx.stream0)
                out += [q, s]
            return out

        op_a, op_b = operands(a), operands(b)
        product = lambda op, c: (ctx.gemm_fp8 if fp8 else ctx.gemm_rowpar)(*op, c, M, N, K, ctx.stream0)
        c, eager = iso.DeviceArray((M, N), dt, fill_byte=0xFF), iso.DeviceArray((M, N), dt, fill_byte=0xFF)
        ctx.set_flags(flags)
        product(op_b, eager)
        ctx.set_flags(flags if flags >> 8 != 6 else 0)          # a forced stream-K launch cannot be recorded
        g = Captured(rt, ctx.stream0.handle, lambda: product(op_a, c))
        ctx.set_flags(flags)
        ctx.sync()
        assert g.nodes() == 1
        for rep in range(3):
            c.fill(0xFF)
            eager.fill(0xFF)
            for _ in range(4):
                product(op_b, eager)
                g.launch(other.handle)
            iso.device_sync()
            assert orc.max_rel_err(iso_inputs.to_f64(c.numpy(), dt), ref_a) <= 1e-2, rep
            assert orc.max_rel_err(iso_inputs.to_f64(eager.numpy(), dt), ref_b) <= 1e-2, rep
        g.destroy()


def test_captured_attention_with_heads_of_64_beside_eager_attention():
    """Few rows over a long cache, where an eager launch deals the keys to many workgroups: the recorded launch does not."""
    dt, d, nq, nkv, Tc, q_offset = "bf16", 64, 4, 2, 33, 4095
    kv = q_offset + Tc
    k, v = (iso_inputs.randn((kv, nkv, d), seed=s, dtype=dt) for s in (91, 92))
    qs = [iso_inputs.randn((Tc, nq, d), seed=s, dtype=dt) for s in (93, 94)]
    refs = [orc.attention_chunk(*(iso_inputs.to_f64(t, dt) for t in (q, k, v)), q_offset, kv).reshape(Tc, nq * d) for q in qs]
    rt = hip_runtime()
    with iso.Context(iso.make_cfg(256, nq, nkv, d, 64, dt, kv)) as ctx:
        other = iso.Stream()
        kd, vd, qd = dev(k, dt), dev(v, dt), [dev(q, dt) for q in qs]
        outs = [iso.DeviceArray((Tc, nq * d), dt, fill_byte=0xFF) for _ in qs]
        attend = lambda i: ctx.attn_chunk(qd[i], kd, vd, outs[i], Tc, q_offset, kv, ctx.stream0)
        attend(1)
        g = Captured(rt, ctx.stream0.handle, lambda: attend(0))
        ctx.sync()
        for rep in range(3):
            for o in outs:
                o.fill(0xFF)
            for _ in range(8):
                attend(1)
                g.launch(other.handle)
            iso.device_sync()
            for o, ref in zip(outs, refs):
                assert orc.max_rel_err(iso_inputs.to_f64(o.numpy(), dt), ref) <= 1e-2, rep
        g.destroy()
