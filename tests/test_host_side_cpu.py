"""The host side of libiso without a GPU: the library's HIP calls go to tests/fake_hip.cpp, which records them.  Each case runs in a
process of its own (the stand-in has to be there before the library is loaded)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WORKSPACE = 4096 + 256 * 256 * 1024          # stream-K / split-product workspace of a stream on 256 compute units

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_refuse.argtypes = [ctypes.c_size_t]
import paper_2409_11155_amd as iso
def log():
    lines = [l.split(" ", 2) for l in fake.fake_log().decode().splitlines()]
    fake.fake_clear()
    return lines
def array(*shape, dt="bf16"):
    return iso.DeviceArray(shape, dt)
def layer(hidden, nq, nkv, d, ffn, dt="bf16"):
    return {"w_qkv": array((nq + 2 * nkv) * d, hidden, dt=dt), "w_o": array(hidden, nq * d, dt=dt),
            "w_gate_up": array(2 * ffn, hidden, dt=dt), "w_down": array(hidden, ffn, dt=dt), "g_attn": array(hidden, dt=dt),
            "g_mlp": array(hidden, dt=dt)}
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    path = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-o", path,
                    os.path.join(ROOT, "tests", "fake_hip.cpp")], check=True)
    return path


def run(fake, code):
    p = subprocess.run([sys.executable, "-c", PRELUDE + code, fake], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr


def test_a_refused_workspace_of_an_extra_chunk_stream_costs_the_split_products_only(fake):
    """The 64 MiB for partial sums are optional: without them the chunks of that stream run unsplit launches, the call succeeds,
    no error is left behind for the next launch to report, and nothing is launched before the attention counters, cleared by a
    memset on the null stream, are known to be zero."""
    run(fake, f"""
T, hidden, nq, nkv, d, ffn = 400, 512, 4, 1, 128, 768
w = layer(hidden, nq, nkv, d, ffn)
for refuse in (0, {WORKSPACE}):
    with iso.Context(iso.make_cfg(hidden, nq, nkv, d, ffn, "bf16", T)) as ctx:
        ctx.set_flags(iso.ISO_FLAG_KEEP_CUT)
        x, k, v = array(T, hidden), array(1, T, nkv, d), array(1, T, nkv, d)
        fake.fake_refuse(refuse)
        log()
        for call in range(2):
            ctx.stack_prefill_chunks([w], x, k, v, T, [100, 200, 300], iso.ISO_COMM_D2H, iso.ISO_SCHED_STREAM_PER_CHUNK)
            lines = log()
            kinds = [l[0] for l in lines]
            assert kinds.count("refused") == (2 if refuse and call == 0 else 0), kinds
            assert kinds.count("kernel") > 30
            if call == 0:
                zeroed = max(i for i, n in enumerate(kinds) if n == "memset")
                assert "device_sync" in kinds[zeroed:kinds.index("kernel")], kinds
            split = {{l[1] for l in lines if l[0] == "kernel" and "share_sum" in l[2]}}
            assert len(split) == (2 if refuse else 4), split         # streams with split products
        fake.fake_refuse(0)
""")


def test_the_two_kernels_of_a_split_product_stay_together_under_two_threads(fake):
    """Launches take 2 ms here, so that two threads on one stream meet between a kernel that leaves partial sums and the one
    that adds them if nothing keeps them apart."""
    run(fake, """
import threading
with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, "bf16", 256)) as ctx:
    ctx.set_flags((7 << 8) | (3 << 17))
    a, w, c = array(64, 1024), array(64, 1024), array(64, 64)
    log()
    fake.fake_launch_us(2000)
    start = threading.Barrier(2)
    def enqueue():
        start.wait()
        for _ in range(10):
            ctx.gemm_rowpar(a, w, c, 64, 64, 1024, ctx.stream0)
    threads = [threading.Thread(target=enqueue) for _ in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    order = ["sum" if "share_sum" in l[2] else "partial" for l in log() if l[0] == "kernel"]
    assert order == ["partial", "sum"] * 20, order
""")


def test_the_copy_behind_a_row_parallel_product_leaves_the_compute_units_alone(fake):
    """The caller may run anything beside it: more than 1 MB goes by the copy engine, as between two chunks of a layer."""
    run(fake, """
with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, "bf16", 256)) as ctx:
    for M, how in ((32, "kernel"), (64, "kernel"), (65, "copy2d"), (128, "copy2d"), (384, "copy2d"), (512, "copy2d")):
        a, w, c, sink = array(M, 64), array(8192, 64), array(M, 8192), iso.PinnedArray((M, 8192), "bf16")
        log()
        ctx.gemm_rowpar(a, w, c, M, 8192, 64, ctx.stream0, sink.ptr)
        last = log()[-1]
        assert last[0] == how and ("copy_out" in last[2]) == (how == "kernel"), (M, last)
        sink.free()
""")


def test_the_copy_engine_gets_rows_of_at_least_512_bytes(fake):
    """Narrow results: several rows of the matrix to one of the copy (all bytes, each once); a count of rows that nothing divides
    goes by the plain copy."""
    run(fake, """
with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, "bf16", 256)) as ctx:
    for M, N, how in ((70000, 8, "copy2d"), (99999, 8, "copy2d"), (30000, 24, "copy2d"), (100003, 8, "copy"), (5000, 128, "copy2d"),
                      (2050, 264, "copy2d"), (300003, 4, "copy"), (65537, 40, "copy"), (600, 32768, "copy2d")):
        a, w, c, sink = array(M, 64), array(N, 64), array(M, N), iso.PinnedArray((M, N), "bf16")
        log()
        ctx.gemm_rowpar(a, w, c, M, N, 64, ctx.stream0, sink.ptr)
        last = log()[-1]
        assert last[0] == how, (M, N, last)
        if how == "copy2d":
            width, height = map(int, last[2].split("x"))
            assert width * height == 2 * M * N and width >= 512 and width % 16 == 0, (M, N, last)
        else:
            assert int(last[2]) == 2 * M * N
        sink.free()
""")


def test_attention_over_a_handful_of_keys_takes_the_kernel_with_the_least_to_set_up(fake):
    """fp32 up to 16 (heads of 64) or 40 visible keys, bf16 heads of 64 up to 14; bf16 heads of 128 and forced launch shapes keep
    the tiles."""
    run(fake, """
for dt, d, limit in (("f32", 64, 16), ("f32", 128, 40), ("bf16", 64, 14), ("bf16", 128, 0)):
    with iso.Context(iso.make_cfg(256, 4, 2, d, 64, dt, 256)) as ctx:
        q = array(64, 256, dt=dt)
        for keys in (1, 14, 15, 16, 17, 40, 41, 64):
            for Tc, off, kv in ((keys, 0, keys), (1, keys - 1, 200), (50, 30, keys)):
                for flags in (0, 1 << 12, 2 << 14):
                    ctx.set_flags(flags)
                    log()
                    ctx.attn_chunk(q, q, q, q, Tc, off, kv, ctx.stream0)
                    (launch,) = log()
                    assert ("attn_simple" in launch[2]) == (keys <= limit and not flags), (dt, d, keys, Tc, off, kv, flags, launch)
""")


def test_products_of_a_single_k_slice_stay_with_the_whole_tile_rule(fake):
    run(fake, """
with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, "bf16", 256)) as ctx:
    a = array(64, 64)
    for M, N, K, kernel in ((3, 32, 64, "Li128ELi128ELi2"), (86, 560, 64, "Li128ELi128ELi2"), (195, 168, 64, "Li128ELi128ELi2"),
                            (65, 8, 128, "gemm_narrow_kernel")):
        log()
        ctx.gemm_rowpar(a, a, a, M, N, K, ctx.stream0)
        assert kernel in log()[0][2], (M, N, K)
""")


def test_what_is_recorded_into_a_graph_keeps_out_of_the_eager_workspaces(fake):
    """Recorded products are one kernel.  The first recorded layer allocates a workspace of its own and then runs the launches of
    the eager one; if that allocation fails its products are not split."""
    run(fake, f"""
T, hidden, nq, nkv, d, ffn = 200, 512, 4, 1, 128, 768
w = layer(hidden, nq, nkv, d, ffn)
def kernels():
    return [l[2] for l in log() if l[0] == "kernel"]
for refuse in (0, {WORKSPACE}):
    with iso.Context(iso.make_cfg(hidden, nq, nkv, d, ffn, "bf16", T)) as ctx:
        x, k, v, a = array(T, hidden), array(T, nkv, d), array(T, nkv, d), array(64, 64)
        prefill = lambda: ctx.layer_prefill(w, x, k, v, T, 0, iso.ISO_COMM_NONE, iso.ISO_SCHED_OVERLAP)
        product = lambda: ctx.gemm_rowpar(a, a, a, 512, 5120, 8192, ctx.stream0)
        log(); prefill(); eager = kernels()
        assert any("share_sum" in n for n in eager)
        product(); assert len(kernels()) == 2
        fake.fake_capturing(1)
        fake.fake_refuse(refuse)
        product(); assert len(kernels()) == 1
        for call in range(2):
            prefill()
            lines = log()
            assert [l[2] for l in lines if l[0] == "malloc"] == ([] if refuse or call else ["{WORKSPACE}"])
            assert sum(l[0] == "refused" for l in lines) == (1 if refuse and not call else 0)
            recorded = [l[2] for l in lines if l[0] == "kernel"]
            assert recorded == eager if not refuse else not any("share_sum" in n for n in recorded)
        fake.fake_capturing(0)
        fake.fake_refuse(0)
""")


def test_an_error_that_was_reported_is_not_reported_again_by_the_next_launch(fake):
    """The runtime keeps the last error until it is asked for, and every launch asks: a call that failed for lack of memory must
    not make the next one fail (here the retry, whose extra stream then does without the key-split workspace)."""
    run(fake, f"""
T, hidden, nq, nkv, d, ffn = 300, 512, 4, 1, 128, 768
w = layer(hidden, nq, nkv, d, ffn)
with iso.Context(iso.make_cfg(hidden, nq, nkv, d, ffn, "bf16", T)) as ctx:
    ctx.set_flags(iso.ISO_FLAG_KEEP_CUT)
    x, k, v = array(T, hidden), array(1, T, nkv, d), array(1, T, nkv, d)
    call = lambda: ctx.stack_prefill_chunks([w], x, k, v, T, [100, 200], iso.ISO_COMM_D2H, iso.ISO_SCHED_STREAM_PER_CHUNK)
    fake.fake_refuse({512 * (16 * 256 * 16 + 256 * 8)})
    try:
        call()
        raise SystemExit("the allocation was not refused")
    except iso.IsoError as e:
        assert e.code == iso.ISO_ERR_HIP
    call()
""")


def test_an_offset_far_behind_the_cache_reaches_the_kernels_as_the_end_of_the_cache(fake):
    """A chunk may begin behind the last key: every row sees the whole cache then, whatever the offset.  The kernels add row numbers
    to it in 32 bits; a sum that overflows would put the last visible key below zero and the end of the buffer anywhere."""
    run(fake, """
fake.fake_int_argument(5)                    # q_offset of every attention kernel
for dt in ("f32", "bf16"):
    for d in (64, 128):
        with iso.Context(iso.make_cfg(256, 4, 2, d, 64, dt, 700)) as ctx:
            q = array(700, 512, dt=dt)
            for flags in (0, 7 << 14, 1 << 12, 2 << 14, iso.ISO_FLAG_ATTN_STAGED, iso.ISO_FLAG_SIMPLE_ATTN):
                ctx.set_flags(flags)
                for Tc, kv in ((1, 1), (300, 8), (64, 700), (700, 300)):
                    for off in (0, kv - 1, kv, kv + 1, 2 ** 31 - Tc - 1, 2 ** 31 - 1):
                        log()
                        ctx.attn_chunk(q, q, q, q, Tc, off, kv, ctx.stream0)
                        (launch,) = log()
                        assert int(launch[2].split()[-1]) == min(off, kv), (dt, d, flags, Tc, kv, off, launch)
""")


def test_norms_stay_kernels_where_the_fp32_projections_would_repeat_them_too_often(fake):
    """Gate/up computes its norm up to 256 columns of hidden state and two tiles (16 x 16) a unit, QKV up to 768 columns and, beyond
    256 of them, four tiles a unit; both sides of each line."""
    run(fake, """
for hidden, heads, ffn, T, in_qkv, in_gate_up in (
        (256, 4, 688, 128, 1, 1), (256, 4, 688, 176, 1, 1), (256, 4, 688, 192, 1, 0), (256, 4, 688, 1024, 1, 0), (128, 2, 344, 368, 1, 1),
        (128, 2, 344, 400, 1, 0), (264, 4, 688, 16, 1, 0), (512, 8, 1376, 333, 1, 0), (512, 8, 1376, 352, 0, 0), (768, 6, 1024, 400, 1, 0),
        (776, 6, 1024, 16, 0, 0)):
    w = layer(hidden, heads, heads, 64, ffn, "f32")
    with iso.Context(iso.make_cfg(hidden, heads, heads, 64, ffn, "f32", T)) as ctx:
        x, k, v = array(T, hidden, dt="f32"), array(T, heads, 64, dt="f32"), array(T, heads, 64, dt="f32")
        log()
        ctx.layer_prefill(w, x, k, v, T, 0, iso.ISO_COMM_NONE)
        names = [l[2] for l in log() if l[0] == "kernel"]
        norms = [sum("rmsnorm_kernelIfLi%dELb0ELb1E" % deltas in n for n in names) for deltas in (0, 1)]
        assert norms == [1 - in_qkv, 1 - in_gate_up], (hidden, T, norms)
""")


def test_attention_of_few_rows_takes_the_wave_kernel_where_it_is_ahead(fake):
    """Both sides of every line of the rule, on 256 units: keys and rounds, the rows that a second round needs, and the places
    where the other kernel splits the keys over three workgroups."""
    run(fake, """
for d, heads, Tc, keys, wave in (
        (128, 13, 333, 2816, 1), (128, 13, 333, 2817, 0), (128, 8, 1024, 2816, 1), (64, 32, 512, 2816, 1), (64, 8, 32, 2817, 0),
        (64, 12, 704, 1536, 1), (64, 12, 704, 1537, 0), (64, 12, 672, 2816, 1), (64, 12, 897, 2816, 1),
        (128, 16, 513, 960, 1), (128, 20, 480, 480, 0), (128, 20, 481, 481, 1), (64, 40, 480, 480, 0), (64, 40, 481, 481, 1),
        (128, 16, 1024, 1536, 1), (128, 16, 1024, 1537, 0), (128, 16, 1025, 1025, 0),
        (128, 16, 600, 1010, 1), (128, 16, 600, 1011, 0), (128, 16, 700, 1536, 1),
        (64, 32, 800, 2048, 1), (64, 32, 800, 2049, 0), (64, 32, 801, 801, 0)):
    with iso.Context(iso.make_cfg(256, heads, heads, d, 64, "bf16", keys)) as ctx:
        q = array(8, 8)
        log()
        ctx.attn_chunk(q, q, q, q, Tc, keys - Tc if keys >= Tc else 0, keys, ctx.stream0)
        (launch,) = log()
        assert ("attn_bf16_wave" in launch[2]) == bool(wave), (d, heads, Tc, keys, launch)
""")


def test_launches_that_the_estimates_have_to_get_right_by_far(fake):
    """Narrow tiles are not taken for many rounds of the chip (two to three times the time of the large tiles), and a few rows are
    not dealt to more shares than the second kernel adds in the time that they save."""
    run(fake, """
with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, "bf16", 256)) as ctx:
    a = array(64, 64)
    for M, N, K in ((1734, 7976, 128), (5442, 7992, 192), (1744, 9704, 256), (5442, 7992, 128)):
        log()
        ctx.gemm_rowpar(a, a, a, M, N, K, ctx.stream0)
        assert "gemm_narrow_kernel" not in log()[0][2], (M, N, K)
    for M, most in ((1, 8), (16, 8), (31, 8), (48, 8)):
        log()
        ctx.gemm_rowpar(a, a, a, M, 1280, 8192, ctx.stream0)
        name, grid = log()[0][2].rsplit(" ", 1)
        rows = int(name.split("NarrowCfgIN")[1].split("ELi")[1].split("E")[0]) if "NarrowCfgIN" in name else 32
        tiles = -(-M // rows) * 20
        assert int(grid.split("x")[0]) <= most * tiles, (M, name, grid)
""")


def test_the_plain_main_loop_can_be_forced_for_every_tile_that_has_one(fake):
    run(fake, """
with iso.Context(iso.make_cfg(256, 4, 4, 64, 64, "bf16", 256)) as ctx:
    a = array(64, 64)
    for variant, rows, columns in ((1, 256, 256), (2, 256, 128), (3, 128, 128), (4, 128, 256)):
        ctx.set_flags((variant + 8) << 8)
        log()
        ctx.gemm_rowpar(a, a, a, 300, 520, 256, ctx.stream0)
        (launch,) = log()
        assert "gemm_bf16_dtl_kernelILi%dELi%dE" % (rows, columns) in launch[2] and "ELb0ELb0ELb0E" in launch[2], (variant, launch)
""")
