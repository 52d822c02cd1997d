"""CPU tests of what libmx's host code asks of the HIP runtime: which kernels a
call launches, and when a pinned staging buffer is written again.  The calls run
in a process of their own with a stand-in runtime preloaded (fake_hip.cpp), which
records launches and events and runs no kernel, so device pointers are made up."""
import json
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, sys, threading, time
import numpy as np
import paper_2606_16264_amd as mx
fake = ctypes.CDLL(FAKE)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_guard.argtypes = [ctypes.c_size_t]
A = lambda i: ctypes.c_void_p(0x10000000 * (i + 1))   # a device address
BIG = 1 << 40
def log():
    return [l.split() for l in fake.fake_log().decode().splitlines()]
def batch(decodes, prefill=0):
    n = decodes + (prefill > 0)
    need = [3] * decodes + ([-(-prefill // 16)] if prefill else [])
    at = np.cumsum([0] + need)
    pages = np.arange(at[-1], dtype=np.int32)
    return mx.Batch([mx.MX_DECODE] * decodes + [mx.MX_PREFILL] * (prefill > 0),
                    [1] * decodes + [prefill] * (prefill > 0), [40] * decodes + [0] * (prefill > 0),
                    [pages[at[i]:at[i + 1]] for i in range(n)])
def step(b, cfg, stream=None):
    return mx.lib().mx_layer_step(b.ptr, ctypes.byref(cfg), A(0), A(1), A(2), A(3), A(4), A(5), BIG,
                                  stream)
def append(b, shape, stream=None):
    return mx.lib().mx_kv_append(b.ptr, ctypes.byref(shape), A(0), A(1), A(2), A(3), A(5), BIG,
                                 stream)
def attn(b, shape, stream=None):
    return mx.lib().mx_paged_attn(b.ptr, ctypes.byref(shape), A(0), A(1), A(2), A(3), A(5), BIG,
                                  stream)
cfg = mx.layer_cfg(256, 512, 4, 4, 64, 1 << 20)
"""


@pytest.fixture(scope="session")
def fake_hip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-o", so,
                    os.path.join(HERE, "fake_hip.cpp"), "-ldl"], check=True)
    return so


def run(fake_hip, code, timeout=240):
    """The JSON that `code`, run on the stand-in runtime, prints last."""
    src = f"FAKE = {fake_hip!r}\n" + PRELUDE + textwrap.dedent(code)
    # (behind what is preloaded already, such as a sanitizer's runtime)
    preload = " ".join(filter(None, [os.environ.get("LD_PRELOAD"), fake_hip]))
    out = subprocess.run([sys.executable, "-c", src], cwd=ROOT, capture_output=True, text=True,
                         timeout=timeout, env={**os.environ, "LD_PRELOAD": preload})
    assert out.returncode == 0, out.stderr[-3000:]
    return json.loads(out.stdout.strip().splitlines()[-1])


def test_staging_buffers_outlive_their_readers(fake_hip):
    """Calls of every entry point that stages, on the null stream and others in turn."""
    r = run(fake_hip, """
        for i in range(60):
            s = [None, None, None, A(30), None, A(31)][i % 6]
            b = batch(3, 20 + i)
            st = [step(b, cfg, s), append(b, cfg.attn, s), attn(b, cfg.attn, s)]
            assert st == [0, 0, 0], (i, st, mx.last_error())
        print(json.dumps(dict(launches=len(log()), bad=fake.fake_violations())))
        """)
    assert r["launches"] >= 60 * 8 and r["bad"] == 0, r


@pytest.mark.parametrize("stream", ["None", "A(30)"])
def test_staging_buffer_of_a_call_that_fails_behind_its_launch(fake_hip, stream):
    """The event record behind a launch that reads a staging buffer fails (launch timing's own,
    or the ring's): the call reports it, and the buffer, which its kernel may still read, is not
    written again by later calls."""
    r = run(fake_hip, f"""
        bad = []
        for timing in (1, 0):
            mx.mx_profile_enable(timing)
            fake.fake_fail_record_behind(b"prologue_kernel")
            st = [step(batch(3), cfg, {stream})]
            st += [append(batch(3), cfg.attn, {stream}) for _ in range(20)]
            bad.append([st, fake.fake_violations()])
        print(json.dumps(bad))
        """)
    for st, violations in r:
        assert violations == 0, r
    assert r[0][0] == [6] + [0] * 20, r       # MX_ERR_HIP, then the calls go on
    assert r[1][0].count(6) <= 1 and len(r[1][0]) == 21, r


def test_calls_plan_side_by_side(fake_hip):
    """While one thread is still packing the metadata of a large batch (its staging buffer lets
    the first write wait), a call of another thread on another stream goes through; the large
    one follows when it may write."""
    r = run(fake_hip, """
        fake.fake_guard(1 << 20)
        small, large = batch(3), batch(3, 200000)
        assert step(small, cfg, A(30)) == 0     # first call: device state, a buffer
        st = {}
        def call(name, b, s):
            st[name] = step(b, cfg, s)
        t1 = threading.Thread(target=call, args=("large", large, A(31)), daemon=True)
        t1.start()
        while not fake.fake_guard_hit():
            time.sleep(0.001)
        t2 = threading.Thread(target=call, args=("small", small, A(30)), daemon=True)
        t2.start()
        t2.join(20)
        during = dict(st)
        fake.fake_guard_release()
        t1.join(60)
        t2.join(60)
        print(json.dumps(dict(during=during, end=st, bad=fake.fake_violations())))
        """)
    assert r["during"] == {"small": 0}, r
    assert r["end"] == {"small": 0, "large": 0} and r["bad"] == 0, r


def test_staging_ring_under_threads(fake_hip):
    """More threads than the ring has buffers, on the null stream and streams of their own."""
    r = run(fake_hip, """
        bad = []
        def work(t):
            for i in range(40):
                s = None if t % 3 == 0 else A(30 + t)
                st = append(batch(2 + t, 50 * (i % 5)), cfg.attn, s)
                if st: bad.append((t, i, st, mx.last_error()))
        ts = [threading.Thread(target=work, args=(t,)) for t in range(12)]
        [t.start() for t in ts]
        [t.join() for t in ts]
        print(json.dumps(dict(bad=bad, launches=len(log()), violations=fake.fake_violations())))
        """)
    assert r == dict(bad=[], launches=480, violations=0), r


GEMMS = """
def gemm_kernels(M, N, K, epi, tile_cfg=-1, ksplit=0):
    log()
    st = mx.lib().mx_debug_gemm_tiled(M, N, K, A(0), A(20), A(40), A(60), epi, tile_cfg, ksplit,
                                      A(80), BIG, None)
    assert st == 0, mx.last_error()
    return [l[0] for l in log()]
"""


READ_ONCE = [  # tile shape, M, N, K, K split, whether the read-once kernel runs
    # one row of tiles over 16 MB of weights or more, unsplit
    (3, 64, 12288, 4096, 1, True), (1, 128, 12288, 4096, 1, True), (0, 256, 12288, 4096, 1, True),
    (3, 65, 12288, 4096, 1, False), (3, 64, 2048, 4032, 1, False), (2, 64, 12288, 4096, 1, False),
    # split: planes (4 ksplit M N bytes) of up to a quarter of the weights (2 N K bytes)
    (3, 64, 6144, 4096, 8, True), (3, 64, 6144, 4032, 8, False), (1, 102, 6144, 4096, 5, True),
    (1, 103, 6144, 4096, 5, False), (1, 104, 15360, 5120, 4, True), (1, 72, 6144, 4096, 8, False),
    (0, 256, 8192, 28672, 8, True), (0, 170, 10240, 8192, 6, True), (0, 171, 10240, 8192, 6, False)]


def test_read_once_kernels_by_size(fake_hip):
    """Which main-loop kernel a forced tile shape and K split run."""
    r = run(fake_hip, GEMMS + f"""
print(json.dumps([gemm_kernels(M, N, K, 0, c, ks) for c, M, N, K, ks, _ in {READ_ONCE!r}]))
""")
    for case, names in zip(READ_ONCE, r):
        assert len(names) == 1 + (case[4] > 1), (case, names)
        assert ("gemm_once_kernel" in names[0]) == case[5], (case, names)


def test_forced_shapes_run_as_themselves(fake_hip):
    """Shape 4, 128 x 256 tiles through a three-stage ring, is not taken over by the four-stage
    read-once kernel of the same tile."""
    r = run(fake_hip, GEMMS + """
print(json.dumps([gemm_kernels(M, 12288, 4096, 0, c, 1)[0] for c, M in
                  ((0, 257), (1, 129), (2, 100), (3, 65), (4, 128), (4, 129))]))
""")
    shapes = ["256ELi256ELi128ELi64ELi4", "128ELi256ELi64ELi64ELi4", "128ELi128ELi64ELi64ELi4",
              "64ELi128ELi32ELi64ELi4", "128ELi256ELi64ELi64ELi3", "128ELi256ELi64ELi64ELi3"]
    for name, shape in zip(r, shapes):
        assert f"gemm_kernelILi{shape}E" in name and "once" not in name, (name, shape)


STREAM = [  # N, K, epilogue, the row counts of 1, 8 and 16 that stream
    (12288, 4096, 2, (1, 8, 16)), (4096, 4096, 1, (1, 8, 16)), (4096, 11008, 1, (1, 8, 16)),
    (6144, 4096, 2, (1, 8, 16)), (15360, 5120, 2, (1, 8, 16)), (2048, 4096, 1, (1, 8, 16)),
    (10240, 8192, 2, ()), (5120, 13824, 1, ()), (1024, 12288, 2, ()),
    # the sizes of the streaming kernel's own tests
    (48, 64, 0, (1, 8, 16)), (112, 1088, 1, (1, 8, 16)), (192, 64, 2, (1, 8, 16)),
    (320, 1152, 2, (1, 8, 16)), (16, 4160, 0, (1, 8, 16)), (4160, 512, 1, (1, 8, 16))]


def test_streaming_kernel_by_size(fake_hip):
    """Which GEMMs of up to 16 rows stream the weights, and that more rows never do."""
    r = run(fake_hip, GEMMS + f"""
out = []
for N, K, epi, _ in {STREAM!r}:
    out.append([M for M in (1, 8, 16, 17) if "stream" in gemm_kernels(M, N, K, epi)[0]])
print(json.dumps(out))
""")
    for case, rows in zip(STREAM, r):
        assert tuple(rows) == case[3], (case, rows)
