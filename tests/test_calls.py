"""What the library asks of the HIP runtime, call by call (tests/hip_record.py):
set-up work is complete before anything can use it.  CPU only.
"""
import re

import pytest

import hip_record


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    return hip_record.library(str(tmp_path_factory.mktemp("hip_record")))


def test_plan_upload_is_complete_before_any_stream_uses_it(shim):
    # one shape, first on a stream that may have work queued, then on another: the
    # second launch has no order with the first stream, so the upload is over
    # before the first call publishes the plan, and waits for no caller's work
    a, b, c = hip_record.run(shim, """
out = []
for s in (0x1000, 0x2000, 0x1000):
    assert gemm(700, 1024, 1024, stream=s) == 0, comet.comet_last_error()
    out.append(log())
print(json.dumps(out))
""")
    copies = [i for i, l in enumerate(a) if l.startswith("memcpy")]
    assert len(copies) == 1
    stream = a[copies[0]].split()[1]
    assert stream not in (str(0x1000), str(0x2000))
    launch = next(i for i, l in enumerate(a) if l.startswith(f"launch {0x1000} "))
    assert f"synchronize {stream}" in a[copies[0]:launch]
    assert f"synchronize {0x1000}" not in a
    for l in (b, c):
        assert not any(x.startswith("memcpy") for x in l)
        assert any(x.startswith("launch") for x in l)


@pytest.mark.parametrize("entry", ["comet_w4ax_gemm", "comet_w4ax_gemm_noalloc"])
def test_schedule_mode_reaches_shapes_of_row_groups(shim, entry):
    # 49 to 256 rows of a layer with few panels: row groups by default; the modes
    # that name a schedule of the tile kernels run it, an unknown one is refused
    body = f"""
out = {{}}
for mode in ("", "cost", "dp", "natural", "bogus"):
    os.environ["COMET_SCHED"] = mode
    st = gemm(100, 2048, 2048, entry="{entry}")
    out[mode] = [st, [l.split()[2] for l in log() if l.startswith("launch")], comet.comet_last_error()]
print(json.dumps(out))
"""
    out = hip_record.run(shim, body)
    for mode in ("", "cost"):
        st, kernels, _ = out[mode]
        assert st == 0 and len(kernels) == 1 and "skinny_pair_kernel" in kernels[0]
    for mode, natural in (("dp", 0), ("natural", 1)):
        st, kernels, _ = out[mode]
        assert st == 0 and len(kernels) == 1
        assert f"gemm_kernelILi128ELb0ELb0ELb{natural}E" in kernels[0]
    st, kernels, error = out["bogus"]
    assert st == 1 and not kernels and "unknown mode bogus" in error


KERNELS = {"skinny": r"skinny_kernelI", "skinny_shared": r"skinny_shared_kernelI",
           "mid": r"gemm_kernelILi128E", "tile": r"gemm_kernelILi256E",
           "stream": r"skinny_(chunk|stream)_kernelI", "pair": r"skinny_pair_kernelI"}


@pytest.mark.parametrize("mode", ["cost", "dp"])
def test_the_kernel_that_runs_is_the_one_reported(shim, mode):
    # every class and both sides of the rules between them; the three entry points
    # launch what comet_gemm_kernel says
    body = """
out = []
for M in (1, 8, 9, 16, 32, 33, 40, 41, 48, 49, 64, 65, 96, 128, 129, 200, 256, 257, 700, 2000):
    for N, K in ((1024, 1024), (2048, 896), (4096, 4096), (6144, 4096), (8192, 8192), (9616, 4224),
                 (10240, 8192), (16384, 2048), (57344, 8192), (57600, 8192)):
        kind = comet.KERNEL_NAMES[comet.comet_gemm_kernel(M, N, K, 256)]
        names = []
        for entry in ("comet_w4ax_gemm", "comet_w4ax_gemm_noalloc"):
            assert gemm(M, N, K, entry=entry) == 0, comet.comet_last_error()
            names.append([l.split()[2] for l in log() if l.startswith("launch")][-1])
        m = bytes([4] * (K // 128))
        assert comet.lib().comet_w4ax_gemm_acc(P, m, P, P, P, P, M, N, K, 128, 0, 1, 0, 1, 0) == 0
        names.append([l.split()[2] for l in log() if l.startswith("launch")][-1])
        out.append([M, N, K, kind, names])
print(json.dumps(out))
"""
    rows = hip_record.run(shim, body, COMET_SCHED=mode)
    for M, N, K, kind, names in rows:
        for name in names:
            assert re.search(KERNELS[kind], name), (M, N, K, kind, name)
    seen = {(kind, M > 48) for M, _, _, kind, _ in rows}
    want = {("skinny", False), ("skinny_shared", False), ("stream", False), ("stream", True),
            ("mid", False), ("mid", True), ("tile", True), ("pair", False)}
    assert seen == want | ({("pair", True)} if mode == "cost" else set())


def test_new_counters_are_zero_before_the_launch_that_counts(shim):
    # a captured call only records what it enqueues on its stream: counters cleared
    # there would not be zero for an eager call, and a memset in a graph is not
    # reliable on replays
    log = hip_record.run(shim, """
assert gemm(700, 1024, 1024, stream=0x1000) == 0, comet.comet_last_error()
print(json.dumps(log()))
""")
    assert not any(l.startswith("memset") for l in log)
    zero = next(i for i, l in enumerate(log) if l.startswith("launch") and "zero_ints" in l)
    stream = log[zero].split()[1]
    assert stream != str(0x1000)
    gemm = next(i for i, l in enumerate(log) if l.startswith(f"launch {0x1000} "))
    assert f"synchronize {stream}" in log[zero:gemm]


def test_swiglu_is_fused_exactly_where_the_128_row_kernel_runs(shim):
    rows = hip_record.run(shim, """
out = []
for M, N, K in ((8, 512, 1024), (100, 768, 1024), (100, 768, 640), (100, 33280, 1024), (300, 1024, 2048),
                (1024, 20480, 1024), (128, 57344, 8192)):
    kind = comet.KERNEL_NAMES[comet.comet_gemm_kernel(M, N, K, 256)]
    assert swiglu(M, N, K, stream=0x1000) == 0, comet.comet_last_error()
    names = [l.split()[2] for l in log() if l.startswith(f"launch {0x1000} ")]
    out.append([kind, names])
print(json.dumps(out))
""")
    for kind, names in rows:
        assert re.search(KERNELS[kind], names[0]), (kind, names)
        fused = "gemm_kernelILi128ELb0ELb1E" in names[0]
        assert fused == (kind == "mid")
        assert len(names) == (1 if fused else 2)
    assert {kind for kind, _ in rows} == {"skinny", "pair", "mid", "tile"}
