"""What the library asks of the HIP runtime, call by call (tests/hip_record.py):
set-up work is complete before anything can use it.  CPU only.
"""
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
