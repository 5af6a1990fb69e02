"""The tile kernels at the ends of their pipelines: units shorter than the
weight ring, runs of one block, 8-bit blocks first, last, alone and in between,
ragged rows and columns, and scales that are fp16 subnormals (their products
come from a half-precision MFMA).  Every output against the CPU oracle, with the
tolerance of tests/parity.py.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_12168_amd as comet
import synth
from parity import assert_out_close
from test_gpu_parity import dev_u16, host_u16

pytestmark = pytest.mark.gpu

MAPS = {1: ["4", "8"], 2: ["44", "48", "84", "88"], 3: ["444", "484", "888"], 4: ["4444", "4488"],
        5: ["44444", "44448"], 6: ["444444", "848484"], 7: ["4444444", "4888484", "8888888"]}


def run(M, N, prec, x16, w16):
    K = len(prec) * 128
    A, sa = comet.quantize_act(dev_u16(x16), prec)
    Wp, sw = comet.pack_w4(dev_u16(w16))
    return host_u16(comet.w4ax_gemm(A, prec, sa, Wp, sw, M, N, K)).view(np.float16)


def reference(prec, x16, w16):
    qa, sa = oracle.quantize_act(x16, prec)
    qw, sw = oracle.quantize_weight(w16)
    return oracle.dequant_gemm(qa, sa, qw, sw)


@pytest.mark.parametrize("mode", ["dp", "cost", "natural"])
@pytest.mark.parametrize("M,N,kernel", [(100, 272, 2), (300, 272, 3), (513, 2064, 3)])
def test_short_units(monkeypatch, mode, M, N, kernel):
    monkeypatch.setenv("COMET_SCHED", mode)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for NG, maps in MAPS.items():
        w16 = synth.weights(NG, N, NG * 128)
        kind = comet.comet_gemm_kernel(M, N, NG * 128, cus)
        for m in maps:
            prec = np.array([int(c) for c in m], np.uint8)
            print(f"M={M} N={N} map={m} {mode} kernel={kind}", flush=True)
            x16 = synth.activations(NG, M, NG * 128, prec)
            assert_out_close(run(M, N, prec, x16, w16), reference(prec, x16, w16), m)
    assert kind == kernel or cus != 256


@pytest.mark.parametrize("M,N", [(100, 256), (513, 2064)])
def test_subnormal_scales(M, N):
    # activation scales around 1e-5 (fp16 subnormal), weights scaled to match
    prec = np.array([4, 8, 4], np.uint8)
    x16 = synth.normal_fp16(1, synth.TID_X, (M, 384), 3e-5)
    w16 = synth.normal_fp16(1, synth.TID_W, (N, 384), 200.0)
    _, sa = oracle.quantize_act(x16, prec)
    s = np.asarray(sa).view(np.float16).astype(np.float32)
    assert 0 < s.max() < 6.1e-5
    assert_out_close(run(M, N, prec, x16, w16), reference(prec, x16, w16), "subnormal scales")


@pytest.mark.parametrize("M,N", [(100, 256), (513, 2064)])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_scale_not_finite(M, N, bad):
    # one infinite or NaN scale: every other row and column keeps its bits, and its
    # own has (block sum) * scale: signed infinities, NaN where the sum is 0
    prec = np.array([4, 8, 4], np.uint8)
    K = 384
    x16, w16 = synth.activations(3, M, K, prec), synth.weights(3, N, K)
    A, sa = comet.quantize_act(dev_u16(x16), prec)
    Wp, sw = comet.pack_w4(dev_u16(w16))
    good = comet.w4ax_gemm(A, prec, sa, Wp, sw, M, N, K)
    for row, col, g in ((7, None, 0), (40, None, 1), (None, 5, 1), (None, 40, 2), (None, N - 1, 0)):
        s_a, s_w = sa.clone(), sw.clone()
        if col is None:
            s_a[g, row] = bad
            own = (slice(row, row + 1), slice(0, N))
        else:
            s_w[g, col] = bad
            own = (slice(0, M), slice(col, col + 1))
        print(f"M={M} N={N} {bad} row={row} col={col} block={g}", flush=True)
        out = comet.w4ax_gemm(A, prec, s_a, Wp, s_w, M, N, K)
        acc = comet.w4ax_gemm_acc(A, prec, sa, Wp, sw, M, N, K, own[0].start, own[0].stop,
                                  own[1].start, own[1].stop)
        want = good.clone()
        want[own] = (acc[..., g].float() * bad).half()
        assert torch.equal(torch.isnan(out), torch.isnan(want))
        assert torch.equal(out.nan_to_num(0, 60000, -60000), want.nan_to_num(0, 60000, -60000))
