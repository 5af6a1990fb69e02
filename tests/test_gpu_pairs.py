"""The pair kernel of the few-token GEMM (8 < M <= 48, two weight panels per
workgroup, K split over its sixteen waves): row-block edges, an odd panel count,
uneven slots and 8-bit blocks, against the CPU oracle; exact block sums of a
window; and the same bits on a second call.  With more than two panels per CU it
runs from 33 rows on, below them the per-wave kernel.  Then its row groups
(48 < M <= 256).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_12168_amd as comet
import synth
from parity import assert_out_close
from test_gpu_parity import assert_kernel, dev_u16, host, host_u16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [9, 16, 17, 32, 33, 48])
@pytest.mark.parametrize("panels,NG,n8", [(256, 32, 2), (257, 33, 33), (512, 47, 0), (601, 32, 5)])
def test_pair_kernel(M, panels, NG, n8):
    N, K = 16 * panels, 128 * NG
    prec = synth.prec_map(NG, n8, "random", seed=M)
    print(f"M={M} N={N} K={K} n8={n8}", flush=True)
    assert_kernel("pair" if panels <= 512 or M > 32 else "skinny", M, N, K)
    x16, w16 = synth.activations(M, M, K, prec), synth.weights(panels, N, K)
    A, sa = comet.quantize_act(dev_u16(x16), prec)
    Wp, sw = comet.pack_w4(dev_u16(w16))
    out = comet.w4ax_gemm(A, prec, sa, Wp, sw, M, N, K)
    qa, s_a = oracle.quantize_act(x16, prec)
    qw, s_w = oracle.quantize_weight(w16)
    assert_out_close(host_u16(out).view(np.float16), oracle.dequant_gemm(qa, s_a, qw, s_w), f"M={M}")
    assert torch.equal(out, comet.w4ax_gemm(A, prec, sa, Wp, sw, M, N, K))
    n0 = N - 24  # crosses the last two panels
    acc = comet.w4ax_gemm_acc(A, prec, sa, Wp, sw, M, N, K, M - 3, M, n0, N)
    assert np.array_equal(host(acc), oracle.group_acc(qa[M - 3:], qw[n0:]))


@pytest.mark.parametrize("M", [49, 64, 65, 96, 97, 145, 192, 200, 256])
@pytest.mark.parametrize("panels,NG,n8", [(1, 8, 1), (37, 17, 17), (256, 32, 2)])
def test_row_groups(M, panels, NG, n8):
    # more than 48 rows of a shape with too few tiles: groups of 32 or 48 rows, the
    # last one ragged, one panel or an odd count, fewer K-blocks than waves
    N, K = 16 * panels, 128 * NG
    assert_kernel("pair", M, N, K)
    prec = synth.prec_map(NG, n8, "random", seed=M)
    print(f"M={M} N={N} K={K} n8={n8}", flush=True)
    x16, w16 = synth.activations(M, M, K, prec), synth.weights(panels, N, K)
    A, sa = comet.quantize_act(dev_u16(x16), prec)
    Wp, sw = comet.pack_w4(dev_u16(w16))
    out = comet.w4ax_gemm(A, prec, sa, Wp, sw, M, N, K)
    qa, s_a = oracle.quantize_act(x16, prec)
    qw, s_w = oracle.quantize_weight(w16)
    assert_out_close(host_u16(out).view(np.float16), oracle.dequant_gemm(qa, s_a, qw, s_w), f"M={M}")
    noalloc = torch.empty_like(out)
    comet.comet_w4ax_gemm_noalloc(A, prec, sa, Wp, sw, noalloc, M, N, K)
    assert torch.equal(out, noalloc)
    n0 = max(0, N - 24)
    acc = comet.w4ax_gemm_acc(A, prec, sa, Wp, sw, M, N, K, 30, M, n0, N)  # crosses the groups
    assert np.array_equal(host(acc), oracle.group_acc(qa[30:], qw[n0:]))
