"""Calls of one shape on several streams: a schedule built by the first call serves
the others at once."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_12168_amd as comet
import synth
from parity import assert_out_close
from test_gpu_parity import DEV, dev_u16, host_u16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(700, 1024, 1024), (300, 528, 640)])
def test_new_schedule_from_two_streams(M, N, K):
    # the first call comes on a stream with work queued, the second right after it
    # on another, which has no order with the first
    prec = synth.prec_map(K // 128, 1, "random", seed=M)
    x16, w16 = synth.activations(M, M, K, prec), synth.weights(M, N, K)
    A, sa = comet.quantize_act(dev_u16(x16), prec)
    Wp, sw = comet.pack_w4(dev_u16(w16))
    big = torch.ones((4096, 4096), device=DEV)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    comet.comet_release_caches()
    print(f"M={M} N={N} K={K}", flush=True)
    outs = []
    for i, s in enumerate(streams):
        with torch.cuda.stream(s):
            if i == 0:
                for _ in range(20):
                    big = big @ big * 1e-4
            outs.append(comet.w4ax_gemm(A, prec, sa, Wp, sw, M, N, K))
    torch.cuda.synchronize()
    qa, s_a = oracle.quantize_act(x16, prec)
    qw, s_w = oracle.quantize_weight(w16)
    ref = oracle.dequant_gemm(qa, s_a, qw, s_w)
    for out in outs:
        assert_out_close(host_u16(out).view(np.float16), ref, f"{M}x{N}x{K}")
    assert torch.equal(outs[0], outs[1])
