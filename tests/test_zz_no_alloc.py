"""The analysis entry point for callers without vectors for the scale factors, through the raw C ABI, against the oracle: calls in a
row on one stream and of different sizes, so that counts left behind by one, in any of the words that its blocks add to,
would show in the next."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cq():
    import paper_2410_07505_amd as pkg
    return pkg


def static_analysis(cq, X, alpha, bits):
    """(xrk, counters) from crossquant_kernel_analysis_static."""
    import torch
    T, I = X.shape
    Xg = torch.from_numpy(X).cuda()
    t, c = (torch.from_numpy(v).cuda() for v in oracle.absmax(X))
    xrk = torch.full((T, I), 7.0, dtype=torch.float16, device="cuda")
    cnt = torch.full((3,), -1, dtype=torch.int64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    rc = cq.raw.crossquant_kernel_analysis_static(
        ctypes.c_void_p(Xg.data_ptr()), T, I, Xg.stride(0), ctypes.c_void_p(t.data_ptr()), ctypes.c_void_p(c.data_ptr()),
        alpha, bits, ctypes.c_void_p(xrk.data_ptr()), ctypes.c_void_p(cnt.data_ptr()), ctypes.c_void_p(stream))
    assert rc == 0, cq.crossquant_status_string(rc)
    torch.cuda.synchronize()
    return xrk.cpu().numpy(), cnt.cpu().numpy()


def test_static_analysis_matches_the_oracle_call_after_call(cq):
    # 30 blocks, which add to one word; 256, which add in groups; 2; 256 again; 30
    shapes = [((300, 1537), 0.15, 8), ((2048, 2048), 0.15, 8), ((37, 520), 0.45, 4), ((2047, 2045), 1.0, 8), ((300, 1537), 0.0, 8)]
    for (T, I), alpha, bits in shapes:
        print("no-alloc analysis: %d x %d" % (T, I), flush=True)
        X = workloads.activation(T, I, seed=T + I, n_outlier=3, scale_lo=60.0, scale_hi=60.0)
        t, c = oracle.absmax(X)
        ref = oracle.kernel_analysis(X, t, c, alpha, bits)
        xrk, cnt = static_analysis(cq, X, alpha, bits)
        assert [int(v) for v in cnt] == [ref["Z"], ref["n_col_ge_row"], ref["n_bound_smaller"]]
        assert np.array_equal(xrk.view(np.uint16), ref["xrk"].view(np.uint16))
        assert cnt[0] > 0 and cnt[0] < X.size                      # a real kernel, not a degenerate count


def test_static_analysis_limits_and_argument_errors(cq):
    f = cq.raw.crossquant_kernel_analysis_static
    P = 0x10000
    big = (1 << 19) + 1
    assert f(P, big, 8, 8, P, P, 0.15, 8, P, P, None) == -2          # over the limits of its contract: nothing launched
    assert f(P, 8, big, big, P, P, 0.15, 8, P, P, None) == -2
    assert f(P, 4, 8, 8, P, P, 0.15, 8, P, 0, None) == -1
    assert f(P, 4, 8, 8, P, P, 0.15, 5, P, P, None) == -3
    assert f(P, 4, 8, 8, P, P, 1.5, 8, P, P, None) == -4
