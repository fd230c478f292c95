"""The launch shape a scan chooses (time chunks and workgroup size): which
calls need a workspace, and parity at shapes on both sides of the choice."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2608_02560_amd import precog as P
from paper_2608_02560_amd import synth
from precog_testutil import TOL_BF16, TOL_F32, err_rms

DEV = "cuda"


def _reserved(B, L, D, N):
    """Bytes for as many chunks as fill 2048 waves, of at least 8 tokens."""
    waves = B * -(-D * max(N // 16, 1) // 64)
    if waves >= 2048 or L <= 16:
        return 0
    n = -(-L // -(-L // max(1, min(-(-2048 // waves), L // 8))))
    up = lambda v: -(-v // 256) * 256
    return up(B * n * D * N * 4) + up(B * n * D * 4) if n > 1 else 0


@pytest.mark.parametrize("N", [4, 16, 64])
def test_workspace_covers_the_automatic_cut(N):
    """The reported size is never below what filling the GPU with 8-token or
    longer chunks takes, and stays 0 for the calls that are never cut."""
    for B, L, D in itertools.product((1, 3, 20, 34, 64), (1, 16, 17, 30, 512, 1237, 65536),
                                     (8, 520, 1000, 2048)):
        got = P.scan_workspace_bytes(P.scan_desc(B, L, D, N))
        low = _reserved(B, L, D, N)
        assert got >= low and (low > 0 or got == 0), (B, L, D, N)
        if N <= 16:
            c = P.scan_complex_workspace_bytes(P.scan_desc(B, L, D, N))
            assert (c > 0) == (low > 0) and c >= low


# one pass in workgroups of four waves (one wave per SIMD) with a remainder of
# channels, of eight, just past one four-wave workgroup per CU, and cuts by
# either workgroup size
@pytest.mark.gpu
@pytest.mark.parametrize("B,L,D,N,io", [
    (3, 17, 264, 16, "f32"), (2, 40, 520, 16, "bf16"), (1, 33, 72, 64, "bf16"), (5, 30, 8, 4, "f32"),
    (64, 20, 1032, 16, "bf16"), (65, 18, 1000, 16, "f32"), (130, 24, 1024, 16, "bf16"),
    (5, 300, 1000, 16, "f32"), (24, 160, 1032, 16, "bf16"), (3, 200, 264, 32, "bf16")])
def test_scan_parity_over_launch_shapes(B, L, D, N, io):
    t = torch.float32 if io == "f32" else torch.bfloat16
    inp = synth.scan_inputs_host(B, L, D, N, seed=B + L, in_dtype=t, h0_std=1.0)
    d = {k: v.to(DEV) for k, v in inp.items()}
    y, h = P.scan(d["x"], d["dt"], d["A"], d["B"], d["C"], d["z"], d["Dskip"], d["h0"])
    yr, hr = oracle.scan(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["z"], inp["Dskip"],
                         inp["h0"], nthreads=8)
    tol = TOL_F32 if io == "f32" else TOL_BF16
    assert err_rms(y.double().cpu().numpy(), yr) <= tol
    assert err_rms(h.double().cpu().numpy(), hr) <= tol
    again = P.scan(d["x"], d["dt"], d["A"], d["B"], d["C"], d["z"], d["Dskip"], d["h0"])
    assert torch.equal(again[0], y) and torch.equal(again[1], h)


@pytest.mark.gpu
@pytest.mark.parametrize("Q,D,chunk", [(20, 264, 0), (130, 1032, 0), (260, 264, 0), (7, 256, 10)])
def test_query_call_over_launch_shapes(Q, D, chunk):
    """The one-call query path in workgroups of four and of eight waves (past
    two four-wave workgroups per CU) and with time chunks, against the two
    calls, bitwise."""
    M, E, L = 300, 64, 30
    q, K, _, _ = synth.retrieval_inputs_host(Q, M, E, 4, seed=Q)
    store = synth.state_store(M, D * 16, seed=1, device=DEV).reshape(M, D, 16)
    d = {k: v.to(DEV) for k, v in synth.scan_inputs_host(Q, L, D, 16, 2, torch.bfloat16).items()}
    args = (d["x"], d["dt"], d["A"], d["B"])
    tail = (d["C"], d["z"], d["Dskip"])
    idx, y, h = P.query_prefill(q.to(DEV), K.to(DEV), store, *args, *tail, chunk=chunk)
    ref = P.top1(q.to(DEV), K.to(DEV))
    yr, hr = P.scan_from_store(*args, store, ref, *tail, chunk=chunk)
    assert torch.equal(idx, ref) and torch.equal(y, yr) and torch.equal(h, hr)
    assert np.array_equal(ref.cpu().numpy(), oracle.top1(q, K)[0])
