"""The launch shape a scan chooses (time chunks and workgroup size): which
calls need a workspace, and parity at shapes on both sides of the choice."""
import itertools
import os
import random
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_2608_02560_amd import precog as P
from paper_2608_02560_amd import synth
from precog_testutil import TOL_BF16, TOL_F32, err_rms

DEV = "cuda"
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    """The library's rule as a host program: rows of (complex, bf16, B, L, D,
    N, chunk) -> dicts of what it chooses."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("shape") / "shape")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2608_02560_amd", "csrc"),
                    os.path.join(ROOT, "tests", "shape", "shape_driver.cpp"), "-o", exe], check=True)
    names = ("chunk", "chunks", "threads", "waves", "readout", "states", "one_readout", "one_states", "reserved")

    def run(rows):
        text = "".join("%d %d %d %d %d %d %d\n" % r for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [dict(zip(names, map(int, o.split()))) for o in out if o]
    return run


def test_rule_over_random_descriptors(shapes):
    """Chunks cover the sequence, are at least 8 tokens and fit the reserved
    workspace; rows of up to four waves have workgroups without dead waves; a
    cut is expected to be shorter than one pass over both kinds of scan; and a
    complex scan, whose summary pass costs 0.88 of its readout pass, is never
    cut in two."""
    rr = random.Random(1)
    size = lambda lo, hi: int(round(np.exp(rr.uniform(np.log(lo), np.log(hi)))))
    rows = [(rr.randint(0, 1), rr.randint(0, 1), size(1, 400), size(1, 70000), 8 * size(1, 512),
             rr.choice([1, 2, 4, 8, 16]), 0) for _ in range(4000)]
    rows += [(0, rr.randint(0, 1), size(1, 400), size(1, 70000), 8 * size(1, 512), rr.choice([32, 64]), 0)
             for _ in range(2000)]
    for r, s in zip(rows, shapes(rows)):
        cx, _, B, L, D, N, _ = r
        waves = -(-D * max(N // 16, 1) // 64)
        assert -(-L // s["chunk"]) == s["chunks"] <= s["reserved"], r
        assert s["chunks"] == 1 or s["chunk"] >= 8, r
        assert s["threads"] in ((64 * waves,) if waves <= 4 else (256, 512)), r
        if s["chunks"] > 1:
            assert B * waves < 2048 and s["readout"] + s["states"] < s["one_readout"] + s["one_states"], r
        assert not (cx and N == 16 and s["chunks"] == 2), r


# rows of one or two waves: the workgroups' dead waves were counted as work, so
# these were cut into 7, 3, 11 and 5 chunks and took 1.3 to 3 times as long
@pytest.mark.parametrize("desc,least", [((0, 1, 35, 1260, 64, 16, 0), 25), ((0, 1, 68, 2889, 24, 16, 0), 24),
                                        ((0, 1, 22, 1173, 104, 16, 0), 30), ((1, 1, 47, 1052, 88, 16, 0), 16)])
def test_narrow_rows_fill_the_gpu(shapes, desc, least):
    s, = shapes([desc])
    assert s["chunks"] >= least and s["waves"] <= 2


def test_the_fold_limits_the_cut(shapes):
    """One row of few waves: chunks as short as fill the GPU (8 tokens) would
    be folded one by one for longer than they save."""
    for desc in [(0, 1, 5, 2547, 24, 16, 0), (1, 1, 1, 1155, 208, 16, 0)]:
        s, = shapes([desc])
        assert 40 <= s["chunks"] <= 160, (desc, s)


@pytest.mark.gpu
@pytest.mark.parametrize("B,L,D,io", [(38, 80, 264, "f32"), (1, 36, 8, "bf16"), (47, 105, 88, "bf16"),
                                      (20, 150, 520, "f32")])
def test_complex_parity_over_automatic_cuts(B, L, D, io):
    """Three chunks (the fewest), four, and more in one and two waves per SIMD.
    A token's angle dt w is off by three roundings, and a state sums them over
    its memory: sum dt exp(-A sum dt) <= 1 / A + dt, so its error is at most
    3 2^-24 w (1 / A + dt) of the largest state beside the fp32 bar."""
    t = torch.float32 if io == "f32" else torch.bfloat16
    inp = synth.scan_inputs_host(B, L, D, 16, seed=B + L, in_dtype=t)
    A_im = synth.complex_frequencies(D, 16)
    d = {k: v.to(DEV) for k, v in inp.items()}
    y, h = P.scan_complex(d["x"], d["dt"], d["A"], A_im.to(DEV), d["B"], d["C"], d["z"], d["Dskip"],
                          out_dtype=torch.float32, state_dtype=torch.float32)
    yr, hr = oracle.scan_complex(inp["x"], inp["dt"], inp["A"], A_im, inp["B"], inp["C"], inp["z"], inp["Dskip"], None)
    tol = TOL_F32 if io == "f32" else TOL_BF16
    assert err_rms(y.double().cpu().numpy(), np.asarray(yr)) <= tol
    hr = np.asarray(hr)
    turn = 3 * 2.0 ** -24 * A_im.max().item() * (1 / inp["A"].min().item() + inp["dt"].max().item())
    assert np.abs(h.double().cpu().numpy() - hr).max() <= (TOL_F32 + turn) * np.abs(hr).max()


# one pass in workgroups of four waves (one wave per SIMD) with a remainder of
# channels, of eight, just past one four-wave workgroup per CU, and cuts by
# either workgroup size
@pytest.mark.gpu
@pytest.mark.parametrize("B,L,D,N,io", [
    (3, 17, 264, 16, "f32"), (2, 40, 520, 16, "bf16"), (1, 33, 72, 64, "bf16"), (5, 30, 8, 4, "f32"),
    (64, 20, 1032, 16, "bf16"), (65, 18, 1000, 16, "f32"), (130, 24, 1024, 16, "bf16"),
    (5, 300, 1000, 16, "f32"), (24, 160, 1032, 16, "bf16"), (3, 200, 264, 32, "bf16"),
    # rows of one to four waves: workgroups of as many
    (35, 200, 64, 16, "bf16"), (300, 24, 72, 16, "f32"), (9, 130, 40, 64, "bf16"), (7, 90, 104, 32, "f32")])
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
@pytest.mark.parametrize("Q,D,chunk", [(20, 264, 0), (130, 1032, 0), (260, 264, 0), (7, 256, 10), (40, 72, 30),
                                       (600, 40, 30)])
def test_query_call_over_launch_shapes(Q, D, chunk):
    """The one-call query path in workgroups of one, two, four and eight waves
    (past two four-wave workgroups per CU) and with time chunks, against the
    two calls, bitwise."""
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
