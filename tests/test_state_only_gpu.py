"""The readout-free scans over bf16 inputs, whose B_t u comes from the matrix
core, against the readout kind, which multiplies: the products are exact
either way, so every finite state is the same bits; infinities and NaN stay in
their channel and token."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_02560_amd import precog as P
from paper_2608_02560_amd import synth
from precog_testutil import TOL_BF16, err_rms

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _inputs(B, L, D, N, seed):
    inp = synth.scan_inputs_host(B, L, D, N, seed=seed, in_dtype=torch.bfloat16, h0_std=1.0)
    return inp, {k: v.to(DEV) for k, v in inp.items()}


def _both(d, chunk, dtype=torch.float32):
    a = (d["x"], d["dt"], d["A"], d["B"])
    _, h = P.scan(*a, h0=d["h0"], want_y=False, chunk=chunk, state_dtype=dtype)
    _, ref = P.scan(*a, d["C"], d["z"], d["Dskip"], d["h0"], chunk=chunk, state_dtype=dtype)
    return h, ref


# tiles of 4 tokens in pairs: whole, remainders of 1, 3, 4, 5 and 7; channels
# past a wave and past a workgroup
@pytest.mark.parametrize("N", [16, 32, 64])
@pytest.mark.parametrize("B,L,D", [(1, 1, 8), (2, 3, 72), (1, 4, 64), (3, 5, 264), (2, 8, 136), (1, 15, 520),
                                   (2, 16, 1032), (1, 67, 40)])
def test_same_states_as_the_readout_kind(B, L, D, N):
    _, d = _inputs(B, L, D, N, seed=L + D)
    h, ref = _both(d, L)
    assert torch.equal(h, ref)


@pytest.mark.parametrize("N,chunk", [(16, 9), (32, 16), (64, 21), (16, 0)])
def test_chunked_states_match_the_oracle(N, chunk):
    inp, d = _inputs(2, 150, 136, N, seed=chunk + N)
    h, ref = _both(d, chunk)
    assert torch.equal(h, ref)
    want = oracle.scan(inp["x"], inp["dt"], inp["A"], inp["B"], inp["C"], inp["z"], inp["Dskip"], inp["h0"],
                       nthreads=8)[1]
    assert err_rms(h.double().cpu().numpy(), want) <= TOL_BF16


@pytest.mark.parametrize("every", [1, 3])
@pytest.mark.parametrize("N", [16, 64])
def test_trajectory_without_outputs(N, every):
    _, d = _inputs(2, 37, 136, N, seed=every)
    a = (d["x"], d["dt"], d["A"], d["B"], every)
    h0 = d["h0"].half()  # the state dtype
    t, _, _ = P.trajectory(*a, h0=h0, state_dtype=torch.float16, chunk=37)
    r, _, _ = P.trajectory(*a, d["C"], d["z"], d["Dskip"], h0=h0, state_dtype=torch.float16, want_y=True,
                           chunk=37)
    assert torch.equal(t, r)


@pytest.mark.parametrize("N", [16, 32, 64])
@pytest.mark.parametrize("where", ["x", "dt", "B"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_non_finite_inputs_stay_where_they_are(N, where, value):
    """One non-finite x, dt or B: the states equal the readout kind's, NaN for
    NaN, and the untouched channels are finite."""
    B, L, D = 2, 22, 136
    _, d = _inputs(B, L, D, N, seed=5)
    t = d[where]
    t[1, 13, 5] = value
    h, ref = _both(d, L)
    assert torch.equal(h.isnan(), ref.isnan())
    assert torch.equal(torch.where(h.isnan(), 0.0, h), torch.where(ref.isnan(), 0.0, ref))
    bad = ~h.isfinite()
    assert bad.any() and not bad[0].any()
    if where == "B":
        assert not bad[1, :, torch.arange(N, device=DEV) != 5].any()
    else:
        assert not bad[1, torch.arange(D, device=DEV) != 5].any()


def test_products_near_the_smallest_normal():
    """u below 2^-110, where bf16 halves of it end: within 2^-126 |B| a token."""
    B, L, D, N = 1, 40, 64, 16
    _, d = _inputs(B, L, D, N, seed=6)
    d["x"] = (d["x"].float() * 2.0 ** -112).to(torch.bfloat16)
    d["h0"].zero_()
    h, ref = _both(d, L)
    bound = L * 2.0 ** -126 * d["B"].float().abs().max().item()
    assert (h.double() - ref.double()).abs().max().item() <= bound
    d["x"] = (d["x"].float() * 2.0 ** 112).to(torch.bfloat16)
    h, ref = _both(d, L)
    assert torch.equal(h, ref) and np.isfinite(h.cpu().numpy()).all()


@pytest.mark.parametrize("N", [16, 32, 64])
@pytest.mark.parametrize("x,b", [(-112, 0), (-125, 0), (-133, 0), (-90, -50), (60, -130), (100, -128), (-64, -80)])
def test_small_products_keep_their_bits(N, x, b):
    """x and B scaled by powers of two until u = dt x, B or their product is
    subnormal, every fifth x and every seventh B zero: the states equal the
    multiplications' bit for bit."""
    B, L, D = 2, 37, 136
    _, d = _inputs(B, L, D, N, seed=60 + N)
    for key, power in (("x", x), ("B", b)):
        v = d[key].float() * 2.0 ** max(power, -126) * 2.0 ** min(power + 126, 0)
        v.view(-1)[::5 if key == "x" else 7] = 0.0
        d[key] = v.to(torch.bfloat16)
    d["h0"].zero_()
    h, ref = _both(d, L)
    assert torch.equal(h, ref) and h.isfinite().all() and (h != 0).any()
