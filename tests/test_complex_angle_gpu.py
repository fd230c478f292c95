"""The complex-A scan at its tile edges (4-token tiles, 64-channel waves) with
channels whose angles leave the domain of the hardware sine and cosine (256
revolutions) in some tiles, channels just inside it in waves of their own, and
one with a NaN step, beside ordinary channels, against the fp64 oracle.

The special channels start from |h0| = 1 and hardly decay, so their states keep
every rotation, and their steps are powers of two, so the kernel's angle differs
from the exact one by the roundings of 1 / 2 pi and of w / 2 pi alone.  The CPU
test shows that the bounds tell a missing reduction and a missing rotation."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2608_02560_amd import precog as P
from paper_2608_02560_amd import synth
from precog_testutil import TOL_F32, err_rms

WIDE, BAD, EDGE = 5, 7, 70  # channels: past the domain; a NaN step; just inside it (the next wave)
CASES = [(1, 64, 16, True), (4, 72, 16, True), (5, 8, 16, False), (8, 136, 16, True), (9, 136, 16, True),
         (23, 136, 16, False), (9, 72, 8, True)]


def _case(L, D, N, io):
    inp = synth.scan_inputs_host(2, L, D, N, seed=700 + L + D + N, in_dtype=io)
    A_im = synth.complex_frequencies(D, N)
    h0 = torch.zeros(2, D, N, 2)
    sign = np.where(np.arange(N) % 2 == 0, 1.0, -1.0)
    turns = {WIDE: 256.1 + 300.0 * np.arange(N) / N, EDGE: 255.9 - 40.0 * np.arange(N) / N}
    phase = np.linspace(0.3, 5.9, N)
    # 1/2 in every other tile, else 1/4: past the domain there alone
    step = torch.tensor([0.5 if (t // 4) % 2 == 0 else 0.25 for t in range(L)])
    for c, r in turns.items():
        if c >= D:
            continue
        A_im[c] = torch.from_numpy(sign * 2 * math.pi * r / 0.5).float()
        inp["A"][c] = 2.0 ** -12
        inp["dt"][:, :, c] = step.to(io)
        h0[:, c, :, 0] = torch.from_numpy(np.cos(phase)).float()
        h0[:, c, :, 1] = torch.from_numpy(np.sin(phase)).float()
    if L > 2:
        inp["dt"][0, 2, BAD] = float("nan")
    return inp, A_im, h0, [c for c in turns if c < D]


def _roll(inp, A_im, h0, c, cos_sin):
    """States [2, L, N] of channel c in fp64; cos_sin(angles) -> the rotation."""
    A = inp["A"][c].double().numpy()
    w = A_im[c].double().numpy()
    h = h0[:, c, :, 0].double().numpy() + 1j * h0[:, c, :, 1].double().numpy()
    out = []
    for t in range(inp["x"].shape[1]):
        dt = inp["dt"][:, t, c].double().numpy()[:, None]
        x = inp["x"][:, t, c].double().numpy()[:, None]
        co, si = cos_sin(dt * w)
        h = np.exp(-dt * A) * (co - 1j * si) * h + dt * x * inp["B"][:, t].double().numpy()
        out.append(h)
    return np.stack(out, axis=1)


def _exact(a):
    return np.cos(a), np.sin(a)


def _bound(inp, A_im, states, c):
    """Largest error of the modulus of channel c's states: a token's angle of r
    revolutions is off by 2 roundings, 2 pi r 2^-23, the sine and cosine by
    1.25e-7, and the sums stay within the fp32 bar; each acts on the largest
    state so far."""
    r = 0.5 * np.abs(A_im[c].double().numpy()).max() / (2 * math.pi)
    return states.shape[1] * (2 * math.pi * r * 2.0 ** -23 + 2.5e-7) * np.abs(states).max() + TOL_F32


@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("L,D,N,y", CASES)
def test_bounds_tell_a_wrong_rotation(L, D, N, y, io):
    inp, A_im, h0, special = _case(L, D, N, io)
    _, hT = oracle.scan_complex(inp["x"], inp["dt"], inp["A"], A_im, inp["B"], None, None, None, h0, want_y=False)
    hT = np.asarray(hT, dtype=np.float64)

    def unreduced(a):  # the hardware's results past its domain
        out = np.abs(a) >= 512 * math.pi
        return np.where(out, 1.0, np.cos(a)), np.where(out, 0.0, np.sin(a))

    for c in special:
        s = _roll(inp, A_im, h0, c, _exact)
        bound = _bound(inp, A_im, s, c)
        assert bound < 0.05
        assert np.abs(s[:, -1] - (hT[:, c, :, 0] + 1j * hT[:, c, :, 1])).max() < 1e-10
        none = _roll(inp, A_im, h0, c, lambda a: (np.ones_like(a), np.zeros_like(a)))
        assert np.abs(none[:, -1] - s[:, -1]).max() > 3 * bound
        if c == WIDE:
            wrong = _roll(inp, A_im, h0, c, unreduced)
            assert np.abs(wrong[:, -1] - s[:, -1]).max() > 3 * bound


@pytest.mark.gpu
@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("L,D,N,y", CASES)
def test_wide_angles_beside_ordinary_ones(L, D, N, y, io):
    inp, A_im, h0, special = _case(L, D, N, io)
    d = {k: (v.cuda() if v is not None else None) for k, v in inp.items()}
    got = P.scan_complex(d["x"], d["dt"], d["A"], A_im.cuda(), d["B"], d["C"] if y else None, d["z"] if y else None,
                         d["Dskip"] if y else None, h0.cuda(), out_dtype=torch.float32, state_dtype=torch.float32,
                         want_y=y, chunk=L)
    torch.cuda.synchronize()
    ref = oracle.scan_complex(inp["x"], inp["dt"], inp["A"], A_im, inp["B"], inp["C"] if y else None,
                              inp["z"] if y else None, inp["Dskip"] if y else None, h0, want_y=y)
    yg, hg = (None if g is None else g.double().cpu().numpy() for g in got)
    yr, hr = (None if r is None else np.asarray(r, dtype=np.float64) for r in ref)
    plain = [c for c in range(D) if c not in special and c != BAD]
    assert err_rms(hg[:, plain], hr[:, plain]) <= TOL_F32
    if y:
        assert err_rms(yg[:, :, plain], yr[:, :, plain]) <= TOL_F32
    for c in special:
        bound = _bound(inp, A_im, _roll(inp, A_im, h0, c, _exact), c)
        assert np.hypot(*np.moveaxis(hg[:, c] - hr[:, c], -1, 0)).max() <= bound
        if y:  # the readout weighs the states with C and the gate
            z = inp["z"][:, :, c].double().numpy()
            weight = inp["C"].double().abs().sum(dim=2).numpy() * np.abs(z / (1 + np.exp(-z)))
            assert (np.abs(yg[:, :, c] - yr[:, :, c]) <= bound * weight + TOL_F32 * np.abs(yr[:, :, c])
                    + 1e-6).all()
    if L > 2:
        assert np.isnan(hg[0, BAD]).any() and np.isfinite(hg[1, BAD]).all()
