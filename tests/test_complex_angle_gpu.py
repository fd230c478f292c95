"""The complex-A scan at its tile edges (4-token tiles, 64-channel waves) with
one channel whose angles leave the domain of the hardware sine and cosine (256
revolutions) and one with a NaN step, beside ordinary channels of the same
waves, against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2608_02560_amd import precog as P
from paper_2608_02560_amd import synth
from precog_testutil import TOL_F32, err_rms

pytestmark = pytest.mark.gpu

WIDE, BAD = 5, 7  # channels: huge frequencies; a NaN step


@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("L,D,N,y", [(1, 64, 16, True), (4, 72, 16, True), (5, 8, 16, False), (9, 136, 16, True),
                                     (23, 64, 16, False), (9, 72, 8, True)])
def test_wide_angles_beside_ordinary_ones(L, D, N, y, io):
    inp = synth.scan_inputs_host(2, L, D, N, seed=700 + L + D + N, in_dtype=io)
    A_im = synth.complex_frequencies(D, N)
    sign = torch.tensor([1.0, -1.0]).repeat(N)[:N]
    A_im[WIDE] = (sign * 2 * math.pi * (torch.arange(N) * 600.0 + 3000.0)).float()
    dt = inp["dt"]
    dt[:, :, WIDE] = dt[:, :, WIDE].float().clamp(0.1, 0.4).to(io)  # 300 to 5,000 revolutions a token
    wide_rev = 0.4 * (3000.0 + 600.0 * (N - 1))
    if L > 2:
        dt[0, 2, BAD] = float("nan")
    d = {k: (v.cuda() if v is not None else None) for k, v in inp.items()}
    got = P.scan_complex(d["x"], d["dt"], d["A"], A_im.cuda(), d["B"], d["C"] if y else None, d["z"] if y else None,
                         d["Dskip"] if y else None, out_dtype=torch.float32, state_dtype=torch.float32, want_y=y,
                         chunk=L)
    torch.cuda.synchronize()
    ref = oracle.scan_complex(inp["x"], inp["dt"], inp["A"], A_im, inp["B"], inp["C"] if y else None,
                              inp["z"] if y else None, inp["Dskip"] if y else None, None, want_y=y)
    plain = [c for c in range(D) if c not in (WIDE, BAD)]
    # three roundings of the angle (1 / 2 pi, w / 2 pi, dt w / 2 pi) a token
    wide_tol = L * 2 * math.pi * wide_rev * 3 * 2.0 ** -24
    for g, r, axis in zip(got, ref, (2, 1)):
        if g is None:
            continue
        g = g.double().cpu().numpy()
        r = np.asarray(r, dtype=np.float64)
        assert err_rms(g.take(plain, axis), r.take(plain, axis)) <= TOL_F32
        scale = max(1.0, np.abs(r.take([WIDE], axis)).max())
        assert np.abs(g.take([WIDE], axis) - r.take([WIDE], axis)).max() <= (wide_tol + TOL_F32) * scale * math.sqrt(N)
        if L > 2:
            assert np.isnan(g.take([BAD], axis)[0]).any() and np.isfinite(g.take([BAD], axis)[1]).all()
