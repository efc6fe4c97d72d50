"""GPU parity of the float64 direct contraction (the regrouped form at the
FP32 precision, delta bases, the dense adjoint in R) against the FP64 oracle,
at the edges of its tiles, windows and wave splits.

Everything up to the last rounding is float64, so D is within half a float32
ulp of the oracle's: |err| <= 2^-24 |D|, plus the float64 rounding of the sums,
1e-12 of the products' magnitudes (k^2 M <= 1e4 terms at 2^-53)."""

import numpy as np
import pytest

import synth
from tests.helpers import say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _close(got, want, magnitude):
    return np.all(np.abs(got.astype(np.float64) - want) <= 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-12 * magnitude)


def _images(H, W, seed):
    r = np.random.default_rng(seed)
    return (1000 + 60 * r.normal(size=(H, W))).astype(np.float32), (1000 + 60 * r.normal(size=(H, W))).astype(np.float32), r


# one wave per tile from 768 tiles of 64 x 64 (32 above third order) on, four
# waves on a tile's 16 (8) rows from 512 tiles on or below h = 3, eight otherwise
@pytest.mark.parametrize("shape,h,d_s", [
    ((49152, 3), 1, 1), ((49089, 2), 3, 2), ((24577, 2), 1, 4),
    ((8193, 5), 3, 2), ((8192, 1), 4, 0), ((4097, 3), 2, 5), ((17, 66), 2, 3), ((1, 1), 1, 6),
    ((15, 64), 3, 3), ((16, 65), 2, 6), ((33, 130), 6, 1), ((70, 129), 4, 2)])
def test_delta_basis_splits(svc, orc, shape, h, d_s):
    H, W = shape
    k = 2 * h + 1
    R, I, r = _images(H, W, H + W + h)
    a = r.normal(size=(k * k, synth.n_spatial(d_s))).astype(np.float32)
    want = orc.difference(R, I, h, orc.basis_dfb(h), d_s, a)
    say("direct, delta basis", shape, h, d_s)
    for form in ("regrouped", "basis")[:2 if k * k <= 64 else 1]:
        with svc.Plan.dfb(H, W, h, d_s, form=form, pedestal=37.0) as plan:
            D = to_host(plan.difference(to_dev(R), to_dev(I), to_dev(a)))
            C = to_host(plan.forward(to_dev(R), to_dev(a)))
        assert _close(D, want, 1100.0 * np.abs(a).sum())
        assert _close(C, want + I.astype(np.float64), 1100.0 * np.abs(a).sum())


@pytest.mark.parametrize("shape,h,d_s", [
    ((40, 70), 7, 2), ((65, 64), 10, 3), ((20, 129), 15, 2), ((17, 33), 16, 4), ((33, 40), 31, 1),
    ((90, 65), 1, 0), ((30, 30), 3, 6), ((64, 64), 0, 2)])
def test_gaussian_basis_windows_and_adjoint(svc, orc, shape, h, d_s):
    H, W = shape
    sig, deg = (0.9, 2.0), (2, 1)
    frame = (11, 5, 500, 300)
    R, I, r = _images(H, W, H * W + h)
    B = orc.basis(h, sig, deg)
    a = r.normal(size=(len(B), synth.n_spatial(d_s))).astype(np.float32)
    G = r.uniform(-50, 50, size=shape).astype(np.float32)
    want = orc.difference(R, I, h, B, d_s, a, frame=frame)
    gR_want = orc.grad_R(R.shape, h, B, d_s, a, G, frame=frame)
    say("direct, gaussian basis", shape, h, d_s)
    with svc.Plan(H, W, h, sig, deg, d_s, form="regrouped", frame=frame, pedestal=1000.0) as plan:
        D = to_host(plan.difference(to_dev(R), to_dev(I), to_dev(a)))
        gR, _ = plan.backward(to_dev(R), to_dev(a), to_dev(G), want_ga=False)
        gR = to_host(gR)
    # every basis has unit L1 norm and every |P_m| <= 1; the adjoint's filters
    # are expanded around the pixel, (1 + k sx)^i (1 + k sy)^j <= 1.5^6 of that
    assert _close(D, want, 1100.0 * np.abs(a).sum())
    assert _close(gR, gR_want, 12 * 50.0 * np.abs(a).sum())
