"""GPU parity of the normal equations over the plane counts, segments, tails,
masks and bands of the Gram kernel, against the FP64 oracle."""

import numpy as np
import pytest

import synth
from tests.helpers import say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _run(svc, plan, R, I, mask):
    JtJ, rhs = plan.normal_equations(to_dev(R), to_dev(I), None if mask is None else to_dev(mask))
    return to_host(JtJ), to_host(rhs)


# one Gaussian family per degree, so that N + 1 planes (the bases and I) are
# 2, 16, 17, 19, 23, 24 (8 over 16), 35, 38, 49, 52, 56 and 64: every count of
# blocks of 16 with 0, 2, 4 and 8 planes over, and the padded block
@pytest.mark.parametrize("degrees", [(0,), (4,), (4, 0), (4, 1), (5, 0), (5, 0, 0), (6, 2), (7, 0), (8, 1),
                                     (8, 2), (8, 3), (9, 2, 0, 0)])
def test_plane_counts(svc, orc, degrees):
    H, W, h, d_s = 24, 45, 2, 1
    sig = (0.8, 1.3, 2.0, 2.8)[:len(degrees)]
    R = synth.star_field(H, W, 6, seed=sum(degrees) + 1)
    I = synth.star_field(H, W, 6, seed=sum(degrees) + 2)
    B = orc.basis(h, sig, degrees)
    J, b = orc.normal_equations(R, I, h, B, d_s)
    say("gram planes", len(B) + 1)
    with svc.Plan(H, W, h, sig, degrees, d_s, form="separable", pedestal=1000.0) as plan:
        Jg, bg = _run(svc, plan, R, I, None)
    # the responses are float32: a few 2^-24 of each product's magnitude
    assert np.max(np.abs(Jg - J)) <= 2e-6 * np.abs(J).max()
    assert np.max(np.abs(bg - b)) <= 2e-6 * np.abs(b).max()


@pytest.mark.parametrize("H,W", [(9, 8), (7, 7), (6, 40), (21, 4120), (40, 141), (300, 22), (12, 1039)])
@pytest.mark.parametrize("masked,background", [(False, False), (False, True), (True, False), (True, True)])
def test_delta_basis_segments_and_masks(svc, orc, H, W, masked, background):
    """Responses of a delta basis are pixels of R, exact in float32, so the sums
    differ from the oracle's by float64 rounding only; frames without an interior
    (6 rows at h = 3) give zeros."""
    h, d_s, frame = 3, 2, (7, 3, 5000, 400)
    r = np.random.default_rng(H * W)
    R = np.rint(1000 + 30 * r.normal(size=(H, W))).astype(np.float32)
    I = np.rint(1000 + 30 * r.normal(size=(H, W))).astype(np.float32)
    mask = (r.random((H, W)) < 0.3).astype(np.uint8) if masked else None
    B = orc.basis_dfb(h)
    ref = orc.normal_equations_bg if background else orc.normal_equations
    J, b = ref(R, I, h, B, d_s, mask=mask, frame=frame)
    say("gram segments", (H, W), masked, background)
    with svc.Plan.dfb(H, W, h, d_s, frame=frame, pedestal=1000.0) as plan:
        plan.set_background(background)
        for _ in range(2):   # the second call on the scratch the first one left
            Jg, bg = _run(svc, plan, R, I, mask)
            assert np.max(np.abs(Jg - J)) <= 1e-12 * max(np.abs(J).max(), 1e-300)
            assert np.max(np.abs(bg - b)) <= 1e-12 * max(np.abs(b).max(), 1e-300)
