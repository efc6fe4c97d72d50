"""The float64 kernels of the separable form on plans and frames that its rules
leave to them (small frames and kernels go to the direct contraction with
regrouped filters instead): every half-width, the folds of 1 to 4 factors of one
parity and the tap-by-tap f_8 / f_9, both spatial-degree instances, frames that
are ragged in both directions, crops.  Each test first reads from a captured
graph that the kernel it is about is the one that runs."""

import numpy as np
import pytest

import synth
from tests.graph_nodes import kernel_names
from tests.helpers import TOL_FP32, err_stats, sample_pixels, say, to_dev, to_host

pytestmark = pytest.mark.gpu

SIG = (0.7, 1.5, 2.0, 2.6, 3.1)


def _inputs(H, W, deg, d_s, seed):
    R = synth.star_field(H, W, max(20, H * W // 2000), seed=seed)
    I = synth.star_field(H, W, max(20, H * W // 2000), seed=seed + 1)
    a = synth.coefficients(synth.n_basis(deg), synth.n_spatial(d_s), 0, seed=seed)
    return R, I, a


def _names(call):
    return " ".join(kernel_names(call))


D_CASES = [
    (1, (2,), 1), (2, (1,), 0), (3, (2,), 5), (4, (7,), 4), (5, (8, 1), 4), (6, (7,), 4), (7, (4, 2, 0), 2),
    (8, (9,), 2), (9, (6, 2), 3), (10, (6, 4, 2), 2), (11, (3,), 6), (12, (6, 4, 2), 2), (13, (4,), 1),
    (14, (6, 6, 2, 0, 0), 2), (15, (5, 3), 3), (15, (6, 4, 2), 4)]


@pytest.mark.parametrize("h,deg,d_s", D_CASES)
@pytest.mark.parametrize("frame", [None, (311, 40, 4096, 2048)])
def test_difference(svc, orc, h, deg, d_s, frame):
    import torch
    H, W = 1017, 1003
    R, I, a = _inputs(H, W, deg, d_s, seed=h)
    sig = SIG[-len(deg):]
    B = orc.basis(h, sig, deg)
    say("separable route", h, deg, d_s, frame)
    xs, ys = sample_pixels(H, W, 700, seed=h, R=R, h=h)
    edge = np.arange(0, W - 1, 32)   # rows above and below a tile boundary, the last row
    xs = np.concatenate([xs] + 3 * [edge]).astype(np.int32)
    ys = np.concatenate([ys, 0 * edge + 63, 0 * edge + 64, 0 * edge + H - 1]).astype(np.int32)
    want = orc.convolve_at(R, h, B, d_s, a, xs, ys, frame=frame) - I[ys, xs]
    Rd, Id, ad = to_dev(R), to_dev(I), to_dev(a)
    out = torch.empty_like(Rd)
    with svc.Plan(H, W, h, sig, deg, d_s, form="separable", frame=frame, pedestal=synth.SKY_LEVEL) as plan:
        assert "contract_sep_kernel" in _names(lambda: plan.difference(Rd, Id, ad, out=out))
        D = to_host(plan.difference(Rd, Id, ad))
        plan.set_form("regrouped")
        assert "contract_direct_kernel" in _names(lambda: plan.difference(Rd, Id, ad, out=out))
        whole = to_host(plan.difference(Rd, Id, ad))
    mx, rms = err_stats(D[ys, xs], want)
    say("  max %.3e rms %.3e" % (mx, rms))
    assert mx <= TOL_FP32
    # and every pixel against the direct contraction (itself within the tolerance)
    assert np.max(np.abs(D.astype(np.float64) - whole)) <= 2 * TOL_FP32


R_CASES = [(1, (0,), 5), (2, (1,), 4), (3, (2,), 5), (4, (2,), 4), (5, (4,), 5), (6, (3, 1), 4), (7, (4, 2, 0), 5),
           (8, (4, 2, 0), 4), (9, (5, 3), 5), (10, (5, 3), 4), (11, (4, 2, 0), 4), (12, (8, 1), 5), (13, (5, 3), 4),
           (14, (4, 2, 0), 6), (15, (5, 3), 4), (15, (6, 4, 2), 4)]


@pytest.mark.parametrize("h,deg,d_s", R_CASES)
def test_adjoint_in_R(svc, orc, h, deg, d_s):
    H, W, frame = 77, 139, (9, 500, 1100, 900)
    sig = SIG[-len(deg):]
    R, _, a = _inputs(H, W, deg, d_s, seed=h)
    G = synth.uniform_image(H, W, seed=19, lo=-40.0, hi=40.0)
    B = orc.basis(h, sig, deg)
    want = orc.grad_R((H, W), h, B, d_s, a, G, frame=frame)
    sR = orc.grad_R((H, W), h, np.abs(B), 0, np.abs(a).sum(axis=1, keepdims=True), np.abs(G), frame=frame)
    say("separable adjoint in R, route", h, deg, d_s)
    Rd, ad, Gd = to_dev(R), to_dev(a), to_dev(G)
    with svc.Plan(H, W, h, sig, deg, d_s, form="separable", frame=frame) as plan:
        plan.backward(Rd, ad, Gd, want_ga=False)   # torch's memory for dL/dR, outside the capture
        assert "adjoint_r_sep_kernel" in _names(lambda: plan.backward(Rd, ad, Gd, want_ga=False))
        gR = to_host(plan.backward(Rd, ad, Gd, want_ga=False)[0])
    e = np.abs(gR - want)
    say("  max err %.3e (scale %.3e)" % (e.max(), sR.max()))
    assert np.all(e <= 2e-5 * sR + 1e-6)


def test_autograd_against_the_other_route(svc, orc):
    """The gradients of a separable plan, through the factors, and of a basis-form
    plan, directly and by the dense product, agree to float32 rounding."""
    wl = synth.WORKLOADS["c4"]
    H, W, frame = 128, 150, (1000, 700, 4096, 4096)
    R, I, a = _inputs(H, W, wl.degrees, wl.spatial_degree, seed=3)
    grads = {}
    for form, kernel in (("basis", "contract_direct_kernel"), ("separable", "adjoint_r_sep_kernel")):
        with svc.Plan(H, W, wl.half_width, wl.sigmas, wl.degrees, wl.spatial_degree, form=form, frame=frame) as plan:
            Rd, ad = to_dev(R), to_dev(a)
            plan.backward(Rd, ad, Rd)
            assert kernel in _names(lambda: plan.backward(Rd, ad, Rd))
            Rt, at = Rd.requires_grad_(True), ad.requires_grad_(True)
            D = svc.difference(plan, Rt, to_dev(I), at)
            (D.double() ** 2).sum().backward()
            grads[form] = (to_host(Rt.grad), to_host(at.grad))
    for k in range(2):
        g0, g1 = grads["basis"][k], grads["separable"][k]
        assert np.abs(g1 - g0).max() <= 1e-4 * np.abs(g0).max()


@pytest.mark.parametrize("shape", [(1, 1), (9, 130), (45, 67)])
@pytest.mark.parametrize("h,deg,d_s", [(2, (1,), 3), (4, (2,), 4), (3, (3,), 5), (5, (4,), 6), (1, (1, 1, 1), 6),
                                       (6, (2, 1), 6)])
def test_dense_product_in_the_default_form(svc, orc, shape, h, deg, d_s):
    """What the basis form at FP32 leaves to the dense matrix-core product: up to 8
    bases from third order on (packed rows), 9 to 16 from fifth."""
    import torch
    H, W = shape
    sig, frame = SIG[:len(deg)], (5, 6, W + 30, H + 20)
    R, I, a = _inputs(H, W, deg, d_s, seed=h + H)
    B = orc.basis(h, sig, deg)
    say("dense product", shape, h, deg, d_s)
    Rd, Id, ad = to_dev(R), to_dev(I), to_dev(a)
    out = torch.empty_like(Rd)
    with svc.Plan(H, W, h, sig, deg, d_s, frame=frame, pedestal=synth.SKY_LEVEL) as plan:
        assert "contract_f32_kernel" in _names(lambda: plan.difference(Rd, Id, ad, out=out))
        D = to_host(plan.difference(Rd, Id, ad))
    assert err_stats(D, orc.difference(R, I, h, B, d_s, a, frame=frame))[0] <= TOL_FP32
