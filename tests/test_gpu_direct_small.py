"""GPU parity of the direct contraction's instances for 3 x 3 to 9 x 9 kernels
up to second order (half-width known at compile time) and of the wave splits
beside them, on frames on both sides of each rule, against the FP64 oracle.

Everything up to the last rounding is float64: |err| <= 2^-24 |D|, plus 1e-12 of
the products' magnitudes."""

import re

import numpy as np
import pytest

import synth
from tests.graph_nodes import kernel_names
from tests.helpers import sample_pixels, say, to_dev, to_host

pytestmark = pytest.mark.gpu


def _instance(name):
    """(J, rows, waves, waves per pixel, source of the taps, half-width) of a kernel's
    name; the source is 0 a table, 1 the coefficients of a delta basis, 2 formed by
    the kernel."""
    assert "contract_direct_kernel" in name
    return tuple(int(v) for v in re.findall(r"L[ib](\d+)E", name))


def _route(call):
    return [_instance(n) for n in kernel_names(call) if "contract_direct_kernel" in n][0]


def _run(svc, orc, shape, h, d_s, delta):
    """The instance that ran, after its D is compared at sampled pixels."""
    import torch
    H, W = shape
    r = np.random.default_rng(H + W + h + d_s)
    R = (1000 + 60 * r.normal(size=shape)).astype(np.float32)
    I = (1000 + 60 * r.normal(size=shape)).astype(np.float32)
    sig, deg = (0.9, 2.0), (2, 1)
    B = orc.basis_dfb(h) if delta else orc.basis(h, sig, deg)
    a = r.normal(size=(len(B), synth.n_spatial(d_s))).astype(np.float32)
    say("direct", shape, h, d_s, "delta" if delta else "gaussian")
    plan = svc.Plan.dfb(H, W, h, d_s) if delta else svc.Plan(H, W, h, sig, deg, d_s, form="regrouped")
    with plan:
        Rd, Id, ad = to_dev(R), to_dev(I), to_dev(a)
        out = torch.empty_like(Rd)
        route = _route(lambda: plan.difference(Rd, Id, ad, out=out))
        D = to_host(plan.difference(Rd, Id, ad))
    xs, ys = sample_pixels(H, W, 600, seed=1, h=h)
    ty = np.arange(0, H, 8)   # both sides of every tile edge of a column
    xs = np.concatenate([xs, np.full(len(ty), W - 1, np.int32), np.full(len(ty), min(64, W - 1), np.int32)])
    ys = np.concatenate([ys, ty, np.maximum(ty - 1, 0)]).astype(np.int32)
    want = orc.convolve_at(R, h, B, d_s, a, xs.astype(np.int32), ys) - I[ys, xs]
    bound = 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-12 * 1100.0 * np.abs(a).sum()
    assert np.all(np.abs(D[ys, xs].astype(np.float64) - want) <= bound)
    assert np.all(np.isfinite(D))
    return route


# frames of 32-row tiles: 256 and 255, 512 and 511, 1024 and 1023
ABOVE_BELOW = {1: ((8192, 63), (8160, 63)), 2: ((8190, 100), (8160, 128)), 4: ((8180, 250), (10912, 190))}


@pytest.mark.parametrize("delta", [True, False])
@pytest.mark.parametrize("h,d_s", [(h, d) for h in (1, 2, 3, 4) for d in (0, 1, 2)] + [(1, 3), (2, 3)])
def test_small_kernels(svc, orc, h, d_s, delta):
    k2j = (2 * h + 1) ** 2 * (d_s + 1)
    above, below = ABOVE_BELOW[1 if k2j <= 50 else 2 if k2j <= 75 else 4]
    assert _run(svc, orc, above, h, d_s, delta) == (d_s + 1, 8, 4, 1, int(delta), h)
    few = _run(svc, orc, below, h, d_s, delta)
    assert few[5] == (h if h * (d_s + 1) <= 2 else 0)


# tiles of 64 columns x 16 and x 8 rows against 256 compute units: four waves on
# the same pixels above 256 of the first, eight waves below, on half the rows
# where even those number at most 256
@pytest.mark.parametrize("shape,instance", [
    ((512, 513), (16, 4, 4)), ((513, 512), (16, 4, 4)), ((512, 512), (16, 8, 8)), ((257, 511), (16, 8, 8)),
    ((256, 512), (8, 8, 8)), ((2048, 63), (8, 8, 8))])
@pytest.mark.parametrize("h,d_s", [(5, 0), (7, 1), (10, 2), (6, 3)])
def test_wave_splits(svc, orc, shape, instance, h, d_s):
    assert _run(svc, orc, shape, h, d_s, False) == (d_s + 1,) + instance + (0, 0)


# the default form: the kernel forms its filters (one launch, no table) up to 3
# rounds of 256 entries x 8 bases, and up to 8 with few of either, on frames of at
# most 512 tiles of 64 x 32 (256 for more than 3 rounds)
@pytest.mark.parametrize("shape,h,deg,d_s,formed", [
    ((1, 1), 0, (0,), 0, True), ((48, 40), 2, (2,), 2, True), ((64, 65), 5, (2,), 2, True),
    ((256, 256), 7, (0,), 2, True), ((33, 129), 1, (6, 4, 2), 0, True), ((90, 70), 2, (4, 2, 0), 2, True),
    ((90, 70), 3, (6, 4, 2), 2, False), ((8192, 63), 7, (0,), 1, True), ((8193, 64), 9, (0,), 1, False),
    ((16384, 60), 2, (2,), 1, True), ((16385, 60), 2, (2,), 1, False), ((20, 49200), 1, (2,), 1, False),
    ((30, 33000), 1, (2,), 1, False), ((30, 32768), 3, (1,), 0, True)])
def test_filters_formed_by_the_kernel(svc, orc, shape, h, deg, d_s, formed):
    import torch
    H, W = shape
    sig, frame = (0.9, 1.6, 2.4)[:len(deg)], (3, 2, W + 50, H + 60)
    r = np.random.default_rng(H + W)
    R = (1000 + 60 * r.normal(size=shape)).astype(np.float32)
    I = (1000 + 60 * r.normal(size=shape)).astype(np.float32)
    B = orc.basis(h, sig, deg)
    a = r.normal(size=(len(B), synth.n_spatial(d_s))).astype(np.float32)
    say("direct, filters of the kernel's own", shape, h, deg, d_s)
    with svc.Plan(H, W, h, sig, deg, d_s, frame=frame, pedestal=1000.0) as plan:
        Rd, Id, ad = to_dev(R), to_dev(I), to_dev(a)
        out = torch.empty_like(Rd)
        names = kernel_names(lambda: plan.difference(Rd, Id, ad, out=out))
        assert len(names) == (1 if formed else 2)
        assert (_instance(names[-1])[4] == 2) == formed
        D = to_host(plan.difference(Rd, Id, ad))
        plan.set_form("regrouped")
        # the same filters through a table: the same bits
        assert np.array_equal(to_host(plan.difference(Rd, Id, ad)), D)
    xs, ys = sample_pixels(H, W, 400, seed=2, h=h)
    want = orc.convolve_at(R, h, B, d_s, a, xs, ys, frame=frame) - I[ys, xs]
    bound = 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-12 * 1100.0 * np.abs(a).sum()
    assert np.all(np.abs(D[ys, xs].astype(np.float64) - want) <= bound)
