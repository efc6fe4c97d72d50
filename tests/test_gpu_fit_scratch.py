"""The scratch of the normal matrix over calls of different kinds on one plan."""

import pytest

import synth
from tests.helpers import say, to_dev, to_host

pytestmark = pytest.mark.gpu


def test_kinds_of_calls_share_grown_scratch(svc, orc):
    """Once every kind of call has run, none allocates or frees any more, and each
    gives the same sums as on a plan of its own, bit for bit."""
    import numpy as np
    import torch
    H, W, h, d_s = 2048, 2048, 3, 2
    R, I = to_dev(synth.star_field(H, W, 5000, seed=1)), to_dev(synth.star_field(H, W, 5000, seed=2))
    mask = torch.zeros((H, W), dtype=torch.uint8, device="cuda")
    mask[100:1900:3, 50:2000:2] = 1

    def whole(plan):
        return plan.normal_equations(R, I)

    def stamps(plan):
        return plan.normal_equations(R, I, mask)

    def background(plan):
        plan.set_background(True)
        out = plan.normal_matrix(R, mask)
        plan.set_background(False)
        return (out,)
    kinds = (whole, stamps, background)
    want = []
    for f in kinds:
        with svc.Plan.dfb(H, W, h, d_s) as plan:
            want.append([to_host(t) for t in f(plan)])
    with svc.Plan.dfb(H, W, h, d_s) as plan:
        say("normal-matrix scratch")
        for f in kinds + kinds:
            f(plan)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for _ in range(2):
            for f, w in zip(kinds, want):
                got = [to_host(t) for t in f(plan)]
                assert torch.cuda.mem_get_info()[0] == free, f.__name__
                assert all(np.array_equal(a, b) for a, b in zip(got, w)), f.__name__
