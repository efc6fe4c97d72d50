"""Calls of one basis-form plan that overlap: on several streams, and in the
replays of several graphs captured from it.  Every call has its own table of
regrouped filters, so each gives what it gives alone, bit for bit."""

import numpy as np
import pytest

import synth
from tests.graph_nodes import capture, kernels
from tests.helpers import TOL_FP32, err_stats, say, to_dev, to_host

pytestmark = pytest.mark.gpu

H, W, HALF, SIG, DEG, DS = 300, 333, 10, (0.7, 1.5, 2.0), (6, 4, 2), 2


def _case(n):
    R, I = synth.star_field(H, W, 40, seed=1), synth.star_field(H, W, 40, seed=2)
    a = [synth.coefficients(synth.n_basis(DEG), synth.n_spatial(DS), 28, seed=i) for i in range(n)]
    return R, I, a


def _plan(svc):
    return svc.Plan(H, W, HALF, SIG, DEG, DS, pedestal=1000.0)


def _table(graph):
    """Where a captured call's filters are written (None: it has no such table)."""
    k = [k for k in kernels(graph) if "regroup64_kernel" in k.name]
    return k[0].pointer(5) if k else None


def test_each_capture_has_its_own_filters(svc):
    import torch
    R, I, a = _case(2)
    Rd, Id, ad = to_dev(R), to_dev(I), [to_dev(x) for x in a]
    say("captures of a basis-form plan")
    with _plan(svc) as plan:
        alone = [to_host(plan.difference(Rd, Id, x)) for x in ad]
        out = [torch.empty_like(Rd) for _ in ad]
        graphs = [capture(lambda: plan.difference(Rd, Id, ad[i], out=out[i])) for i in range(2)]
        assert _table(graphs[0]) != _table(graphs[1])
        # two branches of one capture
        side, forked = torch.cuda.Stream(), [torch.empty_like(Rd) for _ in ad]

        def both():
            side.wait_stream(torch.cuda.current_stream())
            plan.difference(Rd, Id, ad[0], out=forked[0])
            with torch.cuda.stream(side):
                plan.difference(Rd, Id, ad[1], out=forked[1])
            torch.cuda.current_stream().wait_stream(side)
        fork = capture(both)
        tables = [k.pointer(5) for k in kernels(fork) if "regroup64_kernel" in k.name]
        assert len(tables) == 2 and tables[0] != tables[1]
        streams = [torch.cuda.Stream() for _ in range(3)]
        eager = torch.empty_like(Rd)
        for g in graphs + [fork]:
            g.instantiate()
        torch.cuda.synchronize()
        for _ in range(20):
            for s, g in zip(streams, graphs + [fork]):
                with torch.cuda.stream(s):
                    g.replay()
            plan.difference(Rd, Id, ad[1], out=eager)
        torch.cuda.synchronize()
        for got in (out, forked):
            assert np.array_equal(to_host(got[0]), alone[0]) and np.array_equal(to_host(got[1]), alone[1])
        assert np.array_equal(to_host(eager), alone[1])


def test_streams_overlap(svc):
    import torch
    R, I, a = _case(4)
    Rd, Id, ad = to_dev(R), to_dev(I), [to_dev(x) for x in a]
    say("streams of a basis-form plan")
    with _plan(svc) as plan:
        alone = [to_host(plan.difference(Rd, Id, x)) for x in ad]
        streams, out = [torch.cuda.Stream() for _ in ad], [torch.empty_like(Rd) for _ in ad]
        torch.cuda.synchronize()
        for _ in range(20):
            for s, x, o in zip(streams, ad, out):
                with torch.cuda.stream(s):
                    plan.difference(Rd, Id, x, out=o)
        torch.cuda.synchronize()
        for got, want in zip(out, alone):
            assert np.array_equal(to_host(got), want)


@pytest.mark.parametrize("deg,d_s", [(DEG, 0), (DEG, 2), (DEG, 3), (DEG, 4), ((4, 2, 0), 4), ((7,), 4), ((3,), 4)])
def test_more_captures_than_tables(svc, orc, deg, d_s):
    """Past the last table the kernel forms the filters, to the same bits, or above
    third order a call takes the dense product, which needs none (49, 22, 36 and 10 bases:
    each number of its 16-filter blocks); the streams that hold one keep it."""
    import torch
    R, I, sig = *_case(0)[:2], SIG[:len(deg)]
    a = synth.coefficients(synth.n_basis(deg), synth.n_spatial(d_s), 0, seed=1)
    Rd, Id, ad = to_dev(R), to_dev(I), to_dev(a)
    say("captures past the last table", deg, d_s)
    with svc.Plan(H, W, HALF, sig, deg, d_s, pedestal=1000.0) as plan:
        first, out = to_host(plan.difference(Rd, Id, ad)), torch.empty_like(Rd)
        tables = [_table(capture(lambda: plan.difference(Rd, Id, ad, out=out))) for _ in range(70)]
        had = [t for t in tables if t is not None]
        assert 32 <= len(had) < 70 and len(set(had)) == len(had)
        assert tables[len(had):] == [None] * (70 - len(had))
        past = capture(lambda: plan.difference(Rd, Id, ad, out=out))
        route = "contract_direct_kernel" if d_s <= 3 else "contract_f32_kernel"
        assert any(route in k.name for k in kernels(past))
        past.instantiate()
        past.replay()
        if d_s <= 3:
            assert np.array_equal(to_host(out), first)
        want = orc.difference(R, I, HALF, orc.basis(HALF, sig, deg), d_s, a)
        assert err_stats(to_host(out), want)[0] <= TOL_FP32
        assert np.array_equal(to_host(plan.difference(Rd, Id, ad)), first)


@pytest.mark.parametrize("half,d_s,fits", [(22, 2, True), (23, 2, True), (24, 2, False), (18, 3, True), (19, 3, False)])
def test_filters_formed_in_lds_at_its_limit(svc, half, d_s, fits):
    """The largest table that fits beside a tile, and the first that does not (which
    the dense product takes, to its own accuracy)."""
    import torch
    R, I = _case(0)[:2]
    a = synth.coefficients(synth.n_basis(DEG), synth.n_spatial(d_s), 0, seed=1)
    Rd, Id, ad = to_dev(R), to_dev(I), to_dev(a)
    say("filters formed in LDS, half-width", half, d_s)
    with svc.Plan(H, W, half, SIG, DEG, d_s, pedestal=1000.0) as plan:
        first, out = to_host(plan.difference(Rd, Id, ad)), torch.empty_like(Rd)
        for _ in range(70):
            g = capture(lambda: plan.difference(Rd, Id, ad, out=out))
        assert _table(g) is None
        assert any("contract_direct_kernel" in k.name for k in kernels(g)) == fits
        g.instantiate()
        g.replay()
        if fits:
            assert np.array_equal(to_host(out), first)
        assert err_stats(to_host(out), first)[0] <= TOL_FP32


def test_per_thread_streams_overlap(svc):
    """The per-thread default stream is one handle for every thread's own stream."""
    import ctypes
    import threading
    import torch
    R, I, a = _case(2)
    Rd, Id, ad = to_dev(R), to_dev(I), [to_dev(x) for x in a]
    say("per-thread default streams of a basis-form plan")
    with _plan(svc) as plan:
        alone = [to_host(plan.difference(Rd, Id, x)) for x in ad]
        out = [torch.empty_like(Rd) for _ in ad]
        turn, bad = threading.Lock(), []
        torch.cuda.synchronize()

        def work(i):
            for _ in range(20):
                with turn:   # one thread at a time calls; what they enqueue overlaps
                    if plan._lib.svconv_plan_set_stream(plan._p, ctypes.c_void_p(2)):
                        bad.append(i)
                    args = [ctypes.c_void_p(t.data_ptr()) for t in (Rd, Id, ad[i], out[i])]
                    if plan._lib.svconv_difference(plan._p, *args):
                        bad.append(i)
        threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not bad
        for got, want in zip(out, alone):
            assert np.array_equal(to_host(got), want)


def test_pipelines_give_their_table_back(svc):
    """A pipeline's compute stream is drained when its run returns."""
    import torch
    R, I, a = _case(1)
    host = [torch.from_numpy(x) for x in (R, I, a[0])]
    dev = [x.cuda() for x in host]
    say("pipelines of a basis-form plan")
    with _plan(svc) as plan:
        want = to_host(plan.difference(*dev))
        for _ in range(70):
            D = torch.empty(H, W)
            with svc.Pipeline(plan, depth=1) as q:
                q.run([host[0]], [host[1]], [host[2]], [D])
            assert np.array_equal(D.numpy(), want)
        assert _table(capture(lambda: plan.difference(*dev))) is not None


def test_factor_beside_a_fit_step(svc):
    """A factorisation on one stream while a Gauss-Newton step of the same plan is
    in flight on another: they share no scratch."""
    import torch
    h, w, half, sig, deg, d_s = 96, 112, 3, (1.2,), (3,), 2
    n = synth.n_basis(deg) * synth.n_spatial(d_s)
    R, I = to_dev(synth.star_field(h, w, 30, seed=3)), to_dev(synth.star_field(h, w, 30, seed=4))
    A = torch.from_numpy(np.eye(n) * 4.0 + 1.0 / n).cuda()
    say("factor beside a step")
    with svc.Plan(h, w, half, sig, deg, d_s, pedestal=1000.0) as plan:
        L = plan.cholesky_factor(plan.normal_matrix(R))
        a0 = torch.zeros(plan._fit_coef, dtype=torch.float64).cuda()
        a0[6, 0] = 1.0

        def state():
            return a0.clone(), torch.empty_like(a0, dtype=torch.float32), torch.empty_like(R)

        def step(a64, a32, D):
            plan.gn_step(R, I, L, a64, a32, D, stats=False)
        alone = state()
        step(*alone)
        alone = to_host(alone[0])
        fit, other = torch.cuda.Stream(), torch.cuda.Stream()
        for _ in range(20):
            st, factors = state(), [A.clone() for _ in range(6)]
            torch.cuda.synchronize()
            with torch.cuda.stream(fit):
                step(*st)
            with torch.cuda.stream(other):
                for M in factors:
                    plan.cholesky_factor(M)
            # the adjoint's sums agree to float64 rounding from call to call, and
            # the step takes them through the normal matrix of a star field
            assert np.max(np.abs(to_host(st[0]) - alone)) <= 1e-6 * np.abs(alone).max()
