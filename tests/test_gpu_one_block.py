"""1D grids that one workgroup holds run their steps in a single launch (k_steps_1d).
The same calls with the stage timer on take the launch-by-launch path, which other
tests hold to the oracle: state, control block, tapes and the stage states left in
the workspace must agree, at grids around the workgroup sizes and with steps that are
clipped or skipped, at a fixed step, and replayed.

Bounds: both paths apply the same functions in the same order, so only the compiler's
choice of fused operations can differ, a few ulps of a field's scale per step, which
the limiter's switches may amplify about tenfold over five steps: 1e-13 in FP64, 5e-5
in FP32."""
import pytest
import torch

import hweno_inputs as hi
import paper_2207_05258_amd as h

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-13, torch.float32: 5e-5}


def _setup(physics, n, dtype, **kw):
    if physics == "euler":
        w = hi.euler1d_piecewise(n, 3)
        kw.setdefault("bc_x", h.REFLECT if n >= 2 else h.OUTFLOW)
    else:
        w = hi.scalar_random_1d(n, 3, physics)
        kw.setdefault("bc_x", h.PERIODIC)
    S = torch.as_tensor(w.S).to(dtype).cuda().contiguous()
    return S, h.Problem(dim=1, nx=n, physics=physics, dtype=dtype, dx=w.dx, **kw)


def _both(S0, prob, call):
    """(state, control block, tapes, workspace) of `call` on either path."""
    out = []
    for timed in (False, True):
        S, st = S0.clone(), h.Stepper(prob)
        st.ws.view(torch.uint8).zero_()
        tapes = torch.zeros(8, h.hweno.CTRL_LEN, dtype=torch.float64, device="cuda")
        if timed:
            h.hweno.timing_begin()
        call(st, S, tapes)
        if timed:
            assert h.hweno.timing_end()[0] > 0     # the stage kernels ran
        torch.cuda.synchronize()
        nb = S.numel() * S.element_size()
        o = 256 + (nb + 255) // 256 * 256          # control block, then the stage states
        stages = [st.ws[a:a + nb].view(S.dtype).view(S.shape).clone() for a in (256, o)]
        out.append((S, st.ctrl.clone(), tapes, stages))
    return out


def _close(x, y, tol, m):
    for f in range(x.shape[0]):
        scale = float(y[f].abs().max())
        assert float((x[f] - y[f]).abs().max()) <= tol * max(scale, float(y[f % m].abs().max())), f


def _check(both, prob):
    (A, ca, ta, sa), (B, cb, tb, sb) = both
    tol = TOL[prob.dtype]
    for x, y in [(A, B)] + list(zip(sa, sb)):
        _close(x, y, tol, prob.m)
    for x, y in ((ca, cb), (ta, tb)):
        x, y = x.reshape(-1, 16), y.reshape(-1, 16)
        assert torch.equal(x[:, 8].contiguous().view(torch.int64), y[:, 8].contiguous().view(torch.int64))
        assert torch.equal(x[:, 9], y[:, 9])
        keep = [0, 1, 2, 3, 4, 5, 6, 7, 10, 11]
        assert torch.allclose(x[:, keep], y[:, keep], rtol=tol, atol=0.0)


SIZES = {"euler": [1, 2, 3, 64, 254, 255, 256, 257, 511], "linadv": [1, 2, 5, 255, 256, 1022, 1023],
         "burgers": [4, 255, 1023]}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("physics,n", [(p, n) for p, ns in SIZES.items() for n in ns])
def test_steps_in_one_launch_match_launched_stages(physics, n, dtype):
    S, prob = _setup(physics, n, dtype)
    _check(_both(S, prob, lambda st, X, tp: st.steps(X, 5, tapes=tp)), prob)


OPTIONS = [dict(limiter_on=False), dict(limiter_characteristic=True), dict(characteristic=False),
           dict(characteristic=False, limiter_characteristic=True), dict(bc_x=h.PERIODIC),
           dict(bc_x=h.OUTFLOW)]


@pytest.mark.parametrize("kw", OPTIONS, ids=[",".join(f"{k}={v}" for k, v in o.items()) for o in OPTIONS])
def test_options_in_one_launch(kw):
    S, prob = _setup("euler", 130, torch.float64, **kw)
    _check(_both(S, prob, lambda st, X, tp: st.steps(X, 4, tapes=tp)), prob)


def test_clipped_skipped_fixed_and_replayed_steps():
    S, prob = _setup("euler", 100, torch.float64)
    dt = 2e-4
    _check(_both(S, prob, lambda st, X, tp: st.steps(X, 8, dt=dt, t_end=4.5 * dt, tapes=tp)), prob)

    def single(st, X, tp):
        for n in range(3):
            st.step(X, t_end=1e-3, tape=tp[n])

    both = _both(S, prob, single)
    _check(both, prob)
    tapes = both[0][2]

    def replay(st, X, tp):
        for n in range(3):
            st.step(X, replay=tapes[n], tape=tp[n])

    again = _both(S, prob, replay)
    _check(again, prob)
    assert torch.equal(again[0][0], both[0][0])     # the taped run, exactly


def test_more_steps_than_one_launch_takes():
    S, prob = _setup("linadv", 60, torch.float64)
    A, B = S.clone(), S.clone()
    sa, sb = h.Stepper(prob), h.Stepper(prob)
    sa.steps(A, 600)
    for n in (1, 255, 256, 88):
        sb.steps(B, n)
    assert torch.equal(A, B) and torch.equal(sa.ctrl, sb.ctrl)


def test_inadmissible_state_is_reported_and_skipped():
    S, prob = _setup("euler", 40, torch.float64)
    S[0, 0, 7] = float("nan")
    both = _both(S, prob, lambda st, X, tp: st.steps(X, 2, tapes=tp))
    a, b = both[0][1][8:9].view(torch.int64), both[1][1][8:9].view(torch.int64)
    assert int(a) == int(b) and int(a) & h.hweno.ST_SKIPPED
    assert torch.equal(torch.nan_to_num(both[0][0]), torch.nan_to_num(both[1][0]))
