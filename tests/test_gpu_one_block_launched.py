"""Steps of a 1D grid that one workgroup holds (k_steps_1d) against the same steps by
launches, which larger grids take and other tests hold to the oracle: a periodic grid
repeated, or a grid between walls unfolded into its mirror image and repeated, is a larger
grid with the same cells, speeds and time steps.  State, stage states and tapes must
agree on the first copy, at grids around the workgroup sizes, with each option, and with
steps that are clipped, skipped, fixed and replayed.  And what a caller may rely on around
it: results that do not depend on the stage timer, and capture.

Bounds: both paths apply the same formulas, so only the compiler's choice of fused
operations (and, unfolded, the order of the two sides of an interface) can differ, a few
ulps of a field's scale per step, which the limiter's switches may amplify about
tenfold over five steps: 1e-13 in FP64, 5e-5 in FP32."""
import pytest
import torch

import hweno_inputs as hi
import paper_2207_05258_amd as h

pytestmark = pytest.mark.gpu

C = h.hweno.CTRL_LEN
TOL = {torch.float64: 1e-13, torch.float32: 5e-5}
LAUNCHED = {"euler": 512, "linadv": 1024, "burgers": 1024}   # cells from which steps are launches


def _setup(physics, n, dtype, **kw):
    w = hi.euler1d_piecewise(n, 3) if physics == "euler" else hi.scalar_random_1d(n, 3, physics)
    kw.setdefault("bc_x", h.REFLECT if physics == "euler" and n >= 2 else h.PERIODIC)
    S = torch.as_tensor(w.S).to(dtype).cuda().contiguous()
    return S, h.Problem(dim=1, nx=n, physics=physics, dtype=dtype, dx=w.dx, **kw)


def _large(S, prob):
    """The same cells as the head of a periodic grid of launches."""
    m = prob.m
    if prob.bc_x == h.REFLECT:
        M = S.flip(-1).clone()
        M[1] *= -1.0            # momentum is odd, and so are derivatives of what is even
        M[m:] *= -1.0
        M[m + 1] *= -1.0
        S = torch.cat([S, M], -1)
    times = -(-LAUNCHED[prob.physics] // S.shape[-1])
    S = S.repeat(1, 1, times).contiguous()
    q = h.Problem(**{**prob.__dict__, "nx": S.shape[-1], "bc_x": h.PERIODIC})
    return S, q


def _run(S, prob, call, n):
    X, st = S.clone(), h.Stepper(prob)
    tapes = torch.zeros(8, C, dtype=torch.float64, device="cuda")
    call(st, X, tapes)
    nb = X.numel() * X.element_size()
    o = 256 + (nb + 255) // 256 * 256
    stages = [st.ws[a:a + nb].view(X.dtype).view(X.shape)[..., :n].clone() for a in (256, o)]
    return X[..., :n].clone(), st.ctrl.clone(), tapes, stages


def _check(S, prob, call):
    n, tol = prob.nx, TOL[prob.dtype]
    a = _run(S, prob, call, n)
    b = _run(*_large(S, prob), call, n)
    for x, y in [(a[0], b[0])] + list(zip(a[3], b[3])):
        for f in range(prob.nf):
            scale = max(float(y[f].abs().max()), float(y[f % prob.m].abs().max()))
            assert float((x[f] - y[f]).abs().max()) <= tol * scale, f
    for x, y in ((a[1], b[1]), (a[2], b[2])):
        x, y = x.reshape(-1, C), y.reshape(-1, C)
        assert torch.equal(x[:, 8].contiguous().view(torch.int64), y[:, 8].contiguous().view(torch.int64))
        assert torch.equal(x[:, 9], y[:, 9])
        assert torch.allclose(x[:, [*range(8), 10, 11]], y[:, [*range(8), 10, 11]], rtol=tol, atol=0.0)
    return a


SIZES = {"euler": [1, 2, 3, 64, 255, 256, 511], "linadv": [1, 2, 255, 256, 1023], "burgers": [4, 255, 1023]}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("physics,n", [(p, n) for p, ns in SIZES.items() for n in ns])
def test_one_launch_matches_launched_stages(physics, n, dtype):
    S, prob = _setup(physics, n, dtype)
    _check(S, prob, lambda st, X, tp: st.steps(X, 5, tapes=tp))


OPTIONS = [dict(limiter_on=False), dict(limiter_characteristic=True), dict(characteristic=False),
           dict(characteristic=False, limiter_characteristic=True), dict(bc_x=h.PERIODIC)]


@pytest.mark.parametrize("kw", OPTIONS, ids=[",".join(f"{k}={v}" for k, v in o.items()) for o in OPTIONS])
def test_options_in_one_launch(kw):
    _check(*_setup("euler", 130, torch.float64, **kw), lambda st, X, tp: st.steps(X, 4, tapes=tp))


def test_clipped_skipped_fixed_and_replayed_steps():
    S, prob = _setup("euler", 100, torch.float64)
    _check(S, prob, lambda st, X, tp: st.steps(X, 8, dt=2e-4, t_end=9e-4, tapes=tp))

    def single(st, X, tp):
        for q in range(3):
            st.step(X, t_end=1e-3, tape=tp[q])

    taped = _check(S, prob, single)

    def replay(st, X, tp):
        for q in range(3):
            st.step(X, replay=taped[2][q], tape=tp[q])

    assert torch.equal(_check(S, prob, replay)[0], taped[0])


def test_the_stage_timer_changes_no_result():
    S, prob = _setup("euler", 100, torch.float64)
    for n, launches in ((5, 1), (300, 2)):       # at most 256 steps a launch
        out = []
        for timed in (False, True):
            X, st = S.clone(), h.Stepper(prob)
            if timed:
                h.timing_begin()
            st.steps(X, n)
            if timed:
                assert h.timing_end()[0] == launches
            out.append((X, st.ctrl[:10].clone(), st.ws[256:].clone()))
        for a, b in list(zip(*out))[:2]:
            assert torch.equal(a, b)
    X, st = S.clone(), h.Stepper(prob)
    Y, ctrl = S.clone(), torch.zeros(C, dtype=torch.float64, device="cuda")
    h.timing_begin()
    st.step(X)
    h.rk3_step_static(Y, prob, ctrl)
    h.timing_end()
    assert torch.equal(X, Y) and torch.equal(st.ctrl[:10], ctrl[:10])


@pytest.mark.parametrize("call", ["step", "steps", "static"])
def test_one_launch_under_capture(call):
    """Replays with eager work on the same kernels and a synchronisation between them."""
    S, prob = _setup("euler", 100, torch.float64)
    X, st = S.clone(), h.Stepper(prob)
    E, se = S.clone(), h.Stepper(prob)

    def advance(state, stepper):
        if call == "step":
            for _ in range(3):
                stepper.step(state)
        elif call == "steps":
            stepper.steps(state, 3)
        else:
            h.rk3_step_static(state, prob, stepper.ctrl)

    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            advance(X, st)
    torch.cuda.current_stream().wait_stream(s)
    assert torch.equal(X, S)                    # nothing ran yet
    for _ in range(4):
        g.replay()
        torch.cuda.synchronize()
        advance(E, se)
        torch.cuda.synchronize()
        assert torch.equal(X, E) and torch.equal(st.ctrl[:10], se.ctrl[:10])
