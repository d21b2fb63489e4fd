"""What hweno.h promises of a step on every path that takes it: grids that one workgroup
holds (1D), grids by launches of each way of reading the speeds (1D, 2D, edge-described
sides), the static step and batched grids."""
import dataclasses

import pytest
import torch

import hweno_inputs as hi
import paper_2207_05258_amd as h

pytestmark = pytest.mark.gpu

ST = h.hweno


def _grid(kind, dtype=torch.float64):
    """(state, problem) of one path."""
    if kind.startswith("1d"):
        n = int(kind[2:])
        w = hi.euler1d_piecewise(n, 3)
        S = torch.as_tensor(w.S).to(dtype).cuda().contiguous()
        return S, h.Problem(dim=1, nx=n, physics="euler", dtype=dtype, dx=w.dx, bc_x=h.REFLECT)
    nx, ny = {"2d_few": (33, 31), "2d_lanes": (130, 107), "2d_scalar": (430, 300), "edges": (65, 40)}[kind]
    w = hi.euler2d_random_smooth(nx, ny, 5)
    S = torch.as_tensor(w.S).to(dtype).cuda().contiguous()
    kw = {}
    if kind == "edges":
        kw = dict(bc_x=h.EDGES, bc_y=h.EDGES, edges=[h.Edge() for _ in range(4)])
    return S, h.Problem(dim=2, nx=nx, ny=ny, physics="euler", dtype=dtype, dx=w.dx, dy=w.dy, **kw)


GRIDS = ["1d100", "1d300", "1d700", "2d_few", "2d_lanes", "2d_scalar", "edges"]


# ---- a step whose time step is not finite is skipped, also when t_end clips it ----
def _poison(S):
    S[0, S.shape[1] // 2, S.shape[2] // 2] = float("nan")
    return S


def _assert_skipped(ctrl, S, before, t0, n):
    assert int(ctrl[8:9].view(torch.int64)) & ST.ST_SKIPPED, n
    assert float(ctrl[6]) == 0.0 and float(ctrl[7]) == t0 and float(ctrl[9]) == 0.0, n
    assert torch.equal(torch.nan_to_num(S), torch.nan_to_num(before)), n


@pytest.mark.parametrize("call", ["step", "steps", "static"])
@pytest.mark.parametrize("kind", GRIDS)
def test_nan_speed_skips_a_step_clipped_to_t_end(kind, call):
    S, prob = _grid(kind)
    _poison(S)
    before, st = S.clone(), h.Stepper(prob, t0=0.25)
    if call == "step":
        st.step(S, t_end=0.5)
    elif call == "steps":
        st.steps(S, 3, t_end=0.5)
    else:
        h.rk3_step_static(S, prob, st.ctrl, t_end=0.5)
    _assert_skipped(st.ctrl, S, before, 0.25, kind)


@pytest.mark.parametrize("blocks", [0, 5])
def test_nan_speed_skips_a_batched_step_clipped_to_t_end(blocks):
    ws = hi.batched_instances(3, 3, sizes=[(37, 29), (16, 15), (64, 7)])
    states = [torch.as_tensor(w.S).cuda().contiguous() for w in ws]
    _poison(states[1])
    before = [S.clone() for S in states]
    grids = [dict(dx=w.dx, dy=w.dy, bc_x=w.bc_x, bc_y=w.bc_y, t_end=0.5) for w in ws]
    b = h.BatchedStepper(states, grids, h.Problem(dim=2, nx=1, ny=1, physics="euler", dtype=torch.float64))
    b.step(blocks=blocks)
    _assert_skipped(b.ctrl(1), states[1], before[1], 0.0, blocks)
    for q in (0, 2):    # the others are stepped
        assert float(b.ctrl(q)[6]) > 0.0 and not torch.equal(states[q], before[q])


# ---- cell sizes whose square leaves the range of the type ----
# Lengths of 2^69 and 2^-67 around one, with fields of 2^16 and 2^-16 (in FP32 the square
# of an indicator leaves the range near 2^20): 1 / dx^2 is 2^-138
# and 2^134 in FP32 (11 bits of it and none), while the fields and the operator stay
# normal.  Against the same call in FP64, in the norms of one step in FP32 (1e-5 of the
# size of U; derivatives times their cell size; rates in units of speed over cell size).
SCALES = [(69, 16), (-67, -16)]


def _scaled_grid(dim, k, j):
    w = hi.euler1d_piecewise(64, 3) if dim == 1 else hi.roughened(hi.euler2d_random_smooth(40, 33, 5), 7)
    m, S = dim + 2, torch.as_tensor(w.S).clone()
    if dim == 1:
        S[m:] += 0.05 / w.dx * (2 * torch.rand(S[m:].shape, generator=torch.Generator().manual_seed(7), dtype=S.dtype) - 1)
    for d, (old, new) in enumerate(((w.dx, 1.3), (w.dy, 1.4))[:dim]):
        S[m * (1 + d):m * (2 + d)] *= old / new * 2.0 ** -k
    S = (S * 2.0 ** j).float().cuda().contiguous()
    n = dict(dim=1, nx=64) if dim == 1 else dict(dim=2, nx=40, ny=33)
    return S, h.Problem(physics="euler", dtype=torch.float32, dx=1.3 * 2.0 ** k, dy=1.4 * 2.0 ** k,
                        eps=1e-6 * 2.0 ** (2 * j), bc_x=w.bc_x, bc_y=w.bc_y, **n)


@pytest.mark.parametrize("k,j", SCALES)
@pytest.mark.parametrize("dim", [1, 2])
def test_operator_and_step_at_extreme_cell_sizes(dim, k, j):
    S, prob = _scaled_grid(dim, k, j)
    X, q = S.double(), dataclasses.replace(prob, dtype=torch.float64)
    m, size = prob.m, float(X[:prob.m].abs().max())
    unit = [1.0] * m + [prob.dx] * m + [prob.dy] * m    # of U over each field
    speed = float(h.alpha(X, q).max())
    rate = h.rhs(S, prob).double(), h.rhs(X, q)
    A, B = S.clone(), X.clone()
    h.Stepper(prob).step(A)
    h.Stepper(q).step(B)
    for f in range(prob.nf):
        for name, (a, b), s in (("rhs", rate, min(prob.dx, prob.dy) / speed), ("step", (A.double(), B), 1.0)):
            assert torch.isfinite(a[f]).all(), (name, f)
            err = float((a[f] - b[f]).abs().max()) * unit[f] * s
            assert err <= 1e-5 * size, (name, f, err / size)


# ---- a workspace that ends before the 1 KiB of partial speeds is taken, exactly to its end ----
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("kind", GRIDS)
def test_workspace_without_partial_speeds(kind, dtype):
    S, prob = _grid(kind, dtype)
    need = h.workspace_bytes(prob) - 1024
    out = []
    for short in (False, True):
        X, tapes = S.clone(), torch.zeros(4, h.hweno.CTRL_LEN, dtype=torch.float64, device="cuda")
        raw = torch.full((need + 1024 + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        ws = raw[(-raw.data_ptr()) % 256:]
        ws[:h.hweno.CTRL_LEN * 8] = 0
        st = h.Stepper._over(prob, prob.c(), ws, need if short else need + 1024)
        st.step(X, tape=tapes[0])
        st.steps(X, 2, tapes=tapes[1:3])
        st.step(X, dt=1e-5, tape=tapes[3])
        if short:
            assert bool((ws[need:] == 0xA5).all())     # nothing was written past its end
        out.append((X, tapes[:, :10], st.ctrl[:12].clone(), ws[256:need].clone()))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    with pytest.raises(h.HwenoError, match="workspace too small"):
        h.Stepper._over(prob, prob.c(), ws, need - 1).step(S.clone())


def test_batched_workspaces_hold_no_partial_speeds():
    ws = hi.batched_instances(2, 3, sizes=[(37, 29), (64, 7)])
    states = [torch.as_tensor(w.S).cuda().contiguous() for w in ws]
    b = h.BatchedStepper(states, [dict(dx=w.dx, dy=w.dy) for w in ws],
                         h.Problem(dim=2, nx=1, ny=1, physics="euler", dtype=torch.float64))
    for q, w in enumerate(ws):
        prob = h.Problem(dim=2, nx=w.nx, ny=w.ny, physics="euler", dtype=torch.float64, dx=w.dx, dy=w.dy)
        assert int(b._host[q].ws_bytes) == h.workspace_bytes(prob) - 1024


# ---- the smallest normal epsilon of each type ----
@pytest.mark.parametrize("dim", [1, 2])
def test_smallest_normal_epsilon_in_fp32(dim):
    """A constant state has no rate of change with any positive epsilon: all indicators are
    epsilon, whose reciprocal is finite down to the smallest normal number."""
    m = dim + 2
    S = torch.zeros(m * (1 + dim), 33 if dim == 2 else 1, 40, device="cuda")
    S[0], S[1], S[m - 1] = 1.0, 0.5, 2.5
    prob = h.Problem(dim=dim, nx=40, ny=S.shape[1], physics="euler", dtype=torch.float32, dx=0.1, dy=0.1,
                     eps=float(torch.finfo(torch.float32).tiny))
    X = S.clone()
    assert torch.equal(h.rhs(S, prob), torch.zeros_like(S))
    h.Stepper(prob).step(X)
    assert torch.isfinite(X).all() and float((X - S).abs().max()) <= 1e-6


# ---- FP32: a step whose operator is zero leaves the conserved fields as they are ----
@pytest.mark.parametrize("dim,n", [(1, 300), (1, 1500), (2, 40)])
def test_fp32_step_without_rates_keeps_every_bit(dim, n):
    """Linear advection at rest: no flux, no splitting speed, so each stage combines a value
    with itself, which the difference form returns exactly (3/4 and 1/3 of it rounded first
    do not)."""
    g = torch.Generator().manual_seed(2)
    ny = 33 if dim == 2 else 1
    S = (torch.rand(1 + dim, ny, n, generator=g) + 0.5).cuda()
    prob = h.Problem(dim=dim, nx=n, ny=ny, physics="linadv", dtype=torch.float32, dx=0.1, dy=0.1,
                     adv_speed=(0.0, 0.0))
    X = S.clone()
    h.Stepper(prob).steps(X, 4, dt=0.05)
    assert torch.equal(X[0], S[0]) and torch.isfinite(X).all()
