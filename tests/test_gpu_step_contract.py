"""What hweno.h promises of a step on every path that takes it: grids that one workgroup
holds (1D), grids by launches of each way of reading the speeds (1D, 2D, edge-described
sides), the static step and batched grids."""
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
