"""The global speeds of a step's stages are folded by the workgroups into slots and read
back in three ways, by the number of workgroups (16 x 15 tiles in 2D): slot 0 alone up
to 48, all slots by lanes up to 512 (FP64) or 1024 (FP32), by scalar loads above.  At both
sides of every line the speeds that a step records must be exactly those that
hweno_alpha finds in the states it was taken from: maxima of the same values, which no
order of reduction changes.  A NaN must reach the time step in each way."""
import pytest
import torch

import hweno_inputs as hi
import paper_2207_05258_amd as h

pytestmark = pytest.mark.gpu

WORKGROUPS = [1, 48, 49, 512, 513, 1024, 1025]
TILES = {1: (1, 1), 48: (8, 6), 49: (7, 7), 512: (16, 32), 513: (27, 19), 1024: (32, 32),
         1025: (41, 25)}


def _grid(n):
    tx, ty = TILES[n]
    return 16 * tx - (tx > 1), 15 * ty - 3 * (ty > 1)   # ragged last tiles


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("n", WORKGROUPS)
def test_recorded_speeds_are_those_of_the_states(n, dtype):
    nx, ny = _grid(n)
    w = hi.euler2d_random_smooth(nx, ny, 5)
    S = torch.as_tensor(w.S).to(dtype).cuda().contiguous()
    prob = h.Problem(dim=2, nx=nx, ny=ny, physics="euler", dtype=dtype, dx=w.dx, dy=w.dy)
    st = h.Stepper(prob)
    tapes = torch.zeros(3, h.hweno.CTRL_LEN, dtype=torch.float64, device="cuda")
    states = [S.clone()]
    for k in (1, 1):
        X = states[-1].clone()
        st.steps(X, k)
        states.append(X)
    A, last = states[0].clone(), h.Stepper(prob)
    last.steps(A, 3, tapes=tapes)
    nb = S.numel() * S.element_size()
    o = 256 + (nb + 255) // 256 * 256
    stage = [last.ws[a:a + nb].view(dtype).view(S.shape) for a in (256, o)]  # of the third step
    for k, X in enumerate(states):
        assert torch.equal(tapes[k][:2], h.alpha(X, prob)), k
    assert torch.equal(tapes[2][2:4], h.alpha(stage[0].contiguous(), prob))
    assert torch.equal(tapes[2][4:6], h.alpha(stage[1].contiguous(), prob))
    assert torch.equal(last.ctrl[:6], tapes[2][:6])


@pytest.mark.parametrize("n", [1, 49, 513])
def test_nan_reaches_the_time_step(n):
    nx, ny = _grid(n)
    w = hi.euler2d_random_smooth(nx, ny, 5)
    S = torch.as_tensor(w.S).cuda().contiguous()
    S[3, ny - 1, nx - 1] = float("nan")     # the last workgroup's cell
    prob = h.Problem(dim=2, nx=nx, ny=ny, physics="euler", dtype=torch.float64, dx=w.dx, dy=w.dy)
    st, before = h.Stepper(prob), S.clone()
    st.steps(S, 2)
    assert st.status & h.hweno.ST_SKIPPED and st.last_dt == 0.0
    assert torch.equal(torch.nan_to_num(S), torch.nan_to_num(before))
    assert torch.isnan(st.ctrl[:2]).any()
