"""The adjoint of the linear derivative fluxes alone: linear advection whose speed is far
below the splitting speed (2^-10 and 1), with an adjoint on the derivative rows only, in
FP32 against FP64.

The adjoint of U is a multiple of 2^-10 of 15 (p2 - p1) + p0 - p3 plus (p0 + p3) - (p1 +
p2), p_s the adjoint of the interface at which the cell is point s.  Cell sizes of one
and integer adjoints below 2^22 make the p_s exact, integers below 2^23 (times 1/8), and
their pairwise sums too, so what may round are the difference of the sums and the result
(one unit each, values up to 2^25) and the first term (2^-10 of 16 units): less than three
units a direction, and one more for each further addition to the cell.  Passed through
sums that hold 15 (p2 - p1) first, the difference alone would round by up to 16 units."""
import pytest
import torch

import paper_2207_05258_amd as h

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,units", [(1, 4), (2, 8)])
def test_linear_flux_adjoint_keeps_the_splitting_speed_exact(dim, units):
    nx, ny = (1000, 1) if dim == 1 else (70, 61)
    g = torch.Generator().manual_seed(11)
    S = torch.rand(1 + dim, ny, nx, generator=g).cuda()
    lam = torch.randint(-2 ** 22, 2 ** 22, (1 + dim, ny, nx), generator=g).float()
    lam[0] = 0.0
    lam = lam.cuda()
    out = []
    for dtype in (torch.float32, torch.float64):
        prob = h.Problem(dim=dim, nx=nx, ny=ny, physics="linadv", dtype=dtype, dx=1.0, dy=1.0,
                         adv_speed=(2.0 ** -10, 2.0 ** -10))
        out.append(h.rhs_adjoint(S.to(dtype).contiguous(), prob, [1.0, 1.0 if dim == 2 else 0.0],
                                 lam.to(dtype).contiguous()).double())
    err = float((out[0][0] - out[1][0]).abs().max()) * 8     # in units: the p_s carry 1/8
    print("largest error in units: %.2f" % err)
    assert float(out[1][0].abs().max()) > 2 ** 20 and err <= units
