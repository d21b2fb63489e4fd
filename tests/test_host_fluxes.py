"""What the kernels run around one interface (interface_fluxes and side_vjp, built for the
host by tests/host/flux_host.cpp) against the oracle's interface fluxes: f-hat (Section 2.1
with Remarks 2.1/2.2), the linear derivative flux h-hat and the mixed flux, and the
adjoint of f-hat against torch autograd through the oracle.

Bounds.  The point data carry |F| + alpha |U| + h (|A Dn| + alpha |Dn|); f-hat passes
through the eigenvectors, whose condition number multiplies its rounding.  A few dozen
roundings: 1e-13 in FP64, 5e-6 in FP32 (2e-11 for the oracle's gradients, which invert the
eigenvectors numerically)."""
import hashlib
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import hweno_ref as o

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"
SRC = ["tests/host/flux_host.cpp", "paper_2207_05258_amd/csrc/hweno_math.h",
       "paper_2207_05258_amd/csrc/hweno_adjoint.h"]
LIN = (0.98, 0.01, 0.01)
EPS, GAMMA = 1e-6, 1.4
U24 = 2.0 ** -24     # unit roundoff of FP32


def _exe():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    h = hashlib.sha256()
    for s in SRC:
        with open(os.path.join(ROOT, s), "rb") as fh:
            h.update(fh.read())
    out = os.path.join("/tmp", "hweno_flux_host", h.hexdigest()[:16])
    exe = os.path.join(out, "flux_host")
    if not os.path.exists(exe):
        os.makedirs(out, exist_ok=True)
        cmd = [HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               os.path.join(ROOT, SRC[0]), "-o", exe + ".tmp"]
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stderr[-3000:]
        os.replace(exe + ".tmp", exe)
    return exe


def _run(op, prec, rows, lin=LIN, eps=EPS):
    args = [_exe()] + [repr(x) for x in lin] + [repr(eps), repr(GAMMA)]
    text = "".join(f"{op} {prec} " + " ".join(repr(float(x)) for x in r) + "\n" for r in rows)
    r = subprocess.run(args, input=text, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    out = np.array([[float(x) for x in ln.split()] for ln in r.stdout.splitlines()])
    assert out.shape[0] == len(rows)
    return out


H = 1.0 / 64.0


def _euler_rows(seed, n=800):
    """[n, 2 + 48]: (an, alpha), then four points of (U, H Dn, H Dt): one admissible
    state per row and neighbours close to it, or independent states in a third of
    the rows; speeds up to twice the stencil's own."""
    g = np.random.default_rng(seed)

    def states(k):
        rho, p = 10.0 ** g.uniform(-1, 1, k), 10.0 ** g.uniform(-1, 1.5, k)
        c = np.sqrt(GAMMA * p / rho)
        u, v = g.uniform(-2, 2, k) * c, g.uniform(-2, 2, k) * c
        return np.stack([rho, rho * u, rho * v, p / (GAMMA - 1) + 0.5 * rho * (u * u + v * v)], 1)
    U = np.stack([states(n) for _ in range(4)], 1)
    near = g.random(n) < 2 / 3
    U[near] = U[near][:, :1] * (1 + 0.02 * g.uniform(-1, 1, (int(near.sum()), 4, 1)))
    D = 0.1 * g.standard_normal((n, 4, 8)) * np.abs(U).max((1, 2), keepdims=True)
    pr = (GAMMA - 1) * (U[..., 3] - 0.5 * (U[..., 1] ** 2 + U[..., 2] ** 2) / U[..., 0])
    s = (np.abs(U[..., 1] / U[..., 0]) + np.sqrt(GAMMA * pr / U[..., 0])).max(1)
    al = s * g.uniform(1, 2, n)
    return np.concatenate([np.zeros((n, 1)), al[:, None], np.concatenate([U, D], 2).reshape(n, 48)], 1)


def _oracle(rows, char, X=None):
    """fh, hh, xx in the units of interface_fluxes (2 f-hat, 8 H h-hat, 12 H times the
    mixed flux) of the middle interface of one periodic 4-cell row per stencil."""
    prob = o.Problem(dim=2, physics="euler", dx=H, dy=H, lin_w=LIN, eps=EPS, gamma_gas=GAMMA,
                     characteristic=char)
    P = torch.as_tensor(rows[:, 2:50], dtype=torch.float64).view(-1, 4, 12) if X is None else X
    out = []
    for q in range(len(rows)):       # a speed of its own per row
        S = P[q].T.reshape(12, 1, 4)
        f, hh, xx = o._direction_fluxes(S[:4], S[4:8] / H, S[8:] / H, prob, 0, float(rows[q, 1]))
        out.append(torch.cat([2 * f[:, 0, 2], 8 * H * hh[:, 0, 2], 12 * H * xx[:, 0, 2]]))
    return torch.stack(out)


def _scale(rows):
    """(size of the point data, condition number of the interface's eigenvectors)."""
    P = torch.as_tensor(rows[:, 2:50]).view(-1, 4, 12)
    eu = o.Euler(o.Problem(dim=2, physics="euler", gamma_gas=GAMMA))
    al = torch.as_tensor(rows[:, 1]).view(-1, 1, 1)
    F, A, B = eu.flux(P[..., :4], 0), eu.jvp(P[..., :4], P[..., 4:8], 0), eu.jvp(P[..., :4], P[..., 8:], 0)
    size = (F.abs() + al * P[..., :4].abs() + A.abs() + al * P[..., 4:8].abs() + B.abs()).amax((1, 2))
    cond = torch.linalg.cond(eu.right_eigenvectors(P[:, 1, :4], P[:, 2, :4], 0))
    return size.numpy(), cond.numpy()


@pytest.mark.parametrize("char", [True, False])
@pytest.mark.parametrize("prec,tol", [("d", 1e-13), ("f", 5e-6)])
def test_interface_fluxes_match_the_oracle(prec, tol, char):
    rows = _euler_rows(5)
    if prec == "f":
        rows = rows.astype(np.float32).astype(np.float64)
    got = _run("p" if char else "c", prec, rows)
    ref = _oracle(rows, char).numpy()
    size, cond = _scale(rows)
    err = np.abs(got - ref)
    assert (err[:, :4] / (size * (cond if char else 1.0))[:, None]).max() <= tol
    assert (err[:, 4:] / size[:, None]).max() <= 20 * tol     # weights up to 15


@pytest.mark.parametrize("char", [True, False])
def test_nonlinear_flux_adjoint_matches_autograd(char):
    rows = _euler_rows(6, 300)
    gf = np.random.default_rng(7).standard_normal((len(rows), 4))
    got = _run("P" if char else "C", "d", np.concatenate([rows, gf], 1)).reshape(-1, 4, 8)
    X = torch.as_tensor(rows[:, 2:50], dtype=torch.float64).view(-1, 4, 12).clone().requires_grad_(True)
    (_oracle(rows, char, X)[:, :4] * torch.as_tensor(gf)).sum().backward()
    ref = X.grad[..., :8].numpy()
    _, cond = _scale(rows)
    err = np.abs(got - ref) / (np.abs(ref).max((1, 2), keepdims=True) * (cond if char else np.ones_like(cond))[:, None, None])
    assert err.max() <= 2e-11, (err.max(), np.unravel_index(err.argmax(), err.shape))


def test_linear_flux_keeps_the_splitting_speed_out_of_its_rounding():
    """h-hat of linear advection with a = 2^-10 split with a speed of one, on values within
    a hundredth of one: exactly F0 - 15 F1 + 15 F2 - F3 + alpha (U0 - U1 - U2 + U3) plus
    derivative terms, which are zero here.  Each of the four outer terms may round alpha U once
    on either side of the interface (x+_0, x+_1, x-_2, x-_3): 4 u, and the small differences
    and the fluxes (14 (F2 - F1): 28 u a) add less than one more.  Weights of 7 on F +- alpha U
    would allow 32 u."""
    g = np.random.default_rng(3)
    n = 4000
    U = (1 + 0.01 * g.uniform(-1, 1, (n, 4))).astype(np.float32).astype(np.float64)
    a = 2.0 ** -10
    rows = np.zeros((n, 14))
    rows[:, 0], rows[:, 1] = a, 1.0
    rows[:, 2::3] = U
    got = _run("a", "f", rows)[:, 1]
    ref = a * (U @ [1.0, -15.0, 15.0, -1.0]) + U @ [1.0, -1.0, -1.0, 1.0]
    err = np.abs(got - ref)
    print("h-hat error in u: max %.2f, rms %.2f" % (err.max() / U24, np.sqrt((err ** 2).mean()) / U24))
    assert err.max() <= 5 * U24 * np.abs(U).max()
