"""The marching sweep where a segment begins, against the face-stream sweep, bit
for bit (the decision dump and the mask digest keep the face-stream sweep)."""
import numpy as np
import pytest

from paper_2003_09145_amd import workloads as W

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_09145_amd import binding
    return torch, binding


def _same(torch, a, b):
    return bool(torch.equal(a.isnan(), b.isnan())) and \
        bool(torch.equal(a.nan_to_num(0.0, float("inf"), -float("inf")),
                         b.nan_to_num(0.0, float("inf"), -float("inf"))))


def test_overflowing_flux_at_the_first_row():
    # Energy fluxes near the largest double in steps of three rows: with frozen
    # speeds 0 the linear scheme's overshoot is infinite at every sixth face, the
    # first face of segments among them; the row behind such a face is updated in
    # place and comes out infinite where the face-stream sweep says so, not NaN.
    torch, B = _gpu()
    nx, ny = 128, 51000
    prob = W.uniform_problem(2, [nx, ny], [0.0, 0.0], [nx, ny], "periodic", scheme="linear5")
    rho = 1e-10 * np.where((np.arange(ny) // 3) % 2 == 0, 1.0, 0.5)[:, None] * np.ones((ny, nx))
    u = np.full((ny, nx), 1e106 * (1.7 / 0.57) ** (1 / 3) * (0.9 + 0.005 * 22))
    U = W.conserved(rho, [0.0 * u, u], rho * u * u / 50, 1.4).reshape(4, 1, ny, nx)
    Ud = torch.from_numpy(U).cuda()
    S = B.Solver(prob)
    alpha = torch.zeros(3, dtype=torch.float64, device="cuda")
    R = S.rhs(Ud, alpha_in=alpha)
    Rd, _ = S.rhs(Ud, alpha_in=alpha, decisions=True)
    assert int(Rd[3].isinf().sum()) > ny and not bool(Rd[:3].isinf().any())
    assert _same(torch, R, Rd)
