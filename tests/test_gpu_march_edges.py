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


def _box(n, bc, seed, **kw):
    nd = len(n)
    prob = W.uniform_problem(nd, list(n), [0.0] * nd, [1.0] * nd, bc, **kw)
    return prob, W.random_field(prob, seed=seed)


@pytest.mark.parametrize("shape", [(61, 100003), (12, 160003, 5), (12, 5, 160003)])
def test_narrow_march_equals_oracle(orc, shape):
    # as few columns as the march takes: the last lanes of its one wave a row
    # repeat the last column
    torch, B = _gpu()
    prob, U = _box(shape, "periodic", 11)
    S = B.Solver(prob)
    R = S.rhs(torch.from_numpy(U).cuda())
    assert np.array_equal(R.cpu().numpy(), orc.rhs(prob, U))


@pytest.mark.parametrize("n,bc,kw", [
    ((61, 100003), "transmissive", dict(theta="cut")),
    ((62, 100005), ["reflective", "periodic"], dict(scheme="fixed_ct", ct_fixed=1e-5)),
    ((1281, 4801), ["periodic", "reflective"], dict()),
    ((1100, 5600), "periodic", dict(scheme="teno5a")),
    ((1300, 4800), "transmissive", dict(scheme="linear5"))])
def test_march_equals_face_stream(n, bc, kw):
    # right-hand side and two steps
    torch, B = _gpu()
    prob, U = _box(n, bc, 21, **kw)
    Ud = torch.from_numpy(U).cuda()
    S, D = B.Solver(prob), B.Solver(prob)
    D.g.flags |= B.FLAG_MASK_DIGEST
    R = S.rhs(Ud)
    Rd, _ = D.rhs(Ud, decisions=True)
    assert torch.equal(R, Rd)
    Ua, Ub = Ud.clone(), Ud
    for s, u in ((S, Ua), (D, Ub)):
        s.init(0.0, float("inf"), 0.4)
        for _ in range(2):
            s.step(u)
    torch.cuda.synchronize()
    ca, cb = S.read_ctrl(), D.read_ctrl()
    assert ca.status == 0 and ca.nsteps == 2
    assert (ca.t, ca.dt) == (cb.t, cb.dt) and torch.equal(Ua, Ub)


@pytest.mark.parametrize("n", [(62, 101000), (12, 160003, 5)])
def test_march_in_place_keeps_zero_signs(n):
    torch, B = _gpu()
    prob, _ = _box(n, "periodic", 12)
    U = torch.ones((len(n) + 2, *([1] * (3 - len(n))), *n[::-1]), dtype=torch.float64, device="cuda")
    U[-1] = 9.0
    g = B.Solver(prob).g
    alpha = torch.full((4,), 3.0, dtype=torch.float64, device="cuda")
    Rin = torch.where(torch.arange(U.numel(), device="cuda") % 3 == 0, -0.0, 0.0).double().view(U.shape)
    out = torch.empty_like(Rin)
    B.teno_sweep(g, 1, U, out, alpha, Rin=Rin)
    B.teno_sweep(g, 1, U, Rin, alpha, Rin=Rin)
    assert torch.equal(out.view(torch.int64), Rin.view(torch.int64))
