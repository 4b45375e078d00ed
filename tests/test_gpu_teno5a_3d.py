"""TENO5-A where its kernels are the largest: lines of 252 cells and more (the x
sweep that stages four chunks of a line at once), marched 3D grids, and the 3D
adjoint's fixed-stride chunks (lines of 63 cells and more)."""
import numpy as np
import pytest

from paper_2003_09145_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_09145_amd import binding
    return binding


def _box(n, bc, seed):
    nd = len(n)
    prob = W.uniform_problem(nd, list(n), [0.0] * nd, [1.0] * nd, bc, scheme="teno5a")
    return prob, W.random_field(prob, seed=seed)


@pytest.mark.parametrize("n,bc", [
    ((252, 9, 8), ["periodic", "reflective", "transmissive"]), ((253, 20, 24), "reflective"),
    ((300, 80, 70), ["transmissive", "periodic", "periodic"]), ((256, 66, 64), "periodic"),
    ((252, 33), "transmissive"), ((515, 1100), ["reflective", "periodic"])],
    ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_long_lines_equal_oracle(B, orc, n, bc):
    import torch
    prob, U = _box(n, bc, 41)
    S = B.Solver(prob)
    Ud = torch.from_numpy(U).cuda()
    assert np.array_equal(S.rhs(Ud).cpu().numpy(), orc.rhs(prob, U))
    S.init(0.0, 1e9, 0.4)
    t, Uc = 0.0, U
    for _ in range(2):
        S.step(Ud)
        Uc, t, dt, a9, st = orc.step(prob, Uc, 0.4, t, 1e9)
        assert st == 0
    torch.cuda.synchronize()
    c = S.read_ctrl()
    assert (c.status, c.nsteps, c.t, c.dt) == (0, 2, t, dt) and np.array_equal(Ud.cpu().numpy(), Uc)


def test_marched_long_lines_equal_oracle(B, orc):
    import torch
    prob, U = _box((256, 256, 160), "periodic", 42)
    S = B.Solver(prob)
    Ud = torch.from_numpy(U).cuda()
    S.init(0.0, 1e9, 0.4)
    S.step(Ud)
    Uc, t, dt, a9, st = orc.step(prob, U, 0.4, 0.0, 1e9)
    torch.cuda.synchronize()
    c = S.read_ctrl()
    assert st == 0 and (c.status, c.t, c.dt) == (0, t, dt) and np.array_equal(Ud.cpu().numpy(), Uc)


@pytest.mark.parametrize("n,bc", [
    ((70, 66, 9), ["periodic", "reflective", "transmissive"]),
    ((9, 5, 131), ["reflective", "transmissive", "periodic"]),
    ((64, 65, 66), "periodic")], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_adjoint_dot_product(B, orc, n, bc):
    import torch
    prob, U = _box(n, bc, 43)
    a, _ = orc.alpha(prob, U)
    g = B.grid(prob)
    ws = torch.empty(B.adjoint_workspace_bytes(g), dtype=torch.uint8, device="cuda")
    rng = np.random.default_rng(6)
    lam = rng.normal(size=U.shape)
    v = rng.normal(size=U.shape) * np.abs(U)
    Ud, ad, ld = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (U, a, lam))
    out = torch.empty_like(Ud)
    B.teno_rhs_adjoint(g, Ud, ad, ld, out, ws)
    torch.cuda.synchronize()
    _, jv = orc.rhs_jvp(prob, U, v, a)
    lhs, rhs = float(np.sum(lam * jv)), float(np.sum(out.cpu().numpy() * v))
    assert abs(lhs - rhs) <= 1e-12 * float(np.sum(np.abs(lam * jv)))
