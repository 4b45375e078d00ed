"""Per-end boundaries, splits that move in time and gravity on the routes of a step
that apply them themselves, bit for bit against the oracle: 1D (the short-line
kernel and the sweeps above its size) and the 3D march."""
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


def _steps_equal_oracle(B, orc, prob, U, cfl, steps, t0=0.0):
    import torch
    S = B.Solver(prob)
    Ud = torch.from_numpy(U).cuda()
    assert np.array_equal(S.rhs(Ud).cpu().numpy(), orc.rhs(prob, U))
    S.init(t0, 1e9, cfl)
    t, Uc = t0, U
    for _ in range(steps):
        S.step(Ud)
        Uc, t, dt, a9, st = orc.step(prob, Uc, cfl, t, 1e9)
        assert st == 0
    torch.cuda.synchronize()
    c = S.read_ctrl()
    assert (c.status, c.nsteps, c.t, c.dt) == (0, steps, t, dt)
    assert np.array_equal(Ud.cpu().numpy(), Uc)
    return S, t


ENDS = {
    "fixed_reflective": (("fixed", None, 0.0), ("reflective", None, 0.0)),
    "reflective_transmissive": (("reflective", None, 0.0), ("transmissive", None, 0.0)),
    # the end's kind changes within the second step: at t, t + dt and t + dt / 2 in its stages
    "moving": (("fixed", "reflective", 1.5), ("transmissive", "fixed", 1.2)),
}


@pytest.mark.parametrize("n", [3, 58, 200, 570, 571, 1500, 2300])
@pytest.mark.parametrize("ends", list(ENDS))
def test_lines(B, orc, n, ends):
    import torch
    cfl, steps = 0.4, 4
    prob = W.uniform_problem(1, [n], [0.0], [1.0], "transmissive")
    U = W.random_field(prob, seed=n)
    a = W.conserved(1.2, [0.1], 0.9, prob.gamma).tolist()
    b = W.conserved(0.7, [-0.2], 0.6, prob.gamma).tolist()
    # the coordinate of a 1D end is the first cell's centre; a split that passes it
    # after `when` steps' time changes the end's kind
    dt = cfl * prob.dx[0] / float(orc.alpha(prob, U)[0][0])

    def side(kind_a, kind_b, when, state):
        if kind_b is None:
            return W.Side(kind_a, state_a=state)
        return W.Side(kind_a, kind_b, split_axis=0, split0=prob.dx[0], state_a=state,
                      split_rate=-0.5 * prob.dx[0] / (when * dt), state_b=state)

    lo, hi = ENDS[ends]
    prob = prob.replace(boundary=W.Boundary(
        sides=[[side(*lo, a), side(*hi, b)], [W.Side("periodic")] * 2, [W.Side("periodic")] * 2],
        gravity=(0.3, 0.0, 0.0)))
    S, t = _steps_equal_oracle(B, orc, prob, U, cfl, steps)
    # the same steps in one recorded run
    S.init(0.0, 1e9, cfl)
    u = torch.from_numpy(U).cuda()
    S.run(u, steps, steps_per_graph=steps)
    torch.cuda.synchronize()
    assert S.read_ctrl().t == t
    Uc, tc = U, 0.0
    for _ in range(steps):
        Uc, tc, *_ = orc.step(prob, Uc, cfl, tc, 1e9)
    assert np.array_equal(u.cpu().numpy(), Uc)


@pytest.mark.parametrize("scheme", ["lad", "teno5a"])
def test_marched_3d(B, orc, scheme):
    # 216 x 240 x 200 cells: y and z are marched
    prob = W.uniform_problem(3, [216, 240, 200], [0.0] * 3, [1.0, 1.0, 1.0], "transmissive",
                             scheme=scheme)
    U = W.random_field(prob, seed=14)
    a = W.conserved(1.2, [0.1, -0.2, 0.05], 0.9, prob.gamma).tolist()
    b = W.conserved(0.6, [0.0, 0.3, -0.1], 0.4, prob.gamma).tolist()
    prob = prob.replace(boundary=W.Boundary(sides=[
        [W.Side("fixed", state_a=a), W.Side("transmissive")],
        [W.Side("fixed", "reflective", split_axis=0, split0=0.3, split_rate=2.0, state_a=b),
         W.Side("periodic", "fixed", split_axis=2, split0=0.5, split_rate=-3.0, state_b=a)],
        [W.Side("reflective", "transmissive", split_axis=1, split0=0.7, split_rate=4.0),
         W.Side("transmissive", "fixed", split_axis=1, split0=0.2, split_rate=-1.0, state_b=a)]],
        gravity=(0.1, -0.2, 0.3), time=0.05))
    _steps_equal_oracle(B, orc, prob, U, 0.4, 2)
