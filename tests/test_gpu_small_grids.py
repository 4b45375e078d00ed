"""Steps of small grids, where one block takes whole steps of a 1D line and the
sweeps of other small grids do the work around a stage themselves, bit for bit
against the oracle: sizes on both sides of every line of the dispatch, the
clipped last step, runs recorded with a remainder, and the same steps with the
sweeps as launches of their own."""
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


def _box(n, bc, seed, **kw):
    nd = len(n)
    prob = W.uniform_problem(nd, list(n), [0.0] * nd, [1.0] * nd, bc, **kw)
    return prob, W.random_field(prob, seed=seed)


def _same(c, t, dt, a9, steps):
    return (c.status, c.nsteps, c.active) == (0, steps, 0) and (c.t, c.dt) == (t, dt) \
        and np.array_equal(np.array(c.alpha), a9)


SIZES = [(3,), (57,), (58,), (59,), (64,), (250,), (251,), (506,), (507,), (570,), (571,), (2048,),
         (2049,), (32, 64), (3, 683), (683, 3), (31, 67), (362, 362), (363, 362), (13, 13, 12),
         (13, 13, 13), (50, 51, 51), (52, 51, 50)]


@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_small_steps_equal_oracle(B, orc, n):
    import torch
    k = SIZES.index(n)
    bc = ["periodic", "reflective", "transmissive"][k % 3]
    kw = [dict(), dict(scheme="teno5a"), dict(theta="cut"), dict(scheme="fixed_ct", ct_fixed=1e-5),
          dict(scheme="linear5")][k % 5]
    prob, U = _box(n, bc, 100 + k, **kw)
    S = B.Solver(prob)
    Ud = torch.from_numpy(U).cuda()
    Rc, _ = orc.rhs(prob, U, dump=True)
    assert np.array_equal(S.rhs(Ud).cpu().numpy(), Rc)
    t, Uc, steps = 0.0, U.copy(), 3
    S.init(0.0, 1e9, 0.4)
    for _ in range(steps):
        S.step(Ud)
        Uc, t, dt, a9, st = orc.step(prob, Uc, 0.4, t, 1e9)
        assert st == 0
    torch.cuda.synchronize()
    assert np.array_equal(Ud.cpu().numpy(), Uc)
    assert _same(S.read_ctrl(), t, dt, a9, steps)


@pytest.mark.parametrize("n", [(200,), (570,), (900,), (60, 40)], ids=lambda n: "x".join(map(str, n)))
def test_small_runs_stop_at_the_end_time(B, n):
    # 7 + 7 + 3 steps recorded by sevens, the end time within the third seven,
    # against single steps whose sweeps are launches of their own
    import torch
    prob, U = _box(n, "transmissive", 7)
    a, b = torch.from_numpy(U).cuda(), torch.from_numpy(U).cuda()
    R, T = B.Solver(prob), B.Solver(prob)
    T.init(0.0, 1e9, 0.4)
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(6 * len(n))]
    for e in evs:
        e.record(torch.cuda.current_stream())
    for _ in range(15):
        T.step(b, events=evs)
    t_end = T.read_ctrl().t * (1.0 + 1e-3)
    for s in (R, T):
        s.init(0.0, t_end, 0.4)
    b.copy_(torch.from_numpy(U))
    R.run(a, 17, steps_per_graph=7)
    for _ in range(17):
        T.step(b, events=evs)
    torch.cuda.synchronize()
    ca, cb = R.read_ctrl(), T.read_ctrl()
    assert (ca.t, ca.dt, ca.nsteps, ca.status) == (cb.t, cb.dt, cb.nsteps, cb.status) == (
        t_end, cb.dt, 16, 0)
    assert torch.equal(a, b)
