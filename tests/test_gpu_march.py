"""The marching sweep against the face-stream sweep, bit for bit, over the
forms it accepts: every boundary kind, per-end boundaries that change along
the boundary and in time, gravity, every scheme, ragged column counts (lanes
past the last column, columns that wrap over planes inside a wave) and
segment ends, the plain and the fused stages.  The decision dump and the mask
digest keep the face-stream sweep, so each grid runs both ways."""
import pytest

from paper_2003_09145_amd import workloads as W

pytestmark = pytest.mark.gpu


def _box(n, bc, seed, **kw):
    nd = len(n)
    prob = W.uniform_problem(nd, n, [0.0] * nd, [1.0] * nd, bc, **kw)
    return prob, W.random_field(prob, seed=seed)


CASES = {
    "2d_1281x2900_pr": lambda: _box([1281, 2900], ["periodic", "reflective"], 1),
    "2d_33x60011_tt": lambda: _box([33, 60011], "transmissive", 2, theta="cut"),
    "2d_1100x3400_pp_a5": lambda: _box([1100, 3400], "periodic", 3, scheme="teno5a"),
    "2d_3x60005_rp_ct": lambda: _box([3, 60005], ["reflective", "periodic"], 4,
                                     scheme="fixed_ct", ct_fixed=1e-5),
    "2d_1300x2900_linear": lambda: _box([1300, 2900], "transmissive", 5, scheme="linear5"),
    "2d_1284x2901_literal": lambda: _box([1284, 2901], "periodic", 6),
    "2d_rayleigh_taylor": lambda: W.rayleigh_taylor(1025, 3600, scheme="fixed_ct", ct_fixed=1e-5),
    "2d_double_mach": lambda: W.double_mach(2500, 1510, theta="cut"),
    "3d_5x400x5120_prt": lambda: _box([5, 400, 5120], ["periodic", "reflective", "transmissive"], 7),
    "3d_201x230x230_tpr": lambda: _box([201, 230, 230], ["transmissive", "periodic", "reflective"],
                                       8, scheme="teno5a"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_march_equals_face_stream(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_09145_amd import binding as B
    prob, U = CASES[name]()
    Ud = torch.from_numpy(U).cuda()
    S = B.Solver(prob)
    if name.endswith("literal"):
        S.g.flags |= B.FLAG_LITERAL_DECISIONS
    D = B.Solver(prob)
    D.g.flags = S.g.flags | B.FLAG_MASK_DIGEST
    R = S.rhs(Ud)
    Rd, _ = D.rhs(Ud, decisions=True)
    assert torch.equal(R, Rd)
    Ua, Ub = Ud.clone(), Ud.clone()
    for s, u in ((S, Ua), (D, Ub)):
        s.init(0.0, float("inf"), 0.4)
        for _ in range(2):
            s.step(u)
    torch.cuda.synchronize()
    ca, cb = S.read_ctrl(), D.read_ctrl()
    assert ca.status == 0 and ca.nsteps == 2
    assert (ca.t, ca.dt) == (cb.t, cb.dt) and torch.equal(Ua, Ub)


@pytest.mark.parametrize("shape", [(65, 30001), (5, 160003, 5), (6, 5, 160001)])
def test_march_equals_oracle(orc, shape):
    # few columns, long enough for the march along y (z)
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_09145_amd import binding as B
    prob, U = _box(list(shape), "periodic", 11)
    S = B.Solver(prob)
    R = S.rhs(torch.from_numpy(U).cuda())
    Rc, _ = orc.rhs(prob, U, dump=True)
    assert np.array_equal(R.cpu().numpy(), Rc)


@pytest.mark.parametrize("n", [(70, 31000), (7, 160003, 5)])
def test_march_in_place_keeps_zero_signs(n):
    # a uniform state changes nothing: the signed zeros of the partial
    # right-hand side come out as they went in less +-0, in place as elsewhere
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_09145_amd import binding as B
    prob, U = _box(list(n), "periodic", 12)
    Ud = torch.ones(U.shape, dtype=torch.float64, device="cuda")
    Ud[-1] = 9.0
    g = B.Solver(prob).g
    alpha = torch.full((4,), 3.0, dtype=torch.float64, device="cuda")
    Rin = torch.where(torch.arange(Ud.numel(), device="cuda") % 3 == 0, -0.0, 0.0).double().view(Ud.shape)
    out = torch.empty_like(Rin)
    B.teno_sweep(g, 1, Ud, out, alpha, Rin=Rin)
    B.teno_sweep(g, 1, Ud, Rin, alpha, Rin=Rin)
    assert torch.equal(out.view(torch.int64), Rin.view(torch.int64))
