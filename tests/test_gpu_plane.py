"""The nonlinear term of small planes in one launch (nx, ny of 32 and 64) against
the FP64 oracle and the separate y and x passes, over plane counts that leave part
of an eight-plane group, three and four fields, both precisions and graph replays.

Bar 1e-11 as for every solver output (the transforms add a few 1e-16 to the
continuation's rounding); FP32 transforms: 2e-6, as the mixed-precision step of
any size."""
import numpy as np
import pytest

import workloads as W
from oracle.ns import Oracle, Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(32, 32, 33, 25), (64, 64, 17, 15), (32, 64, 11, 15), (64, 32, 24, 26)]


@pytest.fixture(scope="module")
def fcns():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2002_01392_amd as P
    P.load_library()
    return P


def rel_l2(a, b):
    a = a.detach().cpu().numpy() if hasattr(a, "detach") else np.asarray(a)
    b = b.detach().cpu().numpy() if hasattr(b, "detach") else np.asarray(b)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _table(C, d=5):
    q, a = np.eye(d), np.zeros((C, d))
    a[:, d - 1] = np.linspace(1.0, 0.0, C + 2)[1:-1] ** 2
    return np.concatenate([q.ravel(), a.ravel()])


@pytest.mark.parametrize("nx,ny,nz,C", SHAPES)
@pytest.mark.parametrize("theta", [False, True])
def test_nonlinear_term(fcns, nx, ny, nz, C, theta):
    v = np.stack([W.smooth_field(nx, ny, nz, 2.0, 3.0, 1.3, 3 + i, kmax=3) for i in range(3)])
    th = W.smooth_field(nx, ny, nz, 2.0, 3.0, 1.3, 12, kmax=3)
    # content at every mode, the Nyquist ones included
    v += 0.1 * W.white_field(v.shape, 23)
    th = th + 0.1 * W.white_field(th.shape, 24)
    tv, tt = torch.from_numpy(v), torch.from_numpy(th) if theta else None
    own = C == 26   # (no stored table: against the separate passes only)
    s = fcns.Solver(nx, ny, nz, 2.0, 3.0, 1.3, 0.01, C=C, boussinesq=theta, kappa=0.01,
                    gamma=1.0, table=_table(C) if own else None)
    got = [x for x in s.rhs_nonlinear(tv, tt, filtered=True) if x is not None]
    torch.cuda.synchronize()
    s.set_choices("xvar=1")
    ref = [x for x in s.rhs_nonlinear(tv, tt, filtered=True) if x is not None]
    torch.cuda.synchronize()
    for a, b in zip(got, ref):
        assert rel_l2(a, b) < 1e-12
    if not own:
        o = Oracle(Problem(nx=nx, ny=ny, nz=nz, lx=2.0, ly=3.0, lz=1.3, nu=0.01, C=C,
                           boussinesq=theta, kappa=0.01, gamma=1.0))
        for a, b in zip(got, o.rhs_nonlinear(v, th if theta else None, filtered=True)):
            assert rel_l2(a, b) < 1e-11
    s.close()


@pytest.mark.parametrize("nx,ny,nz,C", SHAPES[:3])
@pytest.mark.parametrize("precision,bar", [("fp64", 1e-11), ("mixed", 2e-6)])
def test_step_and_replays(fcns, nx, ny, nz, C, precision, bar):
    w = W.rayleigh_benard(nx, ny, nz, 1e5, C=C, dt=1e-3, steps=4, seed=31, noise_rms=1e-2,
                          kmax=2, mmax=3, perturbation="curl_eigen")
    w = W.replace(w, dt=W.stable_dt(w))
    v0, th0 = w.initial_state()
    s = fcns.Solver.from_workload(w, precision=precision)
    o = Oracle(Problem(**w.problem_kwargs()))
    s.set_state(torch.from_numpy(v0), torch.from_numpy(th0))
    o.set_state(v0, th0)
    for k in range(4):   # two eager steps between replays of the captured one
        (s.rk_graph if k % 2 else s.rk_step)(w.dt, 1)
        o.rk_step(w.dt, 1)
        v, th, _ = s.get_state()
        s.synchronize()
        rv, rth, _ = o.get_state()
        assert rel_l2(v, rv) < bar and rel_l2(th, rth) < bar
    s.close()


def test_launch_time_is_reported_whole(fcns):
    # in its own class, and the same launches in each of the four whose work it does
    w = W.channel(32, 32, 33, 1500.0, C=25, dt=1e-3, steps=1, seed=61, noise_rms=0.02)
    v0, _ = w.initial_state()
    s = fcns.Solver.from_workload(w)
    s.set_state(torch.from_numpy(v0))
    s.rk_step(w.dt, 1)
    s.set_timing(True)
    s.timing_reset()
    s.rk_step(w.dt, 3)
    rep = s.timing_report()
    assert rep["plane_nl"][0] == 6 and rep["plane_nl"][1] > 0
    for k in ("y_back_dy", "y_back_dz", "x_nl", "y_fwd"):
        assert rep[k] == rep["plane_nl"]
    for k in ("plane_nl", "x_nl"):
        s.set_timing(True, classes=[k])
        s.timing_reset()
        s.rk_step(w.dt, 2)
        one = s.timing_report()
        assert one[k][0] == 4 and one[k][1] > 0
        assert all(n == 0 for c, (n, _) in one.items() if c != k)
    s.close()
