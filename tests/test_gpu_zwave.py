"""The wavefront z pass (N' = 32 K, K = 2..9) against the FP64 oracle and against
the separate z kernels: every length, continuation tables with one and two
registers of continuation rows (C = 31, 15 and 33), every stage pattern (o = 1
runs the separate kernels in place, o >= 3 alternates the stage buffers), grids
whose last 8-pencil groups hold padding pencils, and the transforms alone
(set_state, get_state, the filtered nonlinear term, mixed precision).

Bars: velocity and theta 1e-11 as for every solver output.  Pressure (a
potential divided by c, on grids with few y points): 20 times what a 1e-15
relative change of the oracle's own start moves it by, at least 1e-10."""
import numpy as np
import pytest

import workloads as W
from oracle.ns import Oracle, Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fcns():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2002_01392_amd as P
    P.load_library()
    return P


def rel_l2(a, b):
    a = a.detach().cpu().numpy() if hasattr(a, "detach") else np.asarray(a)
    nb = np.linalg.norm(b)
    return float(np.linalg.norm(a - b) / (nb if nb > 0 else 1.0))


def _workload(kind, nx, ny, npr, C, d, seed):
    nz = npr - C
    if kind == "rb":
        w = W.rayleigh_benard(nx, ny, nz, 1e5, d=d, C=C, dt=1e-3, steps=2, seed=seed,
                              perturbation="curl_eigen", noise_rms=1e-2, kmax=3, mmax=3)
    else:
        w = W.channel(nx, ny, nz, 1500.0, d=d, C=C, dt=1e-3, steps=2, seed=seed, noise_rms=0.02,
                      kmax=3, mmax=3)
    return W.replace(w, dt=W.stable_dt(w))


def _oracle(w, v0, th0, order, steps):
    o = Oracle(Problem(**w.problem_kwargs(), rk_order=order))
    o.set_state(v0, th0)
    o.rk_step(w.dt, steps)
    return o.get_state()


@pytest.mark.parametrize("kind,nx,ny,npr,C,d,order", [
    ("rb", 12, 10, 64, 31, 5, 2), ("channel", 10, 12, 64, 33, 7, 2),
    ("rb", 18, 8, 96, 25, 5, 3), ("channel", 8, 14, 96, 15, 5, 4),
    ("rb", 16, 10, 128, 33, 7, 2), ("channel", 12, 8, 160, 31, 5, 1),
    ("rb", 10, 8, 160, 31, 5, 1), ("rb", 14, 8, 192, 25, 5, 2),
    ("channel", 8, 10, 224, 33, 7, 3), ("rb", 10, 8, 256, 15, 5, 2),
    ("rb", 8, 12, 288, 31, 5, 2), ("channel", 14, 8, 288, 33, 7, 2)])
def test_step_matches_the_oracle(fcns, kind, nx, ny, npr, C, d, order):
    w = _workload(kind, nx, ny, npr, C, d, 900 + npr + order)
    v0, th0 = w.initial_state()
    rv, rth, rp = _oracle(w, v0, th0, order, 2)
    r = W.rng(5)
    pv, pth = v0 * (1 + 1e-15 * r.standard_normal(v0.shape)), th0
    if th0 is not None:
        pth = th0 * (1 + 1e-15 * r.standard_normal(th0.shape))
    bar = max(1e-10, 20 * rel_l2(_oracle(w, pv, pth, order, 2)[2], rp))
    got = {}
    for fused in (True, False):
        s = fcns.Solver.from_workload(w, keep_pressure=True, rk_order=order)
        if order > 1 or not fused:
            s.set_z_fused(fused)
        s.set_state(torch.from_numpy(v0), torch.from_numpy(th0) if th0 is not None else None)
        s.rk_step(w.dt, 2)
        got[fused] = s.get_state(pressure=True)
        s.synchronize()
        v, th, p = got[fused]
        assert rel_l2(v, rv) < 1e-11, fused
        if rth is not None:
            assert rel_l2(th, rth) < 1e-11, fused
        assert rel_l2(p, rp) < bar, fused
        s.close()


def test_default_is_the_wavefront_pass_and_graph_replays_it(fcns):
    w = _workload("rb", 16, 12, 96, 31, 5, 77)
    v0, th0 = w.initial_state()
    out = []
    for graph in (False, True):
        s = fcns.Solver.from_workload(w, rk_order=3)
        assert "zfused=1" in s.choices()
        s.set_state(torch.from_numpy(v0), torch.from_numpy(th0))
        for _ in range(3):   # replays with eager work between them
            (s.rk_graph if graph else s.rk_step)(w.dt, 2)
            s.diagnostics()
        out.append(s.get_state())
        s.synchronize()
        s.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("npr,C,d", [(64, 31, 5), (128, 33, 7), (288, 25, 5)])
def test_transforms_alone(fcns, npr, C, d):
    nx, ny, nz, lz = 14, 10, npr - C, 1.3
    s = fcns.Solver(nx, ny, nz, 2.0, 3.0, lz, 0.01, d=d, C=C)
    v = np.stack([W.smooth_field(nx, ny, nz, 2.0, 3.0, lz, 40 + i) for i in range(3)])
    s.set_state(torch.from_numpy(v))
    back, _, _ = s.get_state()
    spec = s.get_spectral(1)
    nl, _ = s.rhs_nonlinear(torch.from_numpy(v), filtered=True)
    torch.cuda.synchronize()
    o = Oracle(Problem(nx=nx, ny=ny, nz=nz, lx=2.0, ly=3.0, lz=lz, nu=0.01, d=d, C=C))
    o.set_state(v)
    # a 1e-15 relative change of the input moves the oracle's own continued
    # spectrum by 1e-12 to 5e-12 at d = 5 and 2e-10 at d = 7 (table entries to 4e5)
    o2 = Oracle(o.p)
    o2.set_state(v * (1 + 1e-15 * W.rng(3).standard_normal(v.shape)))
    bar = max(1e-11, rel_l2(o2.Vt[1], o.Vt[1]))
    assert rel_l2(back, v) < 1e-12
    assert rel_l2(spec, o.Vt[1]) < bar
    assert rel_l2(nl, o.rhs_nonlinear(v, filtered=True)[0]) < bar
    # the spectral state written back is the state read
    s.set_spectral([s.get_spectral(f) for f in range(3)])
    again, _, _ = s.get_state()
    assert torch.equal(again, back)
    s.close()


def test_mixed_precision_back_transforms(fcns):
    w = _workload("rb", 16, 12, 128, 31, 5, 91)
    v0, th0 = w.initial_state()
    rv, rth, _ = _oracle(w, v0, th0, 2, 2)
    s = fcns.Solver.from_workload(w, precision="mixed")
    s.set_state(torch.from_numpy(v0), torch.from_numpy(th0))
    s.rk_step(w.dt, 2)
    v, th, _ = s.get_state()
    s.synchronize()
    assert rel_l2(v, rv) < 2e-6 and rel_l2(th, rth) < 2e-6
    s.close()
