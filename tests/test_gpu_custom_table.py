"""Continuation tables that the wavefront z kernels do not take (C + d > 64, or
d > 7) at N' = 32 K: the split and the fused workgroup kernels against the
oracle, and such members in a batch beside others.

Bars: 1e-11 as for every solver output, or, where the table amplifies more
(|M| is about 1e5 at (5, 63), 1e6 at (8, 31)), 4 times what a 1e-15 relative
change of the oracle's own start moves its result by."""
import numpy as np
import pytest

import workloads as W
from oracle import fc_table
from oracle.ns import Oracle, Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BANDWIDTHS = {(5, 63): 28, (8, 31): 19}


@pytest.fixture(scope="module")
def fcns():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2002_01392_amd as P
    P.load_library()
    return P


@pytest.fixture(autouse=True)
def bandwidths(monkeypatch):
    for k, v in BANDWIDTHS.items():
        monkeypatch.setitem(fc_table.K_CHOICE, k, v)


def rel_l2(a, b):
    a = a.detach().cpu().numpy() if hasattr(a, "detach") else np.asarray(a)
    b = b.detach().cpu().numpy() if hasattr(b, "detach") else np.asarray(b)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _workload(npr, d, C, seed):
    w = W.rayleigh_benard(12, 10, npr - C, 1e5, d=d, C=C, dt=1e-3, steps=2, seed=seed,
                          perturbation="curl_eigen", noise_rms=1e-2, kmax=3, mmax=3)
    return W.replace(w, dt=W.stable_dt(w))


def _solver(fcns, w, v0, th0, **kw):
    Q, A, _, _ = fc_table.fc_tables(w.d, w.C)
    s = fcns.Solver.from_workload(w, table=np.concatenate([Q.ravel(), A.ravel()]), **kw)
    s.set_state(torch.from_numpy(v0), torch.from_numpy(th0))
    return s


def _oracle(w, v0, th0):
    o = Oracle(Problem(**w.problem_kwargs()))
    o.set_state(v0, th0)
    o.rk_step(w.dt, w.steps)
    return o.get_state()[:2]


# (64 to 224: a compiled plan each in the fused pass, as 288)
@pytest.mark.parametrize("npr,d,C", [(128, 8, 31), (288, 5, 63), (64, 8, 31), (96, 8, 31),
                                     (160, 5, 63), (192, 8, 31), (224, 5, 63)])
def test_step_and_batch(fcns, npr, d, C):
    w = _workload(npr, d, C, 870)
    v0, th0 = w.initial_state()
    ref = _oracle(w, v0, th0)
    rng = np.random.default_rng(871)
    moved = _oracle(w, v0 * (1 + 1e-15 * rng.standard_normal(v0.shape)),
                    th0 * (1 + 1e-15 * rng.standard_normal(th0.shape)))
    bar = [max(1e-11, 4 * rel_l2(m, r)) for m, r in zip(moved, ref)]

    def check(s, what):
        v, th, _ = s.get_state()
        s.synchronize()
        err = [rel_l2(v, ref[0]), rel_l2(th, ref[1])]
        print(npr, d, C, what, err, bar, flush=True)
        assert err[0] < bar[0] and err[1] < bar[1], what

    for fused in (False, True):
        s = _solver(fcns, w, v0, th0)
        s.set_z_fused(fused)
        s.rk_step(w.dt, w.steps)
        check(s, "fused" if fused else "split")
    # beside a wavefront member (64) and a run-time plan (58)
    others = [W.rayleigh_benard(12, 10, n - c, 1e5, C=c, dt=w.dt, steps=2, seed=872)
              for n, c in ((64, 31), (58, 25))]
    states = [x.initial_state() for x in others]
    members = [_solver(fcns, w, v0, th0, stream=torch.cuda.Stream())]
    for x, (v, th) in zip(others, states):
        members.append(fcns.Solver.from_workload(x, stream=torch.cuda.Stream()))
        members[-1].set_state(torch.from_numpy(v), torch.from_numpy(th))
    torch.cuda.synchronize()
    b = fcns.Batch(members, [w.dt] * 3)
    b.run(w.steps)
    check(members[0], "batch")
    for s, x, (v, th) in zip(members[1:], others, states):
        got, _, _ = s.get_state()
        s.synchronize()
        alone = fcns.Solver.from_workload(x)
        alone.set_state(torch.from_numpy(v), torch.from_numpy(th))
        alone.set_z_fused(True)
        alone.rk_step(w.dt, w.steps)
        ref_v, _, _ = alone.get_state()
        alone.synchronize()
        assert rel_l2(got, ref_v) < 1e-13, x.name
    b.close()
