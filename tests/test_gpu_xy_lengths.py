"""The x and y transforms over row lengths: wavefront rows, LDS tiles (with their
radix remainders, prime factors above 7 and the edges where the tile shape
changes: 160 and 162 points in x, 256 and 258, 288 and 290 in y), row counts
that leave partial tiles, against the FP64 oracle.

Bar 1e-11 as for every solver output: these transforms add a few 1e-16 to the
continuation's rounding (d = 5: the oracle's spectrum moves 1e-12 to 5e-12 for a
1e-15 relative change of its input)."""
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


def _fields(nx, ny, nz, seed):
    v = np.stack([W.smooth_field(nx, ny, nz, 2.0, 3.0, 1.3, seed + i, kmax=2) for i in range(3)])
    th = W.smooth_field(nx, ny, nz, 2.0, 3.0, 1.3, seed + 9, kmax=2)
    # content at every mode, the Nyquist ones included
    v += 0.1 * W.white_field(v.shape, seed + 20)
    return v, th + 0.1 * W.white_field(th.shape, seed + 21)


@pytest.mark.parametrize("nx,ny,theta", [
    (4, 6, True), (10, 4, False), (30, 14, True), (84, 6, False), (120, 10, True),
    (158, 8, False), (160, 6, True), (162, 6, True), (256, 6, True), (258, 4, False),
    (512, 4, True), (96, 12, True), (32, 10, False), (6, 84, True), (8, 90, False),
    (6, 256, True), (4, 286, False), (6, 288, True), (4, 290, True), (4, 512, False),
    (6, 518, True)])
def test_nonlinear_term_and_state(fcns, nx, ny, theta):
    nz = 11   # 11 ny rows: partial tiles of 8 and 16 rows
    C = 15
    s = fcns.Solver(nx, ny, nz, 2.0, 3.0, 1.3, 0.01, C=C, boussinesq=theta, kappa=0.01,
                    gamma=1.0)
    v, th = _fields(nx, ny, nz, 7 * nx + ny)
    tv, tt = torch.from_numpy(v), torch.from_numpy(th) if theta else None
    nlv, nlt = s.rhs_nonlinear(tv, tt)
    s.set_state(tv, tt)
    back, bth, _ = s.get_state()
    torch.cuda.synchronize()
    o = Oracle(Problem(nx=nx, ny=ny, nz=nz, lx=2.0, ly=3.0, lz=1.3, nu=0.01, C=C,
                       boussinesq=theta, kappa=0.01, gamma=1.0))
    rv, rt = o.rhs_nonlinear(v, th if theta else None)
    o.set_state(v, th if theta else None)
    sv, st, _ = o.get_state()
    assert rel_l2(nlv, rv) < 1e-11
    assert rel_l2(back, sv) < 1e-11
    if theta:
        assert rel_l2(nlt, rt) < 1e-11
        assert rel_l2(bth, st) < 1e-11
    s.close()


@pytest.mark.parametrize("nx,ny", [(30, 14), (120, 84), (174, 10), (6, 290)])
def test_mixed_precision_step(fcns, nx, ny):
    w = W.rayleigh_benard(nx, ny, 33, 1e5, C=25, dt=1e-3, steps=2, seed=31, noise_rms=1e-2,
                          kmax=2, mmax=3, perturbation="curl_eigen")
    w = W.replace(w, dt=W.stable_dt(w))
    v0, th0 = w.initial_state()
    s = fcns.Solver.from_workload(w, precision="mixed")
    s.set_state(torch.from_numpy(v0), torch.from_numpy(th0))
    s.rk_step(w.dt, 2)
    v, th, _ = s.get_state()
    s.synchronize()
    o = Oracle(Problem(**w.problem_kwargs()))
    o.set_state(v0, th0)
    o.rk_step(w.dt, 2)
    rv, rth, _ = o.get_state()
    assert rel_l2(v, rv) < 2e-6 and rel_l2(th, rth) < 2e-6
    s.close()


# rows loaded ahead into LDS: several rounds of rows per workgroup with a partial
# last one, against the tiled kernel of any length
@pytest.mark.parametrize("nx,ny,nz,theta,precision", [
    (128, 512, 131, True, "fp64"), (192, 258, 131, False, "fp64"), (192, 258, 131, True, "mixed"),
    (256, 258, 131, False, "fp64"), (256, 258, 131, True, "mixed"), (128, 6, 11, False, "mixed")])
def test_rows_loaded_ahead(fcns, nx, ny, nz, theta, precision):
    C = 15
    out = []
    gen = torch.Generator(device="cuda").manual_seed(nx)
    v = torch.randn(3, nz, ny, nx, dtype=torch.float64, device="cuda", generator=gen)
    th = torch.randn(nz, ny, nx, dtype=torch.float64, device="cuda", generator=gen)
    for xvar in (0, 1):
        s = fcns.Solver(nx, ny, nz, 2.0, 3.0, 1.3, 1e-5, C=C, boussinesq=theta, kappa=1e-5,
                        gamma=1.0, precision=precision, rk_order=1)
        s.set_choices(f"xvar={xvar}")
        s.set_state(v, th if theta else None)
        s.rk_step(1e-4, 1)
        out.append([x for x in s.get_state()[:2] if x is not None])
        s.synchronize()
        s.close()
    for a, b in zip(*out):
        assert bool(torch.isfinite(a).all())
        # one step moves the state by dt times the term: FP64 rounding, or FP32's in
        # the term (white noise in a step: up to 1e-1 of the state), 1e-7 of that
        d = float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))
        assert d < (1e-12 if precision == "fp64" else 2e-6), (nx, precision, d)


# compiled y plans: tiles of 8 columns that end inside a plane or span two
@pytest.mark.parametrize("nx,ny,theta", [(4, 64, True), (10, 64, False), (6, 96, True),
                                         (20, 128, False), (4, 128, True), (12, 192, True),
                                         (20, 256, True)])
def test_columns_of_compiled_plans(fcns, nx, ny, theta):
    test_nonlinear_term_and_state(fcns, nx, ny, theta)


@pytest.mark.parametrize("ny", [96, 192])
def test_columns_of_compiled_plans_mixed(fcns, ny):
    test_mixed_precision_step(fcns, 12, ny)


# both forms of prime stages (pairs, matrices) in every kernel that has them, two
# primes in a length, and above the primes with a table
@pytest.mark.parametrize("nx,ny,theta", [
    (22, 6, True), (26, 6, False), (34, 6, True), (220, 4, False), (242, 4, True),
    (260, 4, True), (442, 4, False), (6, 26, False), (6, 34, True), (6, 110, True), (4, 220, True),
    (4, 338, False), (4, 442, True), (4, 514, False)])
def test_prime_forms(fcns, nx, ny, theta):
    test_nonlinear_term_and_state(fcns, nx, ny, theta)


@pytest.mark.parametrize("nx,ny", [(26, 34), (34, 26), (220, 6), (260, 8), (6, 338), (6, 526)])
def test_prime_forms_mixed(fcns, nx, ny):
    test_mixed_precision_step(fcns, nx, ny)


# the same in z, for each number of rows a thread holds, split and fused: pairs at 44,
# 242 and 338, matrices at 76, 92, 276 and 322
@pytest.mark.parametrize("npr", [44, 76, 92, 242, 276, 322, 338])
def test_prime_forms_z(fcns, npr):
    w = W.rayleigh_benard(8, 6, npr - 15, 1e5, C=15, dt=1e-3, steps=2, seed=npr, noise_rms=1e-2,
                          kmax=2, mmax=3, perturbation="curl_eigen")
    w = W.replace(w, dt=W.stable_dt(w))
    v0, th0 = w.initial_state()
    o = Oracle(Problem(**w.problem_kwargs()))
    o.set_state(v0, th0)
    o.rk_step(w.dt, 2)
    rv, rth, _ = o.get_state()
    for precision, fused, bar in (("fp64", False, 1e-11), ("fp64", True, 1e-11),
                                  ("mixed", False, 2e-6)):
        if fused and npr > 288:
            continue
        s = fcns.Solver.from_workload(w, precision=precision)
        s.set_z_fused(fused)
        s.set_state(torch.from_numpy(v0), torch.from_numpy(th0))
        s.rk_step(w.dt, 2)
        v, th, _ = s.get_state()
        s.synchronize()
        assert rel_l2(v, rv) < bar and rel_l2(th, rth) < bar, (precision, fused)
        s.close()


# lengths past the last one with tiles of 8 columns (192), to the last of 4 rows per
# thread (256) and the first of 8
@pytest.mark.parametrize("nx,ny,theta", [(10, 180, True), (4, 194, True), (6, 200, False),
                                         (10, 254, True), (4, 258, True), (6, 270, False)])
def test_columns_of_any_length(fcns, nx, ny, theta):
    test_nonlinear_term_and_state(fcns, nx, ny, theta)


@pytest.mark.parametrize("ny", [200, 270])
def test_columns_of_any_length_mixed(fcns, ny):
    test_mixed_precision_step(fcns, 12, ny)


# what is reported of the y tiles is what runs: a choice at 512 points only
@pytest.mark.parametrize("ny,precision,lines", [(84, "fp64", 8), (192, "fp64", 4),
                                                (192, "mixed", 8), (200, "fp64", 4),
                                                (256, "fp64", 8), (512, "fp64", None)])
def test_reported_columns_per_tile(fcns, ny, precision, lines):
    s = fcns.Solver(8, ny, 11, 2.0, 3.0, 1.3, 0.01, C=15, precision=precision)
    s.set_state(torch.zeros(3, 11, ny, 8, dtype=torch.float64))
    report = s.autotune()
    s.synchronize()
    text = s.choices()
    if lines:
        assert report.count(f" {lines} lines") == 2 and report.count(" lines") == 2
        assert "ylines" not in text
    else:
        assert "ylines=" in text and "ylines1=" in text
    s.set_choices(text + ";ylines=4;ylines1=4")   # as a text saved before may hold
    s.set_choices(text)
    assert s.choices() == text
    s.close()


# the same lengths where few workgroups run without direct loads
@pytest.mark.parametrize("nx,ny,nz,theta,precision", [
    (128, 66, 65, True, "fp64"), (128, 66, 65, False, "fp64"), (128, 96, 97, False, "mixed"),
    (256, 96, 65, False, "mixed")])
def test_rows_not_loaded_ahead(fcns, nx, ny, nz, theta, precision):
    test_rows_loaded_ahead(fcns, nx, ny, nz, theta, precision)
