"""The line operators (fc_extend, fc_derivative) over strides, remainders and
table shapes: contiguous lines run wavefront kernels, other strides the general
ones, and both must match the oracle's operators on the same lines."""
import ctypes

import numpy as np
import pytest

import workloads as W
from oracle.fcgram import FCGram, fc_derivative_lines

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
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _lines(nz, n, seed, lz=1.7):
    z = np.linspace(0, lz, nz)
    r = W.rng(seed)
    return np.stack([np.sin(r.uniform(1, 9) * z + r.uniform()) * np.exp(r.uniform(-1, 1) * z)
                     for _ in range(n)])


def _strided(f, ps, ls, fill=np.nan):
    """Lines f (n, m) laid out with point stride ps and line stride ls, in a
    buffer of exactly the elements they span (gaps hold `fill`)."""
    n, m = f.shape
    buf = np.full((n - 1) * ls + (m - 1) * ps + 1, fill)
    idx = np.arange(n)[:, None] * ls + np.arange(m)[None] * ps
    buf[idx] = f
    return torch.from_numpy(buf).cuda(), idx


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


# strides as functions of (lines, points)
CONTIG = (lambda n, m: (1, m))
PADDED = (lambda n, m: (1, m + 3))
LINE_FASTEST = (lambda n, m: (n, 1))
SPREAD = (lambda n, m: (2, 2 * m + 1))


# rows of the wavefront form: 4 lines per wave, 16 per workgroup (remainders 1,
# 3, 17), d = 5 and 7 in registers, other d and C > 64 read from memory
@pytest.mark.parametrize("nz,d,C,n,ins,outs", [
    (33, 5, 25, 1, CONTIG, CONTIG), (65, 5, 31, 17, PADDED, CONTIG),
    (193, 5, 15, 66, CONTIG, PADDED), (65, 7, 33, 3, CONTIG, CONTIG),
    (64, 4, 10, 19, CONTIG, PADDED), (101, 3, 95, 21, CONTIG, CONTIG),
    (33, 5, 25, 18, LINE_FASTEST, LINE_FASTEST), (65, 5, 31, 9, SPREAD, CONTIG),
    (65, 5, 31, 9, CONTIG, SPREAD)])
def test_fc_extend_strides_and_tables(fcns, nz, d, C, n, ins, outs):
    r = W.rng(31 * nz + C)
    q, a = r.standard_normal((d, d)), r.standard_normal((C, d))
    s = fcns.Solver(8, 8, nz, 1.0, 1.0, 1.0, 0.0, d=d, C=C,
                    table=np.concatenate([q.ravel(), a.ravel()]))
    f = _lines(nz, n, 5 * nz + n)
    m = a @ q.T
    ref = np.concatenate([f, f[:, nz - d:] @ m.T + f[:, :d] @ m[::-1, ::-1].T], axis=1)
    src, _ = _strided(f, *ins(n, nz))
    dst, idx = _strided(np.zeros((n, nz + C)), *outs(n, nz + C), fill=7.0)
    ips, ils = ins(n, nz)
    ops, ols = outs(n, nz + C)
    assert s.lib.fcns_fc_extend(s.ctx, _p(src), n, ips, ils, _p(dst), ops, ols) == 0
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    # the copied points exactly, the sums of 2 d products to rounding, and
    # nothing written between the lines
    assert np.array_equal(got[idx][:, :nz], f)
    assert rel_l2(got[idx], ref) < 1e-14
    gaps = np.ones(got.size, bool)
    gaps[idx.ravel()] = False
    assert np.all(got[gaps] == 7.0)
    s.close()
