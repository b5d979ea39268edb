"""The device solution of the projected complex Hermitian eigenproblems by itself (a solve falls back
to the host QR if it fails, so the solver's results do not show which of the two ran).

Tolerance: the Householder reduction, the divide and conquer and the back-transformation are backward
stable, residual and loss of orthogonality within a modest multiple of m eps; m eps (of the largest
eigenvalue for the residual) is asked for, floor 64 eps.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_2504_10096_amd as bse

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def device_eig(s, a):
    """(w, z) of bse::herm_eig_device on the handle of s; fails if the device path did not run."""
    ok, w, z = call(s, a)
    assert ok
    return w, z


def call(s, a):
    f = bse.load_library()._ZN3bse15herm_eig_deviceEP12bse_handle_siPK15HIP_vector_typeIdLj2EEPdPS3_
    f.argtypes = [ctypes.c_void_p, ctypes.c_int] + 3 * [ctypes.c_void_p]
    f.restype = ctypes.c_bool
    m = a.shape[0]
    at = np.ascontiguousarray(a.T, dtype=np.complex128)  # column-major
    w, zt = np.zeros(m), np.zeros((m, m), complex)
    ok = f(s._h, m, at.ctypes.data, w.ctypes.data, zt.ctypes.data)
    return ok, w, zt.T


def check(a, w, z):
    m = len(w)
    tol = max(64, m) * EPS
    assert np.all(np.diff(w) >= 0)
    ad, zd = (torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in (a, z))
    wd = torch.as_tensor(w).cuda()
    r = torch.linalg.vector_norm(ad @ zd - zd * wd, dim=0).max()
    assert float(r) <= tol * np.abs(w).max()
    g = zd.mH.contiguous() @ zd - torch.eye(m, device="cuda")
    assert float(g.abs().max()) <= tol


def herm(rng, m):
    a = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    return a + a.conj().T


@pytest.fixture(scope="module")
def handle():
    s = bse.Solver("tda", 8)
    yield s
    s.close()


# odd and even orders, one and several batches of 512 rows per lane of the reduction, its largest
# order (2048) and the library's whole solution above; the buffers grow and are used again for less
@pytest.mark.parametrize("m", [2, 3, 48, 129, 131, 257, 511, 512, 513, 514, 608, 1025, 2047, 2048, 2049, 130])
def test_orders(handle, m):
    print(f"device eigensolver order {m}", flush=True)
    a = herm(np.random.default_rng(m), m)
    w, z = device_eig(handle, a)
    check(a, w, z)
    if m <= 608:
        ref = np.linalg.eigvalsh(a)
        assert np.abs(w - ref).max() <= max(64, m) * EPS * np.abs(ref).max()


@pytest.mark.parametrize("kind,m", [("diagonal", 150), ("real", 150), ("degenerate", 150), ("blocks", 150),
                                    ("arrowhead", 150), ("diagonal", 2048)])
def test_structures(handle, kind, m):
    """Columns with nothing to reduce, repeated eigenvalues, and the restart's own shape."""
    print(f"device eigensolver {kind} order {m}", flush=True)
    rng = np.random.default_rng(3)
    a = herm(rng, m)
    if kind == "diagonal":
        a = np.diag(np.diag(a).real).astype(complex)
    elif kind == "real":
        a = a.real.astype(complex)
    elif kind == "degenerate":
        q, _ = np.linalg.qr(a)
        a = (q * np.repeat([1.0, 2.0, 3.0], m // 3)) @ q.conj().T
        a = 0.5 * (a + a.conj().T)
    elif kind == "blocks":
        a[70:, :70] = 0.0
        a[:70, 70:] = 0.0
    else:  # diagonal, one full row and column, tridiagonal after it
        b = np.diag(np.diag(a).real).astype(complex)
        b[60, :61] = a[60, :61]
        b[:61, 60] = a[:61, 60]
        for i in range(60, m - 1):
            b[i + 1, i], b[i, i + 1] = a[i + 1, i], a[i, i + 1]
        a = b
    w, z = device_eig(handle, a)
    check(a, w, z)


@pytest.mark.parametrize("scale", [1e-300, 1e-158, 1.0, 1e153, 1e300])
@pytest.mark.parametrize("col", [1.0, 1e-155, 1e-160, 1e-165, 1e-165j])
def test_range(handle, scale, col):
    """Squares of a column that under- or overflow: no quotient of zeros (col 1e-165j) and no
    reflector that is not unitary (1e-160)."""
    print(f"device eigensolver scale {scale} column {col}", flush=True)
    m = 150
    a = herm(np.random.default_rng(5), m)
    a[1:, 0] *= col
    a[0, 1:] = a[1:, 0].conj()
    w, z = device_eig(handle, scale * a)
    check(a, w / scale, z)


def test_library_solution_of_a_diagonal_matrix(handle):
    """Above order 2048 the whole solution is the library's: right, or refused (the host QR solves it
    then), never vectors that are not numbers."""
    m = 2060
    print(f"device eigensolver diagonal order {m}", flush=True)
    a = np.diag(np.random.default_rng(8).standard_normal(m)).astype(complex)
    ok, w, z = call(handle, a)
    if ok:
        check(a, w, z)


# the reduction and the library's whole solution
@pytest.mark.parametrize("m", [300, 2060])
def test_repeats_are_bitwise_equal(handle, m):
    print(f"device eigensolver repeats order {m}", flush=True)
    a = herm(np.random.default_rng(9), m)
    w0, z0 = device_eig(handle, a)
    w1, z1 = device_eig(handle, a)
    assert np.array_equal(w0, w1) and np.array_equal(z0, z1)


def test_no_buffers_of_the_reduction_above_its_orders():
    """The two m x m buffers of the own reduction come with the first order that it takes."""
    print("device eigensolver buffers", flush=True)
    a = np.diag(np.arange(1.0, 2061.0)).astype(complex)
    s = bse.Solver("tda", 8, allocator="torch")
    call(s, a)
    before = torch.cuda.memory_allocated()
    assert call(s, a[:2048, :2048])[0]
    assert torch.cuda.memory_allocated() - before >= 2 * 16 * 2048 ** 2
    before = torch.cuda.memory_allocated()
    assert call(s, a[:300, :300])[0]
    assert torch.cuda.memory_allocated() == before
    s.close()


def pack(a):
    return np.concatenate([a[: j + 1, j] for j in range(len(a))]).astype(np.complex128)


# orders around the block of the library's back-transformation and the host / device split, and above
# the device reduction
@pytest.mark.parametrize("kind,n", [("real", 66), ("real", 129), ("real", 300), ("diagonal", 66), ("diagonal", 300),
                                    ("diagonal", 2060)])
def test_direct_tda_without_imaginary_parts(kind, n):
    """The dense TDA solve of real and of diagonal blocks, of which the library's whole solution makes
    vectors that are not numbers."""
    print(f"direct tda {kind} n={n}", flush=True)
    rng = np.random.default_rng(n)
    a = np.diag(rng.uniform(1.0, 5.0, n))
    if kind == "real":
        g = rng.standard_normal((n, n))
        a = a + 0.05 * (g + g.T)
    k = 5
    s = bse.Solver("tda", n)
    s.set_packed("A", torch.as_tensor(pack(a)).cuda())
    om, x, _, st = s.direct(k)
    s.close()
    om, x = om.cpu().numpy(), x.cpu().numpy().T
    ref = np.linalg.eigvalsh(a)
    tol = max(64, n) * EPS * np.abs(ref).max()
    assert np.abs(om - ref[:k]).max() <= tol
    assert np.linalg.norm(a @ x - x * om, axis=0).max() <= tol
    assert np.abs(x.conj().T @ x - np.eye(k)).max() <= max(64, n) * EPS
