"""Kernel shapes where a split or a remainder can go wrong, against the dense FP64 definition.

Tolerance of the products: 1e-13 of the largest entry, as in test_gpu_parity (about
eps * sqrt(N) * 10 for these sizes).
"""
import numpy as np
import pytest
import torch

import oracle
from conftest import hi_operator, pack_upper, random_herm, random_sym
from test_gpu_parity import dev, host, make_solver

pytestmark = pytest.mark.gpu


# one block, a full and a ragged block edge, 15 and 16 blocks per edge (the two splits of the sum of
# the partials), and the default edge of that size
@pytest.mark.parametrize("n", [1, 5, 63, 64, 65, 200, 960, 961])
@pytest.mark.parametrize("storage", ["c128", "hilo"])
def test_small_block_products(n, storage):
    print(f"small block products n={n} storage={storage}", flush=True)
    rng = np.random.default_rng(1000 + n)
    A, B = random_herm(rng, n), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B)
    ap32, bp32 = hi_operator(ap, bp)
    s = make_solver("ph", ap, bp, storage)
    for prec in ["fp64"] + (["hi64"] if storage == "hilo" else []):
        pa, pb = (ap32, bp32) if prec == "hi64" else (ap, bp)
        for op in ["A", "K1", "K2", "H"]:
            length = 2 * n if op == "H" else n
            for nvec in [1, 2, 3, 4, 5]:
                x = rng.standard_normal((nvec, length)) + 1j * rng.standard_normal((nvec, length))
                got = host(s.apply(op, dev(x), precision=prec))
                ref = oracle.apply_dense(op, pa, x, pb)
                err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
                assert err < 1e-13, (op, prec, nvec, err)
    s.close()


# lengths at the edges of the orthogonalization kernels: one workgroup per vector up to 4096 rows, one
# launch per dot product up to 12288 (variant 3 works on ld + n rows, twice the matrix order), column
# groups of the updates up to 16384; block 1-4 vectors against the basis
@pytest.mark.parametrize("n,variant,block", [(257, 0, 0), (2048, 3, 2), (2049, 3, 3), (4096, 0, 0), (4097, 1, 0),
                                             (6145, 3, 4), (8200, 3, 1)])
def test_orthogonalization_lengths(n, variant, block):
    """Residuals recomputed here from the definition, and X^H X - Y^H Y = 1 (the solver's own basis
    stays M-orthonormal only if every dot product and update covers all rows)."""
    print(f"orthogonalization lengths n={n} variant={variant} block={block}", flush=True)
    k, tol = 4, 1e-9
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    f = torch.randn((n, 8, 2), dtype=torch.float64, device="cuda", generator=g)
    f = torch.view_as_complex(f) / n ** 0.5
    i = torch.arange(n, device="cuda")
    A = f @ f.mH
    # level spacing that opens towards the lower edge, as in the workloads (a dense lower edge does not
    # converge from so few kept vectors)
    A += torch.diag(1.0 + 13.0 * ((i + 0.5) / n).to(torch.float64) ** (2.0 / 3.0)).to(A.dtype)
    B = 0.2 * (f @ f.T)
    up = i[:, None] >= i[None, :]  # row j, column i <= j: packed column j
    s = make_solver("ph", host(A.T[up]), host(B.T[up]))
    om, x, y, _ = s.solve(k, tol, variant=variant, block=block)
    s.close()
    x, y = x.T.contiguous(), y.T.contiguous()
    top = A @ x + B @ y - om * x
    bot = -(A.conj().resolve_conj() @ y + B.conj().resolve_conj() @ x) - om * y
    res = torch.sqrt((top.abs() ** 2).sum(0) + (bot.abs() ** 2).sum(0))
    nrm = torch.sqrt((x.abs() ** 2).sum(0) + (y.abs() ** 2).sum(0))
    assert float((res / (om * nrm)).max()) <= 1.01 * tol
    assert float(((x.abs() ** 2).sum(0) - (y.abs() ** 2).sum(0) - 1.0).abs().max()) < 1e-12


def _packed_gradients(x, y, g):
    """dL/dA, dL/dB of L = sum g omega from the definition (LAPACK-'U', off-diagonal doubled)."""
    n = x.shape[1]
    j, i = np.tril_indices(n)  # packed order: column j, rows i <= j
    f = np.where(i == j, 1.0, 2.0)
    w = g if y is None else g / (np.sum(np.abs(x) ** 2, 1) - np.sum(np.abs(y) ** 2, 1))
    ga = (x.T * w) @ x.conj()
    if y is None:
        return f * ga[i, j], None
    ga = ga + (y.conj().T * w) @ y
    gb = (x.T * w) @ y.conj() + (y.conj().T * w) @ x
    return f * ga[i, j], f * gb[i, j]


# one tile, its edge and remainder, several tiles; pairs below, at and past the chunks of 8 (16 for TDA)
@pytest.mark.parametrize("n,k", [(7, 1), (63, 3), (64, 7), (65, 8), (130, 9), (200, 16), (129, 17), (257, 33)])
@pytest.mark.parametrize("kind", ["tda", "ph"])
def test_gradient_tiles(kind, n, k):
    """The packed gradients and the packed-component scalars of the handle's own pairs against the
    definition in FP64: sums of 4 k products per entry, so 1e-14 of the largest entry allows for
    about 10 roundings of it (k <= 33)."""
    print(f"gradient tiles {kind} n={n} k={k}", flush=True)
    rng = np.random.default_rng(2000 + n)
    A, B = random_herm(rng, n, lam_min=1.0), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B) if kind == "ph" else None
    s = make_solver(kind, ap, bp)
    _, x, y, _ = s.solve(k, 1e-8)
    g = rng.standard_normal(k)
    da, db = s.backward(dev(g))
    ra, rb = _packed_gradients(host(x), None if y is None else host(y), g)
    assert np.max(np.abs(host(da) - ra)) <= 1e-14 * np.max(np.abs(ra))
    if kind == "ph":
        assert np.max(np.abs(host(db) - rb)) <= 1e-14 * np.max(np.abs(ra))
    c = rng.standard_normal(len(ap)) + 1j * rng.standard_normal(len(ap))
    comps = [("A", "packed", dev(c), 1.0)] + ([("B", "packed", dev(c), -0.5)] if kind == "ph" else [])
    got = s.strength(dev(g), comps)
    # Re sum conj(g_ij) C_ij; a diagonal entry of G_A is real
    for v, ref, sc in zip(got, [ra, rb], [1.0, -0.5]):
        terms = np.real(np.conj(ref) * c)
        assert abs(v - sc * np.sum(terms)) <= 1e-14 * np.sum(np.abs(ref) * np.abs(c))
    s.close()


# the multi-vector products of every larger block edge: one block, ragged block rows, several vectors
# per read and a remainder (7 = 4 + 3)
@pytest.mark.parametrize("block", [128, 256, 512])
@pytest.mark.parametrize("n", [100, 512, 1100])
@pytest.mark.parametrize("storage", ["c128", "hilo"])
def test_large_block_products(block, n, storage, monkeypatch):
    print(f"large block products n={n} block={block} storage={storage}", flush=True)
    rng = np.random.default_rng(3000 + n)
    A, B = random_herm(rng, n), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B)
    ap32, bp32 = hi_operator(ap, bp)
    s = make_solver("ph", ap, bp, storage, block, monkeypatch)
    for prec in ["fp64"] + (["hi64"] if storage == "hilo" else []):
        pa, pb = (ap32, bp32) if prec == "hi64" else (ap, bp)
        for op in ["A", "K1", "K2", "H"]:
            length = 2 * n if op == "H" else n
            for nvec in [1, 2, 3, 4, 7]:
                x = rng.standard_normal((nvec, length)) + 1j * rng.standard_normal((nvec, length))
                got = host(s.apply(op, dev(x), precision=prec))
                ref = oracle.apply_dense(op, pa, x, pb)
                err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
                assert err < 1e-13, (op, prec, nvec, err)
    s.close()


# orders 2 n around the blocks of eight of the back-transformation, the panels of 64 columns and the
# chunks of 256 columns of the reduction; tolerance 1e-12 as in test_gpu_direct
@pytest.mark.parametrize("n", [1, 2, 4, 5, 31, 32, 33, 64, 65, 97, 128, 129, 161])
def test_direct_orders(n):
    import test_gpu_direct as tgd
    print(f"direct orders n={n}", flush=True)
    rng = np.random.default_rng(4000 + n)
    A, B = random_herm(rng, n, lam_min=1.0), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B)
    s = make_solver("ph", ap, bp)
    tgd.check_ph(s, ap, bp, max(1, n // 3))
    s.close()


# orders 2 n whose reduction changes its form at 2048 remaining rows: after one panel with 1986 and
# with exactly 2048 left; tolerance as above
@pytest.mark.parametrize("n", [1025, 1056])
def test_direct_orders_two_forms(n):
    import test_gpu_direct as tgd
    print(f"direct orders, two forms n={n}", flush=True)
    rng = np.random.default_rng(5000 + n)
    A, B = random_herm(rng, n, lam_min=1.0), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B)
    s = make_solver("ph", ap, bp)
    tgd.check_ph(s, ap, bp, 6)
    s.close()


def test_projected_eigensolver_orders():
    """Block full-H solves whose projected problems (order ncv, complex Hermitian) sit on both sides of
    the host / device split (128) and around the 64-row workgroups of the device reduction: the same
    pairs as the dense oracle."""
    n, k = 300, 6
    rng = np.random.default_rng(77)
    A, B = random_herm(rng, n, lam_min=1.0), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B)
    ref, _, _ = oracle.ph(ap, bp, k, vectors=False)
    s = make_solver("ph", ap, bp)
    for ncv in [128, 130, 192, 194, 258]:
        print(f"projected order {ncv}", flush=True)
        om, x, y, st = s.solve(k, 1e-10, variant=3, ncv=ncv, block=2)
        assert np.max(np.abs(host(om) - ref) / ref) < 1e-10
        rel = oracle.residual_ph(ap, bp, host(om), host(x).T, host(y).T)
        assert rel.max() <= 1.01e-10
    s.close()


# products of full-H vectors on block edge 64: one block, a ragged edge, the two splits of the sums of the
# partials, several vectors per read and a remainder
@pytest.mark.parametrize("n", [1, 65, 400, 961, 2001])
@pytest.mark.parametrize("storage", ["c128", "hilo"])
def test_full_h_halves(n, storage):
    """Each half of H [x; y] = [A x + B y; -(conj(B) x + conj(A) y)] against its own largest entry, where
    the halves differ in size (eigenvectors have |y| << |x|, a lone excitation y = 0): a half that is
    formed from A, B, x and y themselves is a sum of 4 N products, some eps sqrt(N) of the largest entry
    (2001: 1e-14); a sum and difference of the halves would leave eps (|A| + |B|)(|x| + |y|) instead,
    1e-11 of the smaller half here (|B| = 1e-3)."""
    print(f"full-H halves n={n} storage={storage}", flush=True)
    rng = np.random.default_rng(6000 + n)
    A, B = random_herm(rng, n), random_sym(rng, n, 1e-3)
    ap, bp = pack_upper(A), pack_upper(B)
    ap32, bp32 = hi_operator(ap, bp)
    s = make_solver("ph", ap, bp, storage)
    for prec in ["fp64"] + (["hi64"] if storage == "hilo" else []):
        pa, pb = (ap32, bp32) if prec == "hi64" else (ap, bp)
        for fx, fy in [(1.0, 0.0), (1.0, 0.02), (0.0, 1.0), (1.0, 1.0)]:
            for nvec in [1, 2, 3, 4, 5]:
                x = rng.standard_normal((nvec, 2 * n)) + 1j * rng.standard_normal((nvec, 2 * n))
                x[:, :n] *= fx
                x[:, n:] *= fy
                got = host(s.apply("H", dev(x), precision=prec))
                ref = oracle.apply_dense("H", pa, x, pb)
                for half in [slice(0, n), slice(n, 2 * n)]:
                    err = np.max(np.abs(got[:, half] - ref[:, half])) / np.max(np.abs(ref[:, half]))
                    assert err < 1e-14, (prec, fx, fy, nvec, half, err)
    s.close()


# four vectors per read on the larger block edges, N not a multiple of the edge
@pytest.mark.parametrize("block,n", [(128, 300), (256, 300), (512, 600)])
@pytest.mark.parametrize("storage", ["c128", "hilo"])
def test_infinite_last_entry(block, n, storage, monkeypatch):
    """An infinite last entry of one of four vectors: the rows of the earlier panels take it times their
    entry of the last column and nothing else that is infinite (the padding past N enters as zero), the
    other vectors stay finite."""
    print(f"infinite last entry n={n} block={block} storage={storage}", flush=True)
    rng = np.random.default_rng(7000 + n)
    A, B = random_herm(rng, n), random_sym(rng, n, 0.5)
    ap, bp = pack_upper(A), pack_upper(B)
    ap32, bp32 = hi_operator(ap, bp)
    s = make_solver("ph", ap, bp, storage, block, monkeypatch)
    top = (n - 1) // block * block  # rows of the panels before the last one
    for prec in ["fp64"] + (["hi64"] if storage == "hilo" else []):
        pa, pb = (ap32, bp32) if prec == "hi64" else (ap, bp)
        for op, sb in [("A", 0.0), ("K1", 1.0), ("K2", -1.0)]:
            x = rng.standard_normal((4, n)) + 1j * rng.standard_normal((4, n))
            ref = oracle.apply_dense(op, pa, x, pb)
            x[1, n - 1] = np.inf
            got = host(s.apply(op, dev(x), precision=prec))
            k = A[:top, n - 1] + sb * B[:top, n - 1]
            assert np.array_equal(got[1, :top].real, np.sign(k.real) * np.inf), (op, prec)
            assert np.array_equal(got[1, :top].imag, np.sign(k.imag) * np.inf), (op, prec)
            rest = [0, 2, 3]
            assert np.max(np.abs(got[rest] - ref[rest])) < 1e-13 * np.max(np.abs(ref[rest])), (op, prec)
    s.close()
