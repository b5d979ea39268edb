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
