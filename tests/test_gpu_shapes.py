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
