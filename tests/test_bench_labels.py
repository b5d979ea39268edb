"""bench.py names the kernel that a run's reads take (CPU)."""
import pytest

import bench


@pytest.mark.parametrize("n,edge", [(320, 64), (5632, 64), (5633, 128), (11392, 256), (23000, 512), (100000, 512)])
def test_block_edge(n, edge, monkeypatch):
    monkeypatch.delenv("BSE_BLOCK_EDGE", raising=False)
    assert bench.block_edge(n) == edge
    nb = -(-n // edge)
    assert edge == 64 or nb * (nb + 1) // 2 >= 1024
    monkeypatch.setenv("BSE_BLOCK_EDGE", "128")
    assert bench.block_edge(n) == 128


@pytest.mark.parametrize("edge,dtype,op,nv,kernel", [
    (64, "c64", "H", 4, "tile64_kernel"), (64, "c128", "A", 1, "tile64_kernel"),
    (512, "c64", "H", 2, "mh_stream_kernel"), (512, "c64", "H", 4, "mfma_pass_kernel"),
    (128, "hi+lo", "H", 4, "mh_stream_kernel"), (128, "c64", "H", 3, "mfma_pass_kernel"),
    (512, "c64", "K", 1, "mv_stream_kernel"), (512, "c64", "A", 2, "mk_block_kernel"),
    (256, "hi+lo", "A", 4, "mfma_pass_kernel"), (128, "c64", "K", 4, "mk_block_kernel")])
def test_pass_kernel(edge, dtype, op, nv, kernel):
    assert bench.pass_kernel(edge, dtype, op, nv) == kernel
