"""GPU: the recompression's small problem (csrc/recompress.hip) at the ranks where its
workgroup changes: blocks whose ACA rank lies at either end of every bucket,
against the SVD of their ACA factors in NumPy."""
import numpy as np
import pytest
import torch

from oracle.core import Grid
from paper_2306_05789_amd import inputs, rte

pytestmark = pytest.mark.gpu
DEV = "cuda"
BUCKETS = [(2, 16), (17, 32), (33, 48), (49, 64), (65, 96)]
EPS = 1e-4


@pytest.fixture(scope="module")
def factors():
    n = (20, 18, 22)
    mesh = rte.rte_mesh_create(n)
    kt = torch.tensor(inputs.smooth_kappa(Grid(n).positions())[None, :], device=DEV)
    got = []
    for rc in (0, 1):
        H = rte.rte_hmat_assemble(mesh, kt, rte.hmat_opts(kind=rte.RTE_VOLUME, leaf_size=48, aca_eps=EPS,
                                                          precision=rte.RTE_FP64, recompress=rc))
        got.append([rte.rte_hmat_block_factors(H, 0, b) for b in range(rte.rte_hmat_stats(H)["n_lowrank"])])
    return list(zip(*got))


@pytest.mark.parametrize("lo,hi", BUCKETS)
def test_truncated_svd_at_every_bucket(factors, lo, hi):
    mine = sorted((p for p in factors if lo <= p[0][0] <= hi), key=lambda p: p[0][0])
    assert len(mine) >= 4
    for (k, U, V), (r, Ur, Vr) in mine[:3] + mine[-3:]:
        A = U @ V.T
        sig = np.linalg.svd(A, compute_uv=False)
        norm = np.linalg.norm(sig)
        tail = np.sqrt(np.cumsum(sig[::-1] ** 2))[::-1]   # tail[c]: what a truncation to c drops
        want = next((c for c in range(1, k) if tail[c] <= EPS * norm), k)
        assert r == want
        if r < k:
            # FP64 and columns orthogonal to 3e-15: what is dropped is the tail, up to a
            # rounding error of order k^2 u (1e-12) of the norm
            assert abs(np.linalg.norm(A - Ur @ Vr.T) - tail[r]) <= 1e-11 * norm
            # k columns of V', each off by the 3e-15 times sigma_1 / sigma_r at most
            assert np.linalg.norm(Vr.T @ Vr - np.eye(r)) <= 1e-14 * k * sig[0] / sig[r - 1]
