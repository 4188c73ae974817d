"""GPU: the accurate product of mixed storage against the FP64 product of the stored (hi +
lo) blocks.  Per 32-wide step the leading BF16 products leave one FP32 rounding of their
sum and the 2^-8 smaller ones round at their own size, so the error stays at 2^-24 of the
row's largest terms, whatever the number of steps."""
import numpy as np
import pytest
import torch

from paper_2306_05789_amd import inputs, rte
from readback import gpu_operator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nrhs", [1, 16, 17])
@pytest.mark.parametrize("n,leaf", [((11, 9, 10), 13), ((15, 14, 16), 32), ((21, 20, 22), 64)])
def test_accurate_product_error(n, leaf, nrhs):
    mesh = rte.rte_mesh_create(n, emit_faces=inputs.ALL_FACES)
    kap = torch.tensor(inputs.smooth_kappa(inputs.grid_positions(n, (0, 0, 0), (1, 1, 1))), device=DEV)
    opts = rte.hmat_opts(kind=rte.RTE_VOLUME, leaf_size=leaf, aca_eps=1e-5, precision=rte.RTE_MIXED_BF16)
    H = rte.rte_hmat_assemble(mesh, kap[None, :], opts)
    A = gpu_operator(mesh, H, opts)
    x = np.random.default_rng(1).uniform(0.5, 2.0, (nrhs, mesh.N))
    y = torch.empty((nrhs, mesh.N), device=DEV, dtype=torch.float64)
    rte.rte_hmat_matvec(H, 0, torch.tensor(x, device=DEV), y)
    ref = np.zeros_like(x)
    for t0, t1, s0, s1, D in A.dense:
        ref[:, A.tgt_perm[t0:t1]] += x[:, A.src_perm[s0:s1]] @ D.T
    for t0, t1, s0, s1, U, V in A.lowrank:
        ref[:, A.tgt_perm[t0:t1]] += (x[:, A.src_perm[s0:s1]] @ V) @ U.T
    err = (y.cpu().numpy() - ref) / ref
    # half a unit (2^-25) for each of the roundings in random directions: a row of S steps of similar size has
    # 2^-25 / sqrt(3 S) of itself, a row that one step makes up 2^-25; the lo parts' own roundings add about as much
    assert np.sqrt((err ** 2).mean()) <= 2.0 ** -26
    assert np.abs(err).max() <= 2.0 ** -23
