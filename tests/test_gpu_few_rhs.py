"""GPU: products of one to four right-hand sides per pass on the vector ALUs (FP64 up to
4, FP32 in groups of 4 with every remainder), against the FP64 product of the stored
blocks read back, on leaves and ranks that are no multiple of anything."""
import numpy as np
import pytest
import torch

from paper_2306_05789_amd import inputs, rte
from readback import gpu_operator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("precision,counts", [(rte.RTE_FP64, (1, 2, 3, 4)), (rte.RTE_FP32, (1, 2, 3, 4, 5, 6, 7, 10))],
                         ids=["fp64", "fp32"])
@pytest.mark.parametrize("kind", [rte.RTE_VOLUME, rte.RTE_SURFACE], ids=["volume", "surface"])
@pytest.mark.parametrize("leaf", [13, 64, 100])
def test_few_right_hand_sides(precision, counts, kind, leaf):
    n = (11, 9, 10)
    mesh = rte.rte_mesh_create(n, emit_faces=inputs.FACE_X_LO | inputs.FACE_Y_HI)
    kap = torch.tensor(inputs.smooth_kappa(inputs.grid_positions(n, (0, 0, 0), (1, 1, 1))), device=DEV)
    opts = rte.hmat_opts(kind=kind, leaf_size=leaf, aca_eps=1e-5, precision=precision)
    H = rte.rte_hmat_assemble(mesh, kap[None, :], opts)
    A = gpu_operator(mesh, H, opts)
    ns = mesh.N if kind == rte.RTE_VOLUME else mesh.L
    x = np.random.default_rng(leaf).uniform(-0.5, 2.0, (max(counts), ns))
    ref, size = np.zeros((len(x), mesh.N)), np.zeros((len(x), mesh.N))
    for t0, t1, s0, s1, D in A.dense:
        ref[:, A.tgt_perm[t0:t1]] += x[:, A.src_perm[s0:s1]] @ D.T
        size[:, A.tgt_perm[t0:t1]] += np.abs(x[:, A.src_perm[s0:s1]]) @ np.abs(D).T
    for t0, t1, s0, s1, U, V in A.lowrank:
        ref[:, A.tgt_perm[t0:t1]] += (x[:, A.src_perm[s0:s1]] @ V) @ U.T
        size[:, A.tgt_perm[t0:t1]] += (np.abs(x[:, A.src_perm[s0:s1]]) @ np.abs(V)) @ np.abs(U).T
    # sums of fewer than 2 ns terms in the accumulation type, x rounded to it
    tol = 2 * ns * 2.0 ** (-53 if precision == rte.RTE_FP64 else -24) * size
    X = torch.tensor(x, device=DEV)
    for nr in counts:
        y = torch.full((nr, mesh.N), float("nan"), device=DEV, dtype=torch.float64)
        rte.rte_hmat_matvec(H, 0, X[:nr].contiguous(), y)
        assert (np.abs(y.cpu().numpy() - ref[:nr]) <= tol[:nr]).all(), nr
