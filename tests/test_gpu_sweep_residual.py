"""GPU: the residual of a sweep and the temperatures after it, on either side of the
mesh size (8192 vertices) up to which one launch does both."""
import numpy as np
import pytest
import torch

from oracle.core import Grid
from paper_2306_05789_amd import inputs, rte

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", [(2, 2, 2), (7, 9, 5), (16, 16, 32), (16, 16, 33)])
@pytest.mark.parametrize("nb,nrhs", [(1, 1), (3, 2)], ids=["grey", "bands"])
def test_residual_of_the_second_sweep(n, nb, nrhs):
    mesh = rte.rte_mesh_create(n)
    kap = inputs.smooth_kappa(Grid(n).positions())
    kt = torch.tensor(np.stack([kap * (1.0 + 0.5 * b) for b in range(nb)]), device=DEV)
    G = rte.rte_hmat_assemble(mesh, kt, rte.hmat_opts(kind=rte.RTE_VOLUME, leaf_size=32, aca_eps=1e-3))
    S = rte.rte_hmat_assemble(mesh, kt, rte.hmat_opts(kind=rte.RTE_SURFACE, leaf_size=32, aca_eps=1e-3))
    Tw = torch.ones((nrhs, mesh.L), device=DEV, dtype=torch.float64) * torch.arange(1, nrhs + 1, device=DEV)[:, None]
    nu = None if nb == 1 else [0.5, 1.0, 2.5]
    Js, Ts = [], []
    for sweeps in (1, 2):
        T = torch.empty((nrhs, mesh.N), device=DEV, dtype=torch.float64)
        J = torch.empty((nrhs, nb, mesh.N), device=DEV, dtype=torch.float64)
        st = rte.rte_fixed_point_solve(mesh, G, S, Tw, T, J, grey=nb == 1, nu=nu, tol=1e-14, max_iter=sweeps,
                                       allow_not_converged=True, history=True)
        Js.append(J.cpu().numpy())
        Ts.append(T.cpu().numpy())
    d = np.linalg.norm(Js[1] - Js[0], axis=2) / np.linalg.norm(Js[1], axis=2)
    assert len(st["residuals"]) == 2 and st["residuals"][0] == 1.0   # from J = 0
    # sums of N squares in two orders: N u relative at most
    assert abs(st["residuals"][1] - d.max()) <= 1e-12 * d.max()
    assert (Ts[1] >= Ts[0] * (1 - 2e-15)).all() and (Ts[0] > 0).all()
