"""GPU: what the library keeps on the device after a call, and that it is given back."""
import gc

import pytest
import torch

from paper_2306_05789_amd import inputs, rte

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MB = 1 << 20


def field(n, bands=1):
    kap = torch.tensor(inputs.smooth_kappa(inputs.grid_positions(n, (0, 0, 0), (1, 1, 1))), device=DEV)
    return torch.stack([kap * (1.0 + 0.5 * b) for b in range(bands)])


def device_free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def fresh():
    gc.collect()
    rte.rte_release_scratch()
    held, idle = rte.rte_memory_info()
    assert idle == 0
    return held


def test_idle_scratch_is_given_back():
    """Products and solves leave their working buffers idle; one call returns them to the device."""
    base = fresh()
    n = (13, 14, 15)
    mesh = rte.rte_mesh_create(n)
    G = rte.rte_hmat_assemble(mesh, field(n), rte.hmat_opts(kind=rte.RTE_VOLUME))
    S = rte.rte_hmat_assemble(mesh, field(n), rte.hmat_opts(kind=rte.RTE_SURFACE))
    x = torch.rand((600, mesh.N), device=DEV, dtype=torch.float64)
    y = torch.empty_like(x)
    rte.rte_hmat_matvec(G, 0, x, y)
    T = torch.empty((1, mesh.N), device=DEV, dtype=torch.float64)
    rte.rte_fixed_point_solve(mesh, G, S, torch.ones((1, mesh.L), device=DEV, dtype=torch.float64), T, grey=True)
    held, idle = rte.rte_memory_info()
    assert idle >= 2 * x.numel() * 8   # the product's vectors
    free = device_free()
    rte.rte_release_scratch()
    now, left = rte.rte_memory_info()
    assert left == 0 and now == held - idle
    assert device_free() - free >= idle // 2   # the runtime may keep part of a freed range
    y2 = torch.empty_like(x)
    rte.rte_hmat_matvec(G, 0, x, y2)   # and everything still runs
    assert torch.equal(y, y2)
    del G, S, mesh
    assert fresh() == base
