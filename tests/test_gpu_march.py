"""GPU: the optical depth by kinks (csrc/march.h) on every pair of vertices of
small grids with random absorption, against the oracle's entries: rays along
axes, in planes of every family, through edges and vertices, on the upper
faces (where the table continues kappa past the grid), grids of one cell and
longer than wide, paths reflected at either side of every axis.  FP64 entries
agree to 1e-12 as everywhere; FP32 ones to 1e-6 (1 + tau)."""
import os

import numpy as np
import pytest
import torch

from oracle.core import Grid, Problem
from paper_2306_05789_amd import rte

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

GRIDS = [(2, 2, 2), (2, 9, 3), (6, 5, 7), (13, 3, 4)]
WALLS = [None, [(0, 0, 0.5)], [(1, 1, 1.0)], [(0, 1, 0.7), (1, 0, 1.0), (2, 0, 0.4), (2, 1, 0.6)]]


@pytest.fixture(params=["table", "points"])
def quadrature(request):
    """The volume quadrature from the mesh's table by offset, or summed point by
    point (what a mesh too large for the table takes)."""
    if request.param == "points":
        os.environ["RTE_STAR_TABLE"] = "0"
    yield request.param
    os.environ.pop("RTE_STAR_TABLE", None)


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("walls", WALLS, ids=["open", "x-", "y+", "four"])
def test_every_pair_matches_oracle(n, walls, quadrature):
    g = Grid(n, (0.0, 0.0, 0.0), (1.0, 0.8, 1.3))
    kap = np.random.default_rng(sum(n)).uniform(0.05, 4.0, g.N)
    taken = {2 * a + s for a, s, _ in walls or []}
    emit = sum(1 << f for f in range(6) if f not in taken)
    P = Problem(g, kap, emit_faces=emit, walls=walls)
    mesh = rte.rte_mesh_create(n, (0.0, 0.0, 0.0), (1.0, 0.8, 1.3), emit_faces=emit, walls=walls)
    kt = torch.tensor(kap, device=DEV)
    pos = g.positions()
    for kind, ref, ids in ((rte.RTE_VOLUME, P.dense_G(), np.arange(g.N)), (rte.RTE_SURFACE, P.dense_S(), P.emitting)):
        rows, cols = (v.ravel() for v in np.meshgrid(np.arange(g.N), np.asarray(ids), indexing="ij"))
        tau = P.tau(pos[rows], pos[cols])
        for w in range(len(walls or [])):
            tau = np.maximum(tau, P.tau(pos[rows], pos[cols], wall=w))
        for precision in (rte.RTE_FP64, rte.RTE_FP32):
            out = torch.empty(len(rows), device=DEV, dtype=torch.float64)
            rte.rte_entries(mesh, kind, kt, torch.tensor(rows, device=DEV), torch.tensor(cols, device=DEV), out, precision)
            tol = np.full(len(rows), 1e-12) if precision == rte.RTE_FP64 else 1e-6 * (1.0 + tau)
            r = ref.ravel()
            err = np.abs(out.cpu().numpy() - r) - tol * np.abs(r)
            k = int(np.argmax(err))
            assert err[k] <= 0, (kind, precision, rows[k], cols[k], out[k].item(), r[k])
