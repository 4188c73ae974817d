"""GPU: the ACA's entry launches with several lanes per entry (k_aca_wide, taken
when a launch would leave most of the chip idle) give the factors of the
one-lane launches bit for bit: open mesh, one wall, three walls, three walls
with a hole; volume and surface; FP64, FP32 and BF16 storage; ranks below and
above the residual terms that a group loads at once (32 and 128)."""
import os

import numpy as np
import pytest
import torch

from paper_2306_05789_amd import inputs, rte

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(n=(13, 12, 15), precision=rte.RTE_FP64),
    dict(n=(13, 12, 15), precision=rte.RTE_MIXED_BF16),
    dict(n=(9, 21, 8), precision=rte.RTE_FP64, walls=[(2, 1, 0.6)], aca_eps=1e-9),
    dict(n=(13, 9, 11), precision=rte.RTE_FP32, walls=[(0, 1, 1.0), (1, 0, 1.0), (2, 0, 0.7)]),
    dict(n=(13, 13, 9), precision=rte.RTE_FP64, walls=[(0, 0, 1.0), (1, 0, 1.0), (2, 0, 1.0)],
         hole=((0, 0, 0), (3, 3, 2)), hole_emit=2 | 8 | 32, emit_faces=2 | 8 | 32),
]


@pytest.mark.parametrize("case", CASES, ids=["open", "mixed", "wall", "walls-fp32", "hole"])
@pytest.mark.parametrize("kind", [rte.RTE_VOLUME, rte.RTE_SURFACE], ids=["volume", "surface"])
def test_lanes_per_entry_do_not_show(case, kind):
    n = case["n"]
    geo = {k: case[k] for k in ("walls", "hole", "hole_emit", "emit_faces") if k in case}
    mesh = rte.rte_mesh_create(n, **{"emit_faces": 1, **geo})
    pos = inputs.grid_positions(n, (0, 0, 0), (1, 1, 1))
    kt = torch.tensor(inputs.smooth_kappa(pos)[None, :], device=DEV)
    opts = rte.hmat_opts(kind=kind, leaf_size=16, aca_eps=case.get("aca_eps", 1e-5), precision=case["precision"])
    got = []
    for wide in ("0", "1"):
        os.environ["RTE_ACA_WIDE"] = wide
        try:
            H = rte.rte_hmat_assemble(mesh, kt, opts)
        finally:
            os.environ.pop("RTE_ACA_WIDE")
        st = rte.rte_hmat_stats(H)
        got.append((st["aca_entries"], [rte.rte_hmat_block_factors(H, 0, b) for b in range(st["n_lowrank"])]))
    assert got[0][0] == got[1][0] and len(got[0][1]) > 0
    for (ka, ua, va), (kb, ub, vb) in zip(got[0][1], got[1][1]):
        assert ka == kb
        if ka > 0:
            assert np.array_equal(ua, ub) and np.array_equal(va, vb)
