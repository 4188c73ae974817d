"""GPU: a sweep with more (request, band) columns than a launch's y dimension may have
(65535) runs them in parts; the columns of the last part get what those of the first do."""
import numpy as np
import pytest
import torch

from paper_2306_05789_amd import inputs, rte
from paper_2306_05789_amd.serve import Server

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_more_columns_than_a_launch_has_rows():
    n, bands, count = (3, 3, 3), 32, 2100
    assert bands * count > 65535
    srv = Server(list(np.geomspace(0.5, 4.0, bands)), leaf_size=8, precision=rte.RTE_FP64, max_active=count, levels_per_decade=4)
    mid = srv.add_mesh(n, torch.tensor(inputs.smooth_kappa(inputs.grid_positions(n, (0, 0, 0), (1, 1, 1))), device=DEV))
    # four operators per request, so that no group of columns alone comes near the limit
    mult = [(1.0, 2.0, 4.0, 8.0)[b % 4] for b in range(bands)]
    walls = [torch.full((inputs.n_emitting(n, inputs.ALL_FACES),), t, device=DEV, dtype=torch.float64) for t in (0.7, 1.3)]
    ids = [srv.submit(mid, list(range(bands)), mult, walls[k % 2], tol=1e-12) for k in range(count)]
    most = 0
    for _ in range(300):
        most = max(most, srv.step()[0])
        if srv.poll(ids[-1])["state"] == rte.RTE_REQ_DONE and all(srv.poll(i)["state"] == rte.RTE_REQ_DONE for i in ids):
            break
    assert most * bands > 65535
    out = [torch.empty(27, device=DEV, dtype=torch.float64) for _ in ids]
    for i, T in zip(ids, out):
        assert srv.poll(i)["converged"]
        srv.fetch(i, T)
    assert not torch.equal(out[0], out[1]) and (out[0] > 0).all()
    assert all(torch.equal(T, out[k % 2]) for k, T in enumerate(out))
