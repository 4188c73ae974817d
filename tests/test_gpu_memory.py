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


def test_a_request_holds_what_it_needs():
    """Wall temperatures of queued requests, states of running ones and results that wait to be fetched take their own
    bytes in whole pages: none of it may exceed the server's budget by a multiple of what it counts."""
    from paper_2306_05789_amd.serve import Server
    n, count = (6, 5, 7), 60
    page = lambda b: -(-b // 4096) * 4096
    srv = Server([0.5, 1.0, 2.0], leaf_size=16, precision=rte.RTE_MIXED_BF16, max_active=20)
    mid = srv.add_mesh(n, field(n)[0].contiguous())
    tw = torch.ones(inputs.n_emitting(n, inputs.ALL_FACES), device=DEV, dtype=torch.float64)
    N, nb = 6 * 5 * 7, 2
    warm = srv.submit(mid, [0, 1], [1.0, 1.0], tw, tol=1e-6)   # assembles the operator
    while srv.poll(warm)["state"] != rte.RTE_REQ_DONE:
        srv.step()
    srv.fetch(warm, torch.empty(N, device=DEV, dtype=torch.float64))
    base = fresh()
    ids = [srv.submit(mid, [0, 1], [1.0, 1.0], tw, tol=1e-6) for _ in range(count)]
    queued = rte.rte_memory_info()[0] - base
    assert queued <= count * page(tw.numel() * 8)
    srv.step()
    running = rte.rte_memory_info()[0] - base
    # 20 states, and the sweep's own small tables
    assert running <= queued + 20 * page(8 * N * (2 + 4 * nb)) + 2 * MB
    while any(srv.poll(i)["state"] != rte.RTE_REQ_DONE for i in ids):
        srv.step()
    held, idle = rte.rte_memory_info()
    assert held - idle - base <= count * page(8 * N) + 2 * MB
    for i in ids:
        srv.fetch(i, torch.empty(N, device=DEV, dtype=torch.float64))
    held, idle = rte.rte_memory_info()
    assert held - idle - base <= 2 * MB


def test_a_mesh_keeps_no_device_memory():
    """What an assembly tabulates by offset goes with it: 23 MB for this mesh."""
    n = (17, 17, 17)
    base = fresh()
    meshes = [rte.rte_mesh_create(n) for _ in range(3)]
    for mesh in meshes:
        H = rte.rte_hmat_assemble(mesh, field(n), rte.hmat_opts(kind=rte.RTE_VOLUME))
        del H
        assert fresh() == base


def test_assembly_does_without_the_table_when_memory_is_short(monkeypatch):
    """At the smallest bound of the library's memory where an operator is assembled point by point, it is assembled by
    default too, to the same bits: its quadrature table (23 MB) is left out where it would not fit.  Without room for the
    operator itself it stays an error, and nothing is lost by it."""
    n = (17, 17, 17)
    opts = rte.hmat_opts(kind=rte.RTE_VOLUME, leaf_size=32, aca_eps=1e-4)
    kap = field(n)
    mesh = rte.rte_mesh_create(n)
    base = fresh()

    def product(H):
        y = torch.empty((1, mesh.N), device=DEV, dtype=torch.float64)
        return rte.rte_hmat_matvec(H, 0, torch.ones_like(y), y)

    def assembled(cap):
        rte.rte_release_scratch()
        monkeypatch.setenv("RTE_MEMORY_CAP", str(base + cap))
        try:
            H = rte.rte_hmat_assemble(mesh, kap, opts)
        except rte.RteError as e:
            assert e.status == rte.RTE_E_OUT_OF_MEMORY
            return None
        finally:
            monkeypatch.delenv("RTE_MEMORY_CAP")
        return product(H)

    monkeypatch.setenv("RTE_STAR_TABLE", "0")
    want = product(rte.rte_hmat_assemble(mesh, kap, opts))
    lo, hi = 0, 2048 * MB
    while hi - lo > 4 * MB:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if assembled(mid) is not None else (mid, hi)
    monkeypatch.delenv("RTE_STAR_TABLE")
    assert 8 * MB < hi < 2048 * MB
    got = assembled(hi)
    assert got is not None and torch.equal(got, want)
    assert assembled(4 * MB) is None
    assert fresh() == base


@pytest.mark.parametrize("precision", [rte.RTE_FP64, rte.RTE_FP32], ids=["fp64", "fp32"])
def test_second_pass_keeps_what_its_bound_allows(monkeypatch, precision):
    """Blocks that reach the first rank cap go on from where they stopped, or start again where their factors would be
    more than the bound: the same operator with all, some and none of them kept.  Where memory is just enough for an
    assembly that keeps none, one that would keep all of them still succeeds."""
    import numpy as np
    n = (15, 14, 13)
    opts = rte.hmat_opts(kind=rte.RTE_VOLUME, leaf_size=24, aca_eps=1e-7, precision=precision)
    kap = field(n)
    mesh = rte.rte_mesh_create(n, emit_faces=inputs.FACE_X_LO, walls=[(2, 0, 0.5)])
    monkeypatch.setenv("RTE_ACA_FIRST_CAP", "16")
    monkeypatch.setenv("RTE_STAR_TABLE", "0")
    base = fresh()

    def assembled(keep, cap=None):
        rte.rte_release_scratch()
        monkeypatch.setenv("RTE_ACA_CARRY", str(keep))
        if cap is not None:
            monkeypatch.setenv("RTE_MEMORY_CAP", str(base + cap))
        try:
            H = rte.rte_hmat_assemble(mesh, kap, opts)
        except rte.RteError as e:
            assert e.status == rte.RTE_E_OUT_OF_MEMORY
            return None
        finally:
            monkeypatch.delenv("RTE_MEMORY_CAP", raising=False)
        st = rte.rte_hmat_stats(H)
        return st["aca_retried"], st["aca_entries"], [rte.rte_hmat_block_factors(H, 0, b) for b in range(st["n_lowrank"])]

    everything = 1 << 40
    retried, all_entries, kept = assembled(everything)
    assert retried > 20
    entries = [all_entries]
    for keep in (32 << 10, 0):
        r, e, got = assembled(keep)
        assert r == retried
        entries.append(e)
        for (ka, ua, va), (kb, ub, vb) in zip(kept, got):
            assert ka == kb and (ka <= 0 or (np.array_equal(ua, ub) and np.array_equal(va, vb)))
    assert entries[0] < entries[1] < entries[2]   # a block that starts again evaluates its rows again
    lo, hi = 0, 2048 * MB
    while hi - lo > 2 * MB:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if assembled(0, mid) is not None else (mid, hi)
    assert assembled(everything, hi) is not None
    assert fresh() == base
