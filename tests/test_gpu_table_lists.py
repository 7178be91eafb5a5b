"""Tabulated forces on target lists with TSC: tables held in LDS (up to 19456
nodes) and larger ones read through the vector caches, with the workgroup
sizes that the list's length selects.

A target's sum runs over the sources in their own order whatever the list, so
every list gives the same bits.  Against the oracle's tabulated scheme and the
pairwise path (the same scheme) the bound is that of the table tests (FP32 pair
terms), 2e-5, here of the rms acceleration: clumped targets can cancel.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import table as ot

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import paper_2602_20787_amd as m
    return m


# 32, 136 and 137 a side hold 1225, 19321 and 19600 nodes with their ghosts; 262144
# targets fill workgroups of 1024 on every CU
@pytest.mark.parametrize("n_grid", [32, 136, 137])
@pytest.mark.parametrize("complete,pot", [(False, False), (False, True), (True, True)])
def test_tsc_lists(sc, n_grid, complete, pot):
    N = 2063
    print(f"[case] TSC lists grid={n_grid} complete={complete} pot={pot}", flush=True)
    p = synth.clustered_load(N, n_clumps=8, clump_frac=0.02, seed=n_grid)
    d = [torch.from_numpy(x).cuda() for x in (p.pos, p.mass, p.eps)]
    tab = (sc.CorrectionTable.ewald(n_grid, n_grid, 4.0, 2.0, 5, 12) if complete
           else sc.CorrectionTable(n_grid, n_grid, 5.0, 64))
    ref_list = torch.arange(N, dtype=torch.int64, device="cuda")
    acc, q = sc.steps_cyl_forces_table(*d, p.L, tab, order=2, targets=ref_list, potential=pot)
    rng = np.random.default_rng(n_grid)
    for n in (1, 63, 257, 65537, 262144, 262209):
        t = torch.from_numpy(rng.integers(0, N, n)).cuda()
        a, b = sc.steps_cyl_forces_table(*d, p.L, tab, order=2, targets=t, potential=pot)
        torch.cuda.synchronize()
        assert torch.equal(a, acc[:, t]), n
        assert not pot or torch.equal(b, q[t]), n
    # the pairwise path evaluates the same scheme
    full, fpot = sc.steps_cyl_forces_table(*d, p.L, tab, order=2, potential=pot)
    torch.cuda.synchronize()
    rms = torch.linalg.norm(full.double(), dim=0).square().mean().sqrt().item()
    assert torch.linalg.norm(acc.double() - full.double(), dim=0).max().item() <= 2e-5 * rms
    if pot:
        assert (torch.abs(q - fpot) / torch.abs(fpot)).max().item() <= 2e-5
    if not complete:
        tg = np.arange(0, N, 64)
        ref = ot.forces_table(p.pos, p.mass, p.eps, p.L, ot.Table(n_grid, n_grid, 5.0, n_far=64), 2, targets=tg)
        err = np.linalg.norm(acc.double().cpu().numpy()[:, tg] - ref, axis=0)
        assert err.max() <= 2e-5 * rms
    tab.close()


# small tables and a large one past one round of 262144 targets: in the caches with
# workgroups of 128 and of 256 threads, in LDS over two and three rounds
@pytest.mark.parametrize("n_grid", [24, 60, 140])
@pytest.mark.parametrize("n", [98305, 280000, 300000, 327681, 480000, 600000, 786432])
def test_long_tsc_lists(sc, n_grid, n):
    N = 257
    print(f"[case] TSC lists grid={n_grid} n={n}", flush=True)
    p = synth.clustered_load(N, n_clumps=4, clump_frac=0.02, seed=n_grid)
    d = [torch.from_numpy(x).cuda() for x in (p.pos, p.mass, p.eps)]
    tab = sc.CorrectionTable(n_grid, n_grid, 5.0, 64)
    every = torch.arange(N, dtype=torch.int64, device="cuda")
    t = torch.from_numpy(np.random.default_rng(n).integers(0, N, n)).cuda()
    for pot in (False, True):
        acc, q = sc.steps_cyl_forces_table(*d, p.L, tab, order=2, targets=every, potential=pot)
        a, b = sc.steps_cyl_forces_table(*d, p.L, tab, order=2, targets=t, potential=pot)
        torch.cuda.synchronize()
        assert torch.equal(a, acc[:, t])
        assert not pot or torch.equal(b, q[t])
    tab.close()
