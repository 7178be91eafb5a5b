"""The forms of the octree walk that the number of groups selects: four, two waves or one per group
of at most 64 particles (CIC up to about 1100, up to 3300 groups and above, TSC 1600 and 16384).

A heap of massless particles in a corner of the root cube adds groups and nothing else: every other
group accepts it as the same massless cell, whatever its number, so its particles keep their list of
sources and its sums their order, and the forces have to be equal bit for bit in all three forms.
The smallest is compared with the oracle elsewhere.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R = synth.r_max()
N = 20000


@pytest.fixture(scope="module")
def sc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_20787_amd as m
    return m


def forces(sc, p, heap, tab, order, leaf, theta):
    rng = np.random.default_rng(1)
    corner = np.array([1.3 * R, 1.3 * R, 0.5 * p.L])
    pos = np.concatenate([p.pos, corner[:, None] + 1e-3 * (rng.random((3, heap)) - 0.5)], axis=1)
    m = np.concatenate([p.mass, np.zeros(heap)])
    e = np.concatenate([p.eps, np.full(heap, 1e-6)])  # small: the heap is not all one softened cell
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (pos, m, e)]
    t = sc.Octree(leaf)
    a = sc.steps_cyl_tree_forces(t, *d, p.L, R, tab, order, theta, 0.0, 0.0)
    torch.cuda.synchronize()
    assert torch.isfinite(a).all()
    t.close()
    return a[:, :p.N]


@pytest.mark.parametrize("complete", [False, True])
@pytest.mark.parametrize("order,heaps", [(1, (70000, 100003, 300000)), (2, (90000, 120007, 1200000))])
@pytest.mark.parametrize("kind", ["plain", "clumps"])
def test_waves_per_group_give_the_same_bits(sc, order, heaps, complete, kind):
    print(f"[case] walk order={order} complete={complete} {kind}", flush=True)
    p = synth.cylinder_load(N, seed=3) if kind == "plain" else synth.clustered_load(N, n_clumps=8, clump_frac=0.05, seed=3)
    # rho up to 4.5: some pairs lie beyond the table
    tab = sc.CorrectionTable.ewald(32, 36, 4.5, 2.0, 5, 12) if complete else sc.CorrectionTable(32, 36, 4.5, 64)
    for leaf, theta in ((16, 0.5), (3, 0.9)):
        ref = forces(sc, p, 100, tab, order, leaf, theta)
        for heap in heaps:
            assert torch.equal(forces(sc, p, heap, tab, order, leaf, theta), ref), (heap, leaf)
    tab.close()
