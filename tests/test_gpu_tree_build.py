"""The octree where its build and walk change form: trees of one cell and one
particle more, leaves of 1 and 64, workgroups of particles full and ragged,
coincident particles down to level 21, the widest frontier (theta = 0), groups
of 1 to 64 particles.

Bars: the structure and the interaction counts are integers and equal the
oracle's; masses and centres to FP64 rounding.  theta = 0 sums the particles
alone: the same FP32 pair terms as the per-target table kernel, both in runs of
at most 64 terms with compensated totals, within 2 x 64 roundings of 6e-8 of the
sum of the terms' sizes.
"""
import numpy as np
import pytest

import synth
from oracle import octree as oc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

R = synth.r_max()


@pytest.fixture(scope="module")
def sc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_20787_amd as m
    return m


def to_dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def load(N, kind):
    p = synth.cylinder_load(N, seed=N + 5)
    pos, eps = p.pos.copy(), p.eps
    if kind == "coincident":
        # two heaps of equal positions: leaves of level 21
        pos[:, : N // 3] = pos[:, :1]
        pos[:, N // 3: N // 2] = pos[:, N // 3: N // 3 + 1]
    return pos, p.mass, eps, p.L


@pytest.mark.parametrize("N,leaf,kind", [(1, 1, "plain"), (2, 1, "plain"), (16, 16, "plain"), (17, 16, "plain"),
                                         (64, 64, "plain"), (65, 64, "plain"), (255, 1, "plain"), (256, 2, "plain"),
                                         (257, 64, "plain"), (513, 3, "plain"), (300, 16, "coincident"),
                                         (700, 64, "coincident"), (90, 1, "coincident")])
@pytest.mark.parametrize("quad", [False, True])
def test_structure_and_counts(sc, N, leaf, kind, quad):
    print(f"[case] N={N} leaf={leaf} {kind} quad={quad}", flush=True)
    pos, m, e, L = load(N, kind)
    t = sc.Octree(leaf, quadrupole=quad)
    tab = sc.CorrectionTable.ewald(16, 12, 6.5, 2.0, 5, 12)
    d = to_dev(pos, m, e)
    a = sc.steps_cyl_tree_forces(t, *d, L, R, tab, 1, 0.6, 0.3, 1.2)
    b = sc.steps_cyl_tree_forces(t, *d, L, R, tab, 1, 0.6, 0.3, 1.2)
    assert torch.equal(a, b) and torch.isfinite(a).all()
    g = sc.steps_cyl_tree_cells(t, N)
    T = oc.Tree(pos, m, e, L, R, 0.3, 1.2, leaf)
    np.testing.assert_array_equal(g["order"], T.order)
    np.testing.assert_array_equal(g["level"], T.level)
    np.testing.assert_array_equal(g["start"], T.start)
    np.testing.assert_array_equal(g["count"], T.end - T.start)
    np.testing.assert_array_equal(g["skip"], T.skip)
    np.testing.assert_array_equal(g["leaf"].astype(bool), T.leaf)
    np.testing.assert_allclose(g["mass"], T.mass, rtol=1e-12)
    np.testing.assert_allclose(g["com"], T.com, rtol=1e-11, atol=1e-12)
    t.close()
    tab.close()


@pytest.mark.parametrize("N,leaf,complete", [(200, 1, True), (3000, 1, False), (9000, 16, True), (20011, 64, False)])
def test_every_cell_opened(sc, N, leaf, complete):
    print(f"[case] theta=0 N={N} leaf={leaf}", flush=True)
    pos, m, e, L = load(N, "plain")
    t = sc.Octree(leaf)
    tab = sc.CorrectionTable.ewald(32, 36, 4.5, 2.0, 5, 12) if complete else sc.CorrectionTable(32, 36, 4.5, 64)
    d = to_dev(pos, m, e)
    a = sc.steps_cyl_tree_forces(t, *d, L, R, tab, 1, 0.0, 0.0, 0.0)
    n_cells, n_c, n_p = sc.steps_cyl_tree_info(t)
    assert n_c == 0 and n_p == N * N
    tg = torch.arange(N, dtype=torch.int64, device="cuda:0")
    ref, _ = sc.steps_cyl_forces_table(*d, L, tab, order=1, targets=tg, potential=False)
    # sizes of the terms: the nearest image, the largest
    size = torch.zeros(N, dtype=torch.float64, device="cuda:0")
    for i in range(0, N, 500):
        s = [d[0][c, i:i + 500, None] - d[0][c][None] for c in range(3)]
        s[2] = s[2] - L * torch.floor(s[2] / L + 0.5)
        h = d[2][i:i + 500, None] + d[2][None]
        size[i:i + 500] = (d[1] / torch.maximum(s[0] ** 2 + s[1] ** 2 + s[2] ** 2, h * h / 2.2)).sum(1)
    err = (torch.linalg.norm(a.double() - ref.double(), dim=0) / size).max().item()
    print(f"difference over the terms' sizes {err:.2e}")
    assert err <= 2 * 64 * 6e-8
    t.close()
    tab.close()


@pytest.mark.parametrize("N", [700, 2500])
@pytest.mark.parametrize("quad", [False, True])
def test_interaction_counts(sc, N, quad):
    # groups of many sizes: what is accepted and opened equals the oracle's
    p = synth.clustered_load(N, n_clumps=4, clump_frac=0.1, seed=9)
    t = sc.Octree(4, quadrupole=quad)
    tab = sc.CorrectionTable.ewald(16, 12, 6.5, 2.0, 5, 12)
    for theta in (0.4, 1.1):
        sc.steps_cyl_tree_forces(t, *to_dev(p.pos, p.mass, p.eps), p.L, R, tab, 2, theta, 0.6, 2.5)
        st = {}
        from oracle import table as ot
        oc.tree_forces(p.pos, p.mass, p.eps, p.L, R, ot.Table(16, 12, 6.5), 1, theta, 0.6, 2.5, leaf_size=4, group=64,
                       stats=st, quadrupole=False)
        assert sc.steps_cyl_tree_info(t) == (st["cells"], st["cell_interactions"], st["particle_interactions"])
    t.close()
    tab.close()
