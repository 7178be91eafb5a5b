"""Small calls evaluate every ordered pair, so a pair's two sides are computed apart: they have to
be each other's negative bit for bit, with images, softened images, and tables inside and beyond
their range, for total momentum to be conserved to the rounding of the FP64 sums.  Two particles
of unit mass show a pair's term alone.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L = 1.0


@pytest.fixture(scope="module")
def sc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_20787_amd as m
    return m


def pairs(n, rho, seed):
    """n pairs of positions [n, 3, 2], separated by up to `rho` across and any way along (some not at all)."""
    rng = np.random.default_rng(seed)
    pos = np.empty((n, 3, 2))
    r, phi = rho * np.sqrt(rng.random(n)), 2.0 * np.pi * rng.random(n)
    first = rng.standard_normal((n, 3))
    pos[:, :, 0] = first
    pos[:, 0, 1] = first[:, 0] + r * np.cos(phi)
    pos[:, 1, 1] = first[:, 1] + r * np.sin(phi)
    # off the half period, where both sides may take the same image
    pos[:, 2, 1] = first[:, 2] + np.where(np.arange(n) % 8 == 0, 0.0, 0.49 * (2.0 * rng.random(n) - 1.0))
    return torch.from_numpy(pos).cuda()


def check(call, pos, eps):
    m, e = torch.ones(2, dtype=torch.float64, device="cuda"), torch.full((2,), eps, dtype=torch.float64, device="cuda")
    acc = torch.stack([call(p.contiguous(), m, e)[0] for p in pos])
    torch.cuda.synchronize()
    assert torch.isfinite(acc).all() and acc.any()
    assert torch.equal(acc[:, :, 0], -acc[:, :, 1])


# softening lengths of 0.01 (plain and softened pairs) and 0.3: images n != 0 softened too
@pytest.mark.parametrize("eps", [0.01, 0.3])
@pytest.mark.parametrize("n_img", [0, 1, 2, 3, 4, 8])
def test_exact_pairs_are_antisymmetric(sc, n_img, eps):
    for rho in (0.02, 2.0):
        check(lambda *d: sc.steps_cyl_forces(*d, L, n_img), pairs(100, rho, n_img), eps)
        check(lambda *d: sc.steps_cyl_forces(*d, L, n_img, potential=False), pairs(50, rho, n_img), eps)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("complete", [False, True])
def test_tabulated_pairs_are_antisymmetric(sc, order, complete):
    tab = sc.CorrectionTable.ewald(32, 36, 4.0, 2.0, 5, 12) if complete else sc.CorrectionTable(32, 36, 4.0, 64)
    for rho, eps in ((0.02, 0.01), (3.0, 0.01), (3.0, 0.3), (12.0, 0.01)):  # the last mostly beyond the table
        for pot in (False, True):
            check(lambda *d: sc.steps_cyl_forces_table(*d, L, tab, order=order, potential=pot), pairs(100, rho, order), eps)
    tab.close()
