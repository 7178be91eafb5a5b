"""The *_ws force calls in less workspace than steps_cyl_forces_workspace() names: two sets of sum
slots per particle (1 KiB of sums; one set with a table, 512 bytes with a network) are enough for
the pairwise paths.

Bars, against the path's default schedule: it adds the same terms in FP64 in another order, and may
take a pair from its other side.  With 4 images a pair has the same terms from either side, and the
results are within one FP32 rounding.  With one (tables, networks) the two sides round apart, each
within 5e-7 of the term, and the results are within 1e-6 of the sum of the terms' sizes.

Lists of targets: up to 4096 sources a target's sum has the same order in every list, mode of
launching and workspace, bit for bit; above, the bars of the short lists.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_20787_amd as m
    return m


def to_dev(p):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (p.pos, p.mass, p.eps)]


def nan_bytes(n):
    # full of NaN: every slot is written before it is added to; off the allocation's alignment
    return torch.full((n + 64,), 255, dtype=torch.uint8, device="cuda:0")[64:]


def order_bytes(sc, N):
    """The spatial order's share: what a tabulated call on a list of N targets takes."""
    tab = sc.CorrectionTable(8, 8, 4.0, 8)
    n = sc.steps_cyl_forces_workspace(sc.STEPS_PATH_TABLE, N, 0, max(N, 4096), 0, table=tab, order=1)
    tab.close()
    return n


def over_terms(a, b, d, L):
    """Largest difference of accelerations over the sum of the terms' sizes."""
    (x, y, z), m, e = d
    worst = 0.0
    for i in range(0, m.numel(), 500):
        dz = z[i:i + 500, None] - z[None]
        dz = dz - L * torch.floor(dz / L + 0.5)
        r2 = (x[i:i + 500, None] - x[None]) ** 2 + (y[i:i + 500, None] - y[None]) ** 2 + dz ** 2
        h = e[i:i + 500, None] + e[None]
        # inside the softening length the spline's force is at most 2.2 / h^2
        size = (m / torch.maximum(r2, h * h / 2.2)).sum(1)
        worst = max(worst, (torch.linalg.norm((a - b)[:, i:i + 500].double(), dim=0) / size).max().item())
    return worst


def one_rounding(a, b):
    scale = torch.linalg.norm(b.double(), dim=0) if b.dim() == 2 else torch.abs(b.double())
    return (torch.abs(a.double() - b.double()) / scale).max().item() <= 1.2e-7


@pytest.mark.parametrize("N", [2305, 4000, 10240, 15296, 31745])
def test_exact(sc, N):
    print(f"[case] exact N={N}", flush=True)
    p = synth.cylinder_load(N, seed=N)
    d = to_dev(p)
    full = sc.steps_cyl_forces_workspace(sc.STEPS_PATH_EXACT, N, 4, 0, sc.STEPS_SUM_PAIRWISE)
    need = order_bytes(sc, N) + (32 + 1 + 64 * 16) * N + 4096
    assert need < full
    acc, pot = sc.steps_cyl_forces(*d, p.L, 4)
    for w in (need, full - 4096):
        a, q = sc.steps_cyl_forces_ws(*d, p.L, 4, nan_bytes(w))
        b, r = sc.steps_cyl_forces_ex_ws(*d, p.L, 4, nan_bytes(w), mode=sc.STEPS_SUM_PAIRWISE)
        assert torch.equal(a, b) and torch.equal(q, r)
        assert one_rounding(a, acc) and one_rounding(q, pot)
    with pytest.raises(sc.StepsError, match="workspace"):
        sc.steps_cyl_forces_ws(*d, p.L, 4, nan_bytes((32 + 64 * 16) * N))


@pytest.mark.parametrize("N", [2305, 4600, 10240, 20011])
@pytest.mark.parametrize("order", [1, 2])
def test_table(sc, N, order):
    print(f"[case] table N={N} order={order}", flush=True)
    p = synth.cylinder_load(N, seed=N)
    d = to_dev(p)
    tab = sc.CorrectionTable(32, 36, 6.4, 64)
    full = sc.steps_cyl_forces_workspace(sc.STEPS_PATH_TABLE, N, 0, 0, 0, table=tab, order=order)
    need = order_bytes(sc, N) + (32 + 1 + 64 * 8) * N + 4096
    assert need < full
    acc, pot = sc.steps_cyl_forces_table(*d, p.L, tab, order=order)
    a, q = sc.steps_cyl_forces_table_ws(*d, p.L, tab, nan_bytes(need), order=order)
    assert over_terms(a, acc, d, p.L) <= 1e-6 and (torch.abs(q - pot) / torch.abs(pot)).max().item() <= 1e-6
    tab.close()


@pytest.mark.parametrize("N", [1, 129, 2049, 5000, 10240, 21633])
def test_learned(sc, N):
    print(f"[case] learned N={N}", flush=True)
    p = synth.cylinder_load(N, seed=N)
    d = to_dev(p)
    net = sc.Mlp.create(synth.mlp_init(seed=21, out_gain=1.0))
    full = sc.steps_cyl_forces_workspace(sc.STEPS_PATH_LEARNED, N, 0, 0, sc.STEPS_SUM_PAIRWISE)
    need = order_bytes(sc, N) + (32 + 64 * 8) * N + 1024
    acc, pot = sc.steps_cyl_forces_learned(*d, p.L, net)
    a, q = sc.steps_cyl_forces_learned_ws(*d, p.L, net, nan_bytes(need))
    if N == 1:
        assert not a.any() and not q.any()
    else:
        assert need < full or N < 1000
        assert over_terms(a, acc, d, p.L) <= 1e-6 and (torch.abs(q - pot) / torch.abs(pot)).max().item() <= 1e-6
    net.close()


# ---- lists of targets: the totals of the source chunks


def lists(N, long):
    rng = np.random.default_rng(N)
    for T in (1, 300, 4097, long):
        yield torch.from_numpy(rng.integers(0, N, T)).cuda()


@pytest.mark.parametrize("N", [256, 257, 1025, 3000, 4096])
@pytest.mark.parametrize("mode", ["compensated", "plain"])
def test_few_sources_give_the_same_bits_in_every_list(sc, N, mode):
    # 131,073 targets and more leave no room for chunks on the device
    print(f"[case] lists N={N} {mode}", flush=True)
    p = synth.cylinder_load(N, seed=N)
    d = to_dev(p)
    m = sc.STEPS_SUM_COMPENSATED if mode == "compensated" else sc.STEPS_SUM_PLAIN
    for n_img in (0, 1, 2, 3, 4, 8):
        acc, pot = sc.steps_cyl_forces_ex(*d, p.L, n_img, mode=m)
        only, _ = sc.steps_cyl_forces_ex(*d, p.L, n_img, mode=m, potential=False)
        for t in lists(N, 140003):
            a, q = sc.steps_cyl_forces_ex(*d, p.L, n_img, targets=t, mode=m)
            assert torch.equal(a, acc[:, t]) and torch.equal(q, pot[t]), (n_img, t.numel())
            # a workspace of the spatial order alone
            n = t.numel()
            w = nan_bytes(order_bytes(sc, n) + 256 if n >= 4096 else 256)
            a, q = sc.steps_cyl_forces_ex_ws(*d, p.L, n_img, w, targets=t, mode=m)
            assert torch.equal(a, acc[:, t]) and torch.equal(q, pot[t]), (n_img, n)
            a, _ = sc.steps_cyl_forces_ex_ws(*d, p.L, n_img, w, targets=t, mode=m, potential=False)
            assert torch.equal(a, only[:, t]), (n_img, n)


@pytest.mark.parametrize("N", [1024, 1025, 4096])
def test_few_sources_give_the_same_bits_with_a_network(sc, N):
    print(f"[case] learned lists N={N}", flush=True)
    p = synth.cylinder_load(N, seed=N)
    d = to_dev(p)
    net = sc.Mlp.create(synth.mlp_init(seed=21, out_gain=1.0))
    acc, pot = sc.steps_cyl_forces_learned_ex(*d, p.L, net)
    for t in lists(N, 350003):
        a, q = sc.steps_cyl_forces_learned_ex(*d, p.L, net, targets=t)
        assert torch.equal(a, acc[:, t]) and torch.equal(q, pot[t]), t.numel()
        n = t.numel()
        a, q = sc.steps_cyl_forces_learned_ex_ws(*d, p.L, net, nan_bytes(order_bytes(sc, n) + 256 if n >= 4096 else 256),
                                                 targets=t)
        assert torch.equal(a, acc[:, t]) and torch.equal(q, pot[t]), n
    net.close()


# chunk totals in the room of 2048 workgroups of at least 4096 sources
@pytest.mark.parametrize("N,T", [(4097, 100), (20011, 300), (60000, 5000)])
def test_lists_in_less_workspace(sc, N, T):
    print(f"[case] lists N={N} T={T}", flush=True)
    p = synth.cylinder_load(N, seed=N)
    d = to_dev(p)
    t = torch.from_numpy(np.random.default_rng(T).choice(N, size=T, replace=False).astype(np.int64)).cuda()
    ref, ref_pot = sc.steps_cyl_forces_f64(*d, p.L, 2, targets=t)
    net = sc.Mlp.create(synth.mlp_init(seed=21, out_gain=1.0))
    far, far_pot = sc.steps_cyl_forces_learned_ex(*d, p.L, net, targets=t)
    for block, path in ((256, sc.STEPS_PATH_EXACT), (128, sc.STEPS_PATH_LEARNED)):
        chunks = min(-(-2048 // -(-T // block)), -(-N // 4096))
        w = nan_bytes((order_bytes(sc, T) if T >= 4096 else 0) + 32 * chunks * T + 512)
        full = sc.steps_cyl_forces_workspace(path, N, 2, T, sc.STEPS_SUM_COMPENSATED)
        assert w.numel() < full
        if path == sc.STEPS_PATH_EXACT:
            a, q = sc.steps_cyl_forces_ex_ws(*d, p.L, 2, w, targets=t)
            r, rq = ref, ref_pot
        else:
            a, q = sc.steps_cyl_forces_learned_ex_ws(*d, p.L, net, w, targets=t)
            r, rq = far, far_pot
        # FP32 sums of 32 terms: 32 roundings of 6e-8, and the terms' own 5e-7
        (x, y, z), m, e = d
        dz = z[t, None] - z[None]
        dz = dz - p.L * torch.floor(dz / p.L + 0.5)
        r2 = (x[t, None] - x[None]) ** 2 + (y[t, None] - y[None]) ** 2 + dz ** 2
        size = (m / torch.maximum(r2, (e[t, None] + e[None]) ** 2 / 2.2)).sum(1)
        assert (torch.linalg.norm((a - r).double(), dim=0) / size).max().item() <= 2.5e-6
        assert (torch.abs(q - rq) / torch.abs(rq)).max().item() <= 2.5e-6
    with pytest.raises(sc.StepsError, match="workspace"):
        sc.steps_cyl_forces_ex_ws(*d, p.L, 2, nan_bytes(32), targets=t)
    net.close()
