"""Gradients of more samples than one pass of the reduction holds (256 partial rows of 32 samples).

The gradient is the sum of the batches of 32 in order, in FP32.  A batch's own gradient differs from
its share in a larger one of 2^k batches by the factor 2^-k, which is exact, so the sum of the shares
gives the gradient, and the loss, bit for bit.  Ragged numbers against the oracle with the bars of the
gradient test; the loss of many samples (its partials too take several passes) within n u of the
forward pass's, n the number of partials.
"""
import numpy as np
import pytest

import synth
from oracle import mlp as om

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_20787_amd as m
    return m


def samples(B):
    rng = np.random.default_rng(B)
    return (rng.uniform(-1, 1, (2, B)).astype(np.float32), (rng.standard_normal((2, B)) * 0.5).astype(np.float32))


@pytest.mark.parametrize("B", [8192, 16384, 32768])
def test_gradient_is_the_sum_of_its_batches_in_order(sc, B):
    print(f"[case] reduction B={B}", flush=True)
    F, T = (torch.from_numpy(a).cuda() for a in samples(B))
    net = sc.Mlp.create(synth.mlp_init(seed=7, out_gain=1.0))
    g, loss = net.grad(F, T)
    again, _ = net.grad(F, T)
    assert torch.equal(g, again)
    rows = []
    for b in range(0, B, 32):
        q, l = net.grad(F[:, b:b + 32].contiguous(), T[:, b:b + 32].contiguous())
        rows.append(np.append(q.cpu().numpy(), l.cpu().numpy().reshape(-1)[:1]))
    rows = np.array(rows, dtype=np.float32) * np.float32(32.0 / B)
    total = np.zeros(rows.shape[1], dtype=np.float32)
    for r in rows:
        total += r
    np.testing.assert_array_equal(g.cpu().numpy(), total[:-1])
    assert float(loss.cpu()) == float(total[-1])
    net.close()


@pytest.mark.parametrize("B", [8191, 8193, 20011])
def test_ragged_gradients_match_the_oracle(sc, B):
    print(f"[case] ragged B={B}", flush=True)
    p = synth.mlp_init(seed=7, out_gain=1.0)
    F, T = samples(B)
    net = sc.Mlp.create(p)
    g, loss = net.grad(torch.from_numpy(F).cuda(), torch.from_numpy(T).cuda())
    g = g.cpu().numpy().astype(np.float64)
    lref, gref = om.loss_and_grad(p.astype(np.float64), F.astype(np.float64), T.astype(np.float64), bf16=True)
    assert float(loss.cpu()) == pytest.approx(lref, rel=1e-4)
    off = 0
    for name, shape in om.param_shapes():
        n = int(np.prod(shape))
        assert np.linalg.norm(g[off:off + n] - gref[off:off + n]) < 1e-3 * np.linalg.norm(gref[off:off + n]), name
        off += n
    net.close()


@pytest.mark.parametrize("B", [524288, 600011])
def test_loss_of_many_samples(sc, B):
    print(f"[case] loss B={B}", flush=True)
    F, T = (torch.from_numpy(a).cuda() for a in samples(B))
    net = sc.Mlp.create(synth.mlp_init(seed=7, out_gain=1.0))
    _, loss = net.grad(F, T)
    ref = ((net.forward(F).double() - T.double()) ** 2).sum().item() / (2 * B)
    assert float(loss.cpu()) == pytest.approx(ref, rel=(B + 31) // 32 * 6e-8)
    net.close()
