"""Training gradients at row counts around the partial sums: one workgroup, a
ragged last tile, sums over 15 to 17, 33 and the most workgroups, and the
fused update against the gradient and the update by themselves."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def data(rows):
    rng = np.random.default_rng(rows)
    p = np.zeros(oracle.N_PARAMS, dtype=np.float32)
    for name, scale in (("W1", 0.5), ("W2", 0.18), ("W3", 0.13), ("b1", 0.1), ("b2", 0.1)):
        a, b = oracle.PARAM_SLICES[name]
        p[a:b] = rng.normal(0, scale, b - a)
    x = rng.random((rows, 8)).astype(np.float32)
    y = (rng.random(rows) < 0.3).astype(np.float32)
    return p, x, y


@pytest.mark.parametrize("rows", [1, 33, 128, 129, 15 * 128, 17 * 128, 33 * 128 - 5, 256 * 128 + 77])
def test_gradient_and_step(rows):
    import paper_2303_02650_amd as P

    p, x, y = data(rows)
    dev = lambda a: torch.from_numpy(a).cuda()
    loss, g = P.mlp_grad(dev(p), dev(x), dev(y))
    L, ref = oracle.mlp_grad(p.astype(np.float64), x.astype(np.float64), y.astype(np.float64))
    # the backward's BF16 operands: 2^-8 per term, in sums whose terms cancel
    assert loss.item() == pytest.approx(L, rel=1e-3)
    g = g.cpu().numpy().astype(np.float64)
    for name, (a, b) in oracle.PARAM_SLICES.items():
        assert np.linalg.norm(g[a:b] - ref[a:b]) <= 1e-2 * np.linalg.norm(ref[a:b]) + 1e-12, name
    A, B = P.MlpTrainer(dev(p), lr=1e-3, max_rows=rows), P.MlpTrainer(dev(p), lr=1e-3, max_rows=rows)
    for t in range(2):
        la = A.train_step(dev(x), dev(y)).item()
        lb, gb = P.mlp_grad(B.params, dev(x), dev(y))
        P.pecc_mlp_adam(B.params, B.m, B.v, gb, B.step, B.hp)
        assert la == lb.item() and torch.equal(A.grad, gb)
        assert A.step.item() == t + 1 == B.step.item()
        assert torch.equal(A.params, B.params) and torch.equal(A.m, B.m) and torch.equal(A.v, B.v)


def test_workspace_holds_every_smaller_row_count():
    import paper_2303_02650_amd as P

    sizes = [P.pecc_mlp_grad_workspace_size(r) for r in (0, 1, 64, 65, 16384, 16385, 32768, 10**7)]
    assert sizes == sorted(sizes)
    p, x, y = data(16384)
    dev = lambda a: torch.from_numpy(a).cuda()
    T = P.MlpTrainer(dev(p), lr=1e-3, max_rows=16400)
    loss = T.train_step(dev(x), dev(y)).item()
    L, _ = oracle.mlp_grad(p.astype(np.float64), x.astype(np.float64), y.astype(np.float64))
    assert loss == pytest.approx(L, rel=1e-3)
