"""Training gradients at the edges of the present split: fewer partial sums than
the reduction has shares, 63 to 65 of them, the most, and the row count where a
wave's turn takes two tiles."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def data(rows):
    rng = np.random.default_rng(rows + 1)
    p = np.zeros(oracle.N_PARAMS, dtype=np.float32)
    for name, scale in (("W1", 0.5), ("W2", 0.18), ("W3", 0.13), ("b1", 0.1), ("b2", 0.1)):
        a, b = oracle.PARAM_SLICES[name]
        p[a:b] = rng.normal(0, scale, b - a)
    return p, rng.random((rows, 8)).astype(np.float32), (rng.random(rows) < 0.3).astype(np.float32)


# one tile per turn: 1 to 5, 63 to 65, 255 and 256 partial sums; two: beyond
@pytest.mark.parametrize("rows", [1, 64, 65, 129, 193, 257, 63 * 64, 63 * 64 + 1, 64 * 64 + 1, 8192, 255 * 64,
                                  16384, 16385, 20000])
def test_partial_sums(rows):
    import paper_2303_02650_amd as P

    p, x, y = data(rows)
    pd, xd, yd = (torch.from_numpy(a).cuda() for a in (p, x, y))
    L, ref = oracle.mlp_grad(p.astype(np.float64), x.astype(np.float64), y.astype(np.float64))
    size = P.pecc_mlp_grad_workspace_size(rows)
    buf = torch.full((size + 1024,), 0x5A, dtype=torch.uint8, device="cuda")
    loss, g = P.mlp_grad(pd, xd, yd, workspace=buf[:size])
    assert (buf[size:] == 0x5A).all()
    # the backward's BF16 operands: 2^-8 per term, in sums whose terms cancel
    assert loss.item() == pytest.approx(L, rel=1e-3)
    h = g.cpu().numpy().astype(np.float64)
    for name, (a, b) in oracle.PARAM_SLICES.items():
        assert np.linalg.norm(h[a:b] - ref[a:b]) <= 1e-2 * np.linalg.norm(ref[a:b]) + 1e-12, name
    T, U = P.MlpTrainer(pd, max_rows=rows), P.MlpTrainer(pd, max_rows=rows)
    assert T.train_step(xd, yd).item() == loss.item() and torch.equal(T.grad, g)
    P.pecc_mlp_adam(U.params, U.m, U.v, g, U.step, U.hp)
    assert torch.equal(T.params, U.params) and torch.equal(T.m, U.m) and torch.equal(T.v, U.v)
