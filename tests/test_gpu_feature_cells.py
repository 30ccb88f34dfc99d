"""Candidate features against the oracle where their search changes its way:
sizes around a wave and a workgroup, cell rows longer than a mask, distances
of exactly 2 and 4 and one FP32 step to either side, points outside the
container, coordinates that are not finite, candidate counts that leave lanes
or threads over."""
import math

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def layout(kind, n, rng):
    R = max(2.5, float(np.sqrt(n / 0.84)))
    x = synth.disk_uniform(n, R, rng)
    m = int(np.ceil(np.sqrt(n)))
    if kind == "dense":                         # rows around the mask's length
        x *= 0.62
    elif kind == "cluster":
        x = rng.uniform(-1.0, 1.0, size=(n, 2)) + 0.3 * R
    elif kind == "outside":
        x = x * rng.uniform(0.5, 3.0, size=(n, 1))
    elif kind == "square":                      # distances 2 and 4 exactly
        x = 2.0 * np.array([(i % m, i // m) for i in range(n)], dtype=np.float64) - m
        R = 1.5 * m + 1.0
    elif kind == "steps":                       # the same, one step off
        x = 2.0 * np.array([(i % m, i // m) for i in range(n)], dtype=np.float64) - m
        x = np.nextafter(x.astype(np.float32), rng.choice([-1e9, 0.0, 1e9], size=x.shape).astype(np.float32))
        x = x.astype(np.float64)
        R = 1.5 * m + 1.0
    return x, R


@pytest.mark.parametrize("kind", ["random", "dense", "cluster", "outside", "square", "steps"])
@pytest.mark.parametrize("n,C", [(1, 1), (2, 63), (63, 64), (65, 65), (511, 513), (513, 1025), (1000, 1023),
                                 (1024, 1536)])
def test_features_match_oracle(kind, n, C):
    import paper_2303_02650_amd as P

    rng = synth.rng_for(11 * n + C)
    x, R = layout(kind, n, rng)
    y, Q = layout(kind, max(1, n // 2), rng)
    inst = synth.pack([x, y], [R, Q])
    cc, cd = synth.candidates(inst, C, rng)
    for b in range(2):                          # some destinations on other circles, or a lattice step away
        p = inst.instance(b)
        pick = rng.integers(0, len(p), size=C // 2)
        cd[b, : C // 2] = p[pick] + rng.choice([0.0, 2.0, 4.0], size=(C // 2, 2)).astype(np.float32)
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    f = P.features(d, torch.from_numpy(inst.xy.reshape(-1).copy()).cuda(),
                   torch.from_numpy(cc.reshape(-1).copy()).cuda(),
                   torch.from_numpy(cd.reshape(-1).copy()).cuda()).cpu().numpy().reshape(2, C, 8)
    for b in range(2):
        ref = oracle.features(inst.instance(b), inst.R[b], cc[b], cd[b])
        for col in (1, 5):
            assert np.array_equal(f[b][:, col], ref[:, col])
        for col in (3, 7):
            assert np.array_equal(np.round(f[b][:, col] * 16 * math.pi), np.round(ref[:, col] * 16 * math.pi))
        # the FP64 sums differ by their order; values of order 1 stored in FP32
        np.testing.assert_allclose(f[b], ref, rtol=2e-7, atol=1e-6)


@pytest.mark.parametrize("bad", [np.nan, -np.nan, np.inf, -np.inf])
def test_non_finite(bad):
    """A circle at no finite place is near nothing: the other circles' features
    are those of the layout without it; a point at no finite place has no
    neighbors."""
    import paper_2303_02650_amd as P

    rng = synth.rng_for(3)
    x, R = layout("random", 300, rng)
    inst = synth.pack([x[:299]], [R])
    C = 200
    cc, cd = synth.candidates(inst, C, rng)
    run = lambda I, c, q: P.features(
        P.DeviceInstances.from_host(I.offset, I.R), torch.from_numpy(I.xy.reshape(-1).copy()).cuda(),
        torch.from_numpy(c.reshape(-1).copy()).cuda(), torch.from_numpy(q.reshape(-1).copy()).cuda())
    want = run(inst, cc, cd)
    x[299] = (bad, 0.5)
    full = synth.pack([x], [R])
    assert torch.equal(run(full, cc, cd), want)
    cd[0, 5] = (0.25, bad)
    cc[0, 6] = 299
    got = run(full, cc, cd).cpu().numpy().reshape(C, 8)
    want = want.cpu().numpy().reshape(C, 8)
    assert np.array_equal(got[:5], want[:5]) and np.array_equal(got[7:], want[7:])
    assert np.array_equal(got[5, :4], want[5, :4]) and got[5, 5] == 0 and got[5, 7] == 0
    assert got[6, 1] == 0 and got[6, 3] == 0
