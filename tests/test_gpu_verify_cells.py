"""FP64 verify against the oracle at the sizes and layouts where its search
for overlapping pairs changes: with and without a grid, cells that hold many
circles, circles outside the container, contacts at distance 2, non-finite
coordinates."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def layout(kind, n):
    rng = synth.rng_for(77 + n)
    R = max(2.5, float(np.sqrt(n / 0.84)))
    x = synth.disk_uniform(n, R, rng)
    if kind == "outside":                       # half the circles past the container
        x = x * rng.uniform(0.5, 3.0, size=(n, 1))
    elif kind == "cluster":                     # one or a few cells hold everything
        x = rng.uniform(-1.0, 1.0, size=(n, 2)) + 0.3 * R
    elif kind == "tiny":                        # one cell for the whole container
        R = 0.9
    elif kind == "contacts":                    # a square lattice at distance 2 -+ one FP32 step
        m = int(np.ceil(np.sqrt(n)))
        x = 2.0 * np.array([(i % m, i // m) for i in range(n)], dtype=np.float64) - m
        x = np.nextafter(x.astype(np.float32), np.float32(0)).astype(np.float64)
        R = 1.5 * m + 1.0
    return x, R


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 66, 255, 256, 257, 511, 1000, 1023, 1024])
@pytest.mark.parametrize("kind", ["random", "outside", "cluster", "tiny", "contacts"])
def test_verify_matches_oracle(kind, n):
    import paper_2303_02650_amd as P

    x, R = layout(kind, n)
    inst = synth.pack([x, x[: max(1, n // 2)]], [R, R])
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    e, mp, mc, f = [t.cpu().numpy() for t in P.verify(d, xy)]
    for b in range(inst.B):
        v = oracle.verify(inst.instance(b), inst.R[b])
        # FP64 sums of at most n^2 / 2 non-negative terms in another order
        assert abs(e[b] - v["E"]) <= 1e-12 * v["E"]
        assert bool(f[b]) == v["feasible"]
        # one rounded difference and one square root each: four FP64 steps of
        # the distance (2) and of the largest |c_i| + 1
        eps = np.finfo(np.float64).eps
        assert abs(mp[b] - v["max_pair_overlap"]) <= 4 * eps * 2.0
        assert abs(mc[b] - v["max_cont_overlap"]) <= 4 * eps * (mc[b] + R + 1.0)


@pytest.mark.parametrize("n", [5, 64, 65, 300])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_coordinate(bad, n):
    import paper_2303_02650_amd as P

    x, R = layout("random", n)
    inst = synth.pack([x, x], [R, R])
    flat = inst.xy.reshape(-1).copy()
    flat[2 * (n // 2) + 1] = bad
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    e, mp, mc, f = [t.cpu().numpy() for t in P.verify(d, torch.from_numpy(flat).cuda())]
    assert np.isnan(e[0]) and np.isnan(mp[0]) and np.isnan(mc[0]) and f[0] == 0
    assert np.isfinite(e[1])
