"""Neighbor lists inside the descent: the listed-pair count of the first
evaluation (a descent with no iterations) against the FP64 oracle's pair set,
at the sizes and densities where the list build changes its way: a last
wave that is nearly empty, cell rows of more than 32 candidates, more than 64
candidates around a circle, lists that do not fit, distances on the cutoff."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def layouts(kind, n):
    rng = synth.rng_for(1000 + n)
    R = max(3.0, np.sqrt(n / 0.84))
    if kind == "random":
        return synth.disk_uniform(n, R, rng), R
    if kind == "strip":            # one long cell row holds 33 .. 64 candidates
        x = synth.disk_uniform(n, R, rng)
        m = min(n, 48)
        x[:m, 0] = rng.uniform(-3.0, 3.0, m)
        x[:m, 1] = rng.uniform(0.0, 0.4, m)
        return x, R
    if kind == "cluster":          # far more candidates than a mask holds
        return rng.uniform(-1.5, 1.5, size=(n, 2)), R
    # a square lattice on the cutoff itself (2.5): exactly at it, one
    # FP32 step inside it, or outside
    m = int(np.ceil(np.sqrt(n)))
    x = 2.5 * np.array([(i % m, i // m) for i in range(n)], dtype=np.float64) - 1.25 * m
    x = x.astype(np.float32)
    step = rng.integers(0, 3, size=x.shape)
    x = np.where(step == 1, np.nextafter(x, np.float32(-1e3)), x)
    x = np.where(step == 2, np.nextafter(x, np.float32(1e3)), x)
    return x.astype(np.float64), 2.0 * m + 2.0


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 256, 257, 511, 512, 513, 1000, 1024])
@pytest.mark.parametrize("kind", ["random", "strip", "cluster", "lattice"])
def test_listed_pairs_of_first_evaluation(kind, n):
    import paper_2303_02650_amd as P

    x, R = layouts(kind, n)
    inst = synth.pack([x], [R])
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    prm = P.DescentParams(max_iter=0, cutoff=2.5, skin_half=0.25, g_tol=0.0, ftol=0.0, tau64=0.0)
    res = P.results(P.lbfgs_descend(d, xy, prm))[0]
    pi, _ = oracle.neighbors(inst.instance(0), 2.5)
    assert res["evals"] == 1
    assert res["pair_evals"] == len(pi)
    E, *_ = oracle.energy_grad(inst.instance(0).astype(np.float64), R)
    # FP32 sums of n circles' terms: 1e-5 relative, the bound of the energy
    # everywhere in these tests
    assert abs(float(res["E32"]) - E) <= 1e-5 * max(E, 1e-6)
