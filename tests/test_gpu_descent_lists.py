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


@pytest.mark.parametrize("adjust", [False, True])
@pytest.mark.parametrize("n", [1, 20, 64, 65, 128, 129, 256, 257, 512])
def test_workgroup_shapes_agree(n, adjust):
    """An instance's results do not depend on the workgroup shape: alone (the
    smallest shape that holds it) and under a bound of 1024 circles (the
    full one) they have the same bits, FP64 regime included (tau64 above the
    start energy); so do a batch of 300 and one too large for the device,
    which takes the work queue."""
    import paper_2303_02650_amd as P

    R = max(2.5, float(np.sqrt(n / 0.8)))
    inst = synth.instance_set(3, n, R, seed=n)
    prm = P.DescentParams(max_iter=60, contact_margin=1e-4, ftol=1e-7, tau64=1e3)

    def run(copies, max_n):
        off = np.arange(3 * copies + 1, dtype=np.int32) * n
        d = P.DeviceInstances.from_host(off, np.tile(inst.R, copies))
        d.max_n = max_n
        xy = torch.from_numpy(np.tile(inst.xy.reshape(-1), copies)).cuda()
        if adjust:
            Ro, out = P.adjust_container(d, xy, prm, rounds=2)
            return xy.cpu().numpy(), P.results(out), Ro.cpu().numpy()
        return xy.cpu().numpy(), P.results(P.lbfgs_descend(d, xy, prm)), None

    x0, r0, R0 = run(1, 1024)
    for copies, max_n in ((1, n), (100, n), (1400 if n <= 64 else 400, n)):
        x, r, Ro = run(copies, max_n)
        assert x.reshape(copies, -1).tobytes() == np.tile(x0, (copies, 1)).tobytes()
        assert r.tobytes() == np.tile(r0, copies).tobytes()
        if adjust:
            assert Ro.tobytes() == np.tile(R0, copies).tobytes()


def test_instance_above_the_bound_is_refused():
    import paper_2303_02650_amd as P

    inst = synth.instance_set(2, 70, 9.5, seed=4)
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    d.max_n = 60
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    res = P.results(P.lbfgs_descend(d, xy, P.DescentParams(max_iter=5)))
    assert (res["status"] == 7).all()
    assert xy.cpu().numpy().tobytes() == inst.xy.reshape(-1).tobytes()
