"""The geometric batch descent's lists and visits where they change their way:
batches of up to one wave's lanes, one more, and the most a batch may hold;
lists that overflow their slots; cells with more candidates than a mask; a
wave's next batch in the same or a later colour."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def layout(kind, n, rng):
    R = max(2.5, float(np.sqrt(n / 0.84)))
    if kind == "random":
        return synth.disk_uniform(n, R, rng), R
    if kind == "crowded":                       # every list longer than its slots
        return rng.uniform(-1.2, 1.2, size=(n, 2)), R
    x = synth.disk_uniform(n, R, rng)           # a crowded part in an ordinary layout
    x[: n // 4] = 0.3 * R + rng.uniform(-1.6, 1.6, size=(n // 4, 2))
    return x, R


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kind,n,blocks", [
    ("random", 1, 1), ("random", 5, 1), ("random", 64, 1), ("random", 65, 1), ("random", 128, 1),
    ("random", 300, 3), ("random", 1024, 5), ("random", 1000, 8), ("random", 40, 8),
    ("crowded", 30, 1), ("crowded", 128, 1), ("crowded", 100, 2), ("mixed", 300, 4), ("mixed", 400, 6)])
def test_first_iterations_follow_oracle(kind, n, blocks, fp64):
    import paper_2303_02650_amd as P

    rng = synth.rng_for(31 * n + blocks)
    x, R = layout(kind, n, rng)
    y, Q = layout("random", max(1, n // 2), rng)
    inst = synth.pack([x, y], [R, Q])
    for outer in (1, 2):
        d = P.DeviceInstances.from_host(inst.offset, inst.R)
        xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
        res = P.results(P.gbo_descend(d, xy, P.DescentParams(max_iter=outer, g_tol=0.0, ftol=0.0),
                                      blocks=blocks, sweep_fp64=fp64))
        got = xy.cpu().numpy().reshape(-1, 2)
        for b in range(2):
            o0, o1 = inst.offset[b], inst.offset[b + 1]
            x64, r64, _ = oracle.gbo_descend(inst.instance(b).astype(np.float64), inst.R[b],
                                             oracle.DescentParams(g_tol=0.0), blocks=blocks, max_outer=outer)
            if res["status"][b] == 1:           # feasible before the budget
                continue
            assert res["iters"][b] == r64["outer"]
            scale = max(1.0, float(np.abs(x64).max()))
            # FP32 trial positions: an ulp of the coordinates per visit, carried
            # on by the next visit's gradient
            assert np.abs(got[o0:o1] - x64).max() / scale < 5e-5 * outer
            # the energy reported before the last iteration's stop test is the
            # energy at the returned positions
            E = oracle.energy(got[o0:o1].astype(np.float64), inst.R[b])
            assert res["E32"][b] == pytest.approx(E, rel=1e-4, abs=1e-9)
