"""Container adjustment with non-finite instances among healthy ones: they
report NONFINITE with their layout and radius as given, and the others have
the bits of a batch without them, also where a workgroup takes one instance
after another from the queue (more instances than the device holds)."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def adjust(xy, n, R):
    import paper_2303_02650_amd as P

    B = len(xy)
    d = P.DeviceInstances.from_host(np.arange(B + 1, dtype=np.int32) * n, np.full(B, R))
    x = torch.from_numpy(xy.reshape(-1).copy()).cuda()
    prm = P.DescentParams(max_iter=6, contact_margin=1e-4, ftol=1e-7)
    Ro, out = P.adjust_container(d, x, prm, rounds=3)
    return x.cpu().numpy().reshape(B, n, 2), Ro.cpu().numpy(), P.results(out)


# one wave, and shapes of 2 to 8 waves with one and two circles per thread
@pytest.mark.parametrize("n,B", [(40, 7), (40, 5000), (70, 7), (70, 3000), (200, 2000), (300, 1500),
                                 (520, 7), (520, 700)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_others_are_untouched(n, B, bad):
    R = float(np.sqrt(n / 0.8))
    base = synth.instance_set(5, n, R, seed=n)
    xy = base.xy.reshape(5, n, 2)[np.arange(B) % 5].copy()
    want_x, want_R, want = adjust(xy[:5], n, R)
    assert (want["status"] != 6).all()
    ill = np.arange(B) % 3 == 1
    xy[ill, n - 1, 1] = bad
    x, Ro, res = adjust(xy, n, R)
    assert (res["status"][ill] == 6).all()
    assert x[ill].tobytes() == xy[ill].tobytes()
    assert (Ro[ill] == np.float32(R)).all()
    k = (np.arange(B) % 5)[~ill]
    assert x[~ill].tobytes() == want_x[k].tobytes()
    assert Ro[~ill].tobytes() == want_R[k].tobytes()
    assert res[~ill].tobytes() == want[k].tobytes()


@pytest.mark.parametrize("n,B", [(40, 300), (300, 300), (520, 300)])
def test_no_rounds(n, B):
    """Nothing is evaluated: layouts and radii as given, zeros in the result, also
    right after calls that leave numbers in the workgroups' memory."""
    import paper_2303_02650_amd as P

    inst = synth.instance_set(B, n, float(np.sqrt(n / 0.8)), seed=n)
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    for _ in range(3):
        xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
        P.adjust_container(d, xy.clone(), P.DescentParams(max_iter=3), rounds=1)
        Ro, out = P.adjust_container(d, xy, P.DescentParams(), rounds=0)
        res = P.results(out)
        assert xy.cpu().numpy().tobytes() == inst.xy.reshape(-1).tobytes()
        assert (Ro.cpu().numpy() == inst.R.astype(np.float32)).all()
        for f in ("status", "iters", "evals", "rebuilds", "pair_evals", "E32", "gnorm", "cell_evals"):
            assert (res[f] == 0).all(), f
