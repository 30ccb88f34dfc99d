"""The host's bound max_n picks the descents' workgroups: instances of up to
their size are computed as under the exact bound, larger ones are refused and
left as they were; the calls without such workgroups compute them."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
PRM = dict(max_iter=6, contact_margin=1e-4, ftol=1e-7)


def run(call, n, max_n):
    import paper_2303_02650_amd as P

    inst = synth.instance_set(2, n, float(np.sqrt(n / 0.8)), seed=n)
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    d.max_n = max_n
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    prm = P.DescentParams(**PRM)
    if call == "descend":
        out = P.lbfgs_descend(d, xy, prm)
    elif call == "noalloc":
        out = torch.empty(2 * P.RESULT_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        P.pecc_lbfgs_descend_noalloc(d, xy, prm.c(), out)
    elif call == "adjust":
        _, out = P.adjust_container(d, xy, prm, rounds=2)
    elif call == "gbo":
        out = P.gbo_descend(d, xy, prm, blocks=4)
    else:
        out = P.gbo_kbatch_descend(d, xy, P.partition(d, xy, "sector", 5), 5, prm)
    return inst.xy.reshape(-1), xy.cpu().numpy(), P.results(out)


@pytest.mark.parametrize("call", ["descend", "noalloc", "adjust", "kbatch"])
@pytest.mark.parametrize("bound,size", [(1, 64), (60, 64), (65, 128), (129, 256), (257, 512)])
def test_size_of_the_workgroup(call, bound, size):
    if call == "kbatch":
        size = 512
    _, x0, r0 = run(call, size, size)
    _, x, r = run(call, size, bound)
    assert (r["status"] != 7).all()
    assert x.tobytes() == x0.tobytes() and r.tobytes() == r0.tobytes()
    before, x, r = run(call, size + 1, bound)
    assert (r["status"] == 7).all()
    assert x.tobytes() == before.tobytes()


def test_geometric_descent_computes_larger_instances():
    _, x0, r0 = run("gbo", 300, 300)
    _, x, r = run("gbo", 300, 20)
    assert (r["status"] != 7).all()
    assert x.tobytes() == x0.tobytes() and r.tobytes() == r0.tobytes()
