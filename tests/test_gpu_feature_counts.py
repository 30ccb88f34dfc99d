"""Candidate features do not depend on how many instances or candidates a call
has: batches on either side of the workgroup size's rule, with candidate
counts that leave whole waves over, against one call per candidate count."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7, 64, 65, 300, 1024])
@pytest.mark.parametrize("C", [1, 63, 64, 65, 128, 255, 256, 257])
def test_batches_agree(n, C):
    import paper_2303_02650_amd as P

    R = float(max(2.5, np.sqrt(n / 0.84)))
    base = synth.instance_set(3, n, R, seed=n)
    cc, cd = synth.candidates(base, 2048, synth.rng_for(n + C))

    def run(copies, count):
        k = np.arange(3 * copies) % 3
        d = P.DeviceInstances.from_host(np.arange(3 * copies + 1, dtype=np.int32) * n, base.R[k])
        xy = base.xy.reshape(3, n, 2)[k]
        f = P.features(d, torch.from_numpy(xy.reshape(-1).copy()).cuda(),
                       torch.from_numpy(cc[k, :count].reshape(-1).copy()).cuda(),
                       torch.from_numpy(cd[k, :count].reshape(-1).copy()).cuda())
        return f.cpu().numpy().reshape(3 * copies, count, 8)

    want = run(1, 2048)[:, :C]
    for copies in (1, 85, 86, 130):             # 255, 258 instances
        got = run(copies, C)
        assert got.tobytes() == np.tile(want, (copies, 1, 1)).tobytes()
