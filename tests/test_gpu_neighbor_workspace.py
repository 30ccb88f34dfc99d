"""Neighbor lists on a workspace that starts at any byte and holds exactly what
the size query asks for: the same lists, and nothing written outside it."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 3, 31, 32, 33, 64, 320])
def test_any_alignment(B):
    import paper_2303_02650_amd as P

    inst = synth.instance_set(B, lambda b, r: r.integers(1, 40), lambda b, n: 1.0 + np.sqrt(n / 0.8), seed=B)
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    size = P.pecc_build_neighbors_workspace_size(d)

    def build(shift, form):
        buf = torch.full((size + 32,), 0xA5, dtype=torch.uint8, device="cuda")
        ws = buf[shift:shift + size]
        assert ws.data_ptr() % 8 == shift % 8
        row = torch.empty(inst.total_n + 1, dtype=torch.int32, device="cuda")
        col = torch.full((20 * inst.total_n,), -7, dtype=torch.int16 if form == 2 else torch.int32, device="cuda")
        need = torch.zeros(1, dtype=torch.int64, device="cuda")
        P.pecc_build_neighbors(d, xy, 2.3, 0.0, form, row, col, col.numel(), need, ws)
        assert (buf[:shift] == 0xA5).all() and (buf[shift + size:] == 0xA5).all()
        return row.cpu().numpy(), col.cpu().numpy(), int(need.item())

    for form in (0, 1, 2):
        row, col, need = build(0, form)
        assert row[-1] == need and (col[need:] == -7).all()
        for shift in (1, 2, 3, 4, 5, 7, 8, 12):
            r, c, m = build(shift, form)
            assert m == need and np.array_equal(r, row) and np.array_equal(c, col)
