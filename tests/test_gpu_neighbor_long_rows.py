"""Neighbor lists beyond the packing cutoff, against the oracle: rows of 15 to
18 and of more neighbors, 60 to 70 and more candidates, wide cells, one or two
such circles in a wave, segments within and beyond their staging, and a
capacity that ends inside a long row."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def check(parts, cutoff, cell, form, cut=0):
    import paper_2303_02650_amd as P

    inst = synth.pack([p[0] for p in parts], [p[1] for p in parts])
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    row, col = [0], []
    for b in range(inst.B):
        o, n = int(inst.offset[b]), int(inst.offset[b + 1] - inst.offset[b])
        pi, pj = oracle.neighbors(inst.instance(b), cutoff)
        a = np.zeros((n, n), dtype=bool)
        a[pi, pj] = True
        if form != 0:
            a |= a.T
        for i in range(n):
            col.append(np.flatnonzero(a[i]) + (0 if form == 2 else o))
            row.append(row[-1] + len(col[-1]))
    col = np.concatenate(col)
    cap = len(col) - cut
    buf = torch.full((len(col) + 8,), -7, dtype=torch.int16 if form == 2 else torch.int32, device="cuda")
    rows = torch.empty(inst.total_n + 1, dtype=torch.int32, device="cuda")
    need = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = torch.empty(P.pecc_build_neighbors_workspace_size(d), dtype=torch.uint8, device="cuda")
    P.pecc_build_neighbors(d, xy, cutoff, cell, form, rows, buf, cap, need, ws)
    got = buf.cpu().numpy().astype(np.int64)
    assert need.item() == len(col)
    assert np.array_equal(rows.cpu().numpy(), row)
    whole = np.array(row)[np.searchsorted(row, cap, side="right") - 1]
    assert np.array_equal(got[:whole], col[:whole])
    assert (got[cap:] == -7).all()


def disk(n, density, seed):
    R = max(2.5, float(np.sqrt(n / density)))
    return synth.disk_uniform(n, R, synth.rng_for(seed)), R


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("cutoff,cell", [(2.3, 6.9), (3.0, 0.0), (4.0, 0.0), (4.0, 8.0), (5.0, 0.0), (8.0, 0.0)])
@pytest.mark.parametrize("n", [70, 300, 1000, 1024])
def test_cutoffs_and_cells(n, cutoff, cell, form):
    parts = [disk(n, 0.84, n), disk(n, 1.5, n + 1)]
    check(parts, cutoff, cell, form)
    check(parts, cutoff, cell, form, cut=7)


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("pocket", [16, 17, 18, 19, 33, 34, 64, 65, 66, 90])
def test_pocket_of_circles(pocket, form):
    """Within a sparse layout, `pocket` circles that are all neighbors of each
    other: rows of pocket - 1 and more, a few candidates more."""
    x, R = disk(600, 0.4, pocket)
    rng = synth.rng_for(pocket + 1)
    who = rng.choice(600, size=pocket, replace=False)
    x[who] = np.array([0.4 * R, 0.1 * R]) + rng.uniform(-0.7, 0.7, size=(pocket, 2))
    check([(x, R), disk(90, 0.8, pocket)], 2.3, 0.0, form)
