"""Neighbor lists against the oracle where the build changes its way: sizes
around a wave and a workgroup, rows longer than the sorted registers, cells
with more candidates than a mask, segments longer than their staging, entries
that start at any alignment, capacities that cut a segment, cutoffs down to
the subnormal range, more instances than one look back covers."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def layout(kind, n, rng):
    R = max(2.5, float(np.sqrt(n / 0.84)))
    x = synth.disk_uniform(n, R, rng)
    if kind == "dense":                         # rows of 10 to 30
        x *= 0.5
    elif kind == "cluster":                     # everything within the cutoff
        x = rng.uniform(-0.7, 0.7, size=(n, 2)) + 0.3 * R
    elif kind == "outside":
        x = x * rng.uniform(0.5, 3.0, size=(n, 1))
    elif kind == "lattice":                     # distances at the cutoff -+ one FP32 step
        m = int(np.ceil(np.sqrt(n)))
        x = 2.3 * np.array([(i % m, i // m) for i in range(n)], dtype=np.float64) - 1.15 * m
        R = 1.7 * m + 1.0
    elif kind == "nan":
        x[:: 3, 0] = np.nan
        x[1 :: 7, 1] = np.inf
    return x, R


def want_lists(inst, cutoff, form):
    row, col = [0], []
    for b in range(inst.B):
        pi, pj = oracle.neighbors(inst.instance(b), cutoff)
        lists = [[] for _ in range(inst.offset[b + 1] - inst.offset[b])]
        for i, j in zip(pi.tolist(), pj.tolist()):
            lists[i].append(j)
            if form != 0:
                lists[j].append(i)
        for l in lists:
            col += [j + (0 if form == 2 else int(inst.offset[b])) for j in sorted(l)]
            row.append(len(col))
    return np.array(row), np.array(col, dtype=np.int64)


def build(P, inst, cutoff, form, capacity, shift):
    """Row table, entries and count, with col shifted by `shift` entries in a
    buffer of sentinels."""
    d = P.DeviceInstances.from_host(inst.offset, inst.R)
    xy = torch.from_numpy(inst.xy.reshape(-1).copy()).cuda()
    dt = torch.int16 if form == 2 else torch.int32
    buf = torch.full((capacity + shift + 8,), -7, dtype=dt, device="cuda")
    row = torch.empty(inst.total_n + 1, dtype=torch.int32, device="cuda")
    need = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = torch.empty(P.pecc_build_neighbors_workspace_size(d), dtype=torch.uint8, device="cuda")
    P.pecc_build_neighbors(d, xy, cutoff, 0.0, form, row, buf[shift:], capacity, need, ws)
    return row.cpu().numpy(), buf.cpu().numpy().astype(np.int64), int(need.item())


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("kind", ["random", "dense", "cluster", "outside", "lattice", "nan"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 511, 1000, 1024])
def test_rows_match_oracle(n, kind, form):
    import paper_2303_02650_amd as P

    rng = synth.rng_for(9 * n + 1)
    parts = [layout(kind, k, rng) for k in (n, max(1, n // 3), n)]
    inst = synth.pack([p[0] for p in parts], [p[1] for p in parts])
    row, col = want_lists(inst, 2.3, form)
    need = len(col)
    # (capacity, shift): all of it, then cut within a segment
    for cap, shift in ((need, 0), (need, 1), (need, 2), (need, 3), (need // 2, 1), (max(0, need - 1), 0)):
        if cap == 0:
            continue
        r, c, got = build(P, inst, 2.3, form, cap, shift)
        assert got == need
        assert np.array_equal(r, row)
        ends = row[np.searchsorted(row, cap, side="right") - 1]       # complete rows
        assert np.array_equal(c[shift:shift + ends], col[:ends])
        assert (c[shift + ends:shift + cap] != -7).all()
        assert (c[:shift] == -7).all() and (c[shift + cap:] == -7).all()


@pytest.mark.parametrize("cutoff", [1e-22, 1e-10, 0.7, 4.0, 60.0, 1e19, 1e30])
def test_cutoff_range(cutoff):
    import paper_2303_02650_amd as P

    rng = synth.rng_for(5)
    x, R = layout("random", 150, rng)
    x[70] = x[10]                               # a pair at distance 0
    x[71] = x[11] + np.array([0.0, 3e-23])
    tiny = np.concatenate([x[:50] * 1e-22, x[50:]])
    inst = synth.pack([x, tiny], [R, R])
    for form in (0, 1, 2):
        row, col = want_lists(inst, cutoff, form)
        if len(col) == 0:
            continue
        r, c, got = build(P, inst, cutoff, form, len(col), 0)
        assert got == len(col)
        assert np.array_equal(r, row)
        assert np.array_equal(c[:len(col)], col)


def test_many_small_instances():
    import paper_2303_02650_amd as P

    rng = synth.rng_for(6)
    parts = [layout("random", int(k), rng) for k in rng.integers(1, 12, size=3000)]
    inst = synth.pack([p[0] for p in parts], [p[1] for p in parts])
    for form in (0, 1, 2):
        row, col = want_lists(inst, 2.3, form)
        for _ in range(3):                      # the same every time
            r, c, got = build(P, inst, 2.3, form, len(col), 0)
            assert got == len(col)
            assert np.array_equal(r, row)
            assert np.array_equal(c[:len(col)], col)
