"""Sizes at which an edge step on tables changes how it shares rows out (four workers of a wavefront to a row up to a number of rows for a compute
unit that the rows' mean length gives, a row each beyond), with rows longer than a wavefront takes at once and rows without an edge; and the
sums over a row's bonds, sixteen at a time, at 32 features."""
import numpy as np
import pytest

import workloads as wl
from oracle import graph as og
from oracle import model as om
from oracle import three_body as tb

from gpu_util import E_RTOL, F_RTOL, gpu_graph

pytestmark = pytest.mark.gpu


def _system(n, a=3.5):
    """n atoms: a ball of 80 with up to 79 neighbours, four far from everything, the rest a jittered lattice, at 3.5 of some 12 neighbours"""
    rng = np.random.default_rng(n)
    ball = [rng.uniform(0, 6.5, 3)]
    while len(ball) < 80:
        p = rng.uniform(0, 6.5, 3)
        if np.linalg.norm(np.array(ball) - p, axis=1).min() >= 1.0:
            ball.append(p)
    lone = np.array([[14.0, 7.0 * k + 22.0, 14.0] for k in range(4)])
    m = int(np.ceil((n - 84) ** (1 / 3)))
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n - 84] * a + 22.0
    pos = np.concatenate([sites + rng.uniform(-0.3, 0.3, sites.shape), np.array(ball) + 4.0, lone])
    return pos[rng.permutation(n)], np.diag([max(a * m, 24.5) + 28.0] * 3)


def _limit(mean):   # rows for a compute unit
    four, one = int(np.ceil((mean + 1) / 16)), int(np.ceil((mean + 1) / 64))
    return min(32, 16 * (four - one) // (4 * one - four)) if 4 * one > four else 32


# 256 compute units: the limit is that of rows times 128 with 64 features in a reverse step, else 256
@pytest.mark.parametrize("n,a,limit", [(513, 3.5, 8), (1023, 2.7, 8), (1024, 2.7, 8), (1025, 2.7, 8), (2048, 2.7, 8), (2049, 2.7, 8), (4000, 4.6, 0),
                                       (4095, 2.2, 32), (4096, 2.2, 32), (4097, 2.2, 32), (8192, 2.2, 32), (8193, 2.2, 32)])
@pytest.mark.parametrize("F", [32, 64])
def test_rows_to_a_wavefront_or_a_worker(n, a, limit, F):
    import torch
    import paper_2506_02023_amd as M
    pos, cell = _system(n, a)
    spec = (np.arange(n) % 4).astype(np.int32)
    w = wl.rmp_weights(4, F, 2, 21)
    ref_g = og.build_graph(pos, cell, 5.0)
    rows = np.diff(ref_g.row_ptr)
    assert rows.max() > 64 and rows.min() == 0 and _limit(np.ceil(rows.mean())) == limit
    ref = om.energy_forces(pos, cell, spec, w, ref_g, 5.0, 8, 6)
    W = M.Weights(w, 6)
    for P in (1, 3):
        g = gpu_graph(pos, cell, spec, 5.0, n_slabs=P)
        first = None
        for call in ("undecided", "on tables"):   # (the first launches hold both ways: the same bits)
            e, f, ae = M.mlip_forward(g, W, M.MODE_SLABS if P > 1 else M.MODE_WHOLE)
            torch.cuda.synchronize()
            got = [x.cpu().numpy() for x in (e, f, ae)]
            assert abs(float(got[0][0]) - ref["energy"]) <= E_RTOL * np.abs(ref["atom_energy"]).sum(), (P, call)
            assert np.abs(got[1] - ref["forces"]).max() <= F_RTOL * np.abs(ref["forces"]).max(), (P, call)
            assert np.abs(got[2] - ref["atom_energy"]).max() <= 1e-5 * np.abs(ref["atom_energy"]).max(), (P, call)
            assert first is None or all(np.array_equal(a, b) for a, b in zip(first, got)), (P, call)
            first = got


@pytest.mark.parametrize("precision,bound", [(0, F_RTOL), (1, 2e-2)])   # (1: bond rows in bf16, the bound of that mode)
@pytest.mark.parametrize("P", [1, 2])
def test_bond_sums_of_long_and_empty_rows(precision, bound, P):
    """Rows of more than sixteen bonds, fewer, and none, 32 features"""
    import torch
    import paper_2506_02023_amd as M
    pos, cell = _system(300)
    spec = (np.arange(300) % 4).astype(np.int32)
    w = wl.rmp_weights(4, 32, 2, 33)
    w.update(wl.three_body_weights(32, 2, 33))
    ref_g = og.build_graph(pos, cell, 5.0)
    _, bptr, _ = tb.bond_graph(pos, cell, ref_g, 3.4)
    assert np.diff(bptr).max() > 32 and np.any(np.diff(bptr) == 0) and np.any((np.diff(bptr) > 0) & (np.diff(bptr) < 8))
    ref = tb.energy_forces3(pos, cell, spec, w, ref_g, 5.0, 3.4, 8, 6)
    g = gpu_graph(pos, cell, spec, 5.0, n_slabs=P)
    W = M.Weights({k: w[k] for k in ("emb", "W1", "W2", "Wm", "Wo", "Wr1", "wr2")}, 6, precision=precision)
    for _ in range(2):
        f = M.mlip_forward_bonds(g, W, M.BondWeights(w, 3.4, 8), M.MODE_SLABS if P > 1 else M.MODE_WHOLE)[1]
        torch.cuda.synchronize()
        assert np.abs(f.cpu().numpy() - ref["forces"]).max() <= bound * np.abs(ref["forces"]).max()


def _irregular():
    """91 atoms in a box of 30: a ball of 80 whose rows go beyond 64 edges, three pairs, five atoms without a neighbour, in an order in which rows
    without an edge come alone and in twos between long ones"""
    rng = np.random.default_rng(11)
    ball = [np.array([10.0, 10.0, 10.0])]
    while len(ball) < 80:
        p = 7.0 + rng.uniform(0, 6.5, 3)
        if np.linalg.norm(np.array(ball) - p, axis=1).min() >= 1.0:
            ball.append(p)
    lone = [np.array([3.0 + 6 * k, 24.0, 3.0]) for k in range(4)] + [np.array([24.0, 14.0, 20.0])]
    pair = [np.array([3.0 + 8 * k, 24.0, 21.0 + d]) for k in range(3) for d in (0.0, 1.1 + k)]
    pos = lone[:2] + ball[:20] + lone[2:3] + ball[20:41] + pair[:3] + lone[3:] + ball[41:] + pair[3:]
    return np.array(pos), np.diag([30.0] * 3)


@pytest.mark.parametrize("F", [32, 64])
def test_items_of_two_irregular_rows(F):
    """Copies of an irregular system, of an odd number of atoms, further apart than the cutoff: more than sixteen rows for a worker, which it takes
    two at a time, whatever is in them: no edge in the first, the second or both, more than four steps in either.  Every copy as the
    system alone."""
    import torch
    import paper_2506_02023_amd as M
    one, box = _irregular()
    spec, side = (np.arange(len(one)) % 4).astype(np.int32), 15
    w = wl.rmp_weights(4, F, 2, 17)
    ref_g = og.build_graph(one, box, 5.0)
    empty = np.diff(ref_g.row_ptr) == 0
    assert len(one) % 2 == 1 and empty.sum() == 5 and np.any(empty[1:] & empty[:-1]) and np.diff(ref_g.row_ptr).max() > 64
    ref = om.energy_forces(one, box, spec, w, ref_g, 5.0, 8, 6)
    at = 30.0 * np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    copies = side ** 3
    assert copies * len(one) > 16 * 256 * 16 * 4
    g = gpu_graph((at + one).reshape(-1, 3), box * side, np.tile(spec, copies), 5.0)
    assert g.sizes()[1] == copies * ref_g.E
    W = M.Weights(w, 6)
    first = None
    for call in ("undecided", "on tables"):
        got = [x.cpu().numpy() for x in M.mlip_forward(g, W)]
        assert np.abs(got[1].reshape(copies, -1, 3) - ref["forces"]).max() <= F_RTOL * np.abs(ref["forces"]).max(), call
        assert np.abs(got[2].reshape(copies, -1) - ref["atom_energy"]).max() <= 1e-5 * np.abs(ref["atom_energy"]).max(), call
        assert first is None or all(np.array_equal(a, b) for a, b in zip(first, got)), call
        first = got
