"""Weights that no filter table represents (W1 four times larger): the edge kernels that evaluate the filter MLP, in every precision, in both
variants and over more partitions than one launch takes, against the oracle.  The first call of a fresh handle goes by the kernels
that hold both ways, the next one by those of the MLP; both have to give the same bits.

Bounds.  fp32 and split fp16: those of the fp32 tests.  bf16: every rounding is within u = 2^-9 of its value, 4 of them in a forward and 4 in
a reverse step of a layer (operands of two products and what they are propagated through): (4 L + 8) u of the largest force, 4 u of
the sum of the atoms' energies."""
import numpy as np
import pytest

import workloads as wl
from oracle import graph as og
from oracle import model as om
from oracle import three_body as tb

from gpu_util import E_RTOL, F_RTOL

pytestmark = pytest.mark.gpu

TWO = ("emb", "W1", "W2", "Wm", "Wo", "Wr1", "wr2")
SCALE = np.float32(4.0)


def _weights(F, L, seed, bonds=False):
    w = wl.rmp_weights(4, F, L, seed)
    if bonds:
        w.update(wl.three_body_weights(F, L, seed))
    w["W1"] = w["W1"] * SCALE
    return w


def _calls(g, call):
    """Results of two calls and whether the second had passes over the lower edges, which only the way by MLP has (bonds apart)."""
    import torch
    out = []
    for k in range(2):
        if k == 1:
            g.profile_enable(True)
            g.profile_read(reset=True)
        e, f, a = call()
        torch.cuda.synchronize()
        out.append((float(e.cpu()[0]), f.cpu().numpy().astype(np.float64), a.cpu().numpy().astype(np.float64)))
    n = g.profile_read(reset=True)["edge_bwd_lower"][1]
    g.profile_enable(False)
    return out, n > 0


def _hold(got, ref, L, precision, what):
    u = 2.0 ** -9
    e_tol, f_tol = (4 * u, (4 * L + 8) * u) if precision == 1 else (E_RTOL, F_RTOL)
    de = abs(got[0] - ref["energy"]) / np.abs(ref["atom_energy"]).sum()
    df = np.abs(got[1] - ref["forces"]).max() / np.abs(ref["forces"]).max()
    print(f"{what}: dE/sum|e| {de:.2e}, dF/max|F| {df:.2e}")
    assert de <= e_tol and df <= f_tol, (what, de, df)
    if precision == 1:
        assert df > 1e-5   # it really is the reduced-precision path


def _same(a, b, what):
    assert a[0] == b[0] and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2]), what


@pytest.mark.parametrize("F,L,slabs", [(32, 2, 1), (64, 1, 2), (64, 3, 3), (64, 8, 1), (32, 3, 9)])
def test_two_body(F, L, slabs):
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=5)
    w = _weights(F, L, 3)
    mode = M.MODE_SLABS if slabs > 1 else M.MODE_WHOLE
    pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
    ref = om.energy_forces(c["positions"], c["cell"], c["species"], w, og.build_graph(c["positions"], c["cell"], c["r_cut"]),
                           c["r_cut"], 8, 6)
    for precision in (0, 1, 2):
        what = f"F {F}, L {L}, {slabs} slabs, precision {precision}"
        W = M.Weights(w, 6, precision=precision)
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=slabs)
        (first, again), by_mlp = _calls(g, lambda: M.mlip_forward(g, W, mode))
        assert by_mlp == (L > 1), what   # (one layer's reverse step has no second pass)
        _same(first, again, what)
        _hold(first, ref, L, precision, what)
        s = M.mlip_forward_static(g, W, mode)
        torch.cuda.synchronize()
        assert float(s[0].cpu()[0]) == first[0] and np.array_equal(s[1].cpu().numpy(), first[1].astype(np.float32)), what


@pytest.mark.parametrize("F,L,slabs", [(32, 2, 1), (64, 3, 3), (64, 2, 9)])
def test_three_body(F, L, slabs):
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(4, n=5)
    w = _weights(F, L, 5, bonds=True)
    mode = M.MODE_SLABS if slabs > 1 else M.MODE_WHOLE
    pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
    ref_g = og.build_graph(c["positions"], c["cell"], c["r_cut"])
    ref = tb.energy_forces3(c["positions"], c["cell"], c["species"], w, ref_g, c["r_cut"], c["r_bond"], c["K"], c["p"])
    BW = M.BondWeights(w, c["r_bond"], c["A"])
    for precision in (0, 1, 2):
        what = f"bonds, F {F}, L {L}, {slabs} slabs, precision {precision}"
        W = M.Weights({k: w[k] for k in TWO}, c["p"], precision=precision)
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=slabs)
        (first, again), _ = _calls(g, lambda: M.mlip_forward_bonds(g, W, BW, mode))
        _, by_mlp = _calls(g, lambda: M.mlip_forward(g, W, mode))   # the same edge kernels without bonds, decided by now
        assert by_mlp, what
        _same(first, again, what)
        _hold(first, ref, L, precision, what)


@pytest.mark.parametrize("F", [32, 64])
def test_both_sides_of_the_limit(F):
    """W1 from its ordinary size to four times that: somewhere in between the tables stop representing the filters.  On either side,
    and at every step, the fp32 bounds hold."""
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=4)
    pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
    ref_g = og.build_graph(c["positions"], c["cell"], c["r_cut"])
    ways = []
    for scale in 4.0 ** (np.arange(9) / 8):
        w = wl.rmp_weights(4, F, 2, 11)
        w["W1"] = (w["W1"] * np.float32(scale)).astype(np.float32)
        ref = om.energy_forces(c["positions"], c["cell"], c["species"], w, ref_g, c["r_cut"], 8, 6)
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"])
        W = M.Weights(w, 6)
        (first, again), by_mlp = _calls(g, lambda: M.mlip_forward(g, W))
        ways.append(by_mlp)
        _same(first, again, scale)
        _hold(first, ref, 2, 0, f"F {F}, W1 x {scale:.2f}, by {'MLP' if by_mlp else 'table'}")
    assert ways[0] is False and ways[-1] is True and ways == sorted(ways)


@pytest.mark.parametrize("slabs", [1, 2])
def test_a_captured_static_call_follows_the_weights_values(slabs):
    """The static call makes packs and tables anew on every replay: with other values in the same arrays, on either side of the verdict and
    back, every replay gives what an uncaptured call gives for them."""
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=4)
    mode = M.MODE_SLABS if slabs > 1 else M.MODE_WHOLE
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
        models = [M.Weights(wl.rmp_weights(4, 64, 3, 1), 6), M.Weights(_weights(64, 3, 2), 6), M.Weights(wl.rmp_weights(4, 64, 3, 3), 6)]
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=slabs)
        want = []
        for W in models:
            e, f, a = M.mlip_forward(M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=slabs), W, mode)
            torch.cuda.synchronize()
            want.append((float(e.cpu()[0]), f.cpu().numpy(), a.cpu().numpy()))
        W = M.Weights(wl.rmp_weights(4, 64, 3, 4), 6)
        M.mlip_forward_static(g, W, mode)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            e, f, a = M.mlip_forward_static(g, W, mode)
        for k in (0, 1, 1, 2, 1, 0):
            for name, t in W.t.items():
                t.copy_(models[k].t[name])
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert float(e.cpu()[0]) == want[k][0] and np.array_equal(f.cpu().numpy(), want[k][1]), k
            assert np.array_equal(a.cpu().numpy(), want[k][2]), k
