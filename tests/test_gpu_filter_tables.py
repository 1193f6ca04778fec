"""The edge steps on tabulated filters against the oracle, where the table's intervals change length, at both ends of the range and among rows
without edges; and the choice between the tables and the filter MLP, which the device makes from the weights."""
import numpy as np
import pytest

import workloads as wl
from oracle import graph as og
from oracle import model as om

from gpu_util import E_RTOL, F_RTOL, table_interval_ends

pytestmark = pytest.mark.gpu

R_CUT = 5.0


def _weights(F, L, seed, scale=1.0):
    w = wl.rmp_weights(4, F, L, seed)
    w["W1"] = (w["W1"] * np.float32(scale)).astype(np.float32)
    return w


def _run(g, W, mode):
    import torch
    import paper_2506_02023_amd as M
    e, f, a = M.mlip_forward(g, W, mode)
    torch.cuda.synchronize()
    return float(e.cpu()[0]), f.cpu().numpy().astype(np.float64), a.cpu().numpy().astype(np.float64)


def _check(got, ref, what):
    """Energy relative to the sum of the atoms' magnitudes (these seeds are not chosen for a large total)."""
    assert abs(got[0] - ref["energy"]) <= E_RTOL * np.abs(ref["atom_energy"]).sum(), what
    assert np.abs(got[1] - ref["forces"]).max() <= F_RTOL * np.abs(ref["forces"]).max(), what


def _by_mlp(g, W, mode):
    """Whether a call with weights that were judged before goes by the MLP: only then are there passes over the lower edges."""
    g.profile_enable(True)
    g.profile_read(reset=True)
    _run(g, W, mode)
    n = g.profile_read(reset=True)["edge_bwd_lower"][1]
    g.profile_enable(False)
    return n > 0


def _pairs(ds):
    """Pairs of atoms far from all others, single atoms (rows without edges) before, between and behind them; the atoms' pairs (-1: single)"""
    pos, kind = [], []
    for k, d in enumerate(ds):
        at = np.array([12.0 * (k % 6), 12.0 * (k // 6), 0.0]) + 3.0
        if k % 3 == 0:
            pos.append(at + [0, 0, 6.0])
            kind.append(-1)
        u = np.array([np.cos(k), np.sin(k), 0.5])
        pos += [at, at + d * u / np.linalg.norm(u)]
        kind += [k, k]
    return np.array(pos + [np.array([70.0, 70.0, 9.0])]), np.array(kind + [-1])


@pytest.mark.parametrize("F", [32, 64])
def test_pairs_at_the_ends_of_intervals(F):
    """A pair's force is held relative to itself, or to what it is a twentieth nearer where that is larger (it may vanish: that of species 3 and 0
    does at 0.417, F = 64): 2e-5 (rounding of the filters' values and slopes, 1e-7 of each, through three layers) and what the
    rounding of the length to fp32, up to 2^-22 at 5, makes of the fourth power of its distance from the cutoff."""
    import torch
    import paper_2506_02023_amd as M
    ends = table_interval_ends(R_CUT)
    length = np.diff(ends)
    edges = [ends[k + 1] for k in range(len(length) - 1) if ends[k] > 0.3 and abs(length[k + 1] - length[k]) > 1e-9] + [4.7]   # where the length changes
    edges += list(ends[-4::2])
    ds = np.array(sorted(x + o for x in edges for o in (-1e-6, 1e-6)) + [0.3, 1.0, 2.5, 4.97, 4.99, 4.999])
    pos, kind = _pairs(ds)
    spec = (np.arange(len(pos)) % 4).astype(np.int32)
    cell = np.diag([84.0, 84.0, 15.0])
    w = _weights(F, 3, 5)
    ref, nearer = (om.energy_forces(x, cell, spec, w, og.build_graph(x, cell, R_CUT), R_CUT, 8, 6) for x in (pos, _pairs(0.95 * ds)[0]))
    g = M.mlip_build_graph(torch.as_tensor(pos, device="cuda"), cell, torch.as_tensor(spec, device="cuda"), R_CUT)
    W = M.Weights(w, 6)
    first, again = _run(g, W, M.MODE_WHOLE), _run(g, W, M.MODE_WHOLE)
    assert first[0] == again[0] and np.array_equal(first[1], again[1])
    assert not _by_mlp(g, W, M.MODE_WHOLE)
    for k, d in enumerate(ds):
        mine = kind == k
        size = np.abs(ref["forces"][mine]).max()
        if d < 4.5:
            size = max(size, np.abs(nearer["forces"][mine]).max())
        err = np.abs(first[1][mine] - ref["forces"][mine]).max() / size
        assert err <= 2e-5 + 4 * 2.0 ** -22 / (R_CUT - d), (d, err)
    assert np.all(first[1][kind < 0] == 0)
    assert np.abs(first[2] - ref["atom_energy"]).max() <= 1e-5 * np.abs(ref["atom_energy"]).max()


@pytest.mark.parametrize("F,L,slabs", [(32, 2, 1), (64, 3, 1), (64, 1, 3), (64, 3, 3)])
def test_the_way_follows_the_weights(F, L, slabs):
    """Filters that bend too fast for the tables (W1 thirty times larger) go by the MLP, ordinary ones by the tables; a handle that
    only knows ordinary ones gets such weights right too, and every order of calls gives a handle's first results again."""
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=4)
    mode = M.MODE_SLABS if slabs > 1 else M.MODE_WHOLE
    pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
    ref_g = og.build_graph(c["positions"], c["cell"], c["r_cut"])
    models = [_weights(F, L, 7), _weights(F, L, 8, 30.0)]
    refs = [om.energy_forces(c["positions"], c["cell"], c["species"], w, ref_g, c["r_cut"], 8, 6) for w in models]
    Ws = [M.Weights(w, 6) for w in models]
    new = lambda: M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=slabs)  # noqa: E731
    fresh = [_run(new(), W, mode) for W in Ws]
    for got, ref in zip(fresh, refs):
        _check(got, ref, "fresh handle")
    for k, W in enumerate(Ws):
        g = new()
        _run(g, W, mode)
        if L > 1:
            assert _by_mlp(g, W, mode) == (k == 1)
    g = new()
    for k in (0, 0, 1):   # the third call learns on the device that the tables do not do
        got = _run(g, Ws[k], mode)
        _check(got, refs[k], f"model {k}")
    scale = np.abs(refs[1]["forces"]).max()
    assert np.abs(got[1] - fresh[1][1]).max() <= F_RTOL * scale
    for k in (1, 0, 1, 0):
        got = _run(g, Ws[k], mode)
        assert got[0] == fresh[k][0] and np.array_equal(got[1], fresh[k][1]) and np.array_equal(got[2], fresh[k][2])
    for k in (0, 1):
        s = M.mlip_forward_static(g, Ws[k], mode)
        torch.cuda.synchronize()
        assert float(s[0].cpu()[0]) == fresh[k][0] and np.array_equal(s[1].cpu().numpy(), fresh[k][1].astype(np.float32))


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("F,L,slabs", [(32, 2, 1), (64, 3, 3)])
def test_results_do_not_depend_on_what_a_handle_saw_before(F, L, slabs, precision):
    """Calls in any order, none of them waited for, give bit for bit what a fresh handle gives for the same weights, whether or not the
    host has heard what the device found about them; the fixed workspace's too."""
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=4)
    mode = M.MODE_SLABS if slabs > 1 else M.MODE_WHOLE
    pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
    new = lambda: M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=slabs)  # noqa: E731
    Ws = [M.Weights(_weights(F, L, 7 + k, 30.0 if k == 1 else 1.0), 6, precision=precision) for k in range(3)]   # the second: by MLP
    fresh = [_run(new(), W, mode) for W in Ws]
    order = (0, 0, 1, 1, 2, 1, 0, 2, 2, 1)
    g = new()
    for k in (0, 0):
        _run(g, Ws[k], mode)   # the host knows that the first model's tables are good
    outs = []
    for n, k in enumerate(order):
        outs.append(M.mlip_forward_static(g, Ws[k], mode) if n % 4 == 3 else M.mlip_forward(g, Ws[k], mode))
    torch.cuda.synchronize()
    for k, (e, f, a) in zip(order, outs):
        assert float(e.cpu()[0]) == fresh[k][0], k
        assert np.array_equal(f.cpu().numpy(), fresh[k][1].astype(np.float32)), k
        assert np.array_equal(a.cpu().numpy(), fresh[k][2].astype(np.float32)), k


def _sharp(F, L, seed, sharper, scale):
    """Four features fed by four hidden units of their own, with W1 `sharper` times larger; their filters scaled by `scale` and their share of
    the sender projection by its inverse (powers of two: the same model)."""
    w, r = _weights(F, L, seed), np.random.default_rng(seed)
    w["W1"][:, :, :4] *= np.float32(sharper)
    w["W2"][:, :4, :] = w["W2"][:, :, :4] = 0
    w["W2"][:, :4, :4] = r.standard_normal((L, 4, 4)).astype(np.float32) / 2
    w["W2"][:, :, :4] *= np.float32(scale)
    w["Wm"][:, :, :4] /= np.float32(scale)
    return w


@pytest.mark.parametrize("F", [32, 64])
def test_small_features_are_judged_by_themselves(F):
    """Features that bend fast and are small beside the others go by the MLP as they do at the others' size, and pairs at short distances have
    its forces.  Bound, of the largest force: 4e-6 for values and slopes rounded to some 4e-7 in three layers forward and back, and for the
    sharp units, whose t is a sum of terms of up to 3 x `sharper`, 2^-24 of those through SiLU'' / SiLU' <= 1/2 in each of the six steps."""
    import torch
    import paper_2506_02023_amd as M
    ds = np.linspace(0.25, 2.45, 45)
    pos = np.concatenate([[at, at + d * np.array([np.cos(k), np.sin(k), 0.5]) / np.sqrt(1.25)]
                          for k, d in enumerate(ds) for at in [np.array([12.0 * (k % 7), 12.0 * (k // 7), 0.0]) + 3.0]])
    spec, cell = (np.arange(len(pos)) % 4).astype(np.int32), np.diag([84.0, 84.0, 15.0])
    g = M.mlip_build_graph(torch.as_tensor(pos, device="cuda"), cell, torch.as_tensor(spec, device="cuda"), R_CUT)
    ref_g = og.build_graph(pos, cell, R_CUT)
    for seed in (1, 2, 3):
        for sharper in (1.0, 2.0, 4.0, 8.0, 30.0):
            way = []
            for scale in (1.0, 2.0 ** -10, 2.0 ** -19):
                w = _sharp(F, 3, seed, sharper, scale)
                W = M.Weights(w, 6)
                got = _run(g, W, M.MODE_WHOLE)
                way.append(_by_mlp(g, W, M.MODE_WHOLE))
            assert way == [way[0]] * 3, (seed, sharper, way)
            assert way[0] if sharper == 30.0 else not way[0] or sharper > 1.0
            ref = om.energy_forces(pos, cell, spec, w, ref_g, R_CUT, 8, 6)
            err = np.abs(got[1] - ref["forces"]).max() / np.abs(ref["forces"]).max()
            assert err <= 4e-6 + 6 * 0.5 * 3 * 2.0 ** -24 * sharper, (seed, sharper, err)


@pytest.mark.parametrize("F", [32, 64])
def test_most_weights_of_twice_the_usual_size_go_by_tables(F):
    """Of sixty models of two layers, W1 twice as large: at most a sixth by the MLP, which takes twice as long.  (With one table for values and slopes it
    was 13 and 22, with one grid of 64 units for three tables 12 and 17.)"""
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=3)
    g = M.mlip_build_graph(torch.as_tensor(c["positions"], device="cuda"), c["cell"], torch.as_tensor(c["species"], device="cuda"), c["r_cut"])
    refused = 0
    for seed in range(60):
        W = M.Weights(_weights(F, 2, seed, 2.0), 6)
        _run(g, W, M.MODE_WHOLE)
        refused += _by_mlp(g, W, M.MODE_WHOLE)
    assert refused <= 10


def test_first_call_on_a_large_graph():
    """From 4.2 million edges on a first call makes the pair lists only if the device finds that its weights need them: the same results as
    the calls after it and, rounding apart, as without slabs, and the lists are complete when they are asked for."""
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=30)
    pos, sp = torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")
    pairs = []
    for scale in (1.0, 30.0):
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=3)
        assert g.sizes()[1] >= 1 << 22
        W = M.Weights(_weights(32, 2, 3, scale), 6)
        first, again = _run(g, W, M.MODE_SLABS), _run(g, W, M.MODE_SLABS)
        assert first[0] == again[0] and np.array_equal(first[1], again[1]) and np.array_equal(first[2], again[2])
        whole = _run(g, W, M.MODE_WHOLE)
        assert abs(whole[0] - first[0]) <= E_RTOL * np.abs(first[2]).sum()
        assert np.abs(whole[1] - first[1]).max() <= F_RTOL * np.abs(first[1]).max()
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=3)
        _run(g, W, M.MODE_SLABS)
        pairs.append(g.pairs(1))
    g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], n_slabs=3)
    for k, x in g.pairs(1).items():
        assert np.array_equal(pairs[0][k], x) and np.array_equal(pairs[1][k], x), k


def test_limit_of_the_fixed_workspace_with_many_edges_and_one_layer():
    """A graph of 77 edges per atom that fills the 64 MiB but for less than 4 bytes per edge: one layer's step sums an edge over all features at a
    time, so there is one sum per edge.  With the pair lists in the handle already (and so not in the workspace) the call gives the same."""
    import torch
    import paper_2506_02023_amd as M
    F = 64
    n = (16, 17, 17)
    corner = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 1, 3)
    fcc = np.array([[0, 0, 0], [0, 0.5, 0.5], [0.5, 0, 0.5], [0.5, 0.5, 0]])
    pos = 3.0 * (corner + fcc).reshape(-1, 3) + 0.1 * np.random.default_rng(3).standard_normal((4 * n[0] * n[1] * n[2], 3))
    cell, spec = 3.0 * np.diag(n).astype(np.float64), (np.arange(len(pos)) % 4).astype(np.int32)
    args = torch.as_tensor(pos, device="cuda"), cell, torch.as_tensor(spec, device="cuda"), R_CUT
    g = M.mlip_build_graph(*args)
    N, E, _ = g.sizes()
    span = 64   # of the pair lists' work-item table, the finest
    blocks = ([4 * (36864 + 1536 + 12288)]                                          # packed weights
              + [8 * (N + 1), 4 * E] + 5 * [2 * E] + [4 * (E // 2 // span + 2)]      # upper edges
              + [8 * (N + 1)] + 2 * [2 * E] + 2 * [4 * (N + 1)] + [2 * (E + 1)]      # lower edges, counts and ranks
              + 6 * [4 * F * N] + [4 * N, 12 * N, 4 * E] + [N // 4 + 8, 2048])       # node rows, sums
    need, room = sum((b + 255) // 256 * 256 for b in blocks), M.lib().mlip_static_scratch_bytes()
    assert E > F * N and room - 4 * E < need <= room - 256, (E / N, need, room)
    W = M.Weights(_weights(F, 1, 4), 6)
    want = _run(g, W, M.MODE_WHOLE)
    for lists in (False, True):
        g = M.mlip_build_graph(*args)
        if lists:
            g.pairs()
        e, f, a = M.mlip_forward_static(g, W, M.MODE_WHOLE)
        torch.cuda.synchronize()
        assert float(e.cpu()[0]) == want[0] and np.array_equal(f.cpu().numpy(), want[1].astype(np.float32))


def test_limit_of_the_fixed_workspace_with_many_edges_and_two_layers():
    """The largest of a row of graphs of 77 edges per atom that fits the 64 MiB, the next one, with 80 atoms more, being refused: the second sums
    per edge of F = 64, four bytes each and more than those atoms take, lie in the place of the filter MLP's kept values.  The
    same bits as with the workspace that grows."""
    import torch
    import paper_2506_02023_amd as M
    fcc = np.array([[0, 0, 0], [0, 0.5, 0.5], [0.5, 0, 0.5], [0.5, 0.5, 0]])
    W = M.Weights(_weights(64, 2, 4), 6)
    fits = []
    for nx in range(40, 90):
        n = (nx, 5, 4)
        corner = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 1, 3)
        pos = 3.0 * (corner + fcc).reshape(-1, 3) + 0.1 * np.random.default_rng(3).standard_normal((80 * nx, 3))
        g = M.mlip_build_graph(torch.as_tensor(pos, device="cuda"), 3.0 * np.diag(n).astype(np.float64),
                               torch.as_tensor((np.arange(len(pos)) % 4).astype(np.int32), device="cuda"), R_CUT)
        N, E, _ = g.sizes()
        try:
            got = M.mlip_forward_static(g, W, M.MODE_WHOLE)
        except M.MlipError:
            break
        torch.cuda.synchronize()
        fits.append((N, E))
        want = _run(g, W, M.MODE_WHOLE)
        assert float(got[0].cpu()[0]) == want[0] and np.array_equal(got[1].cpu().numpy(), want[1].astype(np.float32)), N
        assert not _by_mlp(g, W, M.MODE_WHOLE)
    assert 1 < len(fits) < 50 and 80 * M.lib().mlip_static_scratch_bytes() / N < 4 * fits[-1][1], (N, fits[-1:])
