"""Launch shapes at their edges: systems whose rows are empty, longer than a work item, or fewer than a tile, so that
work items, tiles and slabs come out empty or partly filled; energy and forces against the fp64 oracle."""
import numpy as np
import pytest

import workloads as wl
from oracle import graph as og
from oracle import model as om

from gpu_util import gpu_energy_forces, gpu_graph

pytestmark = pytest.mark.gpu


def _spread(rng, n, side, least):
    """n points in a cube, no two closer than `least`"""
    out = [rng.uniform(0, side, 3)]
    while len(out) < n:
        p = rng.uniform(0, side, 3)
        if min(np.linalg.norm(p - q) for q in out) >= least:
            out.append(p)
    return np.array(out)


def _system(kind):
    rng = np.random.default_rng(31)
    cell = np.diag([90.0, 20.0, 20.0])
    lone = np.array([[60.0 + 6.5 * k, 10.0, 10.0] for k in range(4)])       # no neighbours at all
    if kind == "pair":
        return np.array([[1.0, 1.0, 1.0], [3.0, 1.5, 1.0]]), cell
    if kind == "ball":     # rows of 60 and more edges (more than the shortest work item) between empty rows
        ball = _spread(rng, 70, 7.0, 1.1) + 5.0
        return np.concatenate([lone[:2], ball, lone[2:]]), cell
    if kind == "chain":    # two edges per row: many rows per tile and three rows inside one step
        return np.concatenate([np.array([[4.0 * k + 0.3 * (k % 3), 10.0, 10.0] for k in range(14)]), lone]), cell
    ball = _spread(rng, 33, 9.0, 1.4)   # "halves": two groups far apart, slabs between them own nothing
    return np.concatenate([ball, ball[::-1] + np.array([45.0, 5.0, 5.0])]), cell


@pytest.mark.parametrize("kind", ["pair", "ball", "chain", "halves"])
@pytest.mark.parametrize("F,L", [(32, 1), (64, 3)])
def test_rows_at_the_edges_of_items_and_tiles(kind, F, L):
    import paper_2506_02023_amd as M
    pos, cell = _system(kind)
    species = (np.arange(len(pos)) % 4).astype(np.int32)
    weights = wl.rmp_weights(4, F, L, 77)
    ref_g = og.build_graph(pos, cell, 5.0)
    ref = om.energy_forces(pos, cell, species, weights, ref_g, 5.0, 8, 6)
    for P in (1, 2, 5):
        g = gpu_graph(pos, cell, species, 5.0, n_slabs=P)
        row_ptr, senders, _, _ = g.csr()
        assert np.array_equal(row_ptr, ref_g.row_ptr) and np.array_equal(senders, ref_g.senders)
        for precision in (0, 2):
            e, f, eps = gpu_energy_forces(g, weights, 6, M.MODE_SLABS if P > 1 else M.MODE_WHOLE, precision)
            what = f"{kind} F {F} L {L} P {P} precision {precision}"
            scale = np.abs(ref["atom_energy"]).sum()
            assert abs(e - ref["energy"]) <= 1e-5 * scale, what
            assert np.abs(eps - ref["atom_energy"]).max() <= 1e-5 * np.abs(ref["atom_energy"]).max(), what
            assert np.abs(f - ref["forces"]).max() <= 1e-4 * np.abs(ref["forces"]).max(), what


def _bins(pos, cell, r_cut):
    """Cells per direction as the library's search takes them (orthogonal cell, at least r_cut wide, at most 8 per atom or
    4096) and the number of atoms in every cell."""
    h = np.diag(cell)
    nb = np.clip((h / (r_cut * 1.000001 + 1e-12)).astype(int), 1, 1024)
    while nb.prod() > max(4096, 8 * len(pos)):
        nb[nb.argmax()] //= 2
    b = np.minimum((pos / h % 1.0 * nb).astype(int), nb - 1)
    return nb, np.bincount((b[:, 0] * nb[1] + b[:, 1]) * nb[2] + b[:, 2], minlength=nb.prod())


@pytest.mark.parametrize("case", ["one_cell", "thin", "crowded", "many_cells", "overflow"])
def test_search_over_cells(case):
    """Cells with no, few and more than 64 atoms, one cell in all, more than 64 surrounding cells, images of an atom
    itself, more than 4096 cells, and rows longer than the staging rows hold (the build then falls back to the two-pass
    search): the graph bit for bit."""
    rng = np.random.default_rng(5)
    if case == "one_cell":      # every pair is seen through several images of the one cell
        pos, cell, sp = wl.random_triclinic(9, 3, scale=3.2, skew=0.2, spread=2.0)
    elif case == "thin":        # reach of 4 cells and more along the thin direction: at least 9 x 3 x 3 surrounding cells
        cell = np.array([[1.2, 0.0, 0.0], [0.3, 14.0, 0.0], [0.0, 1.0, 16.0]])
        pos = rng.uniform(0, 1, (11, 3)) @ cell
        heights = 1.0 / np.linalg.norm(np.linalg.inv(cell), axis=0)
        nb = np.maximum((heights / 5.00001).astype(int), 1)
        around = 2 * np.ceil(5.0 / (heights / nb)).astype(int) + 1
        assert around[0] >= 9 and around.prod() > 64
    elif case == "crowded":     # a sparse system whose cells were widened: 150 atoms fall into one of them
        cell = np.diag([900.0, 900.0, 900.0])
        pos = np.concatenate([_spread(rng, 150, 20.0, 1.2) + 415.0, rng.uniform(0, 900, (30, 3))])
        nb, per_cell = _bins(pos, cell, 5.0)
        assert nb.prod() < 4096 and per_cell.max() >= 150
    elif case == "many_cells":  # 17^3 cells, most of them empty, four to a block
        cell = np.diag([86.0, 87.0, 88.0])
        pos = np.concatenate([_spread(rng, 120, 25.0, 1.0) + 70.0, rng.uniform(0, 86, (700, 3))])
        assert _bins(pos, cell, 5.0)[0].prod() > 4096
    else:                       # more than 64 finds of one atom: the build falls back to the two-pass search
        cell = np.diag([30.0, 30.0, 30.0])
        pos = _spread(rng, 260, 8.5, 0.75) + 3.0
    sp = np.zeros(len(pos), np.int32)
    ref = og.build_graph(pos, cell, 5.0)
    if case == "overflow":
        assert np.diff(ref.row_ptr).max() > 128
    for P in (1, 3):
        g = gpu_graph(pos, cell, sp, 5.0, n_slabs=P)
        row_ptr, senders, shifts, d = g.csr()
        assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(senders, ref.senders)
        assert np.array_equal(shifts, ref.shifts)
        assert np.array_equal(d, og.geometry(pos, cell, ref)[0].astype(np.float32))
        m = g.mirror()
        recv = np.repeat(np.arange(len(pos)), np.diff(row_ptr))
        assert np.array_equal(recv[m], senders) and np.array_equal(shifts[m], -shifts) and np.array_equal(m[m], np.arange(len(m)))


@pytest.mark.parametrize("many_cells", [False, True])
def test_search_over_crowded_cells(many_cells):
    """A sparse system, whose cells are much wider than the cutoff: cells with one atom less than a run of the crowded
    cells' blocks holds, exactly as many, one more, one round of lanes and one more, and many rounds; fewer and more than
    4096 cells, above which a wavefront has a cell to itself.  The graph bit for bit."""
    rng = np.random.default_rng(6)
    cell = np.diag([900.0, 900.0, 900.0])
    sizes = [31, 32, 33, 64, 65, 130] if not many_cells else [31, 32, 33, 64, 65, 96, 97, 700]
    lone = rng.uniform(0, 900, (90, 3)) if not many_cells else rng.uniform(0, 900, (300, 3))
    width = 900.0 / 11 if not many_cells else 900.0 / 22      # (of the widest side of a cell, asserted below)
    # one group per cell, every other one next to the one before it
    parts = [_spread(rng, n, 30.0, 1.2) + np.array([width * (2 + k // 2), width * (3 + k % 2), 450.0]) + 2.0 for k, n in enumerate(sizes)]
    pos = np.concatenate([lone] + parts)[rng.permutation(len(lone) + sum(sizes))]
    nb, per_cell = _bins(pos, cell, 5.0)
    assert nb.max() * width >= 899.9 and (nb.prod() >= 4096) == many_cells
    assert all((per_cell >= n).any() for n in sizes) and (per_cell > 64).sum() >= 2
    ref = og.build_graph(pos, cell, 5.0)
    assert np.diff(ref.row_ptr).max() < 64
    for P in (1, 3):
        g = gpu_graph(pos, cell, np.zeros(len(pos), np.int32), 5.0, n_slabs=P)
        row_ptr, senders, shifts, d = g.csr()
        assert np.array_equal(row_ptr, ref.row_ptr) and np.array_equal(senders, ref.senders)
        assert np.array_equal(shifts, ref.shifts)
        assert np.array_equal(d, og.geometry(pos, cell, ref)[0].astype(np.float32))


def test_a_cluster_in_a_large_box_is_searched_by_many_wavefronts():
    """4,000 atoms as a periodic crystal and as a cluster in a box of 500 A, where the cells hold some 340 atoms: the build
    takes about twice as long there; with a crowded cell left to one wavefront it took 40 times as long."""
    import time
    import torch
    import paper_2506_02023_amd as M
    c = wl.make_config(1, n=10)
    times = []
    for cell in (c["cell"], np.diag([500.0, 500.0, 500.0])):
        pos = torch.as_tensor(c["positions"] + (185.0 if cell[0, 0] == 500.0 else 0.0), device="cuda")
        sp = torch.as_tensor(c["species"], device="cuda")
        g, best = None, 1e9
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            g = M.mlip_build_graph(pos, cell, sp, 5.0, graph=g)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        times.append(best)
    assert _bins(c["positions"] + 185.0, np.diag([500.0] * 3), 5.0)[1].max() > 200
    assert times[1] <= 10 * times[0], times


@pytest.mark.parametrize("F", [32, 64])
def test_fp32_products_keep_the_range_of_fp32(F):
    """Activations of the filter MLP far beyond the range of 16-bit floats (their three-part bf16 operands have the
    exponent range of fp32), brought back by the second map."""
    import paper_2506_02023_amd as M
    pos, cell = _system("ball")
    species = (np.arange(len(pos)) % 4).astype(np.int32)
    weights = wl.rmp_weights(4, F, 2, 78)
    weights["W1"] = weights["W1"] * np.float32(2.0 ** 20)
    weights["W2"] = weights["W2"] * np.float32(2.0 ** -20)
    ref_g = og.build_graph(pos, cell, 5.0)
    ref = om.energy_forces(pos, cell, species, weights, ref_g, 5.0, 8, 6)
    e, f, eps = gpu_energy_forces(gpu_graph(pos, cell, species, 5.0), weights, 6, M.MODE_WHOLE, 0)
    assert abs(e - ref["energy"]) <= 1e-5 * np.abs(ref["atom_energy"]).sum()
    assert np.abs(f - ref["forces"]).max() <= 1e-4 * np.abs(ref["forces"]).max()


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_a_non_finite_atom_spoils_only_what_depends_on_it(precision):
    """Two groups out of each other's reach, their atoms alternating in the arrays (so they share tiles): the embedding of a
    species that one group alone has is infinite.  Everything that depends on it comes out non-finite, the other group's
    energies and forces are those of that group by itself."""
    import paper_2506_02023_amd as M
    pos, cell = _system("halves")
    n = len(pos) // 2
    pos = np.stack([pos[:n], pos[n:]], 1).reshape(-1, 3)      # even: one group, odd: the other
    species = np.zeros(2 * n, np.int32)
    species[0::2], species[1::2] = 3, np.arange(n) % 3
    weights = wl.rmp_weights(4, 64, 2, 79)
    _, f_ref, eps_ref = gpu_energy_forces(gpu_graph(pos, cell, species, 5.0), weights, 6, M.MODE_WHOLE, precision)
    weights["emb"][3, 5] = np.inf
    for P in (1, 3):
        mode = M.MODE_SLABS if P > 1 else M.MODE_WHOLE
        e, f, eps = gpu_energy_forces(gpu_graph(pos, cell, species, 5.0, n_slabs=P), weights, 6, mode, precision)
        assert not np.isfinite(e) and not np.isfinite(eps[0::2]).any()
        assert np.array_equal(eps[1::2], eps_ref[1::2])
        assert np.abs(f[1::2] - f_ref[1::2]).max() <= (2e-2 if precision == 1 else 1e-4) * np.abs(f_ref[1::2]).max()


@pytest.mark.parametrize("F,L", [(32, 1), (64, 3)])
def test_bonds_per_centre_at_the_edges(F, L):
    """Clusters whose atoms are all bonded to one another: 0, 1, 2, 3, 4, 5, 15, 16 (the most that the triplet kernels hold in
    registers), 17, 32 (the most that the forward kernel holds in LDS) and 33 bonds per centre, whole and in slabs."""
    import torch
    import paper_2506_02023_amd as M
    from oracle import three_body as tb
    rng = np.random.default_rng(8)
    sizes, parts = [1, 2, 3, 4, 5, 6, 16, 17, 18, 33, 34], []
    for k, n in enumerate(sizes):
        pts = []
        while len(pts) < n:    # in a ball of radius 2.2: no two farther apart than the bonds reach
            q = rng.uniform(-2.2, 2.2, 3)
            if np.linalg.norm(q) < 2.2 and all(np.linalg.norm(q - r) >= 0.9 for r in pts):
                pts.append(q)
        parts.append(np.array(pts) + [6.0 + 12.0 * k, 7.0, 7.0])
    pos, cell, r_cut, r_bond, K, p = np.concatenate(parts), np.diag([12.0 * len(sizes), 14.0, 14.0]), 5.0, 4.6, 8, 6
    species = (np.arange(len(pos)) % 4).astype(np.int32)
    weights = wl.rmp_weights(4, F, L, 78)
    weights.update(wl.three_body_weights(F, L, 78))
    ref_g = og.build_graph(pos, cell, r_cut)
    ref = tb.energy_forces3(pos, cell, species, weights, ref_g, r_cut, r_bond, K, p)
    assert sorted(set(np.diff(ref["bptr"]))) == [n - 1 for n in sizes]
    BW = M.BondWeights(weights, r_bond, 8)
    # fp32 and split fp16: the bounds of the three-body tests.  bf16: every rounding is within 2^-9 of its value, and one cluster
    # carries most of the energy and force, so the roundings on the way may all point one way.  Energy: filter product, P and Q,
    # S, wb; forces: two operands in each of the 2 L filter products and the 8 bond arrays of both directions.
    u = 2.0 ** -9
    for P in (1, 2, 5):
        g = gpu_graph(pos, cell, species, r_cut, n_slabs=P)
        for precision, e_tol, f_tol in ((0, 1e-5, 1e-4), (2, 1e-5, 1e-4), (1, 4 * u, (4 * L + 8) * u)):
            W = M.Weights({k: weights[k] for k in ("emb", "W1", "W2", "Wm", "Wo", "Wr1", "wr2")}, p, precision=precision)
            e, f, eps = M.mlip_forward_bonds(g, W, BW, M.MODE_SLABS if P > 1 else M.MODE_WHOLE)
            torch.cuda.synchronize()
            what = f"F {F} L {L} P {P} precision {precision}"
            assert abs(float(e[0]) - ref["energy"]) <= e_tol * np.abs(ref["atom_energy"]).sum(), what
            assert np.abs(f.cpu().numpy() - ref["forces"]).max() <= f_tol * np.abs(ref["forces"]).max(), what


@pytest.mark.parametrize("F", [32, 64])
def test_readout_products_do_not_shift_the_energy(F):
    """The matrix unit cuts bits off (towards minus infinity) where it aligns the products of one instruction, which shifts
    every sum of the readout the same way; weights wr2 of one sign would carry that into the total energy of any system.
    4,096 atoms of as many species without neighbours: the mean error of dense products against that of exact ones
    (a unit matrix), which have the same sigmoid.  Of the shift, 1.0e-8 of the energy, no more than a third may be left
    (1.9e-9 with fp32 matrix instructions; the means' own scatter is 1e-7 over the square root of 4 x 4,096 x F values)."""
    import paper_2506_02023_amd as M
    n = 16
    pos = np.stack(np.meshgrid(*[np.arange(n) * 6.0] * 3, indexing="ij"), -1).reshape(-1, 3)
    cell, species = np.diag([6.0 * n] * 3), np.arange(n ** 3).astype(np.int32)
    g = gpu_graph(pos, cell, species, 5.0)
    assert g.sizes()[1] == 0
    shift = {}
    for kind in ("exact", "dense"):
        off, scale = 0.0, 0.0
        for seed in range(4):
            rng = np.random.default_rng([seed, 21])
            h = rng.standard_normal((n ** 3, F)).astype(np.float32)
            Wr1 = (rng.standard_normal((F, F)) / np.sqrt(F)).astype(np.float32)
            if kind == "exact":   # one term per sum, both factors with 8 significant bits
                h, Wr1 = (h.view(np.int32) & -65536).view(np.float32), np.eye(F, dtype=np.float32)
            w = {k: v[:0] if k in ("W1", "W2", "Wm", "Wo") else v for k, v in wl.rmp_weights(4, F, 1, seed).items()}
            w.update(emb=h, Wr1=Wr1, wr2=np.full(F, -0.125, np.float32))
            g.invalidate_weights()   # (the next model's arrays may lie where the last one's did)
            e, _, _ = gpu_energy_forces(g, w, 6, M.MODE_WHOLE)
            y = h.astype(np.float64) @ Wr1.astype(np.float64)
            s = y / (1.0 + np.exp(-y))
            off += e + 0.125 * s.sum()
            scale += 0.125 * np.abs(s).sum()
        shift[kind] = off / scale
    print(F, shift)
    assert abs(shift["dense"] - shift["exact"]) <= 1.0e-8 / 3, shift
