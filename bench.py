"""Benchmark: energy + forces throughput of the partitioned hot path on one MI355X.

One step = mlip_build_graph (n_slabs = 8) + mlip_forward in SLABS mode on benchmark
configuration 3 (63^3 fcc cells, 1,000,188 atoms, ~45.8M directed edges, F = 64, L = 3),
i.e. every stage of the path: cell list, CSR, partition, three layers forward with ghost
copies, reverse pass with ghost-gradient add-backs, forces.  Inputs are resident in HBM
before the timed region.  Prints ONE JSON line.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# The radial edge kernels look the filters up in tables (k_edge_fwd_tab, k_edge_bwd_tab, k_edge_last_tab) and run on the vector unit:
# their peak is PEAK_FP32_VECTOR_TFLOPS.  With weights that the tables do not represent they evaluate the filter MLP
# (k_edge_fwd, k_edge_bwd, k_edge_lower): these products run on the bf16 / fp16 matrix pipeline (2.5 PFLOP/s dense), an
# fp32 product as the six terms of operands in three bf16 parts, a split-fp16 one as three.  The precision mode applies
# to the F x F products; those with the K = 8 basis functions are fp32 in every mode.  A kernel's peak is that of the
# pipeline by the terms it executes per counted flop.
PEAK_MFMA16_TFLOPS = 2500.0
PRODUCT_TERMS = {"f32": 6, "f32split": 3, "bf16": 1}
BASIS_TERMS = 6


def matrix_peak_tflops(precision, F, n_basis, K=8):
    """Peak of a kernel with one F x F product and n_basis products with the basis per item."""
    ff, basis = 2 * F * F, n_basis * 2 * K * F
    return PEAK_MFMA16_TFLOPS * (ff + basis) / (PRODUCT_TERMS[precision] * ff + BASIS_TERMS * basis)


# Algorithmic flops per directed edge and layer, i.e. of the operation as it is defined:
#   forward: filter MLP, t = b W1 (2 K F) and w = SiLU(t) W2 (2 F F);
#   reverse: pre-activations t = b W1 (2 K F), sbar = wbar W2^T (2 F F), dt/dd contraction through W1 (2 K F);
#            the filter value w_e itself is not recomputed, the forward pass keeps it in HBM.
# The forward kernel runs on every edge.  The reverse kernel runs its dense work once per edge / reverse-edge pair (both
# have the same length), so the MFMA units execute half of the reverse figure per directed edge; a memory-bound second
# pass adds the lower edges' terms.  A kernel's roofline fraction is taken on what it executes; the rate of the
# operation as defined is reported beside it ("as_defined_tflops").
def flops_fwd_edge(F, K=8):
    return 2 * K * F + 2 * F * F


PEAK_HBM_GBS = 8000.0


def flops_bwd_edge_as_defined(F, K=8):
    return 2 * K * F + 2 * F * F + 2 * K * F


def flops_bwd_edge(F, K=8):
    """Executed per directed edge: the dense work of a pair, shared by its two edges."""
    return flops_bwd_edge_as_defined(F, K) // 2


# Executed on tables per directed edge, layer and feature: forward five multiply-adds for the filter value and one into the
# row's sum; reverse value and slope (nine), the sum, and slope x g_i x abar_j into the edge's sum (3).  Reverse of layer
# 0: slope only (five) and the latter.
def flops_fwd_tab(F):
    return 12 * F


def flops_bwd_tab(F, L):
    """Mean over the layers."""
    return F * (23 * (L - 1) + 13) / L


# HBM bytes per launch (one layer over all 8 slabs) on the default workload, from rocprofv3 --pmc FETCH_SIZE and
# WRITE_SIZE (profiles/edge_traffic_configs3_8slabs.md): KiB x copy-kernel scale (1.9976 for FETCH_SIZE, 1.000 for
# WRITE_SIZE)
TRAFFIC_SOURCE = ("profiled constant, not measured by this run: rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE of this kernel on "
                  "this workload, profiles/edge_traffic_configs3_8slabs.md")
TRAFFIC_BWD_LAUNCH_BYTES = (2470086 * 1.9976 + 811000) * 1024   # k_edge_bwd_tab, k_edge_last_tab, mean of the three layers
TRAFFIC_FWD_LAUNCH_BYTES = (2085393 * 1.9976 + 250047) * 1024    # k_edge_fwd_tab


# fp32 vector peak that applies to this build: 256 CUs x 4 SIMDs x 16 lanes x 2 flop per FMA x 2.4 GHz = 78.6 TFLOP/s.
# (The published 157.3 TFLOP/s counts packed fp32 FMAs, which the library is compiled without.)  It bounds the triplet
# kernels of the three-body variant.
PEAK_FP32_VECTOR_TFLOPS = 78.6


def flops_triplet_fwd(F, A=8):
    """Per ordered triplet: h = P + Q + T(c) Wtc (2 + 2A per feature), SiLU (5), u * SiLU accumulated (2)."""
    return F * (2 + 2 * A + 5 + 2)


def flops_triplet_bwd(F, A=8):
    """Per ordered triplet, each evaluated once: h again (2 + 2A), SiLU and SiLU' (8), hbar = Sbar u SiLU' (2), sums into
    Pbar, Qbar (2), ubar (2), dT/dc Wtc (2A), its product with hbar (2)."""
    return F * (2 + 2 * A + 8 + 2 + 2 + 2 + 2 * A + 2)


def cpu_baseline(cfg_index, n_cells):
    """The oracle, as it stands, timed once on the timed system itself (n_cells = None) or on a smaller box of the
    same recipe."""
    import workloads as wl
    from oracle import _lib as ol
    from oracle import graph as og
    from oracle import model as om
    c = wl.make_config(cfg_index, n=n_cells)
    t0 = time.perf_counter()
    g = og.build_graph(c["positions"], c["cell"], c["r_cut"])
    if c["three_body"]:
        from oracle import three_body as tb
        tb.energy_forces3(c["positions"], c["cell"], c["species"], c["weights"], g, c["r_cut"], c["r_bond"], c["K"], c["p"])
    else:
        om.energy_forces(c["positions"], c["cell"], c["species"], c["weights"], g, c["r_cut"], c["K"], c["p"])
    dt = time.perf_counter() - t0
    n = len(c["species"])
    return {"value": n / dt, "unit": "atoms/s", "cores": int(ol.lib().orc_num_threads()), "kind": "oracle",
            "sample": (f"configs[{cfg_index}] itself" if n_cells is None else
                       f"configs[{cfg_index}] recipe at {n_cells}^3 fcc cells")
                      + f" ({n} atoms, {g.E} directed edges), fp64, graph + energy + forces, one run of {dt:.1f} s"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", type=int, default=3)
    ap.add_argument("--cells", type=int, default=None, help="override fcc cells per side (smaller runs)")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle timing")
    ap.add_argument("--cpu-cells", type=int, default=None,
                    help="fcc cells per side of a smaller sample for the oracle timing (default: the timed system itself)")
    ap.add_argument("--no-whole", action="store_true", help="skip the unpartitioned (whole-graph) run of the same system")
    ap.add_argument("--precision", choices=("f32", "f32split", "bf16"), default="f32",
                    help="f32split: the F x F products of the filter MLP as split-fp16 MFMA triples (fp32-grade results); "
                         "bf16: those products with bf16 operands (fp32 accumulation)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (slabs are processed in sequence on one device); "
              "use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2506_02023_amd as M
    import workloads as wl

    c = wl.make_config(args.config, n=args.cells)
    three_body = c["three_body"]   # configs[4]: whole-graph mode (a secondary workload; the default is configs[3])
    P = 1 if three_body else max(c["n_slabs"], 2)
    torch.cuda.set_device(0)
    pos = torch.as_tensor(c["positions"], device="cuda")
    spec = torch.as_tensor(c["species"], device="cuda")
    W = M.Weights(c["weights"], c["p"], precision={"f32": 0, "bf16": 1, "f32split": 2}[args.precision])
    BW = M.BondWeights(c["weights"], c["r_bond"], c["A"]) if three_body else None
    N = pos.shape[0]
    out = (torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty((N, 3), dtype=torch.float32, device="cuda"),
           None)
    g = None

    def step(mode=None):
        nonlocal g
        g = M.mlip_build_graph(pos, c["cell"], spec, c["r_cut"], n_slabs=P, graph=g)
        if three_body:
            M.mlip_forward_bonds(g, W, BW, M.MODE_WHOLE, out=out, want_atom_energy=False)
        else:
            M.mlip_forward(g, W, M.MODE_SLABS if mode is None else mode, out=out, want_atom_energy=False)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    g.profile_enable(True)
    g.profile_read(reset=True)
    torch.cuda.synchronize()
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]   # step boundaries, on the library's stream
    t0 = time.perf_counter()
    marks[0].record()
    for k in range(args.steps):
        step()
        marks[k + 1].record()
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    per_step = sorted(marks[k].elapsed_time(marks[k + 1]) for k in range(args.steps))
    prof = g.profile_read(reset=True)
    g.profile_enable(False)
    _, E, _ = g.sizes()
    energy = float(out[0].cpu()[0])
    fsum = out[1].double().sum(0).abs().max().item()

    def timed_variant(weights, n_slabs, mode):
        """The same step with other weights / slab count, outside the headline's timed region."""
        gv = None
        t1 = 0.0
        for it in range(2 + args.steps):
            if it == 2:
                torch.cuda.synchronize()
                t1 = time.perf_counter()
            gv = M.mlip_build_graph(pos, c["cell"], spec, c["r_cut"], n_slabs=n_slabs, graph=gv)
            M.mlip_forward(gv, weights, mode, out=out, want_atom_energy=False)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t1) / args.steps * 1e3
        e = float(out[0].cpu()[0])
        gv.destroy()
        return ms, e

    # for the record (not the headline): the unpartitioned run, and the split-fp16 mode of the headline's step
    whole_ms = split_ms = None
    if not three_body and not args.no_whole:
        whole_ms, energy_whole = timed_variant(W, 1, M.MODE_WHOLE)
    if args.precision == "f32" and not three_body:
        split_ms, energy_split = timed_variant(M.Weights(c["weights"], c["p"], precision=2), P, M.MODE_SLABS)

    ms_step = dt / args.steps * 1e3
    L = c["L"]
    default_workload = args.config == 3 and args.cells is None and args.precision == "f32"   # what the traffic constants were profiled on

    # The reverse step has a second pass only with the filters from the MLP.
    on_tables = prof["edge_bwd_lower"][1] == 0

    def table_roofline(group, kernel, flops_edge, as_defined, traffic):
        ms, n = prof[group]
        avg_ms = ms / max(n, 1)
        rate = E * L * args.steps / (ms * 1e-3) / 1e12 if ms > 0 else 0.0   # T edges and layers / s
        return {"kernel": kernel, "bound": "alu", "achieved": rate * flops_edge, "peak": PEAK_FP32_VECTOR_TFLOPS, "unit": "TFLOP/s",
                "frac": rate * flops_edge / PEAK_FP32_VECTOR_TFLOPS, "traffic": traffic if default_workload else None,
                "traffic_source": TRAFFIC_SOURCE if default_workload else None, "avg_launch_ms": avg_ms, "launches": int(n),
                "flops_per_launch": E * flops_edge * L * args.steps / max(n, 1), "ms_per_step": ms / args.steps,
                "as_defined_tflops": rate * as_defined, "flops_per_edge_layer": {"executed": flops_edge, "as_defined": as_defined},
                "note": "filters from tables: no filter MLP per edge; peak: fp32 vector unit without packed instructions"}

    def edge_roofline(group, kernel, flops_edge, n_basis, traffic, as_defined=None):
        ms, n = prof[group]
        per_launch = E * flops_edge * L * args.steps / max(n, 1)
        avg_ms = ms / max(n, 1)
        ach = per_launch / (avg_ms * 1e-3) / 1e12 if avg_ms > 0 else 0.0
        peak = matrix_peak_tflops(args.precision, c["F"], n_basis)
        r = {"kernel": kernel, "bound": "mfma", "achieved": ach, "peak": peak, "unit": "TFLOP/s",
             "frac": ach / peak, "traffic": traffic if default_workload else None,
             "traffic_source": TRAFFIC_SOURCE if default_workload else None,
             "avg_launch_ms": avg_ms, "launches": int(n), "flops_per_launch": per_launch,
             "ms_per_step": ms / args.steps}
        if as_defined is not None:   # rate of the operation as defined (twice the executed work), not a utilisation
            r["as_defined_tflops"] = ach * as_defined / flops_edge
            r["flops_per_edge_layer"] = {"executed": flops_edge, "as_defined": as_defined}
        r["note"] = (f"peak: 16-bit matrix pipeline, {PRODUCT_TERMS[args.precision]} term(s) per F x F product, "
                     f"{BASIS_TERMS} per product with the basis")
        return r

    F = c["F"]
    if on_tables:
        roof_bwd = table_roofline("edge_bwd", f"k_edge_bwd_tab<{F}>, k_edge_last_tab<{F}> (reverse edge step)", flops_bwd_tab(F, L),
                                  flops_bwd_edge_as_defined(F), TRAFFIC_BWD_LAUNCH_BYTES)
        roof_fwd = table_roofline("edge_fwd", f"k_edge_fwd_tab<{F}> (forward edge step)", flops_fwd_tab(F), flops_fwd_edge(F),
                                  TRAFFIC_FWD_LAUNCH_BYTES)
    else:
        roof_bwd = edge_roofline("edge_bwd", f"k_edge_bwd<{F}> (reverse edge step)", flops_bwd_edge(F), 2, None,
                                 flops_bwd_edge_as_defined(F))
        roof_fwd = edge_roofline("edge_fwd", f"k_edge_fwd<{F}> (forward edge step)", flops_fwd_edge(F), 1, None)
        # the reverse operation as defined takes both of its passes
        both_ms = prof["edge_bwd"][0] + prof["edge_bwd_lower"][0]
        roof_bwd["kernel"] = f"k_edge_bwd<{F}> on the upper-edge graphs (reverse edge step, first pass)"
        roof_bwd["as_defined_tflops"] = E * flops_bwd_edge_as_defined(F) * L * args.steps / (both_ms * 1e-3) / 1e12
        roof_bwd["as_defined_ms_per_step"] = both_ms / args.steps
    roof = roof_fwd if roof_fwd["ms_per_step"] >= roof_bwd["ms_per_step"] else roof_bwd   # the dominant kernel
    roof_lower = {}
    ms, n = prof["edge_bwd_lower"]
    if n > 0 and not on_tables:   # bound by its row traffic; compulsory bytes: per lower edge the kept filter values (read once),
                # per atom the row that is gathered (once if the caches were perfect) and the sum (read, written)
        per_launch = E / 2 * F * 4 + N * 3 * F * 4
        avg_ms = ms / n
        ach = per_launch / (avg_ms * 1e-3) / 1e9 if avg_ms > 0 else 0.0
        roof_lower["edge_bwd_lower"] = {"kernel": f"k_edge_lower<{F}> (reverse edge step, second pass: lower edges)",
                                        "bound": "hbm", "achieved": ach, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                        "frac": ach / PEAK_HBM_GBS,
                                        "traffic": None, "traffic_source": None,
                                        "avg_launch_ms": avg_ms, "launches": int(n),
                                        "bytes_per_launch": per_launch, "ms_per_step": ms / args.steps}
    roof_trip = {}
    if three_body:
        _, bptr = g.bonds()
        cnt = np.diff(bptr).astype(np.int64)
        n_triplets = int((cnt * (cnt - 1)).sum())
        for group, kernel, fl in (("triplet_fwd", f"k_triplet_fwd<{F}>", flops_triplet_fwd(F)),
                                  ("triplet_bwd", f"k_triplet_bwd<{F}>", flops_triplet_bwd(F))):
            ms, n = prof[group]
            per_launch = n_triplets * fl * args.steps / max(n, 1)
            avg_ms = ms / max(n, 1)
            ach = per_launch / (avg_ms * 1e-3) / 1e12 if avg_ms > 0 else 0.0
            roof_trip[group] = {"kernel": kernel, "bound": "alu", "achieved": ach, "peak": PEAK_FP32_VECTOR_TFLOPS,
                                "unit": "TFLOP/s", "frac": ach / PEAK_FP32_VECTOR_TFLOPS, "traffic": None,
                                "avg_launch_ms": avg_ms, "launches": int(n), "flops_per_launch": per_launch,
                                "ms_per_step": ms / args.steps, "triplets": n_triplets}
        if roof_trip["triplet_bwd"]["ms_per_step"] > roof["ms_per_step"]:
            roof = roof_trip["triplet_bwd"]

    res = {
        "metric": "atoms/s (energy+forces)", "value": N / (dt / args.steps), "unit": "atoms/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step, "ms_per_step_min": per_step[0],
        "ms_per_step_median": per_step[len(per_step) // 2], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None,
        "dtype": {"f32": "f32", "bf16": "f32 with W2 of the filter MLP and the bond MLPs' F x F products in bf16",
                  "f32split": "f32 (split-fp16 products where the filter MLP is evaluated per edge)"}[args.precision],
        "data": "synthetic",
        "config": {"workload": c["name"] + f", {N} atoms, {E} directed edges, r_cut 5.0, F={c['F']} L={L} K=8, "
                               + (f"three-body variant (bonds within {c['r_bond']}), graph build + whole-graph energy+forces"
                                  if three_body else f"graph build + {P}-slab sequential energy+forces"), "n_slabs": P},
        "edges_per_s": E / (dt / args.steps),
        "us_per_atom_step": ms_step * 1e3 / N,
        "breakdown_ms_per_step": {k: v[0] / args.steps for k, v in prof.items()},
        "energy": energy, "net_force_max_component": fsum,
        "roofline": roof, "roofline_edge_fwd": roof_fwd, "roofline_edge_bwd": roof_bwd,
    }
    for k, v in roof_trip.items():
        res["roofline_" + k] = v
    for k, v in roof_lower.items():
        res["roofline_" + k] = v
    if split_ms is not None:
        res["split_fp16_products"] = {"ms_per_step": split_ms, "value": N / (split_ms * 1e-3), "unit": "atoms/s",
                                      "energy": energy_split,
                                      "note": "MLIP_PRECISION_FP32_SPLIT: same step; on filter tables the fp32 mode's own, otherwise "
                                              "W2 products as three fp16 MFMA products of split operands"}
    if whole_ms is not None:
        res["whole_graph"] = {"ms_per_step": whole_ms, "value": N / (whole_ms * 1e-3), "unit": "atoms/s",
                              "energy": energy_whole, "rel_energy_difference_to_slabs": abs(energy_whole - energy) / abs(energy),
                              "note": "graph build without partition + unpartitioned energy+forces of the same system"}
    if not args.no_cpu:
        res["cpu_baseline"] = cpu_baseline(args.config, args.cpu_cells if args.cpu_cells else args.cells)
    print(json.dumps(res))


if __name__ == "__main__":
    main()
