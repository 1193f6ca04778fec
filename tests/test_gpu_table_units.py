"""The tables' units: lengths at and next to every limit between two of the 64 units of [0, rc], on whose sides the intervals have different
lengths, so that an interval of one unit taken in the other's measure shows as a wrong slope; first by the launch that holds both ways, then by
the kernels on tables."""
import numpy as np
import pytest

import workloads as wl
from oracle import graph as og
from oracle import model as om

pytestmark = pytest.mark.gpu

R_CUT = 5.0


@pytest.mark.parametrize("F,L", [(32, 1), (32, 3), (64, 1), (64, 2)])
def test_pairs_at_the_limits_of_units(F, L):
    """Bound per pair, of the largest force at its limit and the ones beside it (a pair's own may vanish): 2e-5 (rounding of the filters' values and
    slopes, 1e-7 of each, through the layers) and what the rounding of the length to fp32 makes of the fourth power of its distance
    from the cutoff.  A slope in the wrong measure is off by a third at least."""
    import torch
    import paper_2506_02023_amd as M
    at_limit = (np.arange(5, 64) * R_CUT / 64).astype(np.float32)
    ds = np.concatenate([np.nextafter(at_limit, np.float32(0)), at_limit, np.nextafter(at_limit, np.float32(9))]).astype(np.float64)
    at = np.array([[12.0 * (k % 14), 12.0 * (k // 14), 0.0] for k in range(len(ds))]) + 3.0
    pos = np.stack([at, at + np.stack([0 * ds, 0 * ds, ds], 1)], 1).reshape(-1, 3)
    spec, cell = (np.arange(len(pos)) % 4).astype(np.int32), np.diag([168.0, 168.0, 20.0])
    w = wl.rmp_weights(4, F, L, 9)
    ref = om.energy_forces(pos, cell, spec, w, og.build_graph(pos, cell, R_CUT), R_CUT, 8, 6)
    g = M.mlip_build_graph(torch.as_tensor(pos, device="cuda"), cell, torch.as_tensor(spec, device="cuda"), R_CUT)
    W = M.Weights(w, 6)
    for call in ("undecided", "on tables"):
        f = M.mlip_forward(g, W)[1]
        torch.cuda.synchronize()
        size = np.abs(ref["forces"]).reshape(3, -1, 6).max((0, 2))
        size = np.tile(np.maximum(size, np.maximum(np.roll(size, 1), np.roll(size, -1))), 3)
        err = np.abs(f.cpu().numpy() - ref["forces"]).reshape(-1, 6).max(1) / size
        bound = 2e-5 + 4 * 2.0 ** -22 / (R_CUT - ds)
        assert np.all(err <= bound), (call, ds[err > bound], err[err > bound])
