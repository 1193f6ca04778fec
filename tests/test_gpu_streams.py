"""One handle on several streams: a rebuild on another stream begins after what the handle queued on the old one."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _systems():
    """a large system (its build's last kernels run on for a while after the call returns) and a small one"""
    import torch
    for index, n in ((2, 24), (1, 9)):
        c = wl.make_config(index, n=n)
        yield c, torch.as_tensor(c["positions"], device="cuda"), torch.as_tensor(c["species"], device="cuda")


def _arrays(g):
    return (*g.csr(), g.mirror())


@pytest.mark.parametrize("forward_between", [False, True])
@pytest.mark.parametrize("allocator", [None, False])
def test_rebuild_on_another_stream(allocator, forward_between):
    """Two builds of one handle, on one stream and then on another with no synchronisation between them, with the
    caller's allocator and with the library's: the second graph bit for bit that of a handle of its own, and energy and
    forces with it."""
    import torch
    import paper_2506_02023_amd as M
    systems = list(_systems())
    weights = [M.Weights(c["weights"], c["p"]) for c, _, _ in systems]
    fresh = []
    for (c, pos, sp), W in zip(systems, weights):
        g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"])
        e, f, _ = M.mlip_forward(g, W)
        fresh.append((_arrays(g), e.cpu(), f.cpu()))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    g = M.Graph(allocator=allocator)
    for turn, order in enumerate([(0, 1), (1, 0), (0, 1), (0, 1), (1, 0), (0, 0)]):
        for k, s in zip(order, streams):
            c, pos, sp = systems[k]
            with torch.cuda.stream(s):
                g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"], graph=g)
                if forward_between or s is streams[1]:
                    e, f, _ = M.mlip_forward(g, weights[k])
        assert all(np.array_equal(a, b) for a, b in zip(_arrays(g), fresh[k][0])), turn
        torch.cuda.synchronize()
        assert torch.equal(e.cpu(), fresh[k][1]) and torch.equal(f.cpu(), fresh[k][2]), turn
    g.destroy()
