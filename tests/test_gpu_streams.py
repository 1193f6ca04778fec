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


class _DeviceArray:
    """a borrowed device pointer as torch takes it"""

    def __init__(self, ptr, count, typestr):
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": (count,), "typestr": typestr, "version": 2}


@pytest.mark.parametrize("which", ["csr", "mirror"])
def test_edge_arrays_are_complete_when_handed_out(which):
    """The whole graph's arrays read on another stream right after the call that returns their addresses."""
    import ctypes
    import torch
    import paper_2506_02023_amd as M
    c, pos, sp = next(_systems())
    ref = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"])
    _, senders, _, d = ref.csr()
    want = [senders, d] if which == "csr" else [ref.mirror()]
    side = torch.cuda.Stream()
    g = M.mlip_build_graph(pos, c["cell"], sp, c["r_cut"])
    E, a, b = g.sizes()[1], ctypes.c_void_p(), ctypes.c_void_p()
    if which == "csr":
        assert M.lib().mlip_graph_csr(g._h, None, ctypes.byref(a), ctypes.byref(b)) == 0
        views = [_DeviceArray(a.value, E, "<i4"), _DeviceArray(b.value, E, "<f4")]
    else:
        assert M.lib().mlip_graph_mirror(g._h, ctypes.byref(a)) == 0
        views = [_DeviceArray(a.value, E, "<i4")]
    with torch.cuda.stream(side):
        got = [torch.as_tensor(v, device="cuda").clone() for v in views]
    side.synchronize()
    assert all(np.array_equal(x.cpu().numpy(), y) for x, y in zip(got, want))


def _graph_node_types(graph):
    """hipGraphNodeType of every node of a captured graph"""
    import ctypes
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(w for line in f for w in line.split()[-1:] if "libamdhip64" in w))
    raw, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    nodes, out = (ctypes.c_void_p * n.value)(), []
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(n)) == 0
    for node in nodes:
        t = ctypes.c_int()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(t)) == 0
        out.append(t.value)
    return out


@pytest.mark.parametrize("n_slabs", [1, 3, 64])
def test_static_call_under_capture(n_slabs):
    """mlip_forward_static captured and replayed, other work and synchronisations between the replays: every replay gives
    the eager result, and the graph holds kernels only, also where whole batches of slabs own nothing (64)."""
    import torch
    import paper_2506_02023_amd as M
    rng = np.random.default_rng(4)
    pos = np.concatenate([rng.uniform(0.5, 9.5, (40, 3)) * np.array([1.0, 0.6, 0.6]), np.array([[41.0, 3.0, 3.0]])])
    cell, species = np.diag([64.0, 7.0, 7.0]), (np.arange(41) % 4).astype(np.int32)
    W = M.Weights(wl.rmp_weights(4, 32, 2, 12), 6)
    mode = M.MODE_SLABS if n_slabs > 1 else M.MODE_WHOLE
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        tp, ts = torch.as_tensor(pos, device="cuda"), torch.as_tensor(species, device="cuda")
        g = M.mlip_build_graph(tp, cell, ts, 5.0, n_slabs=n_slabs)
        eager = [x.clone() for x in M.mlip_forward_static(g, W, mode)]
        out = [torch.empty_like(x) for x in eager]
        M.mlip_forward_static(g, W, mode, out=out)
        side.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph, stream=side):
            M.mlip_forward_static(g, W, mode, out=out)
    assert set(_graph_node_types(graph)) == {0}     # hipGraphNodeTypeKernel
    c = wl.make_config(0)
    other = M.mlip_build_graph(torch.as_tensor(c["positions"], device="cuda"), c["cell"], torch.as_tensor(c["species"], device="cuda"), 5.0)
    for k in range(4):
        for x in out:
            x.fill_(float("nan"))
        if k % 2:      # a call from another handle leaves its contents in the shared workspace
            M.mlip_forward_static(other, W)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, eager)), k
