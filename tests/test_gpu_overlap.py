"""Outputs that overlap their inputs: every input is read before an output is
written, in the adjoints too, and a captured call consists of kernels alone."""
import ctypes

import numpy as np
import pytest

import parity

torch = pytest.importorskip("torch")
import paper_1710_11259_amd as fps  # noqa: E402

pytestmark = pytest.mark.gpu

KERNEL_NODE, EMPTY_NODE = 0, 5  # hipGraphNodeType


def _node_types(raw):
    hip = fps.lib()  # its own libamdhip64
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(raw), None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(raw), nodes, ctypes.byref(n)) == 0
    types = []
    for v in nodes:
        t = ctypes.c_int()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(v), ctypes.byref(t)) == 0
        types.append(t.value)
    return types


def _buffers(b, adjoint, shift):
    """Input and output views that start `shift` entries apart."""
    n_in, n_out = (b.out_entries, b.in_entries) if adjoint else (b.in_entries, b.out_entries)
    buf = torch.zeros(max(n_in, n_out) + 8, dtype=torch.float64, device="cuda")
    return buf[shift:shift + n_in], buf[:n_out]


CASES = pytest.mark.parametrize("ns", [[1], [1, 2, 1], [40, 128], [33, 200, 1]])


@CASES
@pytest.mark.parametrize("adjoint", [False, True])
def test_captured_batch_is_kernels_only(ns, adjoint):
    b = fps.batch(ns, tol=1e-13)
    run = fps.batch_solve_adjoint if adjoint else fps.batch_solve
    x, y = _buffers(b, adjoint, 0)
    X = torch.from_numpy(np.random.default_rng(len(ns)).standard_normal(x.numel())).cuda()
    ws = torch.empty(b.workspace_bytes, dtype=torch.uint8, device="cuda")
    x.copy_(X)
    want = run(b, x, out=y, ws=ws).cpu().numpy()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        run(b, x, out=y, ws=ws)
    types = _node_types(g.raw_cuda_graph())
    assert KERNEL_NODE in types and set(types) <= {KERNEL_NODE, EMPTY_NODE}, types
    g.instantiate()
    for rep in range(3):
        ws.fill_(255)
        x.copy_(X)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), want), f"replay {rep}"


@CASES
@pytest.mark.parametrize("out", ["cheb", "native"])
@pytest.mark.parametrize("shift", [0, 3])
def test_adjoint(ns, out, shift):
    rng = np.random.default_rng(len(ns))
    b = fps.batch(ns, tol=1e-13, out=out)
    X = torch.from_numpy(rng.standard_normal(b.out_entries)).cuda()
    want = fps.batch_solve_adjoint(b, X).cpu().numpy()
    x, y = _buffers(b, True, shift)
    x.copy_(X)
    parity.check(fps.batch_solve_adjoint(b, x, out=y).cpu().numpy(), want, 1e-13, "batch")
    n = ns[-1]
    p = fps.plan(n, tol=1e-13, out=out)
    e = p.out_shape()[0]
    X1 = torch.from_numpy(rng.standard_normal((e, e))).cuda()
    want = fps.solve_adjoint(p, X1).cpu().numpy()
    buf = torch.zeros(e * e + 8, dtype=torch.float64, device="cuda")
    x = buf[shift:shift + e * e].view(e, e)
    x.copy_(X1)
    y = fps.solve_adjoint(p, x, out=buf[:n * n].view(n, n))
    parity.check(y.cpu().numpy(), want, 1e-13, "single")
