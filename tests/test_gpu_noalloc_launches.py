"""red_sum_noalloc under its own plan: the kernel that reads the data is the
first one launched, with nothing cleared before it, and the result has the
bits of red_sum under its own plan, at sizes on both sides of the line between
the ticket and the two-kernel plan."""
import ctypes
import sys

import pytest

from paper_2004_05371_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class KernelNodeParams(ctypes.Structure):
    _fields_ = [("blockDim", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("gridDim", Dim3),
                ("kernelParams", ctypes.c_void_p), ("sharedMemBytes", ctypes.c_uint)]


def recorded_kernels(hip, stream, call):
    """(workgroups of the first kernel, number of kernels) that `call` puts on
    the stream, recorded with a stream capture."""
    vp = ctypes.c_void_p
    graph = vp()
    assert hip.hipStreamBeginCapture(vp(stream), 1) == 0
    try:
        call()
    finally:
        assert hip.hipStreamEndCapture(vp(stream), ctypes.byref(graph)) == 0
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    roots = (vp * n.value)()
    r = ctypes.c_size_t(n.value)
    assert hip.hipGraphGetRootNodes(graph, roots, ctypes.byref(r)) == 0 and r.value == 1
    p = KernelNodeParams()
    assert hip.hipGraphKernelNodeGetParams(vp(roots[0]), ctypes.byref(p)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return p.gridDim.x, n.value


@pytest.mark.parametrize("kind", ["f32", "i32", "bf16"])
@pytest.mark.parametrize("nbytes", [800_000, (1 << 20) + 4, 8_000_004, 32 << 20, (32 << 20) + 4])
def test_reads_at_once_and_gives_the_bits_of_red_sum(lib, kind, nbytes):
    n = nbytes // (2 if kind == "bf16" else 4)
    print("noalloc launches", kind, n, file=sys.stderr, flush=True)
    code = {"f32": lib.RED_F32, "i32": lib.RED_I32, "bf16": lib.RED_BF16}[kind]
    h = inputs.uniform_i32(n, sub=90) if kind == "i32" else inputs.normal_f32(n, sub=90)
    x = torch.from_numpy(h).to("cuda")
    if kind == "bf16":
        x = x.to(torch.bfloat16)
    out, ref = (torch.full((), -1, dtype=torch.int64 if kind == "i32" else torch.float64, device="cuda")
                for _ in range(2))
    torch.cuda.synchronize()
    s = torch.cuda.Stream().cuda_stream

    def call():
        assert lib.red_sum_noalloc(code, x.data_ptr(), n, out.data_ptr(), s) == lib.RED_OK
    call()
    lib.red_sum_ex(code, x.data_ptr(), n, ref.data_ptr(), s, None)
    torch.cuda.synchronize()
    assert out.item() == ref.item(), (kind, n, out.item(), ref.item())
    grid, kernels = recorded_kernels(lib.load(), s, call)
    assert grid > 1 and kernels == 2, (kind, n, grid, kernels)
