"""morph_warmup launches every kernel that a dense linear of at most 64 rows, or a 4-bit one in the native order, can come to: whatever it leaves out has its
first launch while serving, or inside a capture.  What it launches is read from a captured graph, which is not replayed."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint), ("y", ctypes.c_uint), ("z", ctypes.c_uint)]


class KernelNodeParams(ctypes.Structure):                  # hipKernelNodeParams
    _fields_ = [("blockDim", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("gridDim", Dim3), ("kernelParams", ctypes.c_void_p),
                ("sharedMemBytes", ctypes.c_uint)]


def kernel_names(graph):
    hip = ctypes.CDLL("libamdhip64.so", mode=ctypes.RTLD_GLOBAL)
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    count = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph), None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph), nodes, ctypes.byref(count)) == 0
    names = set()
    for n in nodes:
        p = KernelNodeParams()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(n), ctypes.byref(p)) == 0        # (a node of another type is an error)
        names.add(hip.hipKernelNameRefByPtr(p.func, None).decode())
    return names


def test_every_kernel_of_decode_linears_is_warmed():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2506_02006_amd import binding as B
    L = B.lib()
    buf = torch.empty(int(L.morph_warmup_bytes()), dtype=torch.uint8, device="cuda")
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        rc = L.morph_warmup(buf.data_ptr(), buf.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    names = kernel_names(g.raw_cuda_graph())
    print(len(names), "kernels", flush=True)
    want = ["decode_dense_kernelILi%dELb%dELb%dELi%dEE" % (mt, bf, steps, cw) for bf in (0, 1)
            for mt, steps, cw in ((1, 1, 1), (2, 1, 1), (4, 1, 1), (1, 1, 2), (2, 1, 2), (1, 0, 2), (2, 0, 2))]
    want += ["decode_small_kernelILi%dELb%dELb1EE" % (rl, bf) for bf in (0, 1) for rl in (1, 4)] + ["decode_mid_kernelILb%dELb1EE" % bf for bf in (0, 1)]
    missing = [w for w in want if not any(w in n for n in names)]
    assert not missing, missing
