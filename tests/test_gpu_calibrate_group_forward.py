"""The binary16 forward of layers that read the same activation, in one launch of the tiled GEMM, against a launch for each: to the bit.  Two to
four layers, with and without biases; rows, columns and tiles at the edges of tiles of 128 and of 256 tokens x 256 channels, rows that share lines
(256-token tiles on more than 224 compute units store these through the caches), one round of workgroups and several, where a workgroup goes from one
layer to the next; one panel of K and many; zero points beyond the short epilogue's.  Which form ran is read from a captured graph: kernels of
the call, and the GEMM's among them."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class _KernelNode(C.Structure):   # hipKernelNodeParams
    _fields_ = [("block", C.c_uint * 3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", C.c_uint * 3), ("params", C.c_void_p), ("shared", C.c_uint)]


def _kernels(run):
    """(function, dynamic LDS) of every kernel that `run` launches, from a capture of it."""
    from paper_2311_01305_amd import binding as B
    hip = B.load_library()   # (its dependencies' symbols with it: the runtime that torch has loaded)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        run()
    raw, n = C.c_void_p(graph.raw_cuda_graph()), C.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(n)) == 0
    out = []
    for node in nodes:
        p = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        out.append((p.func, p.shared))
    return out


def _calibrate(n, T, N, K, shift=0.0):
    from paper_2311_01305_amd import pipeline
    g = torch.Generator(device=DEV)
    g.manual_seed(T + N + K)
    X = (torch.randn(T, K, generator=g, device=DEV) * 2 + 0.3).half()
    W = [(torch.randn(N, K, generator=g, device=DEV) * 0.02 + shift).half() for _ in range(n)]
    b = [torch.randn(N, generator=g, device=DEV) if i != 1 else None for i in range(n)]
    gb = pipeline.GroupBuffers(T, K, (N,) * n, torch.float16, want_out_deq=True, device=DEV)
    for p in gb.per:
        p["out_deq"].fill_(7.0)
    run = lambda: pipeline.calibrate_group(X, W, b, gb)
    run()
    return gb, b, run


_form = {}   # tokens of a tile: the kernel


# (tokens of a tile as the plan has it)
@pytest.mark.parametrize("n,T,N,K,shift,tile", [(3, 700, 256, 64, 0.0, 128), (3, 1000, 260, 512, 0.0, 128), (4, 2100, 508, 136, 0.0, 128),
                                                (3, 2048, 1024, 1024, 0.0, 128), (2, 1537, 2300, 640, 0.0, 128), (3, 8200, 768, 320, 0.0, 128),
                                                (2, 5000, 4092, 128, 0.0, 128), (2, 1500, 1280, 256, 40.0, 128), (2, 4096, 2048, 64, 0.0, 256),
                                                (2, 4000, 2044, 64, 0.0, 256), (2, 8192, 4096, 64, 0.0, 256), (3, 4000, 2300, 72, 0.0, 256),
                                                (4, 4096, 4092, 64, 0.0, 256), (2, 4000, 2044, 200, 40.0, 256)])
def test_group_forward(n, T, N, K, shift, tile):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    gb, b, run = _calibrate(n, T, N, K, shift)
    t = gb.t
    for i, p in enumerate(gb.per):
        out = torch.full_like(p["out_deq"], 9.0)
        B.aweq_w8a8_gemm(t["xq"], B.AWEQ_I8, T, K, K, None, t["act_step"], t["act_zero"], None, t["rowsum_x"], None, p["codes"], N, p["step_w"],
                         p["zero_w"], 0, p["rowsum_w"], b[i], None, out, B.AWEQ_F16, N, None, None, t["status"])
        assert torch.equal(out.view(torch.int16), p["out_deq"].view(torch.int16)), i
    torch.cuda.synchronize()
    kernels = _kernels(run)
    assert len(kernels) == 5, "statistics, their merge, the activation quantizer, the pass over the weights, one GEMM"
    gemm = [f for f, lds in kernels if lds == 160 * 1024]
    assert len(gemm) == 1
    assert _form.setdefault(tile, gemm[0]) == gemm[0] and len(set(_form.values())) == len(_form)


@pytest.mark.parametrize("n,T,N,K", [(2, 700, 256, 64), (2, 10, 976, 80), (2, 16, 256, 1024), (2, 128, 1024, 1024), (4, 16, 1024, 4096), (3, 16, 2048, 2048), (3, 6000, 1024, 4096), (2, 6274, 2048, 4096),
                                     (4, 2048, 8192, 8192)])
def test_a_launch_each(n, T, N, K):
    """Small layers, whose own kernels take less than a round of the tiled GEMM, long rows in rounds that are not full (tiles of 128 and of 256
    tokens), and weights that do not fit the memory-side cache together."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gb, b, run = _calibrate(n, T, N, K)
    torch.cuda.synchronize()
    assert len(_kernels(run)) == 4 + n
