"""The codes brought to natural order by the kernels that multiply straight from them: 17 to 32 tokens with 16 channels a workgroup, and the
64 x 128 and 128 x 128 tiles for some hundred tokens.  One-hot activations, so that an output is one de-quantised weight, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("T,N,K,group", [(17, 260, 256, 128), (32, 132, 2112, 32), (200, 4100, 512, 128), (256, 4096, 576, 0), (240, 11012, 384, 128)])
def test_one_hot(orc, bits, T, N, K, group):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    B.load_library()
    print(f"[wonly natural order] W{bits} T={T} {N} x {K} g={group}", flush=True)
    rng = np.random.default_rng(bits * 1000 + T + N + K)
    W = (rng.standard_normal((N, K)) * 0.02 * rng.uniform(0.3, 3.0, (1, K))).astype(np.float16)
    q = orc.quant_weight(W, bits, group)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    at = (np.arange(T) * 37 + 5) % K                      # every place of a word, a chunk and a wavefront's share
    X = np.zeros((T, K), np.float16)
    X[np.arange(T), at] = 1.0
    out = torch.full((T, N), 7.0, dtype=torch.float16, device=DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, T, K, N), dtype=torch.uint8, device=DEV)
    B.aweq_wonly_gemm(dev(X), T, K, K, dev(orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)), bits, group,
                      dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1)), N, None, out, B.AWEQ_F16, N, ws)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint16), np.ascontiguousarray(Wh[:, at].T).view(np.uint16))
