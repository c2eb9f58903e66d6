"""Weight-only forward with few input channels, on both sides of the sizes where the few-token kernel gives way to the tiled form, for
groups that only these two take, against the oracle's fp64 product within the bound of fp32 accumulation in any order,
|y - ref| <= K 2^-24 sum_k |x w| plus one rounding of the output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("T,N,K", [(512, 4096, 64), (512, 4096, 256), (300, 4096, 768), (300, 4096, 2048), (65, 11008, 192), (65, 11008, 1088)])
def test_few_input_channels(orc, bits, T, N, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    print(f"[gpu-wonly-short] W{bits} T={T} {N} x {K}", flush=True)
    rng = np.random.default_rng(T + N + K + bits)
    q = orc.quant_weight((rng.standard_normal((N, K)) * 0.02).astype(np.float16), bits, 64)
    Wh = orc.dequant_weight_h(q["codes_u"], 64, q["step"], q["zero"])
    X, bias = rng.standard_normal((T, K)).astype(np.float16), rng.standard_normal(N).astype(np.float32)
    ref, mag = orc.wonly_forward(X, Wh, bias)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    out = torch.full((T, N), 7.0, dtype=torch.float16, device=DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, T, K, N), dtype=torch.uint8, device=DEV)
    B.aweq_wonly_gemm(dev(X), T, K, K, dev(orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)), bits, 64, dev(q["step"].reshape(-1)),
                      dev(q["zero"].reshape(-1)), N, dev(bias), out, B.AWEQ_F16, N, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= K * 2.0 ** -24 * mag + 2.0 ** -11 * np.abs(ref) + 2.0 ** -24)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("T,N,K", [(312, 2532, 64), (1309, 616, 128), (512, 1024, 8192), (512, 1024, 8256)])
def test_on_both_sides_of_the_added_launch(orc, bits, T, N, K):
    """Calls so small that the de-quantising launch decides, and K beyond which the few-token kernel's cost has no offset."""
    test_few_input_channels(orc, bits, T, N, K)
