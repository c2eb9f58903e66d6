"""The weight-only forward from some hundred tokens on, where its plans change: 64 x 128 and 128 x 128 tiles straight from the
codes, the pass that de-quantises the weight with tiles of 128 and of 256 tokens behind it, one round of workgroups and
several, 1 .. 5 stages of K (every load ring holds three), columns that end inside a stage, a panel of 512 codes or a tile,
zero points outside the packed path.  Against the oracle's fp64 product within the bound of fp32 accumulation in any order,
|y - ref| <= K 2^-24 sum_k |x w| plus one rounding of the output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("bits,T,N,K,group", [
    (4, 200, 4100, 64, 0), (3, 200, 4100, 256, 128), (4, 200, 4100, 512, 256), (3, 200, 4100, 832, -1), (4, 193, 4228, 1280, 128),   # 64 x 128
    (3, 256, 4096, 576, 0),                                                                           # the same, zero points far outside
    (4, 240, 11012, 64, -1), (3, 240, 11012, 128, 128), (3, 250, 10884, 320, 0), (4, 256, 11008, 384, 128), (4, 129, 22020, 640, 128),   # 128 x 128
    (4, 900, 7172, 64, 64), (3, 1000, 7936, 192, 96), (4, 1024, 8192, 320, 64), (3, 900, 7172, 576, -1),   # 128 tokens a tile, one round
    (4, 2500, 7684, 128, 128),                                                                        # the same, three rounds
    (4, 2100, 4100, 64, 0), (3, 2100, 4100, 192, 64), (4, 2304, 4352, 320, 32),                       # 256 tokens a tile, one round
    (3, 4000, 8100, 128, 128),                                                                        # the same, two rounds
])
def test_tiled_parity(B, orc, bits, T, N, K, group):
    print(f"[gpu-wonly-tiles] W{bits} T={T} N={N} K={K} g={group}", flush=True)
    rng = np.random.default_rng(bits + T + N + K)
    shift = 30.0 if K == 576 else 0.0                            # zero points far outside the packed path
    W = (rng.standard_normal((N, K)) * 0.02 * rng.uniform(0.3, 3.0, (1, K)) + shift).astype(np.float16)
    q = orc.quant_weight(W, bits, group)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    X = rng.standard_normal((T, K + 8)).astype(np.float16)       # a pitched view
    bias = rng.standard_normal(N).astype(np.float32)
    ref, mag = orc.wonly_forward(np.ascontiguousarray(X[:, :K]), Wh, bias)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, T, K, N), dtype=torch.uint8, device=DEV)
    for odt in (torch.float16, torch.float32):
        out = torch.full((T, N + 4), 7.0, dtype=odt, device=DEV)
        B.aweq_wonly_gemm(dev(X), T, K, K + 8, dev(packed), bits, group, dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1)), N,
                          dev(bias), out, B.AWEQ_F32 if odt == torch.float32 else B.AWEQ_F16, N + 4, ws)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(got[:, N:] == 7.0)                         # nothing outside the row is touched
        ulp = 2.0 ** -24 if odt == torch.float32 else 2.0 ** -11
        bound = K * 2.0 ** -24 * mag + ulp * np.abs(ref) + 2.0 ** -24
        assert np.all(np.abs(got[:, :N] - ref) <= bound), float(np.max(np.abs(got[:, :N] - ref) / bound))
