"""Weight-only forward for few tokens (the kernel that multiplies straight from the packed codes): token counts at the
edges of its tiles, output channels and K with remainders, every group form, against the oracle's fp64 product within
the bound of fp32 accumulation in any order, |y - ref| <= K 2^-24 sum_k |x w| plus one rounding of the output."""
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


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,group", [
    (4, 64, 64), (20, 128, 32), (36, 192, 96), (260, 320, 64),   # groups no multiple of 128; K short of a chunk of 256
    (100, 2048 + 128, 128), (48, 4096 + 64, 0), (52, 640, -1),   # one chunk beyond the eight wavefronts; per row; per tensor
    (68, 1024, 512), (12292, 256, 128),                          # long groups; more channels than the narrow tile takes
])
def test_few_tokens_parity(B, orc, bits, N, K, group):
    rng = np.random.default_rng(bits * 100 + N + K)
    shift = 30.0 if N == 36 else 0.0                             # zero points far outside the packed path
    W = (rng.standard_normal((N, K)) * 0.02 * rng.uniform(0.3, 3.0, (1, K)) + shift).astype(np.float16)
    q = orc.quant_weight(W, bits, group)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    codes, step, zero = dev(packed), dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1))
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, 1, K, N), dtype=torch.uint8, device=DEV)
    for T in (1, 4, 5, 16, 17, 32, 33, 65, 256, 257):
        print(f"[gpu-wonly-few] W{bits} T={T} N={N} K={K} g={group}", flush=True)
        X = rng.standard_normal((T, K + 8)).astype(np.float16)   # a pitched view
        bias = rng.standard_normal(N).astype(np.float32) if T % 2 else None
        odt = torch.float32 if T in (4, 17, 65) else torch.float16
        ldo = N + 4
        out = torch.full((T, ldo), 7.0, dtype=odt, device=DEV)
        B.aweq_wonly_gemm(dev(X), T, K, K + 8, codes, bits, group, step, zero, N, dev(bias) if bias is not None else None, out,
                          B.AWEQ_F32 if odt == torch.float32 else B.AWEQ_F16, ldo, ws)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(got[:, N:] == 7.0)                         # nothing outside the row is touched
        ref, mag = orc.wonly_forward(np.ascontiguousarray(X[:, :K]), Wh, bias)
        ulp = 2.0 ** -24 if odt == torch.float32 else 2.0 ** -11
        bound = K * 2.0 ** -24 * mag + ulp * np.abs(ref) + 2.0 ** -24
        assert np.all(np.abs(got[:, :N] - ref) <= bound), (T, float(np.max(np.abs(got[:, :N] - ref) / bound)))
