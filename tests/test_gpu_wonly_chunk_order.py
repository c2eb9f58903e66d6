"""Weight-only forward of few tokens: rows a multiple of 4 KiB apart, whose workgroups begin their rounds over K at different places, and token
counts on both sides of those from which quads of tokens are not left out, against the oracle's fp64 product within the bound of fp32
accumulation in any order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits,N,K,tokens", [(4, 2052, 8192, (1, 5, 12, 13, 16, 17, 24, 25, 33)),     # more workgroups than an XCD's round has places
                                             (4, 276, 16384, (2, 12, 13, 32)), (3, 260, 32768, (1, 16, 17, 25)),   # 16 wavefronts; two chunks and more
                                             (3, 516, 448, (12, 13, 16, 24, 25, 33)), (4, 516, 320, (13, 25)),    # a last chunk of which there is half
                                             (4, 8212, 320, (1, 4, 5, 12, 13, 16)), (3, 12288, 1088, (1, 5, 16)), (4, 12292, 64, (4, 5)), (3, 16384, 128, (4,))])   # four wavefronts, and past them
def test_chunk_order(orc, bits, N, K, tokens):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    B.load_library()
    rng = np.random.default_rng(bits * 100 + N + K)
    group = 128 if K % 128 == 0 else 64
    W = (rng.standard_normal((N, K)) * 0.02 * rng.uniform(0.3, 3.0, (1, K))).astype(np.float16)
    q = orc.quant_weight(W, bits, group)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    codes, step, zero = dev(orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)), dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1))
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, 1, K, N), dtype=torch.uint8, device=DEV)
    for T in tokens:
        print(f"[gpu-wonly-chunk-order] W{bits} T={T} N={N} K={K}", flush=True)
        X = rng.standard_normal((T, K)).astype(np.float16)
        out = torch.full((T, N), 7.0, dtype=torch.float32, device=DEV)
        B.aweq_wonly_gemm(dev(X), T, K, K, codes, bits, group, step, zero, N, None, out, B.AWEQ_F32, N, ws)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        ref, mag = orc.wonly_forward(X, Wh, None)
        assert np.all(np.abs(got - ref) <= K * 2.0 ** -24 * mag + 2.0 ** -24), T
