"""Weight-only forward of few tokens in tiles of 8, 12, 20 and 24 tokens (the last tile of the matrix operand is not whole) and of 16
wavefronts: token counts at the edges of these tiles, K with one chunk of 256 a wavefront, a remainder, and one chunk less; against the oracle's
fp64 product within the bound of fp32 accumulation in any order, K 2^-24 sum_k |x w| plus one rounding of the output.  A token that holds
infinities next to the tile's edge changes no other row."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits,N,K,group", [(4, 52, 4096, 128), (3, 36, 4096 + 128, 128), (4, 20, 3840, 64), (3, 8228, 256, 128), (4, 12292, 320, 0), (3, 8228, 320, 0), (3, 12292, 256, 64)])
def test_token_quads(orc, bits, N, K, group):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    rng = np.random.default_rng(bits * 7 + N + K)
    W = (rng.standard_normal((N, K)) * 0.02 * rng.uniform(0.3, 3.0, (1, K))).astype(np.float16)
    q = orc.quant_weight(W, bits, group)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    codes, step, zero = dev(packed), dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1))
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, 1, K, N), dtype=torch.uint8, device=DEV)
    for T in (6, 8, 9, 12, 13, 16, 17, 20, 21, 24, 25, 32):
        print(f"[gpu-wonly-quads] W{bits} T={T} N={N} K={K} g={group}", flush=True)
        X = rng.standard_normal((T, K)).astype(np.float16)
        out = torch.empty((T, N), dtype=torch.float32, device=DEV)
        run = lambda x: B.aweq_wonly_gemm(dev(x), T, K, K, codes, bits, group, step, zero, N, None, out, B.AWEQ_F32, N, ws)
        run(X)
        got = out.cpu().numpy().astype(np.float64)
        ref, mag = orc.wonly_forward(X, Wh, None)
        assert np.all(np.abs(got - ref) <= K * 2.0 ** -24 * mag + 2.0 ** -23 * np.abs(ref))
        X[T - 1] = np.inf
        run(X)
        assert np.array_equal(out[: T - 1].cpu().numpy(), got[: T - 1].astype(np.float32))
