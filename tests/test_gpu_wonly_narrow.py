"""Weight-only forward of a narrow layer on millions of tokens: more 32-token tiles than a grid's y dimension holds (65535), on
both sides of that limit, against the oracle's fp64 product within the bound of fp32 accumulation in any order,
|y - ref| <= K 2^-24 sum_k |x w| plus one rounding of the output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits,T", [(4, 65535 * 32), (4, 65535 * 32 + 1), (3, 65535 * 32 + 77)])
@pytest.mark.parametrize("N", [16, 32])
def test_more_token_tiles_than_a_grid_dimension(orc, bits, T, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    print(f"[gpu-wonly-narrow] W{bits} T={T} N={N}", flush=True)
    K = 64
    rng = np.random.default_rng(bits + T + N)
    q = orc.quant_weight((rng.standard_normal((N, K)) * 0.02).astype(np.float16), bits, 64)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    Wh = orc.dequant_weight_h(q["codes_u"], 64, q["step"], q["zero"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    X = torch.randn(T, K, generator=torch.Generator(device=DEV).manual_seed(T), device=DEV).half()
    out = torch.full((T, N), 7.0, dtype=torch.float16, device=DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, T, K, N), dtype=torch.uint8, device=DEV)
    B.aweq_wonly_gemm(X, T, K, K, dev(packed), bits, 64, dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1)), N, None, out, B.AWEQ_F16, N, ws)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(512), np.arange(T - 512, T), rng.integers(0, T, 4096)]))
    sel = torch.from_numpy(rows).to(DEV)
    ref, mag = orc.wonly_forward(X[sel].cpu().numpy(), Wh, None)
    got = out[sel].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= K * 2.0 ** -24 * mag + 2.0 ** -11 * np.abs(ref) + 2.0 ** -24)
    assert not torch.any(out == 7.0)
