"""Weight-only forward on rows so far apart that 32-bit offsets do not reach over a tile of them: 256 tokens beyond a pitch of 2^23,
128 beyond 2^24, the few-token kernel's 32 and 16 beyond 2^27 and 2^28.  Against the oracle's fp64 product within the bound of
fp32 accumulation in any order, |y - ref| <= K 2^-24 sum_k |x w| plus one rounding of the output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits,T,N,group,ldx", [
    (4, 513, 21504, 64, (1 << 23) + (1 << 16)), (4, 160, 4100, 0, (1 << 24) - 8), (3, 160, 4100, 0, (1 << 24) + (1 << 18)),
    (4, 513, 21504, 96, (1 << 24) + (1 << 18)), (4, 40, 260, 32, (1 << 27) + (1 << 23)), (3, 12, 20, -1, (1 << 29) + 64), (4, 3, 20, 64, (1 << 31) + 8),
])
def test_rows_far_apart(orc, bits, T, N, group, ldx):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    print(f"[gpu-wonly-pitch] W{bits} T={T} N={N} g={group} ldx={ldx}", flush=True)
    K = 192 if group == 96 else 128
    rng = np.random.default_rng(T + N)
    q = orc.quant_weight((rng.standard_normal((N, K)) * 0.02).astype(np.float16), bits, group)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    X, bias = rng.standard_normal((T, K)).astype(np.float16), rng.standard_normal(N).astype(np.float32)
    home = torch.empty((T - 1) * ldx + K, dtype=torch.float16, device=DEV)
    for t, row in enumerate(dev(X)):
        home[t * ldx:t * ldx + K] = row
    out = torch.full((T, N + 4), 7.0, dtype=torch.float16, device=DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, T, K, N), dtype=torch.uint8, device=DEV)
    B.aweq_wonly_gemm(home, T, K, ldx, dev(packed), bits, group, dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1)), N, dev(bias), out, B.AWEQ_F16,
                      N + 4, ws)
    torch.cuda.synchronize()
    del home
    torch.cuda.empty_cache()
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(got[:, N:] == 7.0)
    ref, mag = orc.wonly_forward(X, Wh, bias)
    assert np.all(np.abs(got[:, :N] - ref) <= K * 2.0 ** -24 * mag + 2.0 ** -11 * np.abs(ref) + 2.0 ** -24)
