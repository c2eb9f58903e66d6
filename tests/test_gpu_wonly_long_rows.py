"""Weight-only forward of a few tokens over long rows: K split between 16 wavefronts, on both sides of the lengths from which it is, against
the oracle's fp64 product within the bound of fp32 accumulation in any order."""
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
@pytest.mark.parametrize("N,K,group", [(20, 8192 - 128, 128), (20, 8192 + 64, 64), (36, 8192 + 128, 128), (4, 16384 - 64, 0), (20, 16384 + 192, 32)])
def test_few_tokens_over_long_rows(B, orc, bits, N, K, group):
    rng = np.random.default_rng(bits * 100 + N + K)
    W = (rng.standard_normal((N, K)) * 0.02 * rng.uniform(0.3, 3.0, (1, K))).astype(np.float16)
    q = orc.quant_weight(W, bits, group)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    Wh = orc.dequant_weight_h(q["codes_u"], group, q["step"], q["zero"])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    codes, step, zero = dev(packed), dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1))
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, 1, K, N), dtype=torch.uint8, device=DEV)
    for T in (1, 3, 4, 5, 16, 17):
        print(f"[gpu-wonly-long] W{bits} T={T} N={N} K={K} g={group}", flush=True)
        X = rng.standard_normal((T, K + 8)).astype(np.float16)   # a pitched view
        out = torch.full((T, N + 4), 7.0, dtype=torch.float16, device=DEV)
        B.aweq_wonly_gemm(dev(X), T, K, K + 8, codes, bits, group, step, zero, N, None, out, B.AWEQ_F16, N + 4, ws)
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.all(got[:, N:] == 7.0)
        ref, mag = orc.wonly_forward(np.ascontiguousarray(X[:, :K]), Wh, None)
        bound = K * 2.0 ** -24 * mag + 2.0 ** -11 * np.abs(ref) + 2.0 ** -24
        assert np.all(np.abs(got[:, :N] - ref) <= bound), T


def test_an_infinite_activation_stays_in_its_token(B, orc):
    """The last values of K stand in for the ones past it, with zero activations: an infinity or NaN among the activations reaches the
    outputs of its own token only, and as the product has it."""
    N, K, bits = 8, 192, 4
    rng = np.random.default_rng(5)
    q = orc.quant_weight((rng.standard_normal((N, K)) * 0.02).astype(np.float16), bits, 64)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    codes, step, zero = dev(orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)), dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1))
    Wh = orc.dequant_weight_h(q["codes_u"], 64, q["step"], q["zero"]).astype(np.float64).reshape(N, K)
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, 1, K, N), dtype=torch.uint8, device=DEV)
    for T in (3, 18):
        X = rng.standard_normal((T, K)).astype(np.float16)
        X[1, K - 1] = np.inf      # the values that are read again past K
        X[2, 5] = np.nan
        out = torch.empty(T, N, dtype=torch.float32, device=DEV)
        B.aweq_wonly_gemm(dev(X), T, K, K, codes, bits, 64, step, zero, N, None, out, B.AWEQ_F32, N, ws)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        with np.errstate(invalid="ignore"):
            ref = X.astype(np.float64) @ Wh.T
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        keep = [t for t in range(T) if t not in (1, 2)]
        assert np.all(np.abs(got[keep] - ref[keep]) <= K * 2.0 ** -24 * (np.abs(X[keep].astype(np.float64)) @ np.abs(Wh).T))


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("K,group", [(192, 0), (192, 64), (64, 32), (320, 0), (8192 + 64, 0)])
def test_an_infinite_weight_is_not_met_by_the_zeros_past_k(B, bits, K, group):
    """A weight beyond binary16's range is infinite as a GEMM operand.  Among the last values of K, which stand in for the ones past it, it
    is multiplied with its activation only: an infinite output, not the NaN of infinity times zero."""
    N, top, zero = 20, 2 ** bits - 1, 3
    rng = np.random.default_rng(K + bits)
    step = np.float32(65504 // (top - 1 - zero) // 64 * 64)   # (a binary16 value)  the highest code is beyond the range, the others are not
    u = rng.integers(0, top, (N, K)).astype(np.uint8)
    u[5, K - 1] = u[9, K - 17] = top
    packed = np.packbits(np.unpackbits(u[..., None], axis=-1, bitorder="little")[..., :bits].reshape(N, K * bits), axis=-1, bitorder="little").reshape(-1)
    ng = N * (K // group) if group else N
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    codes, steps, zeros = dev(packed), torch.full((ng,), float(step), device=DEV), torch.full((ng,), zero, dtype=torch.int32, device=DEV)
    with np.errstate(over="ignore"):
        Wh = ((u.astype(np.float32) - zero) * step).astype(np.float16).astype(np.float64)
    assert np.isinf(Wh).sum() == 2
    ws = torch.empty(B.aweq_workspace_size(B.OP_WONLY_GEMM, 1, K, N), dtype=torch.uint8, device=DEV)
    for T in (1, 4, 5, 12, 13, 16, 17, 25, 40, 64):
        print(f"[gpu-wonly-inf] W{bits} T={T} K={K} g={group}", flush=True)
        X = (np.abs(rng.standard_normal((T, K))) + 0.01).astype(np.float16)
        out = torch.empty(T, N, dtype=torch.float32, device=DEV)
        B.aweq_wonly_gemm(dev(X), T, K, K, codes, bits, group, steps, zeros, N, None, out, B.AWEQ_F32, N, ws)
        torch.cuda.synchronize()
        got, ref = out.cpu().numpy(), X.astype(np.float64) @ Wh.T
        assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and not np.isnan(got).any(), T
        ok = np.isfinite(ref)
        assert np.all(np.abs(got[ok] - ref[ok]) <= (K * 2.0 ** -24 * (np.abs(X.astype(np.float64)) @ np.where(np.isinf(Wh), 0, np.abs(Wh)).T))[ok]), T
