"""W8A8 forward for few tokens (whole-row activation quantizer, few-token int8 GEMM): token counts at the edges of the
tiles and of the rows per block, output channels and K with remainders, against the oracle.  Everything is exact: codes,
sums, int32 accumulator; the outputs equal the oracle's fp64 value rounded once (binary32) or to within one unit in the
last place (binary16, whose fp64 operation is fused on the GPU)."""
import numpy as np
import pytest

from conftest import from_panels, to_panels

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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("K", [8, 72, 512, 4104, 8192 + 56])
def test_row_quantizer(B, orc, dtype, K):
    rng = np.random.default_rng(K)
    for T in (1, 2, 255, 257, 258, 1025, 1027):
        print(f"[gpu-w8a8-few] rows T={T} K={K} {dtype.__name__}", flush=True)
        X = (rng.standard_normal((T, K)) * 3).astype(dtype)
        inv_s = rng.uniform(0.2, 2.0, K).astype(np.float32)
        if K == 512:
            inv_s[3] = 2.0e12                                    # outside every division-free path
        step, zero = np.float32(0.0371), 117
        ref = orc.quant_act(X, inv_s, step, zero)
        xq = torch.full((B.aweq_panel_bytes(T, K),), 5, dtype=torch.int8, device=DEV)
        rs = torch.full((T,), 5, dtype=torch.int32, device=DEV)
        ws = torch.empty(B.aweq_workspace_size(B.OP_QUANT_ACT, T, K), dtype=torch.uint8, device=DEV)
        B.aweq_quant_act(dev(X), B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, T, K, K, dev(inv_s), dev(np.float32([step])),
                         dev(np.int32([zero])), xq, rs, None, ws)
        torch.cuda.synchronize()
        assert np.array_equal(from_panels(xq.cpu().numpy(), T, K), ref["xq"]), T
        assert np.array_equal(rs.cpu().numpy(), ref["rowsum_x"]), T


@pytest.mark.parametrize("N,K,w_group", [(4, 64, 0), (20, 200, -1), (36, 520, 0), (260, 64 * 33, 0), (6148, 136, -1), (2052, 1024, 0)])
def test_few_token_gemm(B, orc, N, K, w_group):
    rng = np.random.default_rng(N + K)
    wq = rng.integers(-128, 128, (N, K), dtype=np.int8)
    ng = N if w_group == 0 else 1
    step_w = rng.uniform(1e-3, 2e-2, ng).astype(np.float32)
    zero_w = rng.integers(0, 256, ng).astype(np.int32)
    if N == 36:
        zero_w[5] = -700                                         # outside [0, 255]: flagged, still exact at this K
    rw = wq.astype(np.int64).sum(1).astype(np.int32)
    step_x, zero_x = np.float32(0.02), 131
    for T in (1, 15, 16, 17, 32, 33, 63, 65, 130):
        print(f"[gpu-w8a8-few] gemm T={T} N={N} K={K}", flush=True)
        xq = rng.integers(-128, 128, (T, K), dtype=np.int8)
        rx = xq.astype(np.int64).sum(1).astype(np.int32)
        bias = rng.standard_normal(N).astype(np.float32) if T % 2 else None
        acc = orc.gemm_i8(xq, wq)
        zx, zw = zero_x - 128, (zero_w.astype(np.int64) - 128) * np.ones(N, np.int64)
        iv = acc.astype(np.int64) - zx * rw.astype(np.int64) - zw * rx.astype(np.int64)[:, None] + K * zx * zw
        ref = iv.astype(np.float64) * (np.float64(step_x) * step_w.astype(np.float64)) + (0.0 if bias is None else bias.astype(np.float64))
        for odt in (torch.float16, torch.float32):
            oi = torch.full((T, N + 4), 7, dtype=torch.int32, device=DEV)
            od = torch.full((T, N + 4), 7.0, dtype=odt, device=DEV)
            cs = torch.full((N,), 7, dtype=torch.int64, device=DEV)
            st = torch.zeros(1, dtype=torch.int32, device=DEV)
            want_i32, want_cs = T != 16, T != 17
            B.aweq_w8a8_gemm(dev(to_panels(xq)), B.AWEQ_I8, T, K, K, None, dev(np.float32([step_x])), dev(np.int32([zero_x])), None, dev(rx),
                             None, dev(to_panels(wq)), N, dev(step_w), dev(zero_w), w_group, dev(rw), dev(bias) if bias is not None else None,
                             oi if want_i32 else None, od, B.AWEQ_F16 if odt == torch.float16 else B.AWEQ_F32, N + 4,
                             cs if want_cs else None, None, st)
            torch.cuda.synchronize()
            got = od.cpu().numpy()
            if want_i32:
                g = oi.cpu().numpy()
                assert np.array_equal(g[:, :N], acc) and np.all(g[:, N:] == 7)
            if want_cs:
                assert np.array_equal(cs.cpu().numpy(), acc.astype(np.int64).sum(0))
            assert np.all(got[:, N:] == 7.0)
            if odt == torch.float32:
                assert np.array_equal(got[:, :N], ref.astype(np.float32))
            else:
                r16 = ref.astype(np.float32).astype(np.float16)
                assert np.all(np.abs(got[:, :N].astype(np.float64) - r16.astype(np.float64)) <= np.spacing(np.abs(r16)).astype(np.float64))
            assert int(st.item()) == (B.ST_ZEROPOINT if N == 36 else 0)
