"""aweq_w8a8_gemm on one to five binary16 / binary32 tokens (up to four are quantised by the GEMM's own launch): codes, row
sums, status and every output equal those of the two separate calls bit for bit, and the codes the oracle's."""
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
@pytest.mark.parametrize("N,K", [(4, 8), (20, 200), (260, 2112), (6148, 136), (100, 4096), (36, 16384), (36, 16392)])
def test_equals_separate_calls(B, orc, dtype, N, K):
    rng = np.random.default_rng(N + K)
    dt = B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32
    wq = rng.integers(-128, 128, (N, K), dtype=np.int8)
    dw, rw = dev(to_panels(wq)), dev(wq.astype(np.int64).sum(1).astype(np.int32))
    sw, zw, bias = dev(rng.uniform(1e-3, 2e-2, N).astype(np.float32)), dev(rng.integers(0, 256, N).astype(np.int32)), dev(rng.standard_normal(N).astype(np.float32))
    for T in (1, 2, 3, 4, 5):
        print(f"[gpu-own-quant] {dtype.__name__} T={T} N={N} K={K}", flush=True)
        X = (rng.standard_normal((T, K + 8)) * 3).astype(dtype)          # a pitched view
        inv_s = rng.uniform(0.2, 2.0, K).astype(np.float32)
        step, zero = np.float32(0.0371), 117
        if K == 200:
            inv_s[3] = 2.0e12 if T % 2 else 1.0                          # outside every division-free path; big quotients
        if K == 136:
            zero = 5000                                                  # outside the screened quotient
        dX, di, ds, dz = dev(X), dev(inv_s), dev(np.float32([step])), dev(np.int32([zero]))
        ref = orc.quant_act(np.ascontiguousarray(X[:, :K]), inv_s, step, zero)
        for odt, i32, cs, rows in ((torch.float16, False, False, True), (torch.float32, True, True, True), (None, True, False, False)):
            new = lambda: dict(xq=torch.full((B.aweq_panel_bytes(T, K),), 5, dtype=torch.int8, device=DEV),
                               rs=torch.full((T,), 5, dtype=torch.int32, device=DEV) if rows else None,
                               oi=torch.full((T, N + 4), 7, dtype=torch.int32, device=DEV) if i32 else None,
                               od=torch.full((T, N + 4), 7.0, dtype=odt, device=DEV) if odt else None,
                               cs=torch.full((N,), 7, dtype=torch.int64, device=DEV) if cs else None,
                               st=torch.zeros(1, dtype=torch.int32, device=DEV))
            ws = torch.empty(max(16, B.aweq_workspace_size(B.OP_W8A8_GEMM, T, K, N)), dtype=torch.uint8, device=DEV)
            out_dt = B.AWEQ_F32 if odt == torch.float32 else B.AWEQ_F16
            a, b = new(), new()
            B.aweq_w8a8_gemm(dX, dt, T, K, K + 8, di, ds, dz, a["xq"], a["rs"], None, dw, N, sw, zw, 0, rw, bias, a["oi"], a["od"], out_dt,
                             N + 4, a["cs"], ws, a["st"])
            B.aweq_quant_act(dX, dt, T, K, K + 8, di, ds, dz, b["xq"], b["rs"], None, ws, b["st"])
            B.aweq_w8a8_gemm(b["xq"], B.AWEQ_I8, T, K, K, None, ds, dz, None, b["rs"], None, dw, N, sw, zw, 0, rw, bias, b["oi"], b["od"], out_dt,
                             N + 4, b["cs"], None, b["st"])
            torch.cuda.synchronize()
            for k in a:
                assert (a[k] is None and b[k] is None) or torch.equal(a[k], b[k]), (T, k)
            assert np.array_equal(from_panels(a["xq"].cpu().numpy(), T, K), ref["xq"])
            if rows:
                assert np.array_equal(a["rs"].cpu().numpy(), ref["rowsum_x"])
            assert int(a["st"].item()) & B.ST_BIGQUOT == ref["status"] & B.ST_BIGQUOT
