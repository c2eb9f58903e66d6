"""Few-token int8 GEMM: numbers of panels around what its wavefronts have in flight (rings of 1 to 4 panels for each of 8 wavefronts), every
tile, against the exact integer product."""
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


@pytest.mark.parametrize("panels", [1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 33, 39, 47, 48, 49, 56, 95, 97])
def test_panels_around_the_ring(B, orc, panels):
    from conftest import from_panels, to_panels
    rng = np.random.default_rng(panels)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    K = 64 * panels - 8 * (panels % 2)
    for N in (20, 6148):                      # 16 channels a workgroup, 32 (and 64 with more tokens)
        W = rng.integers(-128, 128, (N, K)).astype(np.int8)
        wq = dev(to_panels(W))
        for T in (1, 4, 16, 17, 33, 64):
            if N > 20 and (T == 16 or panels > 50):
                continue
            print(f"[gpu-few-ring] panels={panels} T={T} N={N}", flush=True)
            X = (rng.standard_normal((T, K)) * 2).astype(np.float16)
            inv_s = rng.uniform(0.5, 1.5, K).astype(np.float32)
            a = orc.quant_act(X, inv_s, np.float32(0.04), 120)
            xq = torch.empty(B.aweq_panel_bytes(T, K), dtype=torch.int8, device=DEV)
            rs = torch.empty(T, dtype=torch.int32, device=DEV)
            out = torch.full((T, N), 7, dtype=torch.int32, device=DEV)
            ws = torch.empty(max(16, B.aweq_workspace_size(B.OP_W8A8_GEMM, T, K, N)), dtype=torch.uint8, device=DEV)
            B.aweq_w8a8_gemm(dev(X), B.AWEQ_F16, T, K, K, dev(inv_s), dev(np.array([0.04], np.float32)), dev(np.array([120], np.int32)), xq, rs, None,
                             wq, N, None, None, 0, None, None, out, None, B.AWEQ_F16, N, None, ws)
            torch.cuda.synchronize()
            assert np.array_equal(from_panels(xq.cpu().numpy(), T, K), a["xq"]) and np.array_equal(rs.cpu().numpy(), a["rowsum_x"])
            ref = (a["xq"].astype(np.float64) @ W.astype(np.float64).T).astype(np.int64)
            assert np.array_equal(out.cpu().numpy().astype(np.int64), ref), (T, N)
