"""The activation quantizer on binary32 input against the oracle's true division, exactly, in its three forms (whole rows per
block, panels with column sums, column sums only): elements within a few units in the last place of rounding ties, zero
points inside and outside the screened range, Steps that force the division, subnormal and huge elements (BIGQUOT)."""
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


@pytest.mark.parametrize("step,zero", [
    (0.03, 128), (0.0371, 0), (2.0 ** -7, 255), (1.7e-3, -3900), (0.9, 4096), (0.11, 4097), (0.25, -9000),
    (float(np.nextafter(np.float32(0.5), np.float32(0))), 100), (2.0 ** 59, 3), (2.0 ** 61, 3), (2.0 ** -59, 140), (1e-25, 7),
])
def test_binary32_near_ties(B, orc, step, zero):
    rng = np.random.default_rng(int(abs(zero)) + 1)
    step = np.float32(step)
    for T, K, huge in ((1, 8, False), (5, 520, False), (37, 1096, True), (300, 2048, False)):
        print(f"[gpu-act-f32] step={step} zero={zero} T={T} K={K}", flush=True)
        inv_s = rng.uniform(0.2, 5.0, K).astype(np.float32)
        inv_s[::3] = 1.0
        c = rng.integers(-3, 259, (T, K))
        with np.errstate(over="ignore"):
            X = ((c - zero + 0.5) * np.float64(step) / inv_s.astype(np.float64)).astype(np.float32)
            for _ in range(3):
                X = np.where(rng.random((T, K)) < 0.5, np.nextafter(X, np.float32(rng.choice([-np.inf, np.inf]))), X)
        X[:, 5] = np.float32(1e-42)
        if huge:
            X[3, 7], X[T - 1, K - 1], X[8, 64] = 3e38, -3e38, np.float32(step) * np.float32(2.0 ** 23)
        X = np.ascontiguousarray(np.clip(X, -3.3e38, 3.3e38).astype(np.float32))
        o = orc.quant_act(X, inv_s, float(step), zero)
        dX, ds = torch.from_numpy(X).to(DEV), torch.from_numpy(inv_s).to(DEV)
        dst, dz = torch.tensor([step], dtype=torch.float32, device=DEV), torch.tensor([zero], dtype=torch.int32, device=DEV)
        ws = torch.full((max(16, B.aweq_workspace_size(B.OP_QUANT_ACT, T, K)),), 0x5A, dtype=torch.uint8, device=DEV)
        for codes, sums in ((True, False), (True, True), (False, True)):
            xq = torch.full((B.aweq_panel_bytes(T, K),), 0x5A, dtype=torch.int8, device=DEV) if codes else None
            rs = torch.empty(T, dtype=torch.int32, device=DEV) if codes else None
            cs = torch.empty(K, dtype=torch.int64, device=DEV) if sums else None
            st = torch.zeros(1, dtype=torch.int32, device=DEV)
            B.aweq_quant_act(dX, B.AWEQ_F32, T, K, K, ds, dst, dz, xq, rs, cs, ws, st)
            torch.cuda.synchronize()
            if codes:
                kp = -(-K // 64)
                got = xq.cpu().numpy()[:kp * T * 64].reshape(kp, T, 64).transpose(1, 0, 2).reshape(T, kp * 64)
                assert not got[:, K:].any()
                assert np.array_equal(got[:, :K], o["xq"]) and np.array_equal(rs.cpu().numpy(), o["rowsum_x"])
            if sums:
                assert np.array_equal(cs.cpu().numpy(), o["colsum_xq"])
            assert int(st.item()) == o["status"]
