"""Activation quantizer without column sums at the token counts and widths where whole rows per block give way to panels: codes and row
sums equal the oracle's."""
import numpy as np
import pytest

from conftest import from_panels

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("K", [8, 512, 520])
@pytest.mark.parametrize("T", [2048, 2049, 4096, 4097])
def test_rows_and_panels(orc, dtype, T, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    print(f"[gpu-act-narrow] {dtype.__name__} T={T} K={K}", flush=True)
    rng = np.random.default_rng(T + K)
    X, inv_s = (rng.standard_normal((T, K)) * 3).astype(dtype), rng.uniform(0.2, 2.0, K).astype(np.float32)
    ref = orc.quant_act(X, inv_s, np.float32(0.0371), 117)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    xq = torch.full((B.aweq_panel_bytes(T, K),), 5, dtype=torch.int8, device=DEV)
    rs = torch.full((T,), 5, dtype=torch.int32, device=DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_QUANT_ACT, T, K), dtype=torch.uint8, device=DEV)
    B.aweq_quant_act(dev(X), B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, T, K, K, dev(inv_s), dev(np.float32([0.0371])), dev(np.int32([117])),
                     xq, rs, None, ws)
    torch.cuda.synchronize()
    assert np.array_equal(from_panels(xq.cpu().numpy(), T, K), ref["xq"]) and np.array_equal(rs.cpu().numpy(), ref["rowsum_x"])


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("T,K", [(2049, 512), (4096, 8), (4097, 512)])
def test_rows_and_panels_without_sums(orc, dtype, T, K):
    """Without row sums whole rows stay the form for up to 4096 narrow tokens."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    rng = np.random.default_rng(T + K)
    X, inv_s = (rng.standard_normal((T, K)) * 3).astype(dtype), rng.uniform(0.2, 2.0, K).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    xq = torch.full((B.aweq_panel_bytes(T, K),), 5, dtype=torch.int8, device=DEV)
    B.aweq_quant_act(dev(X), B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, T, K, K, dev(inv_s), dev(np.float32([0.0371])), dev(np.int32([117])),
                     xq, None, None)
    torch.cuda.synchronize()
    assert np.array_equal(from_panels(xq.cpu().numpy(), T, K), orc.quant_act(X, inv_s, np.float32(0.0371), 117)["xq"])
