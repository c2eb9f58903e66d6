"""The activation quantizer's row form around the token counts where a block's rows change (one up to 256, two up to 1536, four beyond), the last
block not full, against the oracle: codes and row sums exact, nothing written past the panels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("T", [256, 257, 1024, 1025, 1535, 1536, 1537, 1539])
def test_rows_edges(orc, T, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B, layout
    K = 600                                                     # more than one panel chunk, a ragged last panel
    rng = np.random.default_rng(T)
    X = (rng.standard_normal((T, K)) * rng.uniform(0.5, 8.0, (1, K))).astype(dtype)
    inv_s = rng.uniform(0.3, 2.0, K).astype(np.float32)
    step, zero = np.float32(0.07), 119
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    nb = B.aweq_panel_bytes(T, K)
    xq = torch.full((nb + 64,), 77, dtype=torch.int8, device=DEV)
    rs = torch.full((T + 1,), 77, dtype=torch.int32, device=DEV)
    ws = torch.empty(B.aweq_workspace_size(B.OP_QUANT_ACT, T, K, 0), dtype=torch.uint8, device=DEV)
    B.aweq_quant_act(dev(X), B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, T, K, K, dev(inv_s), dev(np.array([step])),
                     dev(np.array([zero], np.int32)), xq, rs, None, ws, None)
    ref = orc.quant_act(X, inv_s, step, zero)
    got = xq.cpu().numpy()
    assert np.array_equal(layout.from_panels(got[:nb], T, K), ref["xq"]) and np.all(got[nb:] == 77)
    assert np.array_equal(rs.cpu().numpy()[:T], ref["rowsum_x"]) and int(rs[T]) == 77
