"""Activation quantizer at the edges of what its blocks have in flight: rows around the groups of 8 and the ring of two of them, columns
around panels, a wavefront's pair of panels and a block's chunk, for the panel form (column sums asked for) and the row form around
its limits; against the oracle, exactly.  1 / s at an address that is no multiple of 16 where the call takes it."""
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


def _check(B, orc, dtype, T, K, codes, rowsum, colsum, shift, step=0.041, zero=117):
    from conftest import from_panels
    print(f"[gpu-act-ring] {dtype.__name__} T={T} K={K} codes={codes} rowsum={rowsum} colsum={colsum}", flush=True)
    rng = np.random.default_rng(T * 31 + K)
    wide = abs(zero) > 4096
    X = (rng.standard_normal((T, K + 8)) * 2 + ((128 - zero) * step if wide else 0.0)).astype(dtype)     # a pitched view
    inv_s = rng.uniform(*((0.9999, 1.0001) if wide else (0.4, 1.6)), K).astype(np.float32)
    step = np.float32(step)
    a = orc.quant_act(np.ascontiguousarray(X[:, :K]), inv_s, step, zero)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to(DEV)
    inv = torch.zeros(K + 4, dtype=torch.float32, device=DEV)[shift:shift + K]
    inv.copy_(dev(inv_s))
    i32, i64 = torch.int32, torch.int64
    xq = torch.full((B.aweq_panel_bytes(T, K),), 9, dtype=torch.int8, device=DEV) if codes else None
    rs = torch.full((T,), 9, dtype=i32, device=DEV) if rowsum else None
    cs = torch.full((K,), 9, dtype=i64, device=DEV) if colsum else None
    ws = torch.empty(max(16, B.aweq_workspace_size(B.OP_QUANT_ACT, T, K)), dtype=torch.uint8, device=DEV)
    B.aweq_quant_act(dev(X), B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, T, K, K + 8, inv, dev(np.array([step])),
                     dev(np.array([zero], dtype=np.int32)), xq, rs, cs, ws)
    torch.cuda.synchronize()
    if codes:
        assert np.array_equal(from_panels(xq.cpu().numpy(), T, K), a["xq"])
    if rowsum:
        assert np.array_equal(rs.cpu().numpy(), a["rowsum_x"])
    if colsum:
        assert np.array_equal(cs.cpu().numpy(), a["colsum_xq"])


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("T,K", [(1, 8), (7, 64), (8, 120), (15, 128), (16, 136), (17, 192), (31, 512), (33, 520), (64 + 9, 640), (513, 1032), (40, 4104), (70, 1024 + 56)])
def test_panel_form(B, orc, dtype, T, K):
    _check(B, orc, dtype, T, K, True, True, True, 1)
    _check(B, orc, dtype, T, K, False, False, True, 0)


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("T,K", [(1, 8), (3, 4088), (5, 4096), (257, 4104), (1027, 520), (2, 8200), (4097, 2040), (4097, 2048), (6, 12288)])
def test_row_form(B, orc, dtype, T, K):
    _check(B, orc, dtype, T, K, True, True, False, 0)


@pytest.mark.parametrize("zero", [6000, -6000, 1 << 21])
@pytest.mark.parametrize("T,K", [(3, 4096), (15, 128), (16, 128), (17, 256), (40, 1032), (70, 512), (513, 1152), (4097, 640)])
def test_zero_points_beyond_the_screen(B, orc, zero, T, K):
    """Quotients that need the exact form: whole groups of rows one at a time, and what the ring leaves over."""
    step = 0.041 if abs(zero) < 10000 else 0.0041   # (inputs within binary16)
    for dtype in (np.float16, np.float32):
        _check(B, orc, dtype, T, K, True, True, True, 0, step, zero)
        _check(B, orc, dtype, T, K, False, False, True, 1, step, zero)
        _check(B, orc, dtype, T, K, True, True, False, 0, step, zero)
