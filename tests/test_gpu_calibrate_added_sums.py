"""The calibration in one call, whose activation quantizer adds its code sums up in place: column and row sums against the codes that it wrote,
where blocks change (one column chunk of 512 or several, slices of 16 and 32 rows, a ragged last panel), the accumulator's sums against the
weight's codes, on buffers and a workspace that hold something else before each call.  Integers: all exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("T,N,K", [(1, 4, 8), (15, 20, 512), (17, 33, 520), (257, 100, 1032), (2048, 64, 512), (2081, 64, 512), (4097, 36, 1088),
                                   (520, 68, 4096), (300, 40, 11008)])
def test_added_sums(T, N, K, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import layout, pipeline
    g = torch.Generator(device=DEV)
    g.manual_seed(T + N + K)
    X = (torch.randn(T, K, generator=g, device=DEV) * (1 + 20 * torch.rand(K, generator=g, device=DEV)) + 0.3).to(dtype)
    W = (torch.randn(N, K, generator=g, device=DEV) * 0.02).to(dtype)
    buf = pipeline.LayerBuffers(T, K, N, dtype, device=DEV)
    full = buf.t["ws"]
    for fill in (0x55, 0xff):
        # (room for one copy of a narrow matrix's sums only, then for all)
        buf.t["ws"] = full[:full.numel() - 12 * K].contiguous() if fill == 0x55 and K <= 1024 and full.numel() > 16 * K else full
        for t in buf.t.values():
            if t is not None and t.numel():
                t.view(torch.uint8).fill_(fill)
        buf.t["status"].zero_()
        t = pipeline.calibrate_layer(X, W, None, buf, fused_weight_pass=True)
        torch.cuda.synchronize()
        xq = layout.from_panels(t["xq"].cpu().numpy(), T, K).astype(np.int64)
        wq = layout.from_panels(t["codes"].cpu().numpy(), N, K).astype(np.int64)
        assert np.array_equal(t["rowsum_x"].cpu().numpy(), xq.sum(1))
        assert np.array_equal(t["colsum_xq"].cpu().numpy(), xq.sum(0))
        assert np.array_equal(t["rowsum_w"].cpu().numpy(), wq.sum(1))
        assert np.array_equal(t["colsum_acc"].cpu().numpy(), wq @ xq.sum(0))
        assert np.array_equal(t["out_i32"].cpu().numpy(), xq @ wq.T)
