"""The calibration in one call, whose activation quantizer adds its code sums up in place: column and row sums against the codes that it wrote,
where blocks change (one column chunk of 512 or several, slices of 16 and 32 rows, a ragged last panel) and where the copies of a narrow matrix's sums
change from one to four, the accumulator's sums against the weight's codes, on buffers and a workspace that hold something else before each call.
Integers: all exact.  Every call takes the five launches in one, which a captured graph shows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_calibrate_group_forward import _kernels  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("T,N,K", [(1, 4, 8), (15, 20, 512), (17, 33, 520), (257, 100, 1032), (1280, 64, 512), (1281, 64, 504), (2048, 64, 512), (2081, 64, 512), (2048, 36, 1024),
                                   (2049, 36, 520), (2111, 36, 1024), (4097, 36, 1088),
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
    whole = lambda n: -(-n // 256) * 256
    less = whole(16 * K) - whole(4 * K) if K <= 1024 else 0   # what three copies of a narrow matrix's sums take
    for fill in (0x55, 0xff):
        # (room for one copy only, then for all)
        buf.t["ws"] = full[:full.numel() - less].contiguous() if fill == 0x55 else full
        for t in buf.t.values():
            if t is not None and t.numel():
                t.view(torch.uint8).fill_(fill)
        buf.t["status"].zero_()
        t = pipeline.calibrate_layer(X, W, None, buf, fused_weight_pass=True)
        torch.cuda.synchronize()
        assert len(_kernels(lambda: pipeline.calibrate_layer(X, W, None, buf, fused_weight_pass=True))) == 5
        xq = layout.from_panels(t["xq"].cpu().numpy(), T, K).astype(np.int64)
        wq = layout.from_panels(t["codes"].cpu().numpy(), N, K).astype(np.int64)
        assert np.array_equal(t["rowsum_x"].cpu().numpy(), xq.sum(1))
        assert np.array_equal(t["colsum_xq"].cpu().numpy(), xq.sum(0))
        assert np.array_equal(t["rowsum_w"].cpu().numpy(), wq.sum(1))
        assert np.array_equal(t["colsum_acc"].cpu().numpy(), wq @ xq.sum(0))
        assert np.array_equal(t["out_i32"].cpu().numpy(), xq @ wq.T)
