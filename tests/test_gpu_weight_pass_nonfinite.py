"""The pass over the weights of a calibration in one call, where weights hold NaN, infinities, zeros of both signs and rows far from zero: the
extremes hand a NaN on and are then taken again without it.  Against the stage entry points (a workspace of the stages' size), to the bit: folded
weights, codes, Step, Z, row sums; one and two short rows for a wavefront and rows for a block, a NaN in the first, middle and last unit and lane."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("N,K,bits,group", [(9, 512, 8, 0), (13, 1024, 8, 0), (10, 4096, 8, 0), (11, 5000, 8, 0), (7, 11008, 8, 0), (5, 13000, 8, 0),
                                            (9, 512, 4, 128), (10, 4096, 4, 128), (7, 2048, 3, 32), (6, 1536, 3, 512), (2051, 1024, 8, 0), (2049, 72, 8, 0)])
def test_nonfinite_weights(N, K, bits, group, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B, pipeline
    g = torch.Generator(device=DEV)
    g.manual_seed(N + K)
    T = 96
    X = torch.randn(T, K, generator=g, device=DEV).to(dtype)
    W = (torch.randn(N, K, generator=g, device=DEV) * 0.02).to(dtype)
    W[0, 0] = float("nan")
    W[1, K - 1] = float("nan")
    W[1, 7] = float("inf")
    W[2, K // 2 + 3] = float("-inf")
    W[3] = 0.0
    W[3, ::2] = -0.0
    W[4] += 30.0                          # zero points far outside the screen
    W[N - 1, 1::2] = float("nan")         # every pair of halves
    w8a8 = bits == 8
    outs = []
    for stages in (False, True):
        buf = pipeline.LayerBuffers(T, K, N, dtype, bits=bits, group=group, w8a8=w8a8, device=DEV)
        if stages:
            size = max(B.aweq_workspace_size(B.OP_CALIB_STATS, T, K, 0), B.aweq_workspace_size(B.OP_CALIB_STATS, N, K, N),
                       B.aweq_workspace_size(B.OP_QUANT_ACT, T, K, 0), 16)
            assert size < B.aweq_workspace_size(B.OP_CALIBRATE, T, K, N)
            buf.t["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
        t = pipeline.calibrate_layer(X, W, None, buf, fused_weight_pass=False, forward=False)
        outs.append({k: t[k].cpu() for k in ("W_hat", "codes", "step_w", "zero_w", "status") + (("rowsum_w",) if w8a8 else ())})
    for k, v in outs[0].items():
        assert torch.equal(v.view(torch.uint8), outs[1][k].view(torch.uint8)), k
