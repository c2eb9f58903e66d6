"""The binary16 forward of layers that read the same activation, in one launch of the tiled GEMM, against a launch for each: to the bit.  Two to
four layers, with and without biases; rows, columns and tiles at the edges of tiles of 128 and 256 tokens x 256 channels, rows that share lines,
one round of workgroups and several, one panel of K and many; zero points beyond the short epilogue's."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,T,N,K,shift", [(2, 700, 256, 64, 0.0), (3, 1000, 260, 512, 0.0), (4, 2100, 508, 136, 0.0), (3, 2048, 1024, 1024, 0.0),
                                           (2, 1537, 2300, 640, 0.0), (3, 8200, 768, 320, 0.0), (2, 5000, 4092, 128, 0.0), (2, 1500, 1280, 256, 40.0)])
def test_group_forward(n, T, N, K, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B, pipeline
    g = torch.Generator(device=DEV)
    g.manual_seed(T + N + K)
    X = (torch.randn(T, K, generator=g, device=DEV) * 2 + 0.3).half()
    W = [(torch.randn(N, K, generator=g, device=DEV) * 0.02 + shift).half() for _ in range(n)]
    b = [torch.randn(N, generator=g, device=DEV) if i != 1 else None for i in range(n)]
    gb = pipeline.GroupBuffers(T, K, (N,) * n, torch.float16, want_out_deq=True, device=DEV)
    for p in gb.per:
        p["out_deq"].fill_(7.0)
    pipeline.calibrate_group(X, W, b, gb)
    t = gb.t
    for i, p in enumerate(gb.per):
        out = torch.full_like(p["out_deq"], 9.0)
        B.aweq_w8a8_gemm(t["xq"], B.AWEQ_I8, T, K, K, None, t["act_step"], t["act_zero"], None, t["rowsum_x"], None, p["codes"], N, p["step_w"],
                         p["zero_w"], 0, p["rowsum_w"], b[i], None, out, B.AWEQ_F16, N, None, None, t["status"])
        assert torch.equal(out.view(torch.int16), p["out_deq"].view(torch.int16)), i
