"""Int8 GEMM of a narrow layer on millions of tokens: more 64-token tiles than a grid's y dimension holds (65535), on both sides of
that limit.  Accumulator and column sums equal the product formed in binary32, which holds these integers (below 2^24) exactly."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T", [65535 * 64, 65535 * 64 + 1, 65535 * 64 + 130])
@pytest.mark.parametrize("N", [16, 64])
def test_more_token_tiles_than_a_grid_dimension(T, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    print(f"[gpu-w8a8-narrow] T={T} N={N}", flush=True)
    K = 8
    g = torch.Generator(device=DEV).manual_seed(T + N)
    codes = lambda rows: torch.nn.functional.pad(torch.randint(-128, 128, (rows, K), generator=g, dtype=torch.int8, device=DEV), (0, 64 - K))
    xq, wq = codes(T), codes(N)       # K <= 64: the panel layout is one panel
    out = torch.full((T, N), 1 << 30, dtype=torch.int32, device=DEV)
    cs = torch.zeros(N, dtype=torch.int64, device=DEV)
    B.aweq_w8a8_gemm(xq, B.AWEQ_I8, T, K, K, None, None, None, None, None, None, wq, N, None, None, 0, None, None, out, None, B.AWEQ_F16, N, cs)
    want = (xq[:, :K].float() @ wq[:, :K].float().T).int()
    assert torch.equal(out, want)
    assert torch.equal(cs, want.sum(0, dtype=torch.int64))
