"""The int8 GEMM where the choice of its tile turns on the rounds of workgroups: six and seven rounds of 256-token tiles, three and
four rounds of the 128 x 128 tiles for some hundred tokens, rows of up to 512 channels in several rounds and longer ones.  Codes of at most
64 in magnitude and K <= 1024: every sum is below 2^23, so that a binary32 product is exact."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("T,N,K", [(3072, 32768, 64), (3073, 32768, 64), (8200, 14720, 72), (6100, 2048, 640), (6581, 2432, 640),
                                   (8583, 1920, 512), (8583, 1920, 520), (2987, 2688, 160), (2987, 2688, 576)])
def test_rounds(T, N, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    B.load_library()
    print(f"[w8a8 rounds] T={T} {N} x {K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(T + N + K)
    x, w = (torch.randint(-64, 65, (n, K), generator=g, device=DEV, dtype=torch.int8) for n in (T, N))
    xq, wq = (torch.zeros(B.aweq_panel_bytes(n, K), dtype=torch.int8, device=DEV) for n in (T, N))
    B.aweq_pack_panels_i8(x, T, K, K, xq)
    B.aweq_pack_panels_i8(w, N, K, K, wq)
    out, colsum = torch.full((T, N), 7, dtype=torch.int32, device=DEV), torch.full((N,), 7, dtype=torch.int64, device=DEV)
    B.aweq_w8a8_gemm(xq, B.AWEQ_I8, T, K, K, None, None, None, None, None, None, wq, N, None, None, 0, None, None, out, None, B.AWEQ_F16, N, colsum)
    wf = w.float().t().contiguous()
    for t in range(0, T, 1024):
        assert torch.equal(out[t:t + 1024], (x[t:t + 1024].float() @ wf).to(torch.int32))
    assert torch.equal(colsum, out.sum(0, dtype=torch.int64))
