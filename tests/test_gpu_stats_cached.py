"""Column statistics on both sides of the size up to which the matrix is read through the caches (96 MiB), with integer
entries, whose sums are exact in every order."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,rows", [(torch.float16, 49152), (torch.float16, 49153), (torch.float32, 24576), (torch.float32, 24577)])
def test_around_the_limit(dtype, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    B.load_library()
    K = 1024
    print(f"[stats] {dtype} {rows} x {K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(rows)
    M = torch.randint(-60, 61, (rows, K), generator=g, device=DEV, dtype=torch.int32).to(dtype)
    M[rows - 1, K - 1], M[rows - 1, 0] = 1000.0, -1000.0
    e = lambda *s, dtype=torch.float32: torch.empty(s, dtype=dtype, device=DEV)
    cmin, cmax, csum, count, r, R, p = e(K), e(K), e(K, dtype=torch.float64), e(1, dtype=torch.int64), e(K), e(1), e(K)
    ws = torch.full((B.aweq_workspace_size(B.OP_CALIB_STATS, rows, K),), 0x5A, dtype=torch.uint8, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    B.aweq_calib_stats(M, B.AWEQ_F16 if dtype == torch.float16 else B.AWEQ_F32, rows, K, K, cmin, cmax, csum, count, 0, 1, r, R, p, ws, st)
    assert torch.equal(cmin, M.amin(0).float()) and torch.equal(cmax, M.amax(0).float())
    assert torch.equal(csum, M.to(torch.int32).sum(0).double())
    assert count.item() == rows and R.item() == 2000.0
