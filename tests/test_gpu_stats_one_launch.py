"""Column statistics whose R and p come from the merge kernel's last block (up to 1024 channels) and from a launch of their own
(beyond), one row to many row slices, both entry points, several calls on the same scratch memory: bit for bit torch's."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("K", [8, 32, 40, 512, 1016, 1024, 1032])
@pytest.mark.parametrize("rows", [1, 65, 3001])
def test_around_one_launch(dtype, K, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    B.load_library()
    print(f"[stats one launch] {dtype} {rows} x {K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(rows + K)
    dt = B.AWEQ_F16 if dtype == torch.float16 else B.AWEQ_F32
    ws = torch.full((B.aweq_workspace_size(B.OP_CALIB_STATS, rows, K),), 0x5A, dtype=torch.uint8, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    for i in range(4):
        M = torch.randn(rows, K, generator=g, device=DEV).to(dtype)
        M[rows - 1, K - 1 if i & 1 else 0] = 50.0 * (i - 1)   # an extreme in the last or the first column
        o = [torch.full((n,), 7.0, dtype=t, device=DEV) for n, t in ((K, torch.float32), (K, torch.float32), (K, torch.float64))]
        count = torch.zeros(1, dtype=torch.int64, device=DEV)
        r, R, p = (torch.full((n,), 7.0, device=DEV) for n in (K, 1, K))
        p_out = p if i else None
        if i < 3:
            B.aweq_calib_stats(M, dt, rows, K, K, *o, count, 0, 1, r, R, p_out, ws, st)
        else:
            B.aweq_calib_stats_static(M, dt, rows, K, K, *o, count, 0, 1, r, R, p_out, st)
        lo, hi = M.amin(0).float(), M.amax(0).float()
        assert torch.equal(o[0], lo) and torch.equal(o[1], hi) and torch.equal(r, hi - lo)
        assert torch.equal(R, (hi.amax() - lo.amin()).reshape(1))
        if i:
            assert torch.equal(p, r / R)
        assert count.item() == rows
