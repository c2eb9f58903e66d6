"""K-vector work at the edges of its launches: the statistics' finishing kernel (blocks of 256 channels, block extremes
every 32 channels) and the equalization scales (one block up to 4096 channels, a block per 1024 and a range launch
beyond), against the oracle."""
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


@pytest.mark.parametrize("K", [8, 40, 256, 4088, 4096, 4104, 8200, 12296, 49160])
def test_ranges_and_scales(B, orc, K):
    print(f"[channel vectors] K={K}", flush=True)
    rng = np.random.default_rng(K)
    T, N = 33, 5
    X = (rng.standard_normal((T, K)) * np.exp(rng.standard_normal(K))).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    X[:, K // 2] = 0.25        # a constant channel: guarded scale
    X[3, K - 1] = 900.0        # the tensor's extremes in the last and the first channel
    X[7, 0] = -1000.0
    e = lambda *s, dtype=torch.float32: torch.empty(s, dtype=dtype, device=DEV)
    d = lambda a: torch.from_numpy(a).to(DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)

    def stats(M, rows, want_sum):
        o = dict(cmin=e(K), cmax=e(K), csum=e(K, dtype=torch.float64) if want_sum else None, count=e(1, dtype=torch.int64),
                 r=e(K), R=e(1), p=e(K))
        ws = torch.full((B.aweq_workspace_size(B.OP_CALIB_STATS, rows, K),), 0x5A, dtype=torch.uint8, device=DEV)
        half = rows // 2
        for r0, r1, acc in ((0, half, 0), (half, rows, 1)):   # merged in two batches, finished with the second
            B.aweq_calib_stats(M[r0:], B.AWEQ_F16, r1 - r0, K, K, o["cmin"], o["cmax"], o["csum"], o["count"], acc, acc, o["r"],
                               o["R"], o["p"], ws, st)
        return o

    gx, gw = stats(d(X), T, True), stats(d(W), N, False)
    for M, g in ((X, gx), (W, gw)):
        ref = orc.col_stats(M, want_sum=False)
        r, R, p = orc.ranges(ref["cmin"], ref["cmax"])
        assert np.array_equal(g["r"].cpu().numpy(), r) and g["R"].item() == R
        assert np.array_equal(g["p"].cpu().numpy(), p)
    s, inv_s, mu, rngx, step, zero = e(K), e(K), e(K), e(2), e(1), e(1, dtype=torch.int32)
    B.aweq_equalize(gx["cmin"], gx["cmax"], gx["csum"], T, gw["cmin"], gw["cmax"], K, 1, s, inv_s, None, None, B.AWEQ_F16, 0, K, K,
                    None, rngx, mu, step, zero, st)
    sx, sw = orc.col_stats(X), orc.col_stats(W, want_sum=False)
    r_x, _, _ = orc.ranges(sx["cmin"], sx["cmax"])
    r_w, _, _ = orc.ranges(sw["cmin"], sw["cmax"])
    s_ref, inv_ref, _ = orc.scales(r_x, r_w)
    np.testing.assert_allclose(s.cpu().numpy(), s_ref, rtol=1e-6)     # fp64 square root and quotient, rounded once
    inv = inv_s.cpu().numpy()
    assert np.array_equal(inv, np.float32(1.0) / s.cpu().numpy())
    lo, hi = (sx["cmin"] * inv).min(), (sx["cmax"] * inv).max()       # binary32 products, as in the kernel
    assert rngx.cpu().numpy().tolist() == [lo, hi]
    assert step.item() == np.float32(hi - lo) / np.float32(255) and zero.item() == -int(np.rint(lo / np.float32(step.item())))
    # 33 binary16 values summed in binary32 runs of 8: 7 2^-24 of the mean magnitude
    bound = 1e-6 * np.abs(X.astype(np.float64)).mean(axis=0) * inv + 1e-30
    assert np.all(np.abs(mu.cpu().numpy() - X.astype(np.float64).mean(axis=0) * inv) <= bound)
    assert st.item() & B.ST_SCALEGUARD


@pytest.mark.parametrize("K", [5120, 7168, 7176])
def test_both_sides_of_one_block_with_a_range(B, orc, K):
    """With the range asked for, one block serves up to 7168 channels; without it, several from 4104 on: the same scales."""
    test_ranges_and_scales(B, orc, K)
    g = torch.Generator(device=DEV).manual_seed(K)
    lo, hi = -torch.rand(2, K, generator=g, device=DEV) - 0.1, torch.rand(2, K, generator=g, device=DEV)
    xsum = torch.randn(K, generator=g, device=DEV, dtype=torch.float64)
    outs = []
    for want in (True, False):
        s, inv_s, mu = (torch.zeros(K, device=DEV) for _ in range(3))
        rng, step, zero = torch.zeros(2, device=DEV), torch.zeros(1, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
        B.aweq_equalize(lo[0], hi[0], xsum, 100, lo[1], hi[1], K, 1, s, inv_s, None, None, B.AWEQ_F16, 0, K, K, None, rng if want else None, mu,
                        step if want else None, zero if want else None)
        outs.append((s, inv_s, mu))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("K,ld,offset", [(192, 192, 0), (200, 200, 0), (192, 200, 0), (192, 256, 8), (2048, 2048, 0), (2056, 2112, 0)])
def test_folded_rows_of_whole_lines_and_others(B, K, ld, offset):
    """The binary16 fold reads rows of whole 128-byte lines non-temporally and others through the caches: RN16(RN32(w s)) either way."""
    N = 37
    g = torch.Generator(device=DEV).manual_seed(K + ld)
    W = torch.randn(N * ld + offset, generator=g, device=DEV).half()[offset:].view(N, ld)
    lo, hi = -torch.rand(2, K, generator=g, device=DEV) - 0.1, torch.rand(2, K, generator=g, device=DEV)
    s, inv_s, out = torch.zeros(K, device=DEV), torch.zeros(K, device=DEV), torch.full((N, K), 9.0, dtype=torch.float16, device=DEV)
    B.aweq_equalize(lo[0], hi[0], None, 0, lo[1], hi[1], K, 1, s, inv_s, W, out, B.AWEQ_F16, N, ld, K, None, None, None, None, None)
    assert torch.equal(out, (W[:, :K].float() * s).half())
