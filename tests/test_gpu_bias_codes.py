"""Bias correction from the weight codes: the sums sum_k wq[n,k] colsum_xq[k] by digits of base 256 and by 64-bit products, for
column sums over the whole range (digit carries, both signs, both sides of 2^30, both kinds in one wavefront), channels that do
not fill a block's rows, short and long rows, the longest rows the 32-bit digit sums are used for and the first beyond.  The
integers are exact, so delta and bias equal, bit for bit, those of the same call given the oracle's column sums of the
accumulator, and the oracle's delta within the rounding of its mean in another order."""
import numpy as np
import pytest

from conftest import to_panels

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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


EDGES = np.array([s * v + d for v in (0, 127, 128, 255, 256, 32767, 32768, 8388607, 8388608, (1 << 30) - 1) for s in (1, -1) for d in (0, 1, -1)
                  if abs(s * v + d) < 1 << 30], dtype=np.int64)
BEYOND = np.array([1 << 30, -(1 << 30), (1 << 30) + 12345, -(1 << 33) - 1, 1 << 38], dtype=np.int64)


def both_forms(B, Wh, mu, T, colsum, csa, rowsum, step_x, zero_x, codes, group, step_w, zero_w, b_in):
    N, K = Wh.shape
    dt = B.AWEQ_F16 if Wh.dtype == np.float16 else B.AWEQ_F32
    dW, dmu, dcol, drow, dsx, dzx = dev(Wh), dev(mu), dev(colsum), dev(rowsum), dev(np.float32([step_x])), dev(np.int32([zero_x]))
    dsw, dzw, db = dev(step_w), dev(zero_w), dev(b_in)
    res = []
    for ca, wq in ((None, dev(to_panels(codes))), (dev(csa), None)):
        delta, out = torch.zeros(N, device=DEV), torch.zeros(N, device=DEV)
        B.aweq_bias_correct(B.BIAS_W8A8, dW, dt, N, K, K, dmu, T, ca, dcol, drow, dsx, dzx, wq, 8, group, dsw, dzw, db, delta, out, 1)
        torch.cuda.synchronize()
        res.append((delta.cpu().numpy(), out.cpu().numpy()))
    return res


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("N,K,group", [(1, 8, 0), (5, 520, 0), (7, 1024, -1), (5, 1032, -1), (7, 2048, 0), (6, 11008, 0)])
def test_sums_from_the_codes(B, orc, dtype, N, K, group):
    rng = np.random.default_rng(N + K)
    T = 262144
    Wh = (rng.standard_normal((N, K)) * 0.02).astype(dtype)
    mu = rng.standard_normal(K).astype(np.float32)
    codes = rng.integers(-128, 128, (N, K), dtype=np.int8)
    codes[0, ::2] = -128
    ng = N if group == 0 else 1
    step_w, zero_w = rng.uniform(1e-3, 2e-2, ng).astype(np.float32), rng.integers(0, 256, ng).astype(np.int32)
    rowsum = codes.astype(np.int64).sum(1).astype(np.int32)
    b_in = rng.standard_normal(N).astype(np.float32)
    wide = rng.integers(-(1 << 29), 1 << 29, K)
    mixed = wide.copy()
    mixed[rng.random(K) < 0.02] = rng.choice(BEYOND)     # some lanes of a wavefront take the 64-bit products
    mixed[K - 1] = BEYOND[0]
    for name, colsum in (("wide", wide), ("edges", rng.choice(EDGES, K)), ("mixed", mixed), ("beyond", rng.choice(BEYOND, K))):
        print(f"[gpu-bias-codes] {np.dtype(dtype).name} N={N} K={K} g={group} {name}", flush=True)
        csa = orc.colsum_acc_from_colsum_xq(codes, colsum)
        a, b = both_forms(B, Wh, mu, T, colsum, csa, rowsum, 0.0371, 117, codes, group, step_w, zero_w, b_in)
        assert np.array_equal(a[0].view(np.int32), b[0].view(np.int32)) and np.array_equal(a[1].view(np.int32), b[1].view(np.int32))
        d_ref, b_ref = orc.bias_w8a8(Wh, mu, T, csa, colsum, rowsum, 0.0371, 117, step_w * np.ones(N, np.float32), zero_w * np.ones(N, np.int32), b_in)
        assert np.max(np.abs(a[0] - d_ref)) <= 1e-5 * np.max(np.abs(d_ref))
        np.testing.assert_allclose(a[1], b_ref, rtol=1e-5, atol=1e-5 * np.max(np.abs(d_ref)))


@pytest.mark.parametrize("K", [(1 << 24) - 1024, (1 << 24) - 1016, (1 << 24) - 8])
def test_longest_rows(B, orc, K):
    """Every code and every lowest digit -128: the largest growth of the 32-bit digit sums, 2^17 per 8 values."""
    print(f"[gpu-bias-codes] K={K}", flush=True)
    Wh, mu = np.zeros((1, K), np.float16), np.zeros(K, np.float32)
    codes, colsum = np.full((1, K), -128, np.int8), np.full(K, -128, np.int64)
    csa, rowsum = np.array([K * 128 * 128], np.int64), np.array([-128 * K], np.int32)
    step_w, zero_w = np.float32([0.01]), np.int32([128])
    a, b = both_forms(B, Wh, mu, 1, colsum, csa, rowsum, 0.01, 128, codes, 0, step_w, zero_w, np.zeros(1, np.float32))
    assert np.array_equal(a[0], b[0]) and a[0][0] == np.float32(-float(np.float32(0.01)) * float(step_w[0]) * float(csa[0]))


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("N,K", [(4099, 8200), (16390, 8192), (32774, 4104), (8200, 16384)])   # both sides of 256 MiB, short rows and long
def test_both_sources_of_the_sums_agree(B, dtype, N, K):
    """The launch shapes of large weights: delta from the codes and from the same integers given as colsum_acc is the same, bit for
    bit, and within the rounding of its mean in another order of the 64-bit one."""
    print(f"[gpu-bias-codes] large {dtype} N={N} K={K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(N + K)
    dt, T = (B.AWEQ_F16 if dtype == torch.float16 else B.AWEQ_F32), 4096
    Wh = (torch.randn(N, K, generator=g, device=DEV) * 0.02).to(dtype)
    mu, b_in = torch.randn(K, generator=g, device=DEV), torch.randn(N, generator=g, device=DEV)
    codes = torch.randint(-128, 128, (N, K), generator=g, device=DEV, dtype=torch.int8)
    col = torch.randint(-(1 << 19), 1 << 19, (K,), generator=g, device=DEV)
    panels = torch.empty(B.aweq_panel_bytes(N, K), dtype=torch.int8, device=DEV)
    B.aweq_pack_panels_i8(codes, N, K, K, panels)
    # (exact: every partial sum is an integer below 2^53)
    csa = torch.cat([(c.double() * col.double()).sum(1) for c in codes.split(1024)]).long()
    rowsum = codes.sum(1, dtype=torch.int32)
    sx, zx = torch.tensor([0.0371], device=DEV), torch.tensor([117], dtype=torch.int32, device=DEV)
    sw = torch.rand(N, generator=g, device=DEV) * 0.02 + 1e-3
    zw = torch.randint(0, 256, (N,), generator=g, device=DEV, dtype=torch.int32)
    res = []
    for ca, wq in ((None, panels), (csa, None)):
        delta, out = torch.zeros(N, device=DEV), torch.zeros(N, device=DEV)
        B.aweq_bias_correct(B.BIAS_W8A8, Wh, dt, N, K, K, mu, T, ca, col, rowsum, sx, zx, wq, 8, 0, sw, zw, b_in, delta, out, 1)
        res.append((delta, out))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    mean = torch.cat([(w.double() * mu.double()).sum(1) for w in Wh.split(1024)])
    a = csa - T * (117 - 128) * rowsum.long() - (zw.long() - 128) * col.sum() + T * K * (117 - 128) * (zw.long() - 128)
    ref = mean - sx.double() * sw.double() * a.double() / T
    assert torch.max(torch.abs(res[0][0].double() - ref)) <= 1e-6 * torch.max(torch.abs(ref))
