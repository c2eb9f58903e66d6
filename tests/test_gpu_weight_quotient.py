"""The weight quantizer's division-free quotient against the oracle's true division, exactly: slices whose elements sit
within a few units in the last place of rounding ties, with zero points inside and outside the screened range, Steps that
force the division (huge, tiny, an all-ones significand), subnormal elements, ranges that overflow, and slices beside one
with infinities or NaN (whose own codes are unspecified)."""
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


def tie_slices(rng, dtype, S, n, bits):
    """[S, n]: slice i has extremes of its own, and elements next to the ties of the Step they give."""
    levels = (1 << bits) - 1
    out = np.empty((S, n), dtype)
    with np.errstate(over="ignore", invalid="ignore"):
        for i in range(S):
            if dtype == np.float16:
                step = 2.0 ** rng.uniform(-14, -2)
                z = float(rng.choice([0, levels // 2, levels, -40, 300, 1500]))
            else:
                step = 2.0 ** rng.choice([rng.uniform(-30, 30), -59.5, -61.0, -75.0, 59.5, 63.0, 119.0, -140.0])
                z = float(rng.choice([0, levels // 2, -3900, 3900, 4200, -9000, 1 << 21, 1 << 24]))
            if i % 7 == 3:
                step = np.nextafter(np.float32(2.0 ** np.round(np.log2(step))), np.float32(0))   # significand all ones
            lo, hi = dtype(-z * step), dtype((levels - z) * step)
            st = (np.float32(hi) - np.float32(lo)) / np.float32(levels)
            st = float(st) if np.isfinite(st) and st > 0 else 1.0
            zi = -np.rint(np.float32(lo) / np.float32(st))
            c = rng.integers(0, levels + 1, n)
            x = ((c - zi + 0.5) * st).astype(dtype)
            for _ in range(3):   # up to three steps of the type away from the tie
                x = np.where(rng.random(n) < 0.5, np.nextafter(x, dtype(rng.choice([-np.inf, np.inf]))), x)
            x = np.clip(x, min(lo, hi), max(lo, hi))
            x[rng.integers(0, n)] = lo
            x[(int(np.argmin(x)) + 1) % n] = hi
            out[i] = x
    return np.where(np.isfinite(out), out, dtype(1.0))


@pytest.mark.parametrize("bits", [8, 4, 3])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_near_ties(B, orc, dtype, bits):
    rng = np.random.default_rng(bits + (50 if dtype == np.float32 else 0))
    dt = B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32
    for group, N, K in ((0, 160, 2080), (0, 96, 96), (128, 40, 2176), (32, 24, 288), (-1, 40, 544)):
        print(f"[gpu-weight-quotient] {dtype.__name__} b={bits} g={group} N={N} K={K}", flush=True)
        if group > 0:
            W = tie_slices(rng, dtype, N * (K // group), group, bits).reshape(N, K)
        elif group == 0:
            W = tie_slices(rng, dtype, N, K, bits)
        else:
            W = tie_slices(rng, dtype, 1, N * K, bits).reshape(N, K)
        for poison in (False, True):
            if poison:
                if group < 0:
                    continue
                W = W.copy()
                W[5, 3], W[5, 40], W[11, 17] = np.nan, np.inf, -np.inf
            W = np.ascontiguousarray(W)
            ng = 1 if group < 0 else (N if group == 0 else N * (K // group))
            panel = bits == 8 and group <= 0
            codes = torch.full((B.aweq_panel_bytes(N, K) if panel else N * K * bits // 8,), 0x5a, dtype=torch.uint8, device=DEV)
            step, zero = torch.empty(ng, device=DEV), torch.empty(ng, dtype=torch.int32, device=DEV)
            rowsum = torch.empty(N, dtype=torch.int32, device=DEV) if panel else None
            ws, status = torch.empty(64, dtype=torch.uint8, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
            B.aweq_quant_weight(torch.from_numpy(W).to(DEV), dt, N, K, K, bits, group, codes, step, zero, rowsum, ws, status)
            torch.cuda.synchronize()
            o = orc.quant_weight(W, bits, group)
            keep = np.ones((N, K), bool)
            if poison:
                keep[[5, 11]] = False     # (a row is one slice or more of them)
            ks = keep[:, 0] if group <= 0 else np.repeat(keep[:, 0], K // group)
            if group < 0:
                ks = np.ones(1, bool)
            assert np.array_equal(step.cpu().numpy()[ks], o["step"].reshape(-1)[ks])
            assert np.array_equal(zero.cpu().numpy()[ks], o["zero"].reshape(-1)[ks])
            got = codes.cpu().numpy()
            want = np.asarray(orc.pack_codes(o["codes_u"], bits)).view(np.uint8).reshape(N, -1)
            if panel:
                kp = -(-K // 64)
                got = got.reshape(kp, N, 64).transpose(1, 0, 2).reshape(N, kp * 64)
                assert not got[:, K:].any()
                got = got[:, :K]
                assert np.array_equal(rowsum.cpu().numpy()[keep[:, 0]], o["rowsum_w"][keep[:, 0]])
            got = got.reshape(N, -1)
            assert np.array_equal(got[keep[:, 0]], want[keep[:, 0]])
            if not poison:
                assert int(status.item()) == o["status"]
