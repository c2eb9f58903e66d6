"""The tiled int8 GEMM where its plan changes: tiles of 64, 128 and 256 tokens, one round of workgroups and several, the
sequence walk and the patches, and numbers of K-panels around the depth of the load ring.  The int32 accumulator and its
column sums are exact against the oracle; the binary16 / binary32 output is the fp64 value of the exact integer, rounded
once (binary32) or within one unit in the last place (binary16: one fused fp64 operation)."""
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


@pytest.mark.parametrize("T,N,Ks", [
    (1153, 4352, (8, 64, 192, 256, 264, 320, 504, 512, 584)),  # 128 tokens a tile, one round; 1 .. 10 panels
    (1280, 4108, (200, 1000)),                                 # whole tiles of tokens, a ragged last column
    (2300, 4100, (40, 192, 256, 328, 456)),                    # 256 tokens a tile, one round
    (2100, 11008, (136, 584)),                                 # 128 tokens a tile, three rounds
    (6100, 4100, (136, 520)),                                  # 256 tokens a tile, two rounds
    (385, 4100, (8, 64, 200, 320, 512, 776, 1096)),            # 64 x 128 tiles; 1 .. 5 stages of four panels, three in the ring
    (512, 4096, (256,)),                                       # whole 64 x 128 tiles
    (900, 4060, (8, 128, 200, 320, 456, 584)),                 # 128 x 128 tiles; 1 .. 5 stages of two panels, four in the ring
    (65, 22020, (136, 328)),                                   # few tokens, 64 x 128 tiles
])
def test_tiled_gemm(B, orc, T, N, Ks):
    rng = np.random.default_rng(T + N)
    step_w = rng.uniform(1e-3, 2e-2, N).astype(np.float32)
    zero_w = rng.integers(0, 256, N).astype(np.int32)
    bias = rng.standard_normal(N).astype(np.float32)
    step_x, zero_x = np.float32(0.02), 131
    for i, K in enumerate(Ks):
        print(f"[gpu-gemm-tiles] T={T} N={N} K={K}", flush=True)
        xq, wq = rng.integers(-128, 128, (T, K), dtype=np.int8), rng.integers(-128, 128, (N, K), dtype=np.int8)
        rx, rw = xq.sum(1, dtype=np.int32), wq.sum(1, dtype=np.int32)
        acc = orc.gemm_i8(xq, wq)
        zx, zw = zero_x - 128, zero_w.astype(np.int64) - 128
        iv = acc.astype(np.int64) - zx * rw.astype(np.int64) - zw * rx.astype(np.int64)[:, None] + K * zx * zw
        ref = iv.astype(np.float64) * (np.float64(step_x) * step_w.astype(np.float64)) + bias.astype(np.float64)
        dx, dw = dev(to_panels(xq)), dev(to_panels(wq))
        for odt, want_i32, want_cs in ((torch.float16, False, False), (torch.float16, i % 2 == 0, True), (torch.float32, i % 2 == 1, True),
                                       (None, True, True)):
            oi = torch.full((T, N + 4), 7, dtype=torch.int32, device=DEV) if want_i32 else None
            od = torch.full((T, N + 4), 7.0, dtype=odt, device=DEV) if odt else None
            cs = torch.full((N,), 7, dtype=torch.int64, device=DEV) if want_cs else None
            st = torch.zeros(1, dtype=torch.int32, device=DEV)
            B.aweq_w8a8_gemm(dx, B.AWEQ_I8, T, K, K, None, dev(np.float32([step_x])), dev(np.int32([zero_x])), None, dev(rx), None, dw, N,
                             dev(step_w), dev(zero_w), 0, dev(rw), dev(bias), oi, od, B.AWEQ_F16 if odt == torch.float16 else B.AWEQ_F32,
                             N + 4, cs, None, st)
            torch.cuda.synchronize()
            if want_i32:
                g = oi.cpu().numpy()
                assert np.array_equal(g[:, :N], acc) and np.all(g[:, N:] == 7)
            if want_cs:
                assert np.array_equal(cs.cpu().numpy(), acc.sum(0, dtype=np.int64))
            if odt:
                got = od.cpu().numpy()
                assert np.all(got[:, N:] == 7.0)
                r32 = ref.astype(np.float32)
                if odt == torch.float32:
                    assert np.array_equal(got[:, :N], r32)
                else:
                    r16 = r32.astype(np.float16)
                    assert np.all(np.abs(got[:, :N].astype(np.float32) - r16.astype(np.float32)) <= np.spacing(np.abs(r16)).astype(np.float32))
            assert int(st.item()) == 0
