"""Per-group weight quantizer on both sides of the sizes that decide how many rows and units of a group a thread takes, for groups of one
unit up to a whole wavefront of units, with a ragged last row: codes, Step and Z equal the oracle's, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("N,K", [(5, 512), (8191, 512), (8193, 512), (1023, 4096), (1025, 4096), (4097, 1536)])
def test_groups(orc, dtype, N, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    W = (np.random.default_rng(N + K).standard_normal((N, K)) * 0.02).astype(dtype)
    dW = torch.from_numpy(W).to(DEV)
    for bits, group in ((4, 8), (4, 32), (4, 64), (3, 128), (8, 128), (4, 512)):
        print(f"[gpu-weight-groups] {dtype.__name__} {N} x {K} W{bits} g={group}", flush=True)
        ref = orc.quant_weight(W, bits, group)
        codes = torch.zeros(N * K * bits // 8, dtype=torch.uint8, device=DEV)
        step, zero = torch.zeros(N * K // group, device=DEV), torch.zeros(N * K // group, dtype=torch.int32, device=DEV)
        B.aweq_quant_weight(dW, B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, N, K, K, bits, group, codes, step, zero, None)
        torch.cuda.synchronize()
        assert np.array_equal(step.cpu().numpy(), ref["step"].reshape(-1)) and np.array_equal(zero.cpu().numpy(), ref["zero"].reshape(-1))
        assert np.array_equal(codes.cpu().numpy(), orc.pack_codes(ref["codes_u"], bits).view(np.uint8).reshape(-1))
