"""Weight-only bias correction: two and four channels a block (binary16 from 8192 channels on), a last block that is not full, every
code width's loads, K that ends inside a quad of threads and rows of more than one pass, against the oracle.  Tolerance: delta is a
sum in binary64 rounded once to binary32; 1e-6 of its largest value leaves room for the order of a sum that cancels."""
import numpy as np
import pytest

from conftest import to_panels

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bits,group", [(8, 0), (8, 32), (4, -1), (4, 32), (3, 0), (3, 32)])
@pytest.mark.parametrize("dtype,N,K", [(np.float16, 1, 1056), (np.float16, 7, 4128), (np.float16, 8191, 1056), (np.float16, 8193, 1056), (np.float16, 8198, 2080),
                                       (np.float32, 7, 4128), (np.float32, 8193, 1056)])
def test_bias_weight_only(orc, dtype, N, K, bits, group):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding as B
    print(f"[gpu-bias-wonly] {np.dtype(dtype).name} N={N} K={K} W{bits} g={group}", flush=True)
    rng = np.random.default_rng(N + K + bits)
    Wh = (rng.standard_normal((N, K)) * 0.02).astype(dtype)
    mu, b_in = rng.standard_normal(K).astype(np.float32), rng.standard_normal(N).astype(np.float32)
    q = orc.quant_weight(Wh, bits, group)
    packed = orc.pack_codes(q["codes_u"], bits).view(np.uint8).reshape(-1)
    if bits == 8 and group <= 0:
        packed = to_panels(packed.view(np.int8).reshape(N, K))
    d_ref, b_ref = orc.bias_wonly(Wh, mu, q["codes_u"], group, q["step"], q["zero"], b_in)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    delta, out = torch.zeros(N, device=DEV), torch.zeros(N, device=DEV)
    B.aweq_bias_correct(B.BIAS_WEIGHT_ONLY, dev(Wh), B.AWEQ_F16 if dtype == np.float16 else B.AWEQ_F32, N, K, K, dev(mu), 96, None, None, None, None, None,
                        dev(packed), bits, group, dev(q["step"].reshape(-1)), dev(q["zero"].reshape(-1)), dev(b_in), delta, out, 1)
    scale = np.max(np.abs(d_ref))
    assert np.max(np.abs(delta.cpu().numpy() - d_ref)) <= 1e-6 * scale
    assert np.max(np.abs(out.cpu().numpy() - b_ref)) <= 1e-6 * max(scale, np.max(np.abs(b_ref)))


@pytest.mark.parametrize("bits,group", [(8, 0), (8, 64), (4, -1), (4, 64), (3, 0), (3, 64)])
@pytest.mark.parametrize("dtype,N,K", [(np.float16, 1, 8256), (np.float32, 3, 8192), (np.float32, 3, 8256), (np.float32, 5, 22016), (np.float16, 1281, 8256), (np.float16, 513, 8256)])
def test_few_channels_of_long_rows(orc, dtype, N, K, bits, group):
    """512 threads on one channel (more than 8192 values, few channels), and both sides of the limits of K and N."""
    test_bias_weight_only(orc, dtype, N, K, bits, group)
