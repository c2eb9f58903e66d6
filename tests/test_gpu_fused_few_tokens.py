"""aweq_w8a8_gemm_fused without statistics for up to some hundred tokens (64 x 128 and 128 x 128 tiles) and just beyond
(128 x 256 tiles): codes, row and column sums and the stored output equal the oracle's activation quantizer over the
output of the separate path, bit for bit."""
import numpy as np
import pytest

from conftest import from_panels
from test_gpu_fused import B, Dev, fused, host, make_case, next_layer_params, unfused   # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,N", [
    (1, 64, 4), (17, 200, 132), (64, 264, 1024), (65, 1096, 4100), (200, 520, 260),   # 64 x 128
    (900, 328, 4060), (1000, 72, 3908),                                               # 128 x 128
    (1153, 136, 4352), (2300, 200, 4100),                                             # the tiled kernel: 128, 256 tokens
])
@pytest.mark.parametrize("act,store", [(0, True), (1, False)])
def test_quantising_epilogue(B, orc, T, K, N, act, store):   # noqa: F811
    print(f"[gpu-fused-few] T={T} K={K} N={N} act={act} store={store}", flush=True)
    c = make_case(orc, T + K + N, T, K, N, with_bias=act == 1)
    d = Dev(B, c)
    y, cs = unfused(B, c, d)
    if act == 1:
        y = np.maximum(y, np.float16(0))
    nxt = next_layer_params(orc, c["rng"], y)
    if K == 520:
        nxt["zero"] = 5000      # outside the screened quotient
    f = fused(B, c, d, act=act, store=store, stats=False, nxt=nxt)
    a = orc.quant_act(y, nxt["inv_s"], nxt["step"], nxt["zero"])
    assert np.array_equal(from_panels(host(f["yq"]), T, N), a["xq"])
    assert np.array_equal(host(f["rowsum_y"]), a["rowsum_x"]) and np.array_equal(host(f["colsum_yq"]), a["colsum_xq"])
    assert np.array_equal(host(f["colsum_acc"]), cs)
    if store:
        assert np.array_equal(host(f["y"]).astype(np.float32), y.astype(np.float32))
    assert int(host(f["status"])[0]) == a["status"]
