"""A calibration in one call against the stage entry points one after the other (the same call with a workspace of the stages' own
size, which takes them one by one): every output to the bit, except sums in binary64, which are added in another order, and what is
rounded from them."""
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


F16, F32 = torch.float16, torch.float32
CASES = [   # dtype, tokens, channels of each weight, K, bits, group, int8 path, with the GEMM, bias over the corrected bias
    (F16, 1, (1,), 8, 8, 0, True, True, False), (F16, 33, (5,), 72, 8, 0, True, True, False), (F16, 700, (130, 3), 1032, 8, 0, True, True, False),
    (F16, 257, (9,), 1024, 8, 0, True, False, False), (F16, 257, (9,), 4096, 8, 0, True, True, False), (F16, 90, (9, 5, 4, 1), 4104, 8, 0, True, True, False),
    (F16, 300, (6,), 8200, 8, 0, True, False, False), (F16, 64, (7,), 12296, 8, 0, True, True, False), (F16, 40, (5,), 24576, 8, 0, True, False, False),
    (F16, 40, (3, 4, 5, 6, 7), 520, 8, 0, True, True, False),      # more weights than one launch takes: the stages
    (F16, 40, (12,), 520, 8, 0, True, True, True),                 # overlapping buffers: the stages
    (F32, 31, (3,), 520, 8, 0, True, True, False), (F32, 65, (5, 4, 3, 2), 4104, 8, 0, True, True, False), (F32, 33, (3,), 8200, 8, 0, True, False, False),
    (F32, 33, (3,), 12288, 8, 0, True, False, False), (F32, 3000, (65,), 24, 8, 0, True, True, False),
    (F16, 100, (5,), 520, 8, -1, True, True, False), (F16, 100, (5,), 520, 8, -1, True, False, False),   # one scale for the weight
    (F16, 70, (5,), 520, 8, 0, False, False, False),                                                     # 8-bit weight-only: no fused pass
    (F16, 65, (5,), 96, 4, 32, False, False, False), (F16, 65, (6,), 1088, 4, 64, False, False, False), (F16, 65, (7,), 1152, 4, 128, False, False, False),
    (F16, 65, (8,), 2560, 4, 512, False, False, False), (F16, 65, (9,), 2304, 3, 256, False, False, False), (F16, 65, (1,), 256, 3, 32, False, False, False),
    (F32, 65, (5,), 1152, 4, 128, False, False, False), (F32, 65, (5,), 4224, 3, 64, False, False, False), (F16, 65, (5,), 96, 4, 8, False, False, False),
]


def _calibrate(B, X, Ws, biases, K, bits, group, w8a8, forward, alias, small):
    T, dt = X.shape[0], X.dtype
    Ns = [W.shape[0] for W in Ws]
    e = lambda *s, dtype=F32: torch.full(s, 7, dtype=dtype, device=DEV)
    i32, i64 = torch.int32, torch.int64
    v = {n: e(K) for n in ("xmin", "xmax", "r_x", "p_x", "wmin", "wmax", "r_w", "p_w", "s", "inv_s", "mu_xhat")}
    v.update(xsum=e(K, dtype=torch.float64), count=e(1, dtype=i64), wcount=e(1, dtype=i64), R_x=e(1), R_w=e(1), xhat_range=e(2), act_step=e(1),
             act_zero=e(1, dtype=i32), status=torch.zeros(1, dtype=i32, device=DEV), colsum_xq=e(K, dtype=i64),
             xq=e(B.aweq_panel_bytes(T, K), dtype=torch.int8), rowsum_x=e(T, dtype=i32))
    if not w8a8:
        del v["colsum_xq"]
    if not forward:
        del v["xq"], v["rowsum_x"]
    size = max([B.aweq_workspace_size(B.OP_CALIB_STATS, r, K, 0) for r in [T] + Ns] + [B.aweq_workspace_size(B.OP_W8A8_GEMM, T, K, max(Ns)), 16])
    full = B.aweq_workspace_size(B.OP_CALIBRATE, T, K, sum(Ns))
    ws = torch.empty(size if small else max(size, full), dtype=torch.uint8, device=DEV)
    ws_bytes = min(size, full - 1) if small else ws.numel()
    members = []
    for W, b in zip(Ws, biases):
        N = W.shape[0]
        ng = N * (K // group) if group > 0 else N if group == 0 else 1
        codes = torch.zeros(B.aweq_panel_bytes(N, K) if bits == 8 and group <= 0 else N * K // 8 * bits, dtype=torch.int8, device=DEV)
        m = {"W_hat": e(N, K, dtype=dt), "codes": codes, "step_w": e(ng), "zero_w": e(ng, dtype=i32), "rowsum_w": e(N, dtype=i32), "delta": e(N),
             "bias_out": b.clone() if alias else e(N), "out_i32": e(T, N, dtype=i32), "out_deq": e(T, N, dtype=dt), "colsum_acc": e(N, dtype=i64)}
        if not forward:
            del m["out_i32"], m["out_deq"], m["colsum_acc"]
        members.append((W, b, m))
    g = v.get
    B.aweq_calibrate((X, B.AWEQ_F16 if dt == F16 else B.AWEQ_F32, T, K, X.stride(0), v["xmin"], v["xmax"], v["xsum"], v["count"], v["r_x"], v["R_x"],
                      v["p_x"], v["wmin"], v["wmax"], v["wcount"], v["r_w"], v["R_w"], v["p_w"], v["s"], v["inv_s"], v["xhat_range"], v["mu_xhat"],
                      v["act_step"], v["act_zero"], g("xq"), g("rowsum_x"), g("colsum_xq"), 1, 1, bits, group, int(w8a8), int(forward), 0, ws, ws_bytes,
                      v["status"]),
                     [(W, W.shape[0], W.stride(0), m["W_hat"], K, m["codes"], m["step_w"], m["zero_w"], m["rowsum_w"] if bits == 8 and group <= 0 else None,
                       m["bias_out"] if alias else b, m["delta"], m["bias_out"], m.get("out_i32"), m.get("out_deq"), m.get("colsum_acc"))
                      for W, b, m in members])
    torch.cuda.synchronize()
    return {k: t.cpu().numpy() for k, t in v.items()}, [{k: t.cpu().numpy() for k, t in m.items()} for _, _, m in members]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x).replace("torch.", "") for x in c))
def test_one_call_gives_what_the_stages_give(B, case):
    dt, T, Ns, K, bits, group, w8a8, forward, alias = case
    print(f"[calibrate] {case}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K + T)
    r = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    X = (r(T, K) * 2 + 0.1).to(dt)
    X[:, K // 2] *= 40
    Ws = [(r(N, K + 8) * 0.05).to(dt)[:, :K] for N in Ns] if K % 16 else [(r(N, K) * 0.05).to(dt) for N in Ns]   # pitched, or whole rows
    biases = [r(N) for N in Ns]
    one, stages = (_calibrate(B, X, Ws, biases, K, bits, group, w8a8, forward, alias, small) for small in (False, True))
    loose = {"xsum", "mu_xhat", "delta", "bias_out"}
    for a, b in [(one[0], stages[0])] + list(zip(one[1], stages[1])):
        for k in a:
            if k not in loose:
                assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k
    # binary64 sums of T terms in two orders; mu: one rounding of them to binary32
    size = X.double().abs().sum(0).cpu().numpy()
    assert np.all(np.abs(one[0]["xsum"] - stages[0]["xsum"]) <= T * 2.0**-52 * size)
    mu = stages[0]["mu_xhat"].astype(np.float64)
    assert np.all(np.abs(one[0]["mu_xhat"] - mu) <= 2.0**-23 * np.abs(mu) + T * 2.0**-52 * size / T * stages[0]["inv_s"])
    # delta: a rounding of mu in any column, and its own
    for a, b in zip(one[1], stages[1]):
        bound = 2.0**-22 * (np.abs(b["W_hat"].astype(np.float64)) @ np.abs(mu)) + 2.0**-22 * np.abs(b["delta"])
        if not w8a8:   # (the rounding error of the weight takes the place of the weight)
            bound = 2.0**-22 * (np.abs(b["W_hat"].astype(np.float64)).max(1) * np.abs(mu).sum()) + 2.0**-22 * np.abs(b["delta"])
        assert np.all(np.abs(a["delta"].astype(np.float64) - b["delta"]) <= bound)
        assert np.all(np.abs(a["bias_out"].astype(np.float64) - b["bias_out"]) <= bound + 2.0**-23 * np.abs(b["bias_out"]))
