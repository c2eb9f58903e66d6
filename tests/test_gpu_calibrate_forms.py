"""A calibration in one call against the stage entry points called one after the other, on both of its routes (with the workspace of the
fused passes, and with the stages' own): every option that changes what a launch does.  Outputs are compared to the bit, except sums in
binary64, which are added in another order, and what is rounded from them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
F16, F32, I32, I64 = torch.float16, torch.float32, torch.int32, torch.int64
GUARD = 7


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_01305_amd import binding
    binding.load_library()
    return binding


def _e(*shape, dtype=F32):
    return torch.full(shape, GUARD, dtype=dtype, device=DEV)


def _copy(W):
    out = W.new_empty(W.shape[0], W.stride(0))[:, :W.shape[1]]   # with its pitch
    return out.copy_(W)


class Call:
    """Buffers of one call.  codes, Step and Z are longer than the call needs them: what lies behind has to stay."""

    def __init__(self, B, X, Ws, biases, bits, group, w8a8, forward, awe=1, bc=1, in_place=False, nulls=()):
        self.__dict__.update(B=B, X=X, biases=biases, bits=bits, group=group, w8a8=w8a8, forward=forward, awe=awe, bc=bc, nulls=nulls)
        T, K = X.shape
        self.T, self.K, self.dt = T, K, B.AWEQ_F16 if X.dtype == F16 else B.AWEQ_F32
        self.Ws = [_copy(W) if in_place else W for W in Ws]
        v = {n: _e(K) for n in ("xmin", "xmax", "r_x", "p_x", "wmin", "wmax", "r_w", "p_w", "s", "inv_s", "mu_xhat")}
        v.update(xsum=_e(K, dtype=torch.float64), count=_e(1, dtype=I64), wcount=_e(1, dtype=I64), R_x=_e(1), R_w=_e(1), xhat_range=_e(2),
                 act_step=_e(1), act_zero=_e(1, dtype=I32), status=torch.zeros(1, dtype=I32, device=DEV))
        if w8a8:
            v["colsum_xq"] = _e(K, dtype=I64)
        if forward:
            v.update(xq=_e(B.aweq_panel_bytes(T, K), dtype=torch.int8), rowsum_x=_e(T, dtype=I32))
        self.v = {k: t for k, t in v.items() if k not in nulls}
        self.m = []
        for W in self.Ws:
            N = W.shape[0]
            ng = N * (K // group) if group > 0 else N if group == 0 else 1
            panels = bits == 8 and group <= 0
            nc = B.aweq_panel_bytes(N, K) if panels else N * K // 8 * bits
            m = {"W_hat": W if in_place else _e(N, K, dtype=X.dtype), "codes": _e(nc + 64 * N, dtype=torch.int8), "step_w": _e(ng + N),
                 "zero_w": _e(ng + N, dtype=I32), "delta": _e(N), "bias_out": _e(N)}
            if panels:
                m["rowsum_w"] = _e(N, dtype=I32)
            if forward:
                m.update(out_i32=_e(T, N, dtype=I32), out_deq=_e(T, N, dtype=X.dtype), colsum_acc=_e(N, dtype=I64))
            self.m.append(m)
        rows = [T] + [W.shape[0] for W in Ws]
        self.small = max([B.aweq_workspace_size(B.OP_CALIB_STATS, r, K, 0) for r in rows] + [B.aweq_workspace_size(B.OP_W8A8_GEMM, T, K, max(rows[1:])), 16])
        self.full = B.aweq_workspace_size(B.OP_CALIBRATE, T, K, sum(rows[1:]))

    def one(self, small):
        B, v, g = self.B, self.v, self.v.get
        ws = torch.empty(max(self.small, self.full), dtype=torch.uint8, device=DEV)
        ws_bytes = min(self.small, self.full - 1) if small else self.full
        B.aweq_calibrate((self.X, self.dt, self.T, self.K, self.X.stride(0), v["xmin"], v["xmax"], v["xsum"], g("count"), v["r_x"], v["R_x"], g("p_x"),
                          v["wmin"], v["wmax"], g("wcount"), v["r_w"], v["R_w"], g("p_w"), v["s"], v["inv_s"], v["xhat_range"], v["mu_xhat"],
                          v["act_step"], v["act_zero"], g("xq"), g("rowsum_x"), g("colsum_xq"), self.awe, self.bc, self.bits, self.group,
                          int(self.w8a8), int(self.forward), 0, ws, ws_bytes, g("status")),
                         [(W, W.shape[0], W.stride(0), m["W_hat"], m["W_hat"].stride(0), m["codes"], m["step_w"], m["zero_w"], m.get("rowsum_w"), b,
                           m["delta"], m["bias_out"], m.get("out_i32"), m.get("out_deq"), m.get("colsum_acc"))
                          for W, b, m in zip(self.Ws, self.biases, self.m)])
        return self.host()

    def stages(self):
        B, v, g, T, K, dt, X = self.B, self.v, self.v.get, self.T, self.K, self.dt, self.X
        ws = torch.empty(self.small, dtype=torch.uint8, device=DEV)
        st = g("status")
        B.aweq_calib_stats(X, dt, T, K, X.stride(0), v["xmin"], v["xmax"], v["xsum"], g("count"), 0, 1, v["r_x"], v["R_x"], g("p_x"), ws, st)
        last = len(self.Ws) - 1
        for i, W in enumerate(self.Ws):
            B.aweq_calib_stats(W, dt, W.shape[0], K, W.stride(0), v["wmin"], v["wmax"], None, g("wcount"), int(i > 0), int(i == last), v["r_w"],
                               v["R_w"], g("p_w"), ws, st)
        for W, m in zip(self.Ws, self.m):
            B.aweq_equalize(v["xmin"], v["xmax"], v["xsum"], T, v["wmin"], v["wmax"], K, self.awe, v["s"], v["inv_s"], W, m["W_hat"], dt, W.shape[0],
                            W.stride(0), m["W_hat"].stride(0), None, v["xhat_range"], v["mu_xhat"], v["act_step"], v["act_zero"], st)
        if self.w8a8:
            B.aweq_quant_act(X, dt, T, K, X.stride(0), v["inv_s"], v["act_step"], v["act_zero"], g("xq"), g("rowsum_x"), v["colsum_xq"], ws, st)
        wg = min(self.group, 0)
        for W, b, m in zip(self.Ws, self.biases, self.m):
            N, ld = W.shape[0], m["W_hat"].stride(0)
            B.aweq_quant_weight(m["W_hat"], dt, N, K, ld, self.bits, self.group, m["codes"], m["step_w"], m["zero_w"], m.get("rowsum_w"), ws, st)
            if self.forward:
                B.aweq_w8a8_gemm(v["xq"], B.AWEQ_I8, T, K, K, None, v["act_step"], v["act_zero"], None, v["rowsum_x"], None, m["codes"], N, m["step_w"],
                                 m["zero_w"], wg, m["rowsum_w"], b, m["out_i32"], m["out_deq"], dt, N, m["colsum_acc"], None, st)
            if self.w8a8:
                B.aweq_bias_correct(B.BIAS_W8A8, m["W_hat"], dt, N, K, ld, v["mu_xhat"], T, m.get("colsum_acc"), v["colsum_xq"], m["rowsum_w"],
                                    v["act_step"], v["act_zero"], None if self.forward else m["codes"], 8, wg, m["step_w"], m["zero_w"], b, m["delta"],
                                    m["bias_out"], self.bc, st)
            else:
                B.aweq_bias_correct(B.BIAS_WEIGHT_ONLY, m["W_hat"], dt, N, K, ld, v["mu_xhat"], T, None, None, None, None, None, m["codes"], self.bits,
                                    self.group, m["step_w"], m["zero_w"], b, m["delta"], m["bias_out"], self.bc, st)
        return self.host()

    def host(self):
        torch.cuda.synchronize()
        return {k: t.cpu().numpy() for k, t in self.v.items()}, [{k: t.cpu().numpy() for k, t in m.items()} for m in self.m]


def _near(a, b, bound, what):
    """a and b the same where one is infinite or NaN (sums of such values in any order), within `bound` elsewhere"""
    a, b = a.astype(np.float64), b.astype(np.float64)
    bad = ~np.isfinite(b)
    assert np.array_equal(a[bad], b[bad], equal_nan=True), what
    assert np.all(np.abs(a[~bad] - b[~bad]) <= bound[~bad]), what


def _compare(got, want, X, T, w8a8):
    loose = {"xsum", "mu_xhat", "delta", "bias_out"}
    for a, b in [(got[0], want[0])] + list(zip(got[1], want[1])):
        assert a.keys() == b.keys()
        for k in a:
            if k not in loose:
                assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k
    # binary64 sums of T terms in two orders; mu: one rounding of them to binary32; delta: a rounding of mu in any column, and its own
    with np.errstate(invalid="ignore", over="ignore"):
        size = X.double().abs().sum(0).cpu().numpy()
        _near(got[0]["xsum"], want[0]["xsum"], T * 2.0**-52 * size, "xsum")
        mu = want[0]["mu_xhat"].astype(np.float64)
        _near(got[0]["mu_xhat"], want[0]["mu_xhat"], 2.0**-23 * np.abs(mu) + 2.0**-52 * size * want[0]["inv_s"], "mu_xhat")
        for a, b in zip(got[1], want[1]):
            Wh = np.abs(b["W_hat"].astype(np.float64))
            # (weight-only: the rounding error of the weight takes the place of the weight)
            bound = 2.0**-22 * (Wh @ np.abs(mu) if w8a8 else Wh.max(1) * np.abs(mu).sum()) + 2.0**-22 * np.abs(b["delta"].astype(np.float64))
            _near(a["delta"], b["delta"], bound, "delta")
            _near(a["bias_out"], b["bias_out"], bound + 2.0**-23 * np.abs(b["bias_out"].astype(np.float64)), "bias_out")


def _inputs(dtype, T, Ns, K, pitched=False):
    gen = torch.Generator(device=DEV).manual_seed(K + T + sum(Ns))
    r = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    X = (r(T, K) * 2 + 0.1).to(dtype)
    X[:, K // 2] *= 40
    Ws = [(r(N, K + 8) * 0.05).to(dtype)[:, :K] if pitched else (r(N, K) * 0.05).to(dtype) for N in Ns]
    return X, Ws, [r(N) for N in Ns]


def _check(B, X, Ws, biases, bits, group, w8a8, forward, **options):
    print(f"[calibrate forms] {X.dtype} T={X.shape[0]} N={[W.shape[0] for W in Ws]} K={X.shape[1]} bits={bits} group={group} {w8a8} {forward} "
          f"{ {k: v for k, v in options.items()} }", flush=True)
    call = lambda: Call(B, X, Ws, biases, bits, group, w8a8, forward, **options)
    want = call().stages()
    for small in (False, True):
        _compare(call().one(small), want, X, X.shape[0], w8a8)
    return want


@pytest.mark.parametrize("dtype", [F16, F32])
@pytest.mark.parametrize("bits,group,w8a8,forward", [(8, -1, True, True), (8, -1, True, False), (8, 0, True, False), (4, 128, False, False), (3, 64, False, False),
                                                     (4, 8, False, False), (4, -1, False, False), (4, 0, False, False), (8, 128, False, False), (8, 0, False, False)])
def test_several_weights(B, dtype, bits, group, w8a8, forward):
    """Weights of one input in slices of every kind: each has scales of its own."""
    _check(B, *_inputs(dtype, 70, (5, 12, 3), 640), bits, group, w8a8, forward)


FORMS = [(8, 0, True, True), (8, 0, True, False), (4, 128, False, False), (3, 32, False, False), (8, -1, True, False)]
SHAPES = [(33, (5,), 640), (70, (9, 3), 1032), (40, (6,), 4224), (50, (7,), 8200), (40, (1030, 1027), 520)]   # whole 128-byte lines and not; a wavefront to a row, to two rows, and more


def _fits(K, bits, group):
    return group <= 0 or K % group == 0


@pytest.mark.parametrize("dtype", [F16, F32])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("T,Ns,K", SHAPES)
def test_folded_weight_in_its_weights_place(B, dtype, form, T, Ns, K):
    if _fits(K, *form[:2]):
        for pitched in (False, True):
            _check(B, *_inputs(dtype, T, Ns, K, pitched), *form, in_place=True)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("options", [dict(awe=0), dict(awe=2), dict(bc=0), dict(nulls=("count", "wcount", "p_x", "p_w", "status"))], ids=str)
def test_options(B, form, options):
    X, Ws, biases = _inputs(F16, 45, (5, 9), 1152)
    for b in (biases, [None, None]):
        _check(B, X, Ws, b, *form, **options)


def _wide_zero_points(X, Ws):
    Ws[0][1] += 60.0           # a row, a stretch of one far from zero: |Z| beyond what the quotient without a division takes
    Ws[0][2, 128:384] -= 30.0
    X += 50.0


def _degenerate(X, Ws):
    Ws[0][0] = 0.0
    Ws[0][1] = 0.25
    Ws[0][2, 128:384] = 0.0
    Ws[0][3, 128:384] = -0.0
    for W in Ws:
        W[:, 7] = 0.0
        W[:, 11] = 3.0
    X[:, 9] = 0.0
    X[:, 13] = -2.0


def _tiny(X, Ws):
    Ws[0][1] *= 2.0**-12       # (binary16: below its normal numbers)
    Ws[0][2] = 0.0
    Ws[0][2, 40] = 2.0**-24


def _huge(X, Ws):
    Ws[0][1, ::2] = 60000.0
    Ws[0][1, 1::2] = -60000.0
    X[3, 5] = 60000.0


def _infinite_weight(X, Ws):
    Ws[0][1, 20] = float("inf")
    Ws[-1][2, 300] = float("-inf")


def _nan_weight(X, Ws):
    Ws[0][1, 20] = float("nan")
    Ws[-1][2] = float("nan")


def _nonfinite_activation(X, Ws):
    X[3, 20] = float("inf")
    X[5, 40] = float("nan")
    X[:, 41] = float("nan")


@pytest.mark.parametrize("dtype", [F16, F32])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("values", [_wide_zero_points, _degenerate, _tiny, _huge, _infinite_weight, _nan_weight, _nonfinite_activation])
@pytest.mark.parametrize("K", [1152, 8320])
def test_values(B, dtype, form, values, K):
    """Rows, groups and columns without a range, far from zero, near either end of the type's range, with infinities and NaN: the same
    codes, scales and status."""
    print(f"[calibrate forms] {values.__name__}", flush=True)
    X, Ws, biases = _inputs(dtype, 45, (6, 5), K)
    values(X, Ws)
    for awe in (1, 0):
        _check(B, X, Ws, biases, *form, awe=awe)
