"""Convenience driver: allocate the buffers of one linear layer with torch and run the stages in
the order the method applies them (Sec. 3: statistics, equalization, quantization, W8A8 forward,
bias correction) as one call of the C ABI (aweq_calibrate).  No arithmetic of the method happens here.
"""
from dataclasses import dataclass, field
from typing import Optional

import torch

from . import binding as B


def _dt(t: torch.Tensor) -> int:
    if t.dtype == torch.float16:
        return B.AWEQ_F16
    if t.dtype == torch.float32:
        return B.AWEQ_F32
    if t.dtype == torch.int8:
        return B.AWEQ_I8
    raise TypeError(f"unsupported dtype {t.dtype}")


def _layer_args(X, T, K, t, acts, enable_awe, enable_bc, bits, group, w8a8, forward, fused_weight_pass):
    """The fields of aweq_calib_layer (include/aweq.h), in order, from the buffers `t` (acts: xq, rowsum_x, colsum_xq)."""
    ws = t["ws"]
    return (X, _dt(X), T, K, X.stride(0), t["xmin"], t["xmax"], t["xsum"], t["count"], t["r_x"], t["R_x"], t["p_x"], t["wmin"], t["wmax"],
            t["wcount"], t["r_w"], t["R_w"], t["p_w"], t["s"], t["inv_s"], t["xhat_range"], t["mu_xhat"], t["act_step"], t["act_zero"], *acts,
            int(enable_awe), int(enable_bc), bits, group, int(w8a8), int(forward), int(fused_weight_pass), ws, ws.numel() * ws.element_size(),
            t["status"])


@dataclass
class LayerBuffers:
    """Every device buffer one layer's calibration touches (allocated once, reused per step)."""
    T: int
    K: int
    N: int
    dtype: torch.dtype
    bits: int = 8
    group: int = 0
    w8a8: bool = True
    want_out_i32: bool = True
    want_out_deq: bool = False
    device: str = "cuda:0"
    t: dict = field(default_factory=dict)

    def __post_init__(self):
        d, T, K, N = self.device, self.T, self.K, self.N
        f32, i32, i64, f64 = torch.float32, torch.int32, torch.int64, torch.float64
        e = lambda *shape, dtype: torch.empty(shape, dtype=dtype, device=d)
        t = self.t
        for name in ("xmin", "xmax", "wmin", "wmax", "r_x", "p_x", "r_w", "p_w", "s", "inv_s", "mu_xhat"):
            t[name] = e(K, dtype=f32)
        t["xsum"] = e(K, dtype=f64)
        t["count"] = e(1, dtype=i64)
        t["wcount"] = e(1, dtype=i64)
        t["R_x"], t["R_w"] = e(1, dtype=f32), e(1, dtype=f32)
        t["xhat_range"] = e(2, dtype=f32)
        t["act_step"], t["act_zero"] = e(1, dtype=f32), e(1, dtype=i32)
        t["status"] = torch.zeros(1, dtype=i32, device=d)
        t["W_hat"] = e(N, K, dtype=self.dtype)
        ng = 1 if self.group < 0 else (N if self.group == 0 else N * (K // self.group))
        # 8-bit per-row / per-tensor codes are the GEMM operand: K-panel layout
        panel_w = self.bits == 8 and self.group <= 0
        t["codes"] = e(B.aweq_panel_bytes(N, K) if panel_w else N * K * self.bits // 8, dtype=torch.int8)
        t["step_w"], t["zero_w"] = e(ng, dtype=f32), e(ng, dtype=i32)
        t["rowsum_w"] = e(N, dtype=i32)
        t["delta"], t["bias_out"] = e(N, dtype=f32), e(N, dtype=f32)
        ws = max(B.aweq_workspace_size(B.OP_CALIB_STATS, T, K, N), B.aweq_workspace_size(B.OP_CALIB_STATS, N, K, N),
                 B.aweq_workspace_size(B.OP_QUANT_WEIGHT, N, K, N),
                 B.aweq_workspace_size(B.OP_W8A8_GEMM, T, K, N) if self.w8a8 else 0, B.aweq_workspace_size(B.OP_CALIBRATE, T, K, N), 16)
        t["ws"] = e(ws, dtype=torch.uint8)
        if self.w8a8:
            t["xq"] = e(B.aweq_panel_bytes(T, K), dtype=torch.int8)
            t["rowsum_x"] = e(T, dtype=i32)
            t["colsum_xq"] = e(K, dtype=i64)
            t["colsum_acc"] = e(N, dtype=i64)
            if self.want_out_i32:
                t["out_i32"] = e(T, N, dtype=i32)
            if self.want_out_deq:
                t["out_deq"] = e(T, N, dtype=self.dtype)


def calibrate_layer(X: torch.Tensor, W: torch.Tensor, bias: Optional[torch.Tensor], buf: LayerBuffers,
                    enable_awe: bool = True, enable_bc: bool = True, stream=None, fused_weight_pass: bool = False,
                    forward: bool = True):
    """One pass of the whole hot path for one linear layer.  Everything is enqueued on the
    current (or given) stream; nothing synchronises.  forward = False (W8A8) calibrates without
    running the int8 GEMM: the activation quantizer only forms its sums and the bias correction
    takes the accumulator's sums over tokens from the weight codes (the same integers).
    fused_weight_pass matters only where the stages run one by one (include/aweq.h): it fuses fold and quantizer there."""
    t = buf.t
    w8a8, forward = buf.w8a8, buf.w8a8 and forward
    out_i32, out_deq = (t.get("out_i32"), t.get("out_deq")) if forward else (None, None)
    B.aweq_calibrate(
        _layer_args(X, buf.T, buf.K, t, (t["xq"], t["rowsum_x"], t["colsum_xq"]) if forward else (None, None, t["colsum_xq"] if w8a8 else None),
                    enable_awe, enable_bc, buf.bits, buf.group, w8a8, forward, fused_weight_pass),
        [(W, buf.N, W.stride(0), t["W_hat"], t["W_hat"].stride(0), t["codes"], t["step_w"], t["zero_w"],
          t["rowsum_w"], bias, t["delta"], t["bias_out"], out_i32, out_deq,
          t["colsum_acc"] if forward else None)], stream)   # W may be a pitched view (a row slice of a fused qkv weight)
    return t


@dataclass
class GroupBuffers:
    """Buffers of a group of linears that read the same activation (q/k/v, gate/up): one
    statistics pass, one equalization scale (from the merged weight ranges), one activation
    quantization; per linear its folded weight, codes, GEMM output sums and bias."""
    T: int
    K: int
    Ns: tuple
    dtype: torch.dtype
    want_out_i32: bool = False
    want_out_deq: bool = False
    device: str = "cuda:0"
    t: dict = field(default_factory=dict)
    per: list = field(default_factory=list)

    def __post_init__(self):
        d, T, K = self.device, self.T, self.K
        f32, i32, i64, f64 = torch.float32, torch.int32, torch.int64, torch.float64
        e = lambda *shape, dtype: torch.empty(shape, dtype=dtype, device=d)
        t = self.t
        for name in ("xmin", "xmax", "wmin", "wmax", "r_x", "p_x", "r_w", "p_w", "s", "inv_s", "mu_xhat"):
            t[name] = e(K, dtype=f32)
        t["xsum"] = e(K, dtype=f64)
        t["count"], t["wcount"] = e(1, dtype=i64), e(1, dtype=i64)
        t["R_x"], t["R_w"] = e(1, dtype=f32), e(1, dtype=f32)
        t["xhat_range"] = e(2, dtype=f32)
        t["act_step"], t["act_zero"] = e(1, dtype=f32), e(1, dtype=i32)
        t["status"] = torch.zeros(1, dtype=i32, device=d)
        t["xq"] = e(B.aweq_panel_bytes(T, K), dtype=torch.int8)
        t["rowsum_x"] = e(T, dtype=i32)
        t["colsum_xq"] = e(K, dtype=i64)
        ws = max([B.aweq_workspace_size(B.OP_CALIB_STATS, T, K, 0), B.aweq_workspace_size(B.OP_QUANT_ACT, T, K, 0),
                  B.aweq_workspace_size(B.OP_CALIBRATE, T, K, sum(self.Ns))] +
                 [B.aweq_workspace_size(B.OP_CALIB_STATS, N, K, N) for N in self.Ns] + [16])
        t["ws"] = e(ws, dtype=torch.uint8)
        for N in self.Ns:
            p = {"W_hat": e(N, K, dtype=self.dtype), "codes": e(B.aweq_panel_bytes(N, K), dtype=torch.int8), "step_w": e(N, dtype=f32),
                 "zero_w": e(N, dtype=i32), "rowsum_w": e(N, dtype=i32), "colsum_acc": e(N, dtype=i64),
                 "delta": e(N, dtype=f32), "bias_out": e(N, dtype=f32)}
            if self.want_out_i32:
                p["out_i32"] = e(T, N, dtype=i32)
            if self.want_out_deq:
                p["out_deq"] = e(T, N, dtype=self.dtype)
            self.per.append(p)


def calibrate_group(X: torch.Tensor, Ws, biases, gb: GroupBuffers, enable_awe: bool = True, enable_bc: bool = True,
                    stream=None):
    """W8A8 calibration of linears sharing the input X (Sec. 3.1: equalization sits at the
    entrance of the attention block and of the MLP, so layers with a common input share s)."""
    t = gb.t
    B.aweq_calibrate(
        _layer_args(X, gb.T, gb.K, t, (t["xq"], t["rowsum_x"], t["colsum_xq"]), enable_awe, enable_bc, 8, 0, True, True, True),
        [(W, W.shape[0], W.stride(0), p["W_hat"], p["W_hat"].stride(0), p["codes"], p["step_w"], p["zero_w"], p["rowsum_w"], b, p["delta"],
          p["bias_out"], p.get("out_i32"), p.get("out_deq"), p["colsum_acc"]) for W, b, p in zip(Ws, biases, gb.per)], stream)
    return gb
