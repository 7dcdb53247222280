"""Training iterations of the five workloads as sequences of C-ABI calls.

Host control flow only: buffers are torch CUDA tensors used as raw device memory, and every
arithmetic step is a kernel of libmp.so.  The order follows the paper's statement of mixed-precision
training (Sections 3.1, 3.2): forward and loss-scaled backward on the fp16 copies, then one
mp_unscale_check_update over all parameters (inspect, then update masters or skip), then
mp_loss_scale_update.  Nothing here reads device memory, so a whole `step()` can be captured in a
HIP graph (`torch.cuda.graph`) and replayed.
"""
from __future__ import annotations

import math
from typing import Callable, Dict, List, Optional

import numpy as np
import torch

from . import _lib as ML
from . import binding as B

LN_EPS = 1e-5


def _round_up(n: int, k: int) -> int:
    return (n + k - 1) // k * k


class ParamStore:
    """fp32 masters, fp16 copies, fp16 gradients and Adam moments of a model, each kind in one
    contiguous device arena (every tensor starts on a 16-element boundary, gaps stay zero)."""

    def __init__(self, masters: Dict[str, np.ndarray], adam: bool):
        self.names = list(masters)
        self.shapes = {k: tuple(v.shape) for k, v in masters.items()}
        self.offsets, off = {}, 0
        for k, v in masters.items():
            self.offsets[k] = off
            off += _round_up(int(v.size), 16)
        self.total = off
        dev = "cuda"
        self.w32_arena = torch.zeros(off, dtype=torch.float32, device=dev)
        self.w16_arena = torch.zeros(off, dtype=torch.float16, device=dev)
        self.g16_arena = torch.zeros(off, dtype=torch.float16, device=dev)
        self.m_arena = torch.zeros(off, dtype=torch.float32, device=dev) if adam else None
        self.v_arena = torch.zeros(off, dtype=torch.float32, device=dev) if adam else None
        host = np.zeros(off, dtype=np.float32)
        for k, v in masters.items():
            host[self.offsets[k]:self.offsets[k] + v.size] = np.asarray(v, dtype=np.float32).reshape(-1)
        self.w32_arena.copy_(torch.from_numpy(host))
        B.mp_cast_f32_to_f16(off, self.w32_arena, self.w16_arena)     # fp16 copies = RNE16(masters)
        self.w32 = {k: self._view(self.w32_arena, k) for k in self.names}
        self.w16 = {k: self._view(self.w16_arena, k) for k in self.names}
        self.g16 = {k: self._view(self.g16_arena, k) for k in self.names}
        self.m = {k: self._view(self.m_arena, k) for k in self.names} if adam else {}
        self.v = {k: self._view(self.v_arena, k) for k in self.names} if adam else {}
        self.n_params = sum(int(np.prod(s)) for s in self.shapes.values())
        entries = [dict(g16=self.g16[k], w32=self.w32[k], w16=self.w16[k], m=self.m.get(k), v=self.v.get(k))
                   for k in self.names]
        self.tensor_list = B.tensor_list(entries)
        self.n_tensors = len(entries)
        flat = [dict(g16=self.g16_arena, w32=self.w32_arena, w16=self.w16_arena, m=self.m_arena, v=self.v_arena)]
        self.flat_list = B.tensor_list(flat)

    def _view(self, arena, k):
        n = int(np.prod(self.shapes[k]))
        return arena[self.offsets[k]:self.offsets[k] + n].view(self.shapes[k])


class _StepBase:
    def __init__(self, masters: Dict[str, np.ndarray], opt, scale_cfg, prechecked: bool = False, flat_update: bool = False):
        self.P = ParamStore(masters, adam=(opt.kind == "adam"))
        self.cfg = B.opt_cfg(opt.kind, opt.lr, opt.beta1, opt.beta2, opt.eps, opt.weight_decay)
        self.st = B.scale_state_alloc()
        mode = ML.MP_SCALE_BACKOFF if scale_cfg.mode == "backoff" else ML.MP_SCALE_STATIC
        B.mp_scale_state_init(self.st, mode, scale_cfg.init_scale, scale_cfg.growth_interval, scale_cfg.min_scale,
                              scale_cfg.max_scale)
        self.counters = B.update_counters_alloc()
        self.loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        self.prechecked = prechecked
        self.flat_update = flat_update
        self.ws: Optional[torch.Tensor] = None
        # tests may set trace(name, layer, tensor): called right after the kernel that wrote `tensor`
        self.trace: Optional[Callable] = None
        # every gradient producer also reports non-finite outputs into the state itself, which is what
        # `prechecked` relies on to drop the separate inspection pass
        self.st_grad = self.st
        # the loss as partial sums, from the loss call to the end of the iteration (step()); forward_backward() alone finishes it
        self.loss_part: Optional[torch.Tensor] = None
        self._later, self._parts = False, None

    def _alloc_ws(self, nbytes: int, loss_bytes: int):
        """One buffer: the calls' workspace, and the loss's partial sums, which stay from the loss call to the end of step()."""
        n = _round_up(max(nbytes, 1024), 256) // 4
        buf = torch.empty(n + _round_up(loss_bytes, 256) // 4, dtype=torch.float32, device="cuda")
        self.ws, self.loss_part = buf[:n], buf[n:]

    def optimizer(self):
        flags = ML.MP_UPDATE_PRECHECKED if self.prechecked else ML.MP_UPDATE_DEFAULT
        parts, self._parts = self._parts, None
        tensors, n = (self.P.flat_list, 1) if self.flat_update else (self.P.tensor_list, self.P.n_tensors)
        B.mp_unscale_check_update_end(tensors, n, self.cfg, self.st, self.counters, flags, parts, self.loss)

    def _mse(self, rows, cols, y, target, dy):
        """Loss and seed gradient; within step() the loss itself is finished by the launch that ends the iteration."""
        self._parts = None
        if self._later:
            self._parts = B.mp_mse_scaled_parts(rows, cols, y, target, cols, self.st, dy, self.loss_part)
        else:
            B.mp_mse_scaled(rows, cols, y, target, cols, self.st, self.loss, dy, self.loss_part)

    def step(self, inject: Optional[Callable] = None):
        """One iteration.  inject(gradients) runs between backward and update and sees this iteration's loss, and so does an
        `optimizer` of a derived class; otherwise the loss is there when the update is, which finishes it."""
        self._later = inject is None and getattr(self.optimizer, "__func__", None) is _StepBase.optimizer
        try:
            self.forward_backward()
        finally:
            self._later = False
        if inject is not None:
            inject(self.P.g16)
        self.optimizer()

    def state(self) -> B.ScaleState:
        return B.scale_state_read(self.st)

    def _t(self, name, layer, tensor):
        if self.trace is not None:
            self.trace(name, layer, tensor)


def _h16(x: np.ndarray) -> torch.Tensor:
    """Upload fp32 host data and round it to fp16 on the device (RNE, the library's cast)."""
    src = torch.from_numpy(np.ascontiguousarray(np.asarray(x, dtype=np.float32))).cuda()
    dst = torch.empty(src.shape, dtype=torch.float16, device="cuda")
    B.mp_cast_f32_to_f16(src.numel(), src, dst)
    return dst


# ====================================================================================== config 1
class MLPStep(_StepBase):
    """x -> relu(W1 x + b1) -> W2 h + b2, MSE loss (config 1)."""

    def __init__(self, wl, masters=None, **kw):
        super().__init__(masters or wl.masters(), wl.opt, wl.scale, **kw)
        self.wl = wl
        R, di, dh, do = wl.rows, wl.d_in, wl.d_hidden, wl.d_out
        e16 = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda")
        self.x, self.target = e16(R, di), e16(R, do)
        self.h, self.y, self.dy, self.dpre, self.dx = e16(R, dh), e16(R, do), e16(R, do), e16(R, dh), e16(R, di)
        self.d1 = B.gemm_desc(R, dh, di, epilogue=ML.MP_EPI_BIAS_RELU)
        self.d2 = B.gemm_desc(R, do, dh, epilogue=ML.MP_EPI_BIAS)
        self._alloc_ws(max(B.mp_gemm_bwd_dw_workspace_bytes(self.d1, True), B.mp_gemm_bwd_dw_workspace_bytes(self.d2, True)),
                       B.mp_loss_workspace_bytes(R, do))

    def set_batch(self, batch):
        self.x.copy_(_h16(batch["x"]))
        self.target.copy_(_h16(batch["target"]))

    def forward_backward(self):
        w, g, st = self.P.w16, self.P.g16, self.st_grad
        R, do = self.wl.rows, self.wl.d_out
        B.mp_gemm_fwd(self.d1, self.x, w["w1"], w["b1"], None, self.h)
        B.mp_gemm_fwd(self.d2, self.h, w["w2"], w["b2"], None, self.y)
        self._mse(R, do, self.y, self.target, self.dy)
        B.mp_gemm_bwd_both(self.d2, self.dy, w["w2"], self.dpre, self.d2, self.h, g["w2"], g["b2"], st, self.ws,
                           relu_src=self.h, ld_aux=self.wl.d_hidden)
        B.mp_gemm_bwd_both(self.d1, self.dpre, w["w1"], self.dx, self.d1, self.x, g["w1"], g["b1"], st, self.ws)


# ====================================================================================== configs 2, 3
class TransformerStep(_StepBase):
    """Stack of post-LayerNorm encoder layers with an MSE loss on the last output (configs 2, 3)."""

    def __init__(self, wl, masters=None, two_streams=False, fused_attention=True, grouped_dw=True, **kw):
        if masters is None:
            masters = {f"l{i}.{k}": v for i, lay in enumerate(wl.masters()) for k, v in lay.items()}
        super().__init__(masters, wl.opt, wl.scale, **kw)
        self.wl = wl
        self.two_streams = two_streams
        dk_ = wl.d_model // wl.n_heads
        # the fused attention kernels cover head size 64 and sequences up to 128; anything else runs the unfused chain of
        # batched products and softmax kernels (two base layers on 61 sentences of 53 tokens: 671 us that way, 613 us fused)
        self.fused_attention = fused_attention and dk_ == 64 and wl.seq_len <= 128
        self.ld_p = (wl.seq_len + 7) // 8 * 8 if self.fused_attention else wl.seq_len    # rows of the kept probabilities
        self.alpha = 1.0 / math.sqrt(dk_)
        # one launch for the four weight-gradient products of a layer (each alone has too few tiles for the chip);
        # needs weight shapes in multiples of 128 and a token count in multiples of 64, which are the rows these products
        # contract over: their operands have zero rows up to the next such number, written once and never again
        # (two base layers on 3233 tokens: 613 us with four products, their split sums and column sums per layer, 510 us so)
        self.grouped_dw = grouped_dw and wl.d_model % 128 == 0 and wl.d_ff % 128 == 0
        self._groups = {}
        self.side_stream = torch.cuda.Stream() if two_streams else None
        T, d, f, h, S, NB = wl.tokens, wl.d_model, wl.d_ff, wl.n_heads, wl.seq_len, wl.n_seq
        dk = d // h
        e16 = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda")
        e32 = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
        T_dw = self.T_dw = (T + 63) // 64 * 64 if self.grouped_dw else T

        def e16_dw(n):
            t = e16(T_dw, n)
            t[T:].zero_()
            return t[:T]
        self.x0, self.target = e16_dw(d), e16(T, d)
        self.act: List[dict] = []
        for _ in range(wl.n_layers):
            self.act.append(dict(qkv=e16(T, 3 * d), p=e16(NB, h, S, self.ld_p)[..., :S], ctx=e16_dw(d), a=e16(T, d), y1=e16_dw(d),
                                 f=e16_dw(f), g=e16(T, d), y2=e16_dw(d), mean1=e32(T), rstd1=e32(T), mean2=e32(T),
                                 rstd2=e32(T)))
        # backward temporaries, shared by all layers
        self.gbuf = [e16(T, d), e16(T, d)]
        self.tmp = [dict(dz2=e16_dw(d), df=e16_dw(f), dz1=e16_dw(d), dqkv=e16_dw(3 * d)) for _ in range(2)]
        self.dy1, self.dctx, self.dp = e16(T, d), e16(T, d), e16(NB, h, S, S)
        G = B.gemm_desc
        self.d_qkv = G(T, 3 * d, d, epilogue=ML.MP_EPI_BIAS)
        self.d_o = G(T, d, d, epilogue=ML.MP_EPI_BIAS)
        self.d_f1 = G(T, f, d, epilogue=ML.MP_EPI_BIAS_RELU)
        self.d_f2 = G(T, d, f, epilogue=ML.MP_EPI_BIAS)
        alpha = 1.0 / math.sqrt(dk)
        # scores = alpha q k^T and ctx = p v, batched over (sequence, head) with strides into qkv
        self.d_s = G(S, S, dk, ldx=3 * d, ldw=3 * d, ldy=S, alpha=alpha, batch_outer=NB, batch_inner=h,
                     sx=(S * 3 * d, dk), sw=(S * 3 * d, dk), sy=(h * S * S, S * S))
        self.d_c = G(S, dk, S, ldx=S, ldw=3 * d, ldy=d, trans_w=1, batch_outer=NB, batch_inner=h,
                     sx=(h * S * S, S * S), sw=(S * 3 * d, dk), sy=(S * d, dk))
        # a layer small enough for it: both gradients of each linear layer in one launch (then there is no grouped launch
        # and nothing for a second stream).  The grouped launch, where the widths allow it, takes two launches a layer less
        # (it finishes the LayerNorm sums), which call by call is worth 10 us a layer of 128 and 5 of 256 units, whatever the
        # tokens.  On the device they cross between 256 and 320 tokens, and the line is halfway: us of two layers' iteration as a
        # graph, grouped / joint, 128 wide on 128, 256, 320, 384, 512 and 1024 tokens 135.8 / 134.1, 137.9 / 134.9, 140.2 / 140.4,
        # 140.8 / 141.8, 144.1 / 146.8, 166.2 / 170.8; 256 wide on 128, 256, 320, 384 and 512 156.9 / 154.7, 164.4 / 163.0,
        # 164.9 / 168.9, 166.8 / 169.4, 168.6 / 171.3.
        self.joint_bwd = (grouped_dw and not (self.grouped_dw and T > 288) and
                          all(B.mp_gemm_bwd_both_joint(x, x) for x in (self.d_qkv, self.d_o, self.d_f1, self.d_f2)))
        self.grouped_dw = self.grouped_dw and not self.joint_bwd
        need = [B.mp_gemm_bwd_dw_workspace_bytes(x, True) for x in (self.d_qkv, self.d_o, self.d_f1, self.d_f2)]
        need += [B.mp_gemm_bwd_dw_workspace_bytes(self.d_s, False), B.mp_gemm_bwd_dw_workspace_bytes(self.d_c, False),
                 B.mp_layernorm_bwd_workspace_bytes(T, d)]
        self._alloc_ws(max(need), B.mp_loss_workspace_bytes(T, d))
        self.ws_side = torch.empty_like(self.ws)
        # partial column sums of a layer's two LayerNorm backwards, finished by its grouped launch (which alternate by layer)
        self.ln_parts = []
        if self.grouped_dw:
            n = B.mp_layernorm_bwd_workspace_bytes(T, d) // 4
            self.ln_parts = [[e32(n), e32(n)] for _ in range(2)]
            self.ln_nparts = B.mp_layernorm_bwd_nparts(T, d)

    def set_batch(self, batch):
        self.x0.copy_(_h16(batch["x"]))
        self.target.copy_(_h16(batch["target"]))

    def forward(self):
        wl, w = self.wl, self.P.w16
        T, d, h, S, NB = wl.tokens, wl.d_model, wl.n_heads, wl.seq_len, wl.n_seq
        x = self.x0
        for l, a in enumerate(self.act):
            p = f"l{l}."
            B.mp_gemm_fwd(self.d_qkv, x, w[p + "wqkv"], w[p + "bqkv"], None, a["qkv"])
            if self.fused_attention:
                B.mp_attention_fwd_ldp(NB, h, S, d // h, a["qkv"], 3 * d, self.alpha, a["p"], self.ld_p, a["ctx"], d)
            else:
                B.mp_gemm_fwd(self.d_s, a["qkv"], a["qkv"][:, d:], None, None, a["p"])
                self._t("s", l, a["p"])
                B.mp_softmax_fwd(NB * h * S, S, a["p"], a["p"], S)
                B.mp_gemm_fwd(self.d_c, a["p"], a["qkv"][:, 2 * d:], None, None, a["ctx"])
            B.mp_gemm_fwd(self.d_o, a["ctx"], w[p + "wo"], w[p + "bo"], None, a["a"])
            B.mp_layernorm_fwd(T, d, x, a["a"], w[p + "ln1_g"], w[p + "ln1_b"], LN_EPS, a["y1"], a["mean1"], a["rstd1"])
            B.mp_gemm_fwd(self.d_f1, a["y1"], w[p + "w1"], w[p + "b1"], None, a["f"])
            B.mp_gemm_fwd(self.d_f2, a["f"], w[p + "w2"], w[p + "b2"], None, a["g"])
            B.mp_layernorm_fwd(T, d, a["y1"], a["g"], w[p + "ln2_g"], w[p + "ln2_b"], LN_EPS, a["y2"], a["mean2"], a["rstd2"])
            x = a["y2"]
        return x

    def backward(self):
        """Backward pass.  The weight-gradient products do not feed anything else in the backward pass, so
        they are enqueued on a second stream (forked and joined with events, which HIP-graph capture records
        as parallel branches): their prologues, epilogues and partial last rounds overlap the input-gradient
        chain on the main stream.  Temporaries read by the side stream are double-buffered by layer parity, and
        the main stream waits for the side work of two layers back before reusing them."""
        wl, w, g, st, ws = self.wl, self.P.w16, self.P.g16, self.st_grad, self.ws
        T, d, f, h, S, NB = wl.tokens, wl.d_model, wl.d_ff, wl.n_heads, wl.seq_len, wl.n_seq
        main = torch.cuda.current_stream()
        side = self.side_stream if self.two_streams and not self.joint_bwd else None
        done = {}

        def linear_bwd(desc, dy, wname, bname, x, dx, forked, **epi):
            """Gradients of one linear layer.  Jointly in one launch where the model is small enough; else the input
            gradient here, and the weight gradient on the side stream unless the grouped launch takes it (the bias
            gradients `bname` that a LayerNorm backward produces have forked=False)."""
            if self.joint_bwd:
                B.mp_gemm_bwd_both(desc, dy, w[wname], dx, desc, x, g[wname], g[bname], st, ws, **epi)
                return
            if not self.grouped_dw:
                fork(lambda wsx: B.mp_gemm_bwd_dw(desc, dy, x, g[wname], g[bname] if forked else None, st, wsx))
            B.mp_gemm_bwd_dx(desc, dy, w[wname], dx, **epi)

        def fork(fn):
            """Run fn (weight-gradient calls) on the side stream after everything enqueued so far on main."""
            if side is None:
                fn(ws)
                return
            ev = torch.cuda.Event()
            ev.record(main)
            side.wait_event(ev)
            with torch.cuda.stream(side):
                fn(self.ws_side)

        def layernorm_bwd(part, dy, xin, ain, ln, mean, rstd, dz, bname):
            """One LayerNorm backward; its column sums are finished by the layer's grouped launch where there is one."""
            if part is not None:
                B.mp_layernorm_bwd_parts(T, d, dy, xin, ain, w[ln + "_g"], mean, rstd, dz, True, part)
            else:
                B.mp_layernorm_bwd(T, d, dy, xin, ain, w[ln + "_g"], mean, rstd, dz, g[ln + "_g"], g[ln + "_b"], st, ws,
                                   dz_colsum=None if self.joint_bwd else g[bname])

        # the layer-output gradient ping-pongs between two [T, d] buffers; the loss wrote gbuf[0]
        for i, l in enumerate(range(wl.n_layers - 1, -1, -1)):
            dy2, dx = self.gbuf[i % 2], self.gbuf[(i + 1) % 2]
            a, p = self.act[l], f"l{l}."
            tb = self.tmp[i % 2]
            dz2, df, dz1, dqkv = tb["dz2"], tb["df"], tb["dz1"], tb["dqkv"]
            parts = self.ln_parts[i % 2] if self.grouped_dw else (None, None)
            if side is not None and i >= 2:
                main.wait_event(done[i - 2])        # side stream finished reading this parity's temporaries
            x = self.x0 if l == 0 else self.act[l - 1]["y2"]
            # dz2 is the gradient of g = W2 f + b2 too, so its column sums are b2's gradient
            layernorm_bwd(parts[0], dy2, a["y1"], a["g"], p + "ln2", a["mean2"], a["rstd2"], dz2, p + "b2")
            self._t("dy2", l, dy2)
            self._t("dz2", l, dz2)
            linear_bwd(self.d_f2, dz2, p + "w2", p + "b2", a["f"], df, False, relu_src=a["f"], ld_aux=f)
            self._t("df", l, df)
            linear_bwd(self.d_f1, df, p + "w1", p + "b1", a["y1"], self.dy1, True, add=dz2, ld_aux=d)
            self._t("dy1", l, self.dy1)
            layernorm_bwd(parts[1], self.dy1, x, a["a"], p + "ln1", a["mean1"], a["rstd1"], dz1, p + "bo")
            self._t("dz1", l, dz1)
            linear_bwd(self.d_o, dz1, p + "wo", p + "bo", a["ctx"], self.dctx, False)
            self._t("dctx", l, self.dctx)
            # attention: dP = dctx V^T, dV = P^T dctx, dS = softmax', dQ = alpha dS K, dK = alpha dS^T Q
            if self.fused_attention:
                B.mp_attention_bwd_ldp(NB, h, S, d // h, a["qkv"], 3 * d, self.alpha, a["p"], self.ld_p, self.dctx, d, dqkv, 3 * d)
            else:
                B.mp_gemm_bwd_dx(self.d_c, self.dctx, a["qkv"][:, 2 * d:], self.dp)
                self._t("dp", l, self.dp)
                B.mp_gemm_bwd_dw(self.d_c, self.dctx, a["p"], dqkv[:, 2 * d:], None, None, ws)
                B.mp_softmax_bwd(NB * h * S, S, a["p"], self.dp, self.dp, S)
                self._t("ds", l, self.dp)
                B.mp_gemm_bwd_dx(self.d_s, self.dp, a["qkv"][:, d:], dqkv)
                B.mp_gemm_bwd_dw(self.d_s, self.dp, a["qkv"], dqkv[:, d:], None, None, ws)
            self._t("dqkv", l, dqkv)
            linear_bwd(self.d_qkv, dqkv, p + "wqkv", p + "bqkv", x, dx, True, add=dz1, ld_aux=d)
            self._t("dx", l, dx)
            if self.grouped_dw:
                # all four operand pairs of this layer are still in place (the temporaries alternate by layer); the
                # two bias gradients that no LayerNorm backward produced ride in the same launch
                key = (l, i % 2)
                if key not in self._groups:
                    over = lambda x: B.gemm_desc(self.T_dw, x.N, x.K)  # noqa: E731  (the zero rows too)
                    sums = B.colsum_parts([(parts[k], self.ln_nparts, d, (g[p + ln + "_g"], g[p + ln + "_b"], g[p + bias]))
                                           for k, (ln, bias) in enumerate((("ln2", "b2"), ("ln1", "bo")))])
                    self._groups[key] = B.gemm_group([(over(self.d_f2), dz2, a["f"], g[p + "w2"]),
                                                      (over(self.d_f1), df, a["y1"], g[p + "w1"], g[p + "b1"]),
                                                      (over(self.d_qkv), dqkv, x, g[p + "wqkv"], g[p + "bqkv"]),
                                                      (over(self.d_o), dz1, a["ctx"], g[p + "wo"])]), sums
                fork(lambda wsx: B.mp_gemm_bwd_dw_grouped_sums(*self._groups[key], st))
            if side is not None:
                done[i] = torch.cuda.Event()
                done[i].record(side)
        if side is not None:
            main.wait_stream(side)                   # every weight gradient is complete before the update
        self.dx_input = self.gbuf[wl.n_layers % 2]

    def forward_backward(self):
        wl = self.wl
        y = self.forward()
        self._mse(wl.tokens, wl.d_model, y, self.target, self.gbuf[0])
        self.backward()


# ====================================================================================== config 4
class XentStep(_StepBase):
    """Hidden states -> vocabulary logits -> softmax cross-entropy (config 4).  After forward_backward() `logits` [T, V],
    contiguous, holds their gradient."""

    def __init__(self, wl, masters=None, **kw):
        super().__init__(masters or wl.masters(), wl.opt, wl.scale, **kw)
        self.wl = wl
        T, d, V = wl.tokens, wl.d_model, wl.vocab
        self.h = torch.empty(T, d, dtype=torch.float16, device="cuda")
        self.targets = torch.empty(T, dtype=torch.int32, device="cuda")
        # the products work on rows a multiple of 8 elements apart, which every kernel reads in whole 16-byte pieces (pieces at odd
        # addresses arrive at a third of the rate); `logits` then takes dlogits from the pass that writes them
        # (1021 x 12001: an iteration with products on rows of 12001 156 us, so 149)
        self.ld_v = _round_up(V, 8)
        self.rows16 = torch.empty(T, self.ld_v, dtype=torch.float16, device="cuda")
        self.logits = self.rows16 if V == self.ld_v else torch.empty(T, V, dtype=torch.float16, device="cuda")
        self.dh = torch.empty(T, d, dtype=torch.float16, device="cuda")
        self.desc = B.gemm_desc(T, V, d, ldy=self.ld_v, epilogue=ML.MP_EPI_BIAS)
        self.db_with_loss = 16384 < V <= 32768
        self._alloc_ws(max(B.mp_gemm_bwd_dw_workspace_bytes(self.desc, not self.db_with_loss), B.mp_gemm_split_workspace_bytes(self.desc)),
                       B.mp_softmax_xent_db_workspace_bytes(T, V) if self.db_with_loss else B.mp_loss_workspace_bytes(T, V))

    def set_batch(self, batch):
        self.h.copy_(_h16(batch["h"]))
        self.targets.copy_(torch.from_numpy(np.asarray(batch["targets"], dtype=np.int32)).cuda())

    def forward_backward(self):
        wl, w, g = self.wl, self.P.w16, self.P.g16
        T, V = wl.tokens, wl.vocab
        B.mp_gemm_fwd(self.desc, self.h, w["w"], w["b"], None, self.rows16)
        copy = None if V == self.ld_v else self.logits
        # the bias gradient (column sums of dlogits) comes out of the pass that writes dlogits where that pass can, else out of
        # the weight gradient
        self._parts = None
        if self._later:
            self._parts = B.mp_softmax_xent_scaled_parts(T, V, self.rows16, self.ld_v, self.targets, self.st, self.rows16, copy,
                                                         g["b"] if self.db_with_loss else None, self.loss_part)
        elif self.db_with_loss:
            B.mp_softmax_xent_scaled_db_copy(T, V, self.rows16, self.ld_v, self.targets, self.st, self.loss, self.rows16, copy, g["b"], self.loss_part)
        else:
            B.mp_softmax_xent_scaled_copy(T, V, self.rows16, self.ld_v, self.targets, self.st, self.loss, self.rows16, copy, self.loss_part)
        B.mp_gemm_bwd_both(self.desc, self.rows16, w["w"], self.dh, self.desc, self.h, g["w"], None if self.db_with_loss else g["b"],
                           self.st_grad, self.ws)


# ====================================================================================== config 5
def lstm_row_blocks(batch: int, hidden: int, cus: int, seq_len: int) -> List[tuple]:
    """(first row, rows) of the launches that the persistent recurrent kernels of an LSTMStep take a batch in, or [] where
    the step-by-step plan is the faster one.

    All workgroups of a launch (16 units x 8 rows each) wait for each other and have to be resident together, two to a
    compute unit.  A launch takes no more than half of the chip, so that two models (on two streams, or in two processes)
    never leave each other half resident.  Launches follow one another, so their number bounds the gain: us per iteration
    of two layers x 10 steps, persistent / step by step, 512 units: 256 rows (4 launches) 527 / 561, 512 rows (8) 935 / 690;
    1024 units: 64 rows (2) 467 / 640, 128 rows (4) 741 / 784, 256 rows (8) 1295 / 918; 256 units, whose step-by-step
    products have less to do: 256 rows (2) 267 / 348, 512 rows (4) 442 / 384.  Each launch reads the weights anew, which
    short sequences do not make up for: 2, 3 and 4 launches need 3, 5 and 9 time steps (one layer of 1024 units: 64 rows
    (2) x 2 steps 119 / 103, x 3 130 / 126, x 4 142 / 148; 96 rows (3) x 4 172 / 160, x 6 204 / 214; 128 rows (4) x 8
    289 / 276; of 512 units: 128 rows (2) x 2 79 / 68, x 3 88 / 88, 256 rows (4) x 8 214 / 196)."""
    block = 8 * (cus // max(hidden // 16, 1))
    most = min(max(1, (seq_len - 1).bit_length()), 4 if hidden >= 512 else 2)
    if block <= 0 or -(-batch // block) > most:
        return []
    return [(r, min(block, batch - r)) for r in range(0, batch, block)]


class LSTMStep(_StepBase):
    """Stacked LSTM unrolled over time with an MSE loss on the top layer's outputs (config 5).

    Layer l keeps xh[l][t] = [input_t | h_{t-1}] as one row block.  Two launch plans give the same stored tensors:

    persistent (default where the shape allows): per layer ONE large product for the input half of all gate sums
      (fp32, x W_x^T over all T*B rows), then ONE recurrent kernel that runs all T steps with the recurrent weights
      on chip (mp_lstm_layer_fwd); backward likewise one recurrent kernel per layer (mp_lstm_layer_bwd) followed by
      the large input-gradient and weight-gradient products over all T*B rows.
    step by step: per time step one gate product with W[4H, I+H] (mp_gemm_fwd_ws) and one cell kernel; the cell
      kernel writes h_t both into xh[l][t+1] (recurrence) and into the next layer's xh[l+1][t] (or the output).

    A persistent launch may take half of the GPU's workgroup slots, or half of one XCD's, until it is done, so at most two models
    whose iterations may overlap (other streams, other processes on the GPU) run this plan safely; more of them, small ones too,
    need persistent=False.  Where
    that is not kept, a wait ends after 2 s.  What had not arrived by then reads as NaN: the iteration's gradients are
    flagged and its update is skipped, as those of later iterations are until rl_status, which recurrent_kernels_ok()
    looks at, is cleared."""

    def __init__(self, wl, masters=None, persistent=True, **kw):
        if masters is None:
            masters = {f"l{i}.{k}": v for i, lay in enumerate(wl.masters()) for k, v in lay.items()}
        super().__init__(masters, wl.opt, wl.scale, **kw)
        self.wl = wl
        T, Bt, H, NL = wl.seq_len, wl.batch_size, wl.hidden, wl.n_layers
        z16 = lambda *s: torch.zeros(s, dtype=torch.float16, device="cuda")
        z32 = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
        self.in_dims = [wl.d_in if l == 0 else H for l in range(NL)]
        blocks = lstm_row_blocks(Bt, H, torch.cuda.get_device_properties(0).multi_processor_count, T)
        self.persistent = persistent and H % 64 == 0 and H <= 1024 and all(i % 8 == 0 for i in self.in_dims) and bool(blocks)
        self.row_blocks = blocks if self.persistent else []
        self.xh = [z16(T, Bt, self.in_dims[l] + H) for l in range(NL)]      # h_0 = 0 stays in xh[l][0][:, I:]
        self.gates = [z16(T, Bt, 4 * H) for _ in range(NL)]
        self.c = [z32(T + 1, Bt, H) for _ in range(NL)]                      # c_0 = 0
        self.y = z16(T, Bt, H)
        self.target = z16(T, Bt, H)
        self.dy = z16(T, Bt, H)
        self.dxh = [z16(T, Bt, max(self.in_dims) + H) for _ in range(2)]
        self.dgates = z16(T, Bt, 4 * H)
        self.dc = z32(Bt, H)
        self.d_gate = [B.gemm_desc(Bt, 4 * H, self.in_dims[l] + H, epilogue=ML.MP_EPI_BIAS) for l in range(NL)]
        self.d_gate_all = [B.gemm_desc(T * Bt, 4 * H, self.in_dims[l] + H) for l in range(NL)]
        need = [B.mp_gemm_bwd_dw_workspace_bytes(x, True) for x in self.d_gate_all]
        # the recurrent products have only `batch` rows: with a workspace they split their contraction over the chip
        need += [B.mp_gemm_split_workspace_bytes(x) for x in self.d_gate]
        self._alloc_ws(max(need), B.mp_loss_workspace_bytes(T * Bt, H))
        if self.persistent:
            self.gx = z32(T * Bt, 4 * H)                                     # input half of the gate sums, all steps
            self.dx = [z16(T * Bt, max(self.in_dims)) for _ in range(2)]     # input gradient of a layer, all steps
            self.rl_status = torch.zeros(1, dtype=torch.int32, device="cuda")
            rows = self.row_blocks[0][1]
            # two workspaces: every recurrent call of an iteration empties the one that the next call uses
            words = B.mp_lstm_layer_desc_workspace_bytes(B.lstm_layer_desc(T, rows, 0, H, H, H, H, step_rows=Bt)) // 4
            self.rl_ws = [torch.zeros(words, dtype=torch.int32, device="cuda") for _ in range(2)]
            # x W_x^T and dgates W_x: the input columns [0, I) of W[4H, I+H], all T*B rows at once
            self.d_in_all = [B.gemm_desc(T * Bt, 4 * H, self.in_dims[l], ldx=self.in_dims[l] + H, ldw=self.in_dims[l] + H)
                             for l in range(NL)]
            self.d_dx_all = [B.gemm_desc(T * Bt, 4 * H, self.in_dims[l], ldx=self.in_dims[l], ldw=self.in_dims[l] + H)
                             for l in range(NL)]

            # arguments of the recurrent calls: per layer and block of batch rows
            self.rl_fwd, self.rl_bwd = [], []
            for l in range(NL):
                I = self.in_dims[l]
                up, ldup = (self.xh[l + 1], self.in_dims[l + 1] + H) if l + 1 < NL else (self.y, H)
                above, ld_above = (self.dx[(l + 1) % 2].view(-1)[:T * Bt * H].view(T, Bt, H) if l + 1 < NL else self.dy), H
                self.rl_fwd.append([(B.lstm_layer_desc(T, n, I, H, I + H, I + H, ldup, step_rows=Bt), self.gx[r:], self.gates[l][0, r:],
                                     self.c[l][0, r:], self.xh[l][0, r:], up[0, r:]) for r, n in self.row_blocks])
                self.rl_bwd.append([(B.lstm_layer_desc(T, n, I, H, I + H, I + H, ld_above, step_rows=Bt), self.gates[l][0, r:],
                                     self.c[l][0, r:], above[0, r:], self.dgates[0, r:]) for r, n in self.row_blocks])

    def set_batch(self, batch):
        x = _h16(batch["x"])
        self.xh[0][:, :, :self.in_dims[0]].copy_(x)
        self.target.copy_(_h16(batch["target"]))

    def forward_backward(self):
        if self.persistent:
            self._forward_backward_persistent()
        else:
            self._forward_backward_stepwise()

    def recurrent_kernels_ok(self) -> bool:
        """False if a wait of a persistent kernel ever ran out of time (synchronises; tests and logging)."""
        return (not self.persistent) or int(self.rl_status.item()) == 0

    def _forward_backward_persistent(self):
        wl, w, g = self.wl, self.P.w16, self.P.g16
        T, Bt, H, NL = wl.seq_len, wl.batch_size, wl.hidden, wl.n_layers
        ws, ws_next, ready = *self.rl_ws, False          # (nothing is taken over from an earlier iteration)
        for l in range(NL):
            B.mp_gemm_fwd(self.d_in_all[l], self.xh[l], w[f"l{l}.w"], None, None, None, self.gx)
            for d, gx, gates, c, xh, up in self.rl_fwd[l]:
                B.mp_lstm_layer_fwd_placed(d, gx, w[f"l{l}.w"], w[f"l{l}.b"], gates, c, xh, up, self.rl_status, ws, ready, ws_next)
                ws, ws_next, ready = ws_next, ws, True
        self._mse(T * Bt, H, self.y, self.target, self.dy)
        for l in range(NL - 1, -1, -1):
            for d, gates, c, above, dgates in self.rl_bwd[l]:
                B.mp_lstm_layer_bwd_placed(d, w[f"l{l}.w"], gates, c, above, dgates, self.rl_status, ws, ready, ws_next)
                ws, ws_next = ws_next, ws
            B.mp_gemm_bwd_both(self.d_dx_all[l], self.dgates, w[f"l{l}.w"], self.dx[l % 2], self.d_gate_all[l], self.xh[l],
                               g[f"l{l}.w"], g[f"l{l}.b"], self.st_grad, self.ws)
        # gradient of the input: rows of all steps, and with time as a dimension of its own (where the step-by-step plan has
        # [T, batch, I + H]) for the sizes that plan was once the only one for
        lead = (T * Bt,) if Bt <= 32 and H % 128 == 0 else (T, Bt)
        self.dx_input = self.dx[0].view(-1)[:T * Bt * self.in_dims[0]].view(*lead, self.in_dims[0])

    def _forward_backward_stepwise(self):
        wl, w, g = self.wl, self.P.w16, self.P.g16
        T, Bt, H, NL = wl.seq_len, wl.batch_size, wl.hidden, wl.n_layers
        for l in range(NL):
            I = self.in_dims[l]
            ldxh = I + H
            for t in range(T):
                B.mp_gemm_fwd_ws(self.d_gate[l], self.xh[l][t], w[f"l{l}.w"], w[f"l{l}.b"], None, self.gates[l][t], ws=self.ws)
                if l + 1 < NL:
                    up, ldup = self.xh[l + 1][t], self.in_dims[l + 1] + H
                else:
                    up, ldup = self.y[t], H
                rec = self.xh[l][t + 1][:, I:] if t + 1 < T else None
                B.mp_lstm_cell_fwd(Bt, H, self.gates[l][t], 4 * H, self.c[l][t], self.c[l][t + 1], up, ldup, rec, ldxh)
        self._mse(T * Bt, H, self.y, self.target, self.dy)
        above, ld_above = self.dy, H
        for l in range(NL - 1, -1, -1):
            I = self.in_dims[l]
            ldxh = I + H
            dxh = self.dxh[l % 2].view(-1)[:T * Bt * ldxh].view(T, Bt, ldxh)
            B.mp_fill_u32(Bt * H, 0, self.dc)
            for t in range(T - 1, -1, -1):
                rec = dxh[t + 1][:, I:] if t + 1 < T else None
                B.mp_lstm_cell_bwd(Bt, H, self.gates[l][t], 4 * H, self.c[l][t], self.c[l][t + 1], above[t], ld_above,
                                   rec, ldxh, self.dc, self.dgates[t])
                B.mp_gemm_bwd_dx_ws(self.d_gate[l], self.dgates[t], w[f"l{l}.w"], dxh[t], ws=self.ws)
            B.mp_gemm_bwd_dw(self.d_gate_all[l], self.dgates, self.xh[l], g[f"l{l}.w"], g[f"l{l}.b"], self.st_grad, self.ws)
            above, ld_above = dxh, ldxh
        self.dx_input = above


# ====================================================================================== command line
def _main(argv=None):
    """python -m paper_1805_10387_amd.steps <1..5> [--steps N] [--warmup W] [--graph]
    Runs one of the five synthetic workloads for N timed iterations and prints one JSON line (ms per iteration,
    tokens or rows per second, final loss and scale state).  Meant for profiling a workload under rocprofv3."""
    import argparse
    import json
    import sys
    import os
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import mp_inputs as I
    ap = argparse.ArgumentParser(prog="python -m paper_1805_10387_amd.steps")
    ap.add_argument("config", type=int, choices=[1, 2, 3, 4, 5])
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--graph", action="store_true", help="replay the iteration as a HIP graph")
    a = ap.parse_args(argv)
    wl = {1: I.C1, 2: I.C2, 3: I.C3, 4: I.C4, 5: I.C5}[a.config]
    # config 3 in the configuration bench.py times; the others as their parity tests run them
    kw = dict(prechecked=True, flat_update=True) if a.config == 3 else {}
    step = {1: MLPStep, 2: TransformerStep, 3: TransformerStep, 4: XentStep, 5: LSTMStep}[a.config](wl, **kw)
    step.set_batch(wl.batch())
    for _ in range(max(a.warmup, 1)):
        step.step()
    torch.cuda.synchronize()
    run = step.step
    if a.graph:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step.step()
        run = graph.replay
        run()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(a.steps):
        run()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / a.steps
    units = getattr(wl, "tokens", None) or getattr(wl, "rows", None) or 0
    s = step.state()
    print(json.dumps({"config": a.config, "ms_per_step": ms, "units_per_step": units, "units_per_s": units / (ms * 1e-3),
                      "parameters": int(step.P.total), "launch": "HIP graph replay" if a.graph else "eager",
                      "loss": float(step.loss), "loss_scale": s.scale, "opt_steps": s.opt_step, "skipped": s.skipped_steps}))


if __name__ == "__main__":
    _main()
