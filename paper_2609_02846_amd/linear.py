"""FP4 linear layer: Y = X W^T with the UE5M3 recipe in all three GEMMs.

A ``torch.autograd.Function`` over the library's calls (argument marshalling
only; every quantization and product runs in the HIP kernels):

forward (Sec. 2.3, Table 5; eq:delayed-amax)
  * sample-and-hold amax of X and W at the layer's step;
  * X row blocks RN (the fprop operand) and, when W needs a gradient, X
    column blocks RN (the wgrad operand, blocked along tokens) from one
    read;
  * W 16x16 tiles RN, plus the transposed payload when X needs a gradient;
  * fprop GEMM, bf16 Y.

backward (eq:sr: stochastic rounding on the upstream gradient only; RN on
request)
  * sample-and-hold amax of dY;
  * dY row blocks SR -> dgrad GEMM dX = dY W (bf16);
  * dY column blocks SR -> wgrad GEMM dW = dY^T X (in the weight's dtype).

Policies (Table tab:inference-scale-summary):
  * training: every operand refreshes every ``period`` optimizer steps
    (50 in the recipe, 1 = current scaling); the caller sets ``step`` to the
    optimizer-step index;
  * inference (``inference_policy``): the weight amax is measured on the
    first batch and held; activations refresh every 50 batches ("delayed"),
    every batch ("current"), or use a calibrated reference held fixed
    ("calibrated", after ``calibrate``); the batch index is the layer's own
    forward count.

SR randomness: each backward call draws from Philox with key ``seed`` +
(number of earlier backward calls of this layer), counter block
(element index, tensor id); the tensor ids are 2 * layer_id + 1 (dgrad
operand) and 2 * layer_id + 2 (wgrad operand), so layers and the two dY
blockings never share words.

Block-size control (Sec. "Recipe comparison", Table tab:results):
``block=32`` runs every 1D block and weight tile at 32 (one scale code per
32 elements, 32 x 32 weight tiles) with the rest of the recipe unchanged.

Shapes: in_features and out_features multiples of the block (16 or 32);
with W trainable the token count (X's leading dimensions flattened) must
be a multiple of the block too.  Weights are bf16.  There is no bias term.
"""

import ctypes
import functools

import torch

from . import (COL16T, COL32T, NN, NT, OUT_BF16, RN, ROW16, ROW32, SCALE_UE5M3, TILE16, TILE32, TN, AmaxState,
               _MODES, _bf16_2d, _check, _dev_buf, _f32_out, _stream, amax_accumulate, load_library)

# The layer's small calls are bound by the host, so forward and backward
# marshal the library calls themselves: all operands of a pass lie in one or
# two device buffers (``_Layout``), whose shapes and alignment are right by
# construction, instead of some ten tensors that each cost an allocation, a
# check and an argument object.  Measured for 128 x 256 x 256 (host time):
# forward 61 -> 26 us, forward and backward 306 -> 146 us.


class _Layout:
    """Byte offsets of the operands of one pass inside a buffer, each 256-byte
    aligned."""

    def __init__(self):
        self.bytes = 0

    def add(self, nbytes):
        at = self.bytes
        self.bytes += (int(nbytes) + 255) & ~255
        return at


@functools.lru_cache(maxsize=512)
def _forward_layout(T, K, N, B, need_dx, need_dw, shared_dec):
    """(saved, temp): the operands the backward pass needs (X blocked along
    tokens when W needs a gradient, the transposed weight when X does) and
    those only the forward product reads.  ``shared_dec``: one call quantizes
    both blockings of X and writes one decode multiplier."""
    saved, temp = _Layout(), _Layout()
    temp.xr, temp.sxr = temp.add(T * K // 2), temp.add(T * K // B)
    temp.pw, temp.sw = temp.add(N * K // 2), temp.add((N // B) * (K // B))
    temp.dec_x = temp.add(0 if need_dw and shared_dec else 4)
    if need_dw:
        saved.xc, saved.sxc, saved.dec_xc = saved.add(T * K // 2), saved.add(T * K // B), saved.add(4)
    if need_dx:
        saved.pwt, saved.swt = saved.add(N * K // 2), saved.add((N // B) * (K // B))
    (saved if need_dx else temp).dec_w = (saved if need_dx else temp).add(4)
    return saved, temp


@functools.lru_cache(maxsize=512)
def _backward_layout(T, N, B, need_dx, need_dw):
    temp = _Layout()
    if need_dx:
        temp.dr, temp.sdr, temp.dec_r = temp.add(T * N // 2), temp.add(T * N // B), temp.add(4)
    if need_dw:
        temp.dc, temp.sdc, temp.dec_c = temp.add(T * N // 2), temp.add(T * N // B), temp.add(4)
    return temp


def _sample(lib, state, x, numel, step, stream):
    _check(lib.ue5m3_amax_sample(ctypes.byref(state.c), x, numel, step, None, stream), "ue5m3_amax_sample")


def _sample_rht(lib, state, x, rows, cols, mask, step, stream):
    _check(lib.ue5m3_amax_sample_rht(ctypes.byref(state.c), x, rows, cols, mask, step, None, stream),
           "ue5m3_amax_sample_rht")


def _amax(state):
    return _f32_out(state.amax, "amax_dev").data_ptr()


def _quantize(lib, layer, x, rows, cols, axis, state, target, mode, seed, tid, payload, scales, dec, stream):
    args = (x, rows, cols, axis, _amax(state), float(target), mode, seed, tid)
    if layer.block == 16:
        st = lib.ue5m3_quantize_1d(*args, payload, scales, dec, stream)
    else:
        st = lib.ue5m3_quantize_1d_ex(*args, SCALE_UE5M3, layer.block, payload, scales, dec, stream)
    _check(st, "ue5m3_quantize_1d")


def _product(lib, layer, layout, M, N, K, a, a_scales, a_dec, b, b_scales, b_dec, out, stream):
    """One of the layer's three products into the bf16 tensor ``out``, with
    the recipe's blockings for the layout."""
    wide = layer.block == 32
    a_blk = (COL32T if wide else COL16T) if layout == TN else (ROW32 if wide else ROW16)
    b_blk = a_blk if layout == TN else (TILE32 if wide else TILE16)
    args = (layout, M, N, K, a, a_scales, a_blk, a_dec, b, b_scales, b_blk, b_dec, out.data_ptr(), OUT_BF16)
    if layer.pm_grid is not None:
        _check(lib.ue5m3_gemm_pm(*args, SCALE_UE5M3, int(layer.pm_grid), stream), "ue5m3_gemm_pm")
    elif wide:
        _check(lib.ue5m3_gemm_ex(*args, SCALE_UE5M3, stream), "ue5m3_gemm")
    else:
        _check(lib.ue5m3_gemm(*args, stream), "ue5m3_gemm")


class _FP4LinearFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x2d, weight, layer, need_dx, need_dw):
        # need_dx / need_dw are decided by the caller: autograd runs this
        # method with gradients disabled.
        _bf16_2d(x2d, "x")
        _bf16_2d(weight, "weight")
        T, K = x2d.shape
        N = weight.shape[0]
        if weight.shape[1] != K:
            raise ValueError(f"weight has {weight.shape[1]} columns, the input {K}")
        step = int(layer._forward_step())
        lib, stream = load_library(), _stream()
        x, w = x2d.data_ptr(), weight.data_ptr()
        B, target, mask = layer.block, float(layer.target), int(layer.rht_mask)
        dual = B == 16 and not layer.rht_wgrad
        saved, temp = _forward_layout(T, K, N, B, need_dx, need_dw, dual)
        keep = torch.empty(saved.bytes, dtype=torch.uint8, device=x2d.device) if saved.bytes else None
        work = torch.empty(temp.bytes, dtype=torch.uint8, device=x2d.device)
        y = torch.empty((T, N), dtype=torch.bfloat16, device=x2d.device)
        t0 = work.data_ptr()
        s0 = keep.data_ptr() if keep is not None else 0
        xr, sxr, pw, sw = t0 + temp.xr, t0 + temp.sxr, t0 + temp.pw, t0 + temp.sw
        dec_w = s0 + saved.dec_w if need_dx else t0 + temp.dec_w

        _sample(lib, layer.amax_x, x, T * K, step, stream)
        _sample(lib, layer.amax_w, w, N * K, step, stream)
        if need_dw and dual:
            dec_x = s0 + saved.dec_xc
            _check(lib.ue5m3_quantize_dual(x, T, K, _amax(layer.amax_x), target, RN, 0, 0, 0, SCALE_UE5M3,
                                           xr, sxr, s0 + saved.xc, s0 + saved.sxc, dec_x, stream),
                   "ue5m3_quantize_dual")
        else:
            dec_x = t0 + temp.dec_x
            _quantize(lib, layer, x, T, K, 1, layer.amax_x, target, RN, 0, 0, xr, sxr, dec_x, stream)
            if need_dw and layer.rht_wgrad:
                _sample_rht(lib, layer.amax_xt, x, T, K, mask, step, stream)
                _check(lib.ue5m3_quantize_cols_rht(x, T, K, _amax(layer.amax_xt), target, RN, 0, 0, mask,
                                                   s0 + saved.xc, s0 + saved.sxc, s0 + saved.dec_xc, stream),
                       "ue5m3_quantize_cols_rht")
            elif need_dw:
                _quantize(lib, layer, x, T, K, 0, layer.amax_x, target, RN, 0, 0, s0 + saved.xc, s0 + saved.sxc,
                          s0 + saved.dec_xc, stream)
        pwt, swt = (s0 + saved.pwt, s0 + saved.swt) if need_dx else (None, None)
        args = (w, N, K, _amax(layer.amax_w), target, RN, 0, 0)
        if B == 16:
            st = lib.ue5m3_quantize_2d(*args, pw, sw, pwt, swt, dec_w, stream)
        else:
            st = lib.ue5m3_quantize_2d_ex(*args, SCALE_UE5M3, B, pw, sw, pwt, swt, dec_w, stream)
        _check(st, "ue5m3_quantize_2d")
        _product(lib, layer, NT, T, N, K, xr, sxr, dec_x, pw, sw, dec_w, y, stream)
        ctx.layer, ctx.step, ctx.shape, ctx.layout = layer, step, (T, K, N), saved
        ctx.save_for_backward(keep)
        return y

    @staticmethod
    def backward(ctx, dy):
        layer, saved = ctx.layer, ctx.layout
        T, K, N = ctx.shape
        need_dx, need_dw = ctx.needs_input_grad[0], ctx.needs_input_grad[1]
        dy = _bf16_2d(dy.to(torch.bfloat16).contiguous(), "the output gradient")
        keep, = ctx.saved_tensors
        lib, stream = load_library(), _stream()
        d, B, step, mask = dy.data_ptr(), layer.block, ctx.step, int(layer.rht_mask)
        _sample(lib, layer.amax_dy, d, T * N, step, stream)
        seed = layer._next_sr_seed()
        dx = dw = None
        if not (need_dx or need_dw):
            return dx, dw, None, None, None
        mode = _MODES[layer.grad_rounding]
        temp = _backward_layout(T, N, B, need_dx, need_dw)
        work = torch.empty(temp.bytes, dtype=torch.uint8, device=dy.device)
        t0 = work.data_ptr()
        s0 = _dev_buf(keep, torch.uint8, saved.bytes, "the saved operands").data_ptr()
        tid = (2 * layer.layer_id + 1) & 0xFFFFFFFF
        if need_dx:
            dx = torch.empty((T, K), dtype=torch.bfloat16, device=dy.device)
            dr, sdr, dec = t0 + temp.dr, t0 + temp.sdr, t0 + temp.dec_r
            _quantize(lib, layer, d, T, N, 1, layer.amax_dy, layer.target, mode, seed, tid, dr, sdr, dec, stream)
            _product(lib, layer, NN, T, K, N, dr, sdr, dec, s0 + saved.pwt, s0 + saved.swt, s0 + saved.dec_w, dx, stream)
        if need_dw:
            tid = (tid + 1) & 0xFFFFFFFF
            dw = torch.empty((N, K), dtype=torch.bfloat16, device=dy.device)
            dc, sdc, dec = t0 + temp.dc, t0 + temp.sdc, t0 + temp.dec_c
            if layer.rht_wgrad:
                _sample_rht(lib, layer.amax_dyt, d, T, N, mask, step, stream)
                _check(lib.ue5m3_quantize_cols_rht(d, T, N, _amax(layer.amax_dyt), float(layer.target_dy_wgrad),
                                                   mode, seed, tid, mask, dc, sdc, dec, stream),
                       "ue5m3_quantize_cols_rht")
            else:
                _quantize(lib, layer, d, T, N, 0, layer.amax_dy, layer.target_dy_wgrad, mode, seed, tid, dc, sdc, dec,
                          stream)
            _product(lib, layer, TN, N, K, T, dc, sdc, dec, s0 + saved.xc, s0 + saved.sxc, s0 + saved.dec_xc, dw, stream)
        return dx, dw, None, None, None


class Linear(torch.nn.Module):
    """FP4 (E2M1 + UE5M3 block scales) linear layer without bias.

    ``period``: sample-and-hold period D in optimizer steps (50 in the
    recipe).  ``target``: scale target T (448); ``target_dy_wgrad``: T of the
    wgrad dY operand (448, or 2048 for the paper's override).  The weight is
    bf16 and so is its gradient (the wgrad GEMM writes it directly).
    ``grad_rounding``: "sr" (the recipe) or "rn" for the dY quantizers.
    ``pm_grid``: None runs the decoded-operand GEMMs (fp32 accumulation);
    an integer d runs all three products through the probe-matched output
    model with final-grid denominator d (0 = no snap, the paper's 1024).
    ``rht_wgrad``: quantize the two wgrad operands (X and dY blocked along
    tokens) after a 16-point randomized Hadamard transform with one sign mask
    per layer (drawn from ``seed``), each with the amax of its transformed
    tensor as reference (the "UE5M3 with Transformer Engine settings"
    recipe, with ``period`` 1 and ``pm_grid`` 1024).  ``block``: 16 (the
    recipe) or 32 (the block-size control; not with ``rht_wgrad``)."""

    def __init__(self, in_features, out_features, period=50, target=448.0, target_dy_wgrad=448.0,
                 seed=0, layer_id=0, device="cuda", grad_rounding="sr", pm_grid=None, rht_wgrad=False,
                 block=16):
        super().__init__()
        if grad_rounding not in ("sr", "rn"):
            raise ValueError("grad_rounding must be 'sr' or 'rn'")
        if block not in (16, 32):
            raise ValueError("block must be 16 or 32")
        if block == 32 and rht_wgrad:
            raise ValueError("the Hadamard transform works on blocks of 16")
        self.block = int(block)
        self.grad_rounding, self.pm_grid = grad_rounding, pm_grid
        self.rht_wgrad = bool(rht_wgrad)
        self.rht_mask = (((int(seed) * 0x9E3779B97F4A7C15 + 0x632BE59BD9B4E019) % 2 ** 64) >> 48) & 0xFFFF
        if in_features % block or out_features % block or in_features <= 0 or out_features <= 0:
            raise ValueError(f"in_features and out_features must be positive multiples of {block}")
        self.in_features, self.out_features = int(in_features), int(out_features)
        self.weight = torch.nn.Parameter(
            torch.empty(out_features, in_features, dtype=torch.bfloat16, device=device))
        torch.nn.init.normal_(self.weight, std=in_features ** -0.5)
        self.target, self.target_dy_wgrad = float(target), float(target_dy_wgrad)
        self.seed, self.layer_id = int(seed), int(layer_id)
        self.amax_x = AmaxState(period, device)
        self.amax_w = AmaxState(period, device)
        self.amax_dy = AmaxState(period, device)
        self.amax_xt = AmaxState(period, device)     # transformed wgrad operands
        self.amax_dyt = AmaxState(period, device)
        self.step = 0               # optimizer-step index, set by the training loop
        self.sr_calls = 0           # backward calls so far (SR key offset)
        self.batches = 0            # forward calls under an inference policy
        self.policy = None          # None = training

    # -- scale policies -------------------------------------------------
    def inference_policy(self, policy="delayed", calibration=None):
        """Switch to an inference-scale policy: "delayed" (D = 50),
        "current" (D = 1) or "calibrated" (the largest amax over the
        ``calibration`` batches, held fixed).  Caches start empty; the weight
        reference is measured on the first batch and held."""
        if policy not in ("delayed", "current", "calibrated"):
            raise ValueError(policy)
        self.amax_w.set_period(0)
        self.amax_x.set_period(50 if policy == "delayed" else 1)
        if policy == "calibrated":
            if not calibration:
                raise ValueError("the calibrated policy needs calibration batches")
            self.calibrate(calibration)
        self.policy, self.batches = policy, 0
        return self

    def calibrate(self, batches):
        """Hold the largest activation amax over ``batches`` (bf16 tensors of
        [..., in_features]) as X's reference from now on."""
        for i, b in enumerate(batches):
            amax_accumulate(self._flat(b), self.amax_x.amax, clear=(i == 0))
        self.amax_x.freeze()

    def training_policy(self, period=50):
        """Back to training: every operand refreshes every ``period`` steps,
        from empty caches."""
        for st in (self.amax_x, self.amax_w, self.amax_dy, self.amax_xt, self.amax_dyt):
            st.set_period(period)
        self.policy = None
        return self

    # -- internals ------------------------------------------------------
    def _forward_step(self):
        if self.policy is None:
            return self.step
        b = self.batches
        self.batches += 1
        return b

    def _next_sr_seed(self):
        s = (self.seed + self.sr_calls) & (2 ** 64 - 1)
        self.sr_calls += 1
        return s

    def _flat(self, x):
        if x.dtype != torch.bfloat16 or x.shape[-1] != self.in_features:
            raise ValueError(f"input must be bf16 with last dimension {self.in_features}")
        if x.dim() == 2 and x.is_contiguous():
            return x                      # no view node in the autograd graph
        return x.reshape(-1, self.in_features).contiguous()

    def forward(self, x):
        x2d = self._flat(x)
        grad = torch.is_grad_enabled()
        need_dx = grad and x.requires_grad
        need_dw = grad and self.weight.requires_grad
        if need_dw and x2d.shape[0] % self.block:
            raise ValueError("the wgrad operand is blocked along tokens: token count must be a "
                             f"multiple of {self.block}")
        y = _FP4LinearFn.apply(x2d, self.weight, self, need_dx, need_dw)
        return y if x.dim() == 2 else y.reshape(*x.shape[:-1], self.out_features)

    def extra_repr(self):
        return (f"in_features={self.in_features}, out_features={self.out_features}, target={self.target}, "
                f"block={self.block}")
