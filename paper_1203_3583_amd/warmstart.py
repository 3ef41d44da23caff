"""Learned warm start for phase-hologram descent on a curved surface.

A small convolutional encoder-decoder (four levels, base width 32, BF16 weights,
FP32 accumulation on the matrix cores; include/asf_warm.h) maps a target
intensity and the surface height map to a source phase.  It is trained on the
GPU through the diffraction method itself: the predicted phase drives the
forward transform (asf_forward), the loss is the intensity mismatch, and its
gradient comes back through the adjoint (asf_adjoint) into the network's own
backward kernels.  Training pairs are generated by the forward method: random
smooth source phases on random Zernike surfaces give the target intensities.
The network's phase is then a warm start for the adjoint-gradient descent of
``autograd.phase_descent``; zero phase is the fallback, and the forward method
judges both (the same intensity loss).

Tensors are channels-last torch tensors on the GPU: images (B, H, W, C) float32.
Every layer runs in this library's kernels; torch supplies memory and streams.
"""
from __future__ import annotations

import ctypes
import math
from collections.abc import MutableMapping

from . import asf as _asf

_READY = False


def _lib():
    global _READY
    L = _asf.lib()
    if not _READY:
        vp, i32, i64, f32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float
        sig = {
            "asf_warm_conv3x3": [vp, vp, vp, vp, i32, i32, i32, i32, i32, i32, vp],
            "asf_warm_conv3x3_upcat": [vp, i32, vp, i32, vp, vp, vp, i32, i32, i32, i32, i32, vp],
            "asf_warm_conv3x3_wgrad": [vp, vp, vp, vp, i32, i32, i32, i32, i32, vp],
            "asf_warm_flip_weights": [vp, vp, i32, i32, vp],
            "asf_warm_flip_weights_many": [i32, vp, vp, vp, vp, vp],
            "asf_warm_conv3x3_masked": [vp, vp, vp, vp, i32, i32, i32, i32, i32, vp],
            "asf_warm_conv3x3_wgrad_upcat": [vp, i32, vp, i32, vp, vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_up2_backward_relu": [vp, i32, vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_pool2_backward_skip_relu": [vp, vp, i32, i32, vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_relu_backward": [vp, vp, vp, i64, vp],
            "asf_warm_pool2": [vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_pool2_backward": [vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_up2": [vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_up2_backward": [vp, vp, i32, i32, i32, i32, vp],
            "asf_warm_copy_channels": [vp, i32, i32, vp, i32, i32, i32, i64, vp],
            "asf_warm_axpy": [vp, vp, f32, i64, vp],
            "asf_warm_adam": [vp, vp, vp, vp, vp, i64, f32, f32, f32, f32, i32, vp],
        }
        for name, args in sig.items():
            fn = getattr(L, name)
            fn.restype = ctypes.c_int
            fn.argtypes = args
        _READY = True
    return L


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream(torch):
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _ok(rc, what):
    if rc != 0:
        raise RuntimeError(f"{what} failed (invalid arguments or HIP launch error)")


def bf16_bits(torch, w):
    """Round a float32 tensor to BF16 (nearest even) and return the 16-bit patterns (int16)."""
    u = w.contiguous().view(torch.int32).to(torch.int64) & 0xFFFFFFFF
    u = (u + 0x7FFF + ((u >> 16) & 1)) >> 16
    return u.to(torch.int32).to(torch.int16)


def layer_shapes(c=32, cin0=16, cout_head=32):
    """(cin, cout, relu) of the 15 convolutions: two per level on the way down
    (widths c, 2c, 4c, 8c), two per level on the way up after concatenating the
    upsampled features with the skip connection, and a linear head."""
    return [(cin0, c, True), (c, c, True),
            (c, 2 * c, True), (2 * c, 2 * c, True),
            (2 * c, 4 * c, True), (4 * c, 4 * c, True),
            (4 * c, 8 * c, True), (8 * c, 8 * c, True),
            (12 * c, 4 * c, True), (4 * c, 4 * c, True),
            (6 * c, 2 * c, True), (2 * c, 2 * c, True),
            (3 * c, c, True), (c, c, True),
            (c, cout_head, False)]


class _LayerInputs(MutableMapping, dict):
    """The layers' inputs by layer.  A decoder layer whose concatenation was read in place
    has (upsampled half, skip) here, and its tensor is formed when asked for, in whichever
    way a dictionary can be asked; copies are plain dictionaries of tensors.  (The mapping's
    methods go through those below, where a dictionary's own would read past them.)"""

    def __init__(self, net, items):
        dict.__init__(self, items)
        self._net = net

    def parts(self, i):
        """Layer i's input: one tensor, or (low, skip)."""
        return dict.__getitem__(self, i)

    def __getitem__(self, i):
        v = dict.__getitem__(self, i)
        if isinstance(v, tuple):
            v = self._net._cat(self._net._up(v[0]), v[1])
            self[i] = v
        return v

    def __iter__(self):
        return dict.__iter__(self)

    __len__, __contains__, __reversed__ = dict.__len__, dict.__contains__, dict.__reversed__
    __setitem__, __delitem__, clear = dict.__setitem__, dict.__delitem__, dict.clear

    def popitem(self):
        if not self:
            raise KeyError("popitem(): dictionary is empty")
        i = next(reversed(self))
        return i, self.pop(i)

    def copy(self):
        return dict(self)

    def __or__(self, other):
        return dict(self) | other

    def __ror__(self, other):
        return other | dict(self)

    def __ior__(self, other):
        self.update(other)
        return self

    def __repr__(self):
        return repr(dict(self))

    def __reduce_ex__(self, protocol):
        return dict, (dict(self),)


class WarmNet:
    """The encoder-decoder with FP32 master weights, BF16 working copies and Adam state.

    Input (B, H, W, cin0): channel 0 the target intensity over its mean, channel 1 the
    height over 60 um, the rest zero; H and W multiples of 8.  Output channel 0 is
    the source phase (radians) at every sample of the surface grid.
    """

    def __init__(self, base=32, cin0=16, cout_head=32, device="cuda", seed=0, head_scale=0.1):
        import torch

        self.torch = torch
        self.shapes = layer_shapes(base, cin0, cout_head)
        g = torch.Generator(device="cpu").manual_seed(seed)
        self.w, self.b, self.wb, self.gw, self.gb = [], [], [], [], []
        self.mw, self.vw, self.mb, self.vb = [], [], [], []
        for i, (ci, co, relu) in enumerate(self.shapes):
            fan_in = 9 * (2 if i == 0 else ci)   # input layer: two real channels
            std = math.sqrt(2.0 / fan_in) * (1.0 if relu else head_scale)
            w = (torch.randn((co, 9 * ci), generator=g) * std).to(device)
            if i == 0:
                w.view(co, 9, ci)[:, :, 2:] = 0.0   # padded input channels
            self.w.append(w.contiguous())
            self.b.append(torch.zeros(co, device=device))
            self.wb.append(bf16_bits(torch, self.w[-1]))
            self.gw.append(torch.zeros_like(self.w[-1]))
            self.gb.append(torch.zeros_like(self.b[-1]))
            self.mw.append(torch.zeros_like(self.w[-1]))
            self.vw.append(torch.zeros_like(self.w[-1]))
            self.mb.append(torch.zeros_like(self.b[-1]))
            self.vb.append(torch.zeros_like(self.b[-1]))
        self.t = 0

    # -- layers ---------------------------------------------------------------------------
    def _conv(self, i, x, relu=None):
        torch = self.torch
        ci, co, r = self.shapes[i]
        B, H, W, C = x.shape
        assert C == ci and x.is_contiguous()
        out = torch.empty((B, H, W, co), dtype=torch.float32, device=x.device)
        _ok(_lib().asf_warm_conv3x3(_ptr(x), _ptr(self.wb[i]), _ptr(self.b[i]), _ptr(out), B, H, W, ci, co,
                                    int(r if relu is None else relu), _stream(torch)), "conv3x3")
        return out

    def _conv_upcat(self, i, low, skip):
        """Layer i on concat(up2(low), skip), read in place where the kernel takes the
        layer (the same result bit for bit), else concatenated first: the output, and the
        input as _LayerInputs holds it."""
        torch = self.torch
        ci, co, r = self.shapes[i]
        B, h, w, cl = low.shape
        cs = skip.shape[3]
        assert cl + cs == ci and low.is_contiguous() and skip.is_contiguous()
        out = torch.empty((B, 2 * h, 2 * w, co), dtype=torch.float32, device=low.device)
        if _lib().asf_warm_conv3x3_upcat(_ptr(low), cl, _ptr(skip), cs, _ptr(self.wb[i]), _ptr(self.b[i]),
                                         _ptr(out), B, 2 * h, 2 * w, co, int(r), _stream(torch)) == 0:
            return out, (low, skip)
        cat = self._cat(self._up(low), skip)
        return self._conv(i, cat), cat

    def infer(self, x):
        """The output of ``forward`` without keeping activations: the decoder's
        concatenations are read in place by their convolutions.  The activations share one
        allocation (120 floats per pixel at base 32) and the eighteen launches are issued
        with plain addresses (at 512^2 the kernels take about as long as a call per layer
        through torch tensors did)."""
        torch, sh = self.torch, self.shapes
        B, H, W, C = x.shape
        assert C == sh[0][0] and x.is_contiguous()
        L, s = _lib(), torch.cuda.current_stream().cuda_stream
        conv, upcat, pool = L.asf_warm_conv3x3, L.asf_warm_conv3x3_upcat, L.asf_warm_pool2
        # Two places per level, for the first and the second convolution's result, the
        # encoder's and then the decoder's: the first is read by the second convolution only,
        # the second (the skip tensor) last by the decoder's first.  The first also takes the
        # pooled second, the next level's input.
        px = [B * (H >> k) * (W >> k) for k in range(4)]
        enc, dec = (0, 2, 4, 6), (12, 10, 8, 6)   # each level's first layer
        first = [max(px[k] * sh[i][1] for i in (enc[k], dec[k])) for k in range(4)]
        second = [max(px[k] * sh[i + 1][1] for i in (enc[k], dec[k])) for k in range(4)]
        for k in range(3):
            first[k] = max(first[k], px[k + 1] * sh[enc[k] + 1][1])
        starts, total = [], 0
        for n in first + second:
            starts.append(total)
            total += (n + 63) & ~63
        buf = torch.empty(total, dtype=torch.float32, device=x.device)
        at = [buf.data_ptr() + 4 * o for o in starts]
        first, second = at[:4], at[4:]
        out = torch.empty((B, H, W, sh[14][1]), dtype=torch.float32, device=x.device)
        wb, b = [t.data_ptr() for t in self.wb], [t.data_ptr() for t in self.b]

        def layer(i, src, dst, k):
            ci, co, r = sh[i]
            _ok(conv(src, wb[i], b[i], dst, B, H >> k, W >> k, ci, co, int(r), s), "conv3x3")

        src = x.data_ptr()
        for k, i in enumerate(enc):
            layer(i, src, first[k], k)
            layer(i + 1, first[k], second[k], k)
            if k < 3:
                src = first[k]
                _ok(pool(second[k], src, B, H >> k, W >> k, sh[i + 1][1], s), "pool2")
        low, cl = second[3], sh[7][1]
        for k in (2, 1, 0):
            i, skip = dec[k], second[k]
            ci, co, r = sh[i]
            h, w, cs = H >> k, W >> k, sh[enc[k] + 1][1]
            assert cl + cs == ci
            if upcat(low, cl, skip, cs, wb[i], b[i], first[k], B, h, w, co, int(r), s) != 0:
                # layers too small for the tiled kernel are concatenated first
                up = torch.empty(B * h * w * (cl + ci), dtype=torch.float32, device=x.device)
                u, c = up.data_ptr(), up.data_ptr() + 4 * B * h * w * cl
                _ok(L.asf_warm_up2(low, u, B, h // 2, w // 2, cl, s), "up2")
                _ok(L.asf_warm_copy_channels(u, cl, 0, c, ci, 0, cl, B * h * w, s), "concat")
                _ok(L.asf_warm_copy_channels(skip, cs, 0, c, ci, cl, cs, B * h * w, s), "concat")
                layer(i, c, first[k], k)
            layer(i + 1, first[k], second[k], k)
            low, cl = second[k], sh[i + 1][1]
        layer(14, low, out.data_ptr(), 0)
        return out

    def _pool(self, x):
        B, H, W, C = x.shape
        out = self.torch.empty((B, H // 2, W // 2, C), dtype=self.torch.float32, device=x.device)
        _ok(_lib().asf_warm_pool2(_ptr(x), _ptr(out), B, H, W, C, _stream(self.torch)), "pool2")
        return out

    def _up(self, x):
        B, H, W, C = x.shape
        out = self.torch.empty((B, 2 * H, 2 * W, C), dtype=self.torch.float32, device=x.device)
        _ok(_lib().asf_warm_up2(_ptr(x), _ptr(out), B, H, W, C, _stream(self.torch)), "up2")
        return out

    def _cat(self, a, b):
        B, H, W, ca = a.shape
        cb = b.shape[3]
        out = self.torch.empty((B, H, W, ca + cb), dtype=self.torch.float32, device=a.device)
        n = B * H * W
        s = _stream(self.torch)
        _ok(_lib().asf_warm_copy_channels(_ptr(a), ca, 0, _ptr(out), ca + cb, 0, ca, n, s), "concat")
        _ok(_lib().asf_warm_copy_channels(_ptr(b), cb, 0, _ptr(out), ca + cb, ca, cb, n, s), "concat")
        return out

    def _slice(self, x, off, count):
        B, H, W, C = x.shape
        out = self.torch.empty((B, H, W, count), dtype=self.torch.float32, device=x.device)
        _ok(_lib().asf_warm_copy_channels(_ptr(x), C, off, _ptr(out), count, 0, count, B * H * W,
                                          _stream(self.torch)), "slice")
        return out

    # -- forward / backward ------------------------------------------------------------------
    def forward(self, x):
        """Output (B, H, W, cout_head) and the activations the backward needs."""
        a = [None] * 15
        a[0] = self._conv(0, x); a[1] = self._conv(1, a[0])
        p1 = self._pool(a[1]); a[2] = self._conv(2, p1); a[3] = self._conv(3, a[2])
        p2 = self._pool(a[3]); a[4] = self._conv(4, p2); a[5] = self._conv(5, a[4])
        p3 = self._pool(a[5]); a[6] = self._conv(6, p3); a[7] = self._conv(7, a[6])
        a[8], c3 = self._conv_upcat(8, a[7], a[5]); a[9] = self._conv(9, a[8])
        a[10], c2 = self._conv_upcat(10, a[9], a[3]); a[11] = self._conv(11, a[10])
        a[12], c1 = self._conv_upcat(12, a[11], a[1]); a[13] = self._conv(13, a[12])
        a[14] = self._conv(14, a[13])
        cache = {"a": a, "in": _LayerInputs(self, {
            0: x, 1: a[0], 2: p1, 3: a[2], 4: p2, 5: a[4], 6: p3, 7: a[6], 8: c3,
            9: a[8], 10: c2, 11: a[10], 12: c1, 13: a[12], 14: a[13]})}
        return a[14], cache

    def backward(self, dout, cache, record=None):
        """Accumulate the parameter gradients of sum(dout * output) into self.gw, self.gb.
        With a dict `record`, layer i's output gradient, pre-activation gradient and input
        gradient are kept in record[i] (for tests)."""
        if record is None and self._backward_fused(dout, cache):
            return
        torch = self.torch
        L = _lib()
        s = _stream(torch)
        a, inputs = cache["a"], cache["in"]

        def layer(i, dy, need_input=True):
            ci, co, relu = self.shapes[i]
            B, H, W, _ = dy.shape
            if relu:
                dpre = torch.empty_like(dy)
                _ok(L.asf_warm_relu_backward(_ptr(a[i]), _ptr(dy), _ptr(dpre), dy.numel(), s), "relu backward")
            else:
                dpre = dy.contiguous()
            _ok(L.asf_warm_conv3x3_wgrad(_ptr(inputs[i]), _ptr(dpre), _ptr(self.gw[i]), _ptr(self.gb[i]),
                                         B, H, W, ci, co, s), "wgrad")
            dx = None
            if need_input:
                wt = torch.empty_like(self.wb[i])
                _ok(L.asf_warm_flip_weights(_ptr(self.wb[i]), _ptr(wt), ci, co, s), "flip")
                dx = torch.empty((B, H, W, ci), dtype=torch.float32, device=dy.device)
                _ok(L.asf_warm_conv3x3(_ptr(dpre), _ptr(wt), None, _ptr(dx), B, H, W, co, ci, 0, s), "dgrad")
            if record is not None:
                record[i] = (dy, dpre, dx)
            return dx

        def up_back(d):
            B, H2, W2, C = d.shape
            out = torch.empty((B, H2 // 2, W2 // 2, C), dtype=torch.float32, device=d.device)
            _ok(L.asf_warm_up2_backward(_ptr(d), _ptr(out), B, H2 // 2, W2 // 2, C, s), "up2 backward")
            return out

        def pool_back(d, skip):
            B, Hh, Wh, C = d.shape
            out = torch.empty((B, 2 * Hh, 2 * Wh, C), dtype=torch.float32, device=d.device)
            _ok(L.asf_warm_pool2_backward(_ptr(d), _ptr(out), B, 2 * Hh, 2 * Wh, C, s), "pool2 backward")
            _ok(L.asf_warm_axpy(_ptr(skip), _ptr(out), 1.0, out.numel(), s), "axpy")
            return out

        d13 = layer(14, dout)
        d12 = layer(13, d13)
        dc1 = layer(12, d12)
        c = a[11].shape[3]
        d11 = up_back(self._slice(dc1, 0, c)); d1_skip = self._slice(dc1, c, dc1.shape[3] - c)
        d10 = layer(11, d11)
        dc2 = layer(10, d10)
        c = a[9].shape[3]
        d9 = up_back(self._slice(dc2, 0, c)); d3_skip = self._slice(dc2, c, dc2.shape[3] - c)
        d8 = layer(9, d9)
        dc3 = layer(8, d8)
        c = a[7].shape[3]
        d7 = up_back(self._slice(dc3, 0, c)); d5_skip = self._slice(dc3, c, dc3.shape[3] - c)
        d6 = layer(7, d7)
        dp3 = layer(6, d6)
        d5 = pool_back(dp3, d5_skip)
        d4 = layer(5, d5)
        dp2 = layer(4, d4)
        d3 = pool_back(dp2, d3_skip)
        d2 = layer(3, d3)
        dp1 = layer(2, d2)
        d1 = pool_back(dp1, d1_skip)
        d0 = layer(1, d1)
        layer(0, d0, need_input=False)

    def _backward_fused(self, dout, cache):
        """The backward without a record: each input gradient comes out of its kernel
        already past the ReLU below it, the concatenations stay unformed, and one launch
        flips all weights.  The same values as layer by layer, up to the order of the
        weight gradients' atomics.  False (nothing done) where some layer's width is not
        one the fused kernels take."""
        torch, sh = self.torch, self.shapes
        if any(ci % 32 or co % 32 for ci, co, _ in sh[1:]) or sh[0][1] % 32 or any(not r for _, _, r in sh[:14]):
            return False
        if sh[14][2] or any(t % 4 for t in (sh[i][1] for i in range(15))):
            return False
        L, s = _lib(), torch.cuda.current_stream().cuda_stream
        a, inputs = cache["a"], cache["in"]
        if not isinstance(inputs, _LayerInputs):
            return False
        dev, f32 = dout.device, torch.float32
        dout = dout.contiguous()
        # flipped weights of layers 1 .. 14
        n = 14
        wt = torch.empty(sum(self.wb[i].numel() + 8 & ~7 for i in range(1, 15)), dtype=self.wb[1].dtype, device=dev)
        ptrs, at = [], wt.data_ptr()
        for i in range(1, 15):
            ptrs.append(at)
            at += 2 * (self.wb[i].numel() + 8 & ~7)
        _ok(L.asf_warm_flip_weights_many(
            n, (ctypes.c_void_p * n)(*[self.wb[i].data_ptr() for i in range(1, 15)]), (ctypes.c_void_p * n)(*ptrs),
            (ctypes.c_int32 * n)(*[sh[i][0] for i in range(1, 15)]),
            (ctypes.c_int32 * n)(*[sh[i][1] for i in range(1, 15)]), s), "flip")

        def wgrad(i, d):
            ci, co, _ = sh[i]
            B, H, W, _ = d.shape
            v = inputs.parts(i)
            if isinstance(v, tuple):
                low, skip = v
                _ok(L.asf_warm_conv3x3_wgrad_upcat(low.data_ptr(), low.shape[3], skip.data_ptr(), skip.shape[3],
                                                   d.data_ptr(), self.gw[i].data_ptr(), self.gb[i].data_ptr(),
                                                   B, H, W, co, s), "wgrad")
            else:
                _ok(L.asf_warm_conv3x3_wgrad(v.data_ptr(), d.data_ptr(), self.gw[i].data_ptr(),
                                             self.gb[i].data_ptr(), B, H, W, ci, co, s), "wgrad")

        def dgrad(i, d, act=None):
            """Weight gradient of layer i from its pre-activation gradient d, then its input
            gradient, past the ReLU of act."""
            wgrad(i, d)
            ci, co, _ = sh[i]
            B, H, W, _ = d.shape
            dx = torch.empty((B, H, W, ci), dtype=f32, device=dev)
            w = ptrs[i - 1]
            if act is None:
                _ok(L.asf_warm_conv3x3(d.data_ptr(), w, None, dx.data_ptr(), B, H, W, co, ci, 0, s), "dgrad")
            else:
                _ok(L.asf_warm_conv3x3_masked(d.data_ptr(), w, act.data_ptr(), dx.data_ptr(), B, H, W, co, ci, s),
                    "dgrad")
            return dx

        def up_back(dcat, act):
            out = torch.empty_like(act)
            B, H, W, C = act.shape
            _ok(L.asf_warm_up2_backward_relu(dcat.data_ptr(), dcat.shape[3], act.data_ptr(), out.data_ptr(),
                                             B, H, W, C, s), "up2 backward")
            return out

        def pool_back(dpool, dcat, act):
            out = torch.empty_like(act)
            B, H, W, C = act.shape
            cat_c = dcat.shape[3]
            _ok(L.asf_warm_pool2_backward_skip_relu(dpool.data_ptr(), dcat.data_ptr(), cat_c, cat_c - C,
                                                    act.data_ptr(), out.data_ptr(), B, H, W, C, s), "pool2 backward")
            return out

        dc1 = dgrad(12, dgrad(13, dgrad(14, dout, a[13]), a[12]))
        dc2 = dgrad(10, dgrad(11, up_back(dc1, a[11]), a[10]))
        dc3 = dgrad(8, dgrad(9, up_back(dc2, a[9]), a[8]))
        dp3 = dgrad(6, dgrad(7, up_back(dc3, a[7]), a[6]))
        dp2 = dgrad(4, dgrad(5, pool_back(dp3, dc3, a[5]), a[4]))
        dp1 = dgrad(2, dgrad(3, pool_back(dp2, dc2, a[3]), a[2]))
        wgrad(0, dgrad(1, pool_back(dp1, dc1, a[1]), a[0]))
        return True

    def zero_grad(self):
        self.torch._foreach_zero_(self.gw + self.gb)

    def step(self, lr=1e-3, b1=0.9, b2=0.999, eps=1e-8):
        """One Adam step on every layer (FP32 masters, BF16 copies refreshed)."""
        self.t += 1
        L = _lib()
        s = _stream(self.torch)
        for i in range(len(self.shapes)):
            _ok(L.asf_warm_adam(_ptr(self.w[i]), _ptr(self.gw[i]), _ptr(self.mw[i]), _ptr(self.vw[i]),
                                _ptr(self.wb[i]), self.w[i].numel(), lr, b1, b2, eps, self.t, s), "adam")
            _ok(L.asf_warm_adam(_ptr(self.b[i]), _ptr(self.gb[i]), _ptr(self.mb[i]), _ptr(self.vb[i]),
                                None, self.b[i].numel(), lr, b1, b2, eps, self.t, s), "adam")
        if self.shapes[0][0] > 2:
            # keep the padded input channels of the first layer at zero
            co, ci = self.shapes[0][1], self.shapes[0][0]
            self.w[0].view(co, 9, ci)[:, :, 2:] = 0.0
            self.wb[0].copy_(bf16_bits(self.torch, self.w[0]))


# ---------------------------------------------------------------------------------------------
# the phase-hologram problems and training through the diffraction method
# ---------------------------------------------------------------------------------------------

class HoloProblems:
    """A source grid (side^2 samples, 8 um, jittered) with one plan re-binned per surface.

    ``make(rng)`` draws a Zernike surface and a smooth source phase and returns the
    surface height (side^2 float64), the target intensity (side, side) the forward
    method gives for that phase (unit amplitude), and the phase itself.
    """

    def __init__(self, side=512, seed=0, device="cuda"):
        import numpy as np
        import torch

        import synth

        self.torch, self.np, self.synth = torch, np, synth
        x, y, lam, z0, p2, m = synth.warm_pair_geometry(side, seed)
        self.side, self.lam, self.z0, self.p2 = side, lam, z0, p2
        self.x_np, self.y_np = x, y
        self.x = torch.from_numpy(x).to(device)
        self.y = torch.from_numpy(y).to(device)
        self.radius = side * p2 / 2.0
        self.basis = synth.zernike_basis(x, y, self.radius)
        self.amp = torch.ones(side * side, dtype=torch.float32, device=device)
        d0 = torch.zeros_like(self.x)
        self.plan = _asf.Plan(self.x, self.y, d0, lam, z0, p2, p2, m, m)

    def set_surface(self, d):
        """Re-bin the plan for height d (torch float64 [side^2] on the device)."""
        self.plan.setpts(self.x, self.y, d)

    def make(self, rng):
        np, torch = self.np, self.torch
        d = self.synth.zernike_height(rng, self.x_np, self.y_np, self.radius, basis=self.basis)
        phase = self.synth.smooth_phase(rng, self.side, self.side)
        dt = torch.from_numpy(d).to(self.x.device)
        self.set_surface(dt)
        u1 = torch.polar(self.amp, torch.from_numpy(phase.reshape(-1)).float().to(self.x.device))
        u2 = self.plan.forward(u1.contiguous())
        inten = (u2.real ** 2 + u2.imag ** 2).float()
        return dt, inten, phase

    def net_input(self, d, inten, cin0=16):
        """(1, side, side, cin0): intensity over its mean, height over 60 um, zeros."""
        torch = self.torch
        x = torch.zeros((1, self.side, self.side, cin0), dtype=torch.float32, device=inten.device)
        x[0, :, :, 0] = inten / inten.mean()
        x[0, :, :, 1] = (d.reshape(self.side, self.side) / 60e-6).float()
        return x


def physics_loss_and_grad(problems, d, inten, phi):
    """Intensity loss of source phase phi (side, side) on surface d against the target
    inten, and its gradient with respect to phi, through the forward and adjoint
    kernels.  The target is the generated intensity itself, unscaled: the forward
    method produced it from a unit-amplitude source on this surface, so it is exactly
    reachable, and training and both descents of ``compare_descent`` use one scale."""
    torch = problems.torch
    from .autograd import intensity_loss

    problems.set_surface(d)
    theta = phi.reshape(-1).double().detach().requires_grad_(True)
    target = inten.reshape(problems.side, problems.side)
    loss = intensity_loss(problems.plan, theta, problems.amp, target)
    loss.backward()
    return float(loss.detach()), theta.grad.reshape(problems.side, problems.side).float()


def train(net, problems, pairs, steps, lr=1e-3, batch=4, seed=1, log=None):
    """Train on a list of (d, inten) pairs for `steps` Adam steps of `batch` samples;
    each sample's gradient flows through the forward/adjoint kernels into the network."""
    import numpy as np

    torch = problems.torch
    rng = np.random.default_rng(seed)
    losses = []
    for it in range(steps):
        net.zero_grad()
        total = 0.0
        for _ in range(batch):
            d, inten = pairs[int(rng.integers(len(pairs)))]
            x = problems.net_input(d, inten, net.shapes[0][0])
            out, cache = net.forward(x)
            phi = out[0, :, :, 0].contiguous()
            loss, dphi = physics_loss_and_grad(problems, d, inten, phi)
            dout = torch.zeros_like(out)
            dout[0, :, :, 0] = dphi / batch
            net.backward(dout, cache)
            total += loss / batch
        net.step(lr)
        losses.append(total)
        if log is not None:
            log(it, total)
    return losses


def predict_phase(net, problems, d, inten):
    x = problems.net_input(d, inten, net.shapes[0][0])
    out = net.infer(x)
    return out[0, :, :, 0].contiguous()


def compare_descent(net, problems, d, inten, steps=50, lr=0.05):
    """Adjoint-gradient descent from zero phase and from the network's phase on one
    problem, both against the same target (the generated intensity, as in training);
    returns (losses_zero, losses_warm), each a list of `steps` losses."""
    from .autograd import phase_descent

    problems.set_surface(d)
    target = inten.reshape(problems.side, problems.side)
    _, lz = phase_descent(problems.plan, problems.amp, target, steps=steps, lr=lr)
    phi0 = predict_phase(net, problems, d, inten).reshape(-1)
    _, lw = phase_descent(problems.plan, problems.amp, target, steps=steps, lr=lr, theta0=phi0)
    return lz, lw


def iterations_to_reach(losses, level):
    """First iteration (1-based) whose loss is at or below `level`, or None if none is."""
    for i, v in enumerate(losses):
        if v <= level:
            return i + 1
    return None


def main(argv=None):
    """Train on generated pairs and compare descent from zero phase and from the network.

    python -m paper_1203_3583_amd.warmstart --side 512 --pairs 2000 --steps 1500
    prints one JSON line: training time and losses, and per held-out problem the
    losses of 50 descent steps from both starts.
    """
    import argparse
    import json
    import time

    import numpy as np
    import torch

    ap = argparse.ArgumentParser()
    ap.add_argument("--side", type=int, default=512)
    ap.add_argument("--pairs", type=int, default=2000)
    ap.add_argument("--steps", type=int, default=1500)
    ap.add_argument("--batch", type=int, default=4)
    ap.add_argument("--lr", type=float, default=1e-3)
    ap.add_argument("--eval", type=int, default=8)
    ap.add_argument("--descent-steps", type=int, default=50)
    ap.add_argument("--seed", type=int, default=0)
    a = ap.parse_args(argv)
    pr = HoloProblems(side=a.side, seed=a.seed)
    rng = np.random.default_rng(a.seed + 1)
    t0 = time.time()
    pairs = []
    for i in range(a.pairs):
        pairs.append(pr.make(rng)[:2])
        if (i + 1) % 1000 == 0:
            print(f"generated {i + 1} pairs", flush=True)
    torch.cuda.synchronize()
    t_gen = time.time() - t0
    net = WarmNet(base=32, seed=a.seed)
    t0 = time.time()
    losses = train(net, pr, pairs, a.steps, lr=a.lr, batch=a.batch, seed=a.seed + 2,
                   log=lambda it, l: print(f"step {it} loss {l:.4f}", flush=True) if it % 100 == 0 else None)
    torch.cuda.synchronize()
    t_train = time.time() - t0
    erng = np.random.default_rng(a.seed + 1000)
    runs = []
    for _ in range(a.eval):
        d, inten, _ = pr.make(erng)
        lz, lw = compare_descent(net, pr, d, inten, steps=a.descent_steps)
        runs.append({"zero": lz, "warm": lw, "warm_iters_to_zero_final": iterations_to_reach(lw, lz[-1])})
    print(json.dumps({"side": a.side, "pairs": a.pairs, "steps": a.steps, "batch": a.batch,
                      "generate_s": t_gen, "train_s": t_train, "train_loss_first": float(np.mean(losses[:20])),
                      "train_loss_last": float(np.mean(losses[-20:])), "eval": runs}))


if __name__ == "__main__":
    main()
