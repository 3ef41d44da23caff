"""Differentiable forward for PyTorch: gradients through the adjoint transform.

``propagate(plan, u1)`` returns u2 = A u1 (the forward of the C ABI) as a node of
the autograd graph; its backward is the adjoint g1 = A^H g2 (``asf_adjoint``),
which is PyTorch's rule for a complex linear map (the gradient of u1 is A^H
times the gradient of u2).  Both directions run the HIP kernels; the plan's
geometry (x1, y1, d1) is a constant of the graph.

``intensity_loss`` and ``phase_descent`` build the phase-hologram problem on a
curved surface: a phase-only source u1 = a exp(i theta) on the plan's surface and
the loss || |u2|^2 - T ||^2 against a target intensity T.
"""
from __future__ import annotations


def _torch():
    import torch

    return torch


class _Propagate:
    """Holder of the autograd.Function (built lazily so importing needs no torch).  known:
    u2, where the caller has it already."""

    fn = None

    @classmethod
    def get(cls):
        if cls.fn is None:
            torch = _torch()

            class Propagate(torch.autograd.Function):
                @staticmethod
                def forward(ctx, u1, plan, known):
                    ctx.plan = plan
                    return plan.forward(u1.contiguous()) if known is None else known.clone()

                @staticmethod
                def backward(ctx, grad_u2):
                    g = grad_u2
                    if g.dtype != torch.complex64:
                        g = g.to(torch.complex64)
                    return ctx.plan.adjoint(g.contiguous()), None, None

            cls.fn = Propagate
        return cls.fn


def propagate(plan, u1):
    """u2 = A u1 (complex64 [my, mx]) with autograd support through the adjoint."""
    return _Propagate.get().apply(u1, plan, None)


class _IntensityLoss:
    """Holder of the fused loss (an autograd.Function built lazily, as _Propagate's)."""

    fn = None

    @classmethod
    def get(cls):
        if cls.fn is None:
            torch = _torch()
            from . import asf as _asf

            class IntensityLoss(torch.autograd.Function):
                # A graph of the gradient (create_graph) is that of the values the loss was computed
                # from: nothing of the caller's (theta, amp, target may change in place) is read
                # again, and theta only links the graph.  A leaf has no history to change and links
                # it as it is; for any other theta (link) the field u1 is an output beside the loss
                # and, saved as one, links it through this node.  (An output more costs 5 us.)
                @staticmethod
                def forward(ctx, theta, plan, amp, target, link):
                    L = _asf.lib()
                    dev, m = plan.device, plan.mx * plan.my
                    s = _asf._stream_ptr(torch, dev, None)
                    u1 = torch.empty(plan.n, dtype=torch.complex64, device=dev)
                    f64 = int(theta.dtype == torch.float64)
                    _asf._check(L.asf_phase_field(plan.n, amp.data_ptr(), theta.data_ptr(), f64, u1.data_ptr(), s))
                    u2 = plan.forward(u1)
                    # diff, then the sums, then the loss
                    buf = torch.empty(m + _asf.LOSS_SUMS, dtype=torch.float64, device=dev)
                    loss = torch.empty((), dtype=torch.float64, device=dev)
                    diff = buf.data_ptr()
                    _asf._check(L.asf_intensity_loss(m, u2.data_ptr(), target.data_ptr(),
                                                     int(target.dtype == torch.float64), diff, diff + 8 * m,
                                                     loss.data_ptr(), s))
                    ctx.save_for_backward(u1, u2, buf)
                    ctx.plan, ctx.shape, ctx.dtype = plan, theta.shape, theta.dtype
                    if not link:
                        ctx.leaf = theta
                        return loss
                    ctx.leaf = None
                    ctx.set_materialize_grads(False)
                    return loss, u1

                @staticmethod
                def backward(ctx, grad, g1=None):
                    """grad: of the loss, g1: of u1 (from a graph of the gradient); None: none."""
                    plan = ctx.plan
                    u1, u2, buf = ctx.saved_tensors
                    m = plan.mx * plan.my
                    if torch.is_grad_enabled():   # create_graph: the same in differentiable operations
                        if ctx.leaf is not None:   # u1 exp(i (theta - theta))
                            turn = (ctx.leaf - ctx.leaf.detach()).to(torch.float32).reshape(-1)
                            u1 = (u1 * torch.polar(torch.ones_like(turn), turn)).requires_grad_()
                        if grad is not None:
                            u = _Propagate.get().apply(u1, plan, u2)
                            inten = u.real.double() ** 2 + u.imag.double() ** 2
                            # the value saved, the derivative of the intensity
                            d = buf[:m].view(plan.my, plan.mx) + (inten - inten.detach())
                            part = torch.autograd.grad((d ** 2).sum() / buf[m], u1, grad, create_graph=True)[0]
                            g1 = part if g1 is None else g1 + part
                        out = None if g1 is None else (g1.conj() * (1j * u1)).real.to(ctx.dtype).reshape(ctx.shape)
                        return out, None, None, None, None
                    if grad is None and g1 is None:
                        return None, None, None, None, None
                    L = _asf.lib()
                    dev = plan.device
                    s = _asf._stream_ptr(torch, dev, None)
                    if grad is not None:
                        grad = grad.to(torch.float64).contiguous()
                        g2 = torch.empty((plan.my, plan.mx), dtype=torch.complex64, device=dev)
                        diff = buf.data_ptr()
                        _asf._check(L.asf_intensity_loss_backward(m, u2.data_ptr(), diff, diff + 8 * m,
                                                                  grad.data_ptr(), g2.data_ptr(), s))
                        part = plan.adjoint(g2)
                        g1 = part if g1 is None else g1 + part
                    else:
                        g1 = g1.resolve_conj().contiguous()
                    out = torch.empty(ctx.shape, dtype=ctx.dtype, device=dev)
                    _asf._check(L.asf_phase_backward(plan.n, u1.data_ptr(), g1.data_ptr(), out.data_ptr(),
                                                     int(ctx.dtype == torch.float64), s))
                    return out, None, None, None, None

            cls.fn = IntensityLoss
        return cls.fn


def _fused_loss_takes(plan, theta, amp, target):
    """Whether the fused loss computes this call: plain contiguous tensors of the plan's
    sizes on its device, nothing but theta differentiated.  Everything else (broadcast or
    strided arguments, other types, gradients of amp or target) takes the composite of
    elementwise operations.  On every call the fused form takes it is the faster one, five
    launches and 0.09 GB beside the transforms against about thirty and 1.0 GB at 1024^2
    points (there one gradient takes 154 us, against 346)."""
    torch = _torch()
    # tracing and forward-mode levels see the elementwise operations
    if torch.compiler.is_compiling() or torch.jit.is_tracing() or torch.autograd.forward_ad._current_level >= 0:
        return False
    for t in (theta, amp, target):
        if type(t) not in (torch.Tensor, torch.nn.Parameter) or t.device != plan.device or not t.is_contiguous():
            return False
        if t.is_neg() or torch._C._functorch.is_functorch_wrapped_tensor(t):
            return False
    real = (torch.float32, torch.float64)
    return (theta.dtype in real and target.dtype in real and amp.dtype == torch.float32
            and theta.shape == amp.shape and theta.numel() == plan.n and tuple(target.shape) == (plan.my, plan.mx)
            and not amp.requires_grad and not target.requires_grad)


def _intensity_loss_composite(plan, theta, amp, target):
    torch = _torch()
    u1 = torch.polar(amp.to(torch.float32), theta.to(torch.float32))
    u2 = propagate(plan, u1)
    inten = (u2.real.double() ** 2 + u2.imag.double() ** 2)
    t = target.double()
    return ((inten - t) ** 2).sum() / (t * t).sum()


def intensity_loss(plan, theta, amp, target):
    """|| |A (amp exp(i theta))|^2 - target ||^2 / || target ||^2 (float64 scalar).

    theta, amp: real [n] tensors on the plan's device (theta may require grad);
    target: real [my, mx] tensor in the units of |u2|^2 (see ``energy_matched``).
    """
    if _fused_loss_takes(plan, theta, amp, target):
        link = theta.grad_fn is not None
        out = _IntensityLoss.get().apply(theta, plan, amp, target, link)
        return out[0] if link else out
    return _intensity_loss_composite(plan, theta, amp, target)


def energy_matched(plan, amp, target, theta=None):
    """target rescaled so that its sum equals the energy sum |u2|^2 over the destination
    window of the source amp exp(i theta) (default theta = 0).  The window's energy
    depends on theta (the window is finite), so a caller fixes this scale once per
    problem and uses the same target for every iteration and every start it compares."""
    torch = _torch()
    th = torch.zeros_like(amp) if theta is None else theta
    with torch.no_grad():
        u2 = plan.forward(torch.polar(amp.to(torch.float32), th.to(torch.float32)).contiguous())
        e = float((u2.real.double() ** 2 + u2.imag.double() ** 2).sum())
    t = target.double()
    return t * (e / float(t.sum()))


def phase_descent(plan, amp, target, steps=50, lr=0.05, theta0=None, callback=None):
    """Adam on the source phase theta for ``intensity_loss`` against ``target`` as given
    (in units of |u2|^2: an intensity the forward method produced, or a target scaled
    once with ``energy_matched``), from theta0 (default zero phase).  Returns
    (theta, losses); descents from different starts against the same target are
    comparable loss for loss."""
    torch = _torch()
    theta = (torch.zeros_like(amp, dtype=torch.float64) if theta0 is None
             else theta0.detach().to(torch.float64).clone())
    target = target.double()
    theta.requires_grad_(True)
    opt = torch.optim.Adam([theta], lr=lr)
    losses = []
    for it in range(steps):
        opt.zero_grad(set_to_none=True)
        loss = intensity_loss(plan, theta, amp, target)
        loss.backward()
        opt.step()
        losses.append(float(loss.detach()))
        if callback is not None:
            callback(it, losses[-1])
    return theta.detach(), losses
