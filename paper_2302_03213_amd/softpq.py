"""Soft-PQ training operator (arXiv 2302.03213, Sec. 3): a torch.autograd wrapper around the C ABI.

Forward: the hard operator (arg-min encoding + table lookup, lutnn_build_table + lutnn_linear),
with the table quantised as in inference when `table_dtype` is TABLE_I8 / TABLE_I4 (Sec. 3.3: the
forward pass of training uses the quantised table).  Backward: the gradient of the soft output of
Eq. 5-6 (lutnn_softpq_backward) for the centroids, the temperature and the layer input; the weights
W are fixed, as in the paper.  The product Z = dL/dY @ W^T is lutnn_linear_gradient's, or torch's where that is faster.
"""
import torch

from . import binding as _b


class _HostTemperature:
    """The temperature's value for the backward pass, which the C ABI takes by value.  The copy to the host starts in
    the forward pass, ahead of its kernels: when the backward pass asks for the value it has long arrived, instead of
    being waited for behind everything that the stream has been given by then."""

    def __init__(self, temperature):
        self.event = None
        self.value = temperature.detach()
        if temperature.is_cuda:
            with torch.cuda.device(temperature.device):  # whose stream the copy runs on, and the event after it
                if not torch.cuda.is_current_stream_capturing():
                    self.value = torch.empty(temperature.shape, dtype=temperature.dtype, pin_memory=True)
                    self.value.copy_(temperature.detach(), non_blocking=True)
                    self.event = torch.cuda.Event()
                    self.event.record()

    def get(self):
        if self.event is not None:
            if torch.cuda.is_current_stream_capturing():  # replays would keep the value of this pass
                raise RuntimeError("a soft-PQ backward pass cannot be captured: the temperature is read on the host")
            self.event.synchronize()
        return float(self.value)


def _host_temperature(*inputs):
    """For a call whose backward pass may follow, before autograd.Function.forward hides the grad mode."""
    if torch.is_grad_enabled() and any(t is not None and t.requires_grad for t in inputs):
        return _HostTemperature(inputs[2])
    return None


class _SoftPQLinearFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, X, centroids, temperature, W, bias, table_dtype, host_temperature):
        ctx.temperature = host_temperature
        layer = _b.build_table(centroids.detach(), W, table_dtype, bias=bias)
        Y = _b.linear(layer, X)
        ctx.save_for_backward(X, centroids, temperature, W)
        ctx.has_bias = bias is not None
        ctx.table_dtype = table_dtype
        return Y

    @staticmethod
    def backward(ctx, G):
        X, centroids, temperature, W = ctx.saved_tensors
        G = G.contiguous()
        # input gradient of the ordinary linear layer
        Z = _b._input_gradient(G, W)
        dP, dX, dt = _b._softpq_gradients(centroids, W.shape[1], ctx.temperature.get(), X, Z, ctx.needs_input_grad[0])
        dbias = _b._bias_gradient(G) if ctx.has_bias and ctx.needs_input_grad[4] else None
        return dX, dP, dt.reshape(temperature.shape), None, dbias, None, None


class SoftPQLinear(torch.nn.Module):
    """A linear layer replaced by table lookup, in training form: learnable centroids [C, K, V] and
    temperature (Sec. 3.2), fixed weights W [D, M] and optional bias."""

    def __init__(self, centroids, W, bias=None, temperature=1.0, table_dtype=_b.TABLE_I8):
        super().__init__()
        self.centroids = torch.nn.Parameter(centroids.clone())
        self.temperature = torch.nn.Parameter(torch.tensor(float(temperature), device=centroids.device))
        self.register_buffer("W", W.clone())
        self.bias = None if bias is None else torch.nn.Parameter(bias.clone())
        self.table_dtype = table_dtype

    def forward(self, X):
        return _SoftPQLinearFn.apply(X, self.centroids, self.temperature, self.W, self.bias, self.table_dtype,
                                     _host_temperature(X, self.centroids, self.temperature, self.W, self.bias))


class _SoftPQConv2dFn(torch.autograd.Function):
    """The same operator for a convolution (Sec. 4: a convolution is the linear operator on the rows
    of its im2col matrix).  Forward (lutnn_conv2d) and backward (lutnn_softpq_backward_conv2d) read the
    NCHW batch directly; nothing is unfolded, transposed or copied around them."""

    @staticmethod
    def forward(ctx, inp, centroids, temperature, W, bias, table_dtype, kernel, stride, pad, host_temperature):
        ctx.temperature = host_temperature
        layer = _b.build_table(centroids.detach(), W, table_dtype, bias=bias)
        B, _, H, Wd = inp.shape
        Y = _b.conv2d(layer, inp.contiguous(), kernel, stride, pad)  # [B*Ho*Wo, M]
        (kh, kw), (sh, sw), (ph, pw) = _b._pair(kernel), _b._pair(stride), _b._pair(pad)
        Ho, Wo = (H + 2 * ph - kh) // sh + 1, (Wd + 2 * pw - kw) // sw + 1
        ctx.save_for_backward(inp, centroids, temperature, W)
        ctx.has_bias = bias is not None
        ctx.conv = (kernel, stride, pad)
        return Y.view(B, Ho, Wo, -1).permute(0, 3, 1, 2)  # NCHW view of the row-major output

    @staticmethod
    def backward(ctx, G):
        inp, centroids, temperature, W = ctx.saved_tensors
        kernel, stride, pad = ctx.conv
        G = G.contiguous()
        dP, dinp, dt = _b._softpq_gradients_conv2d(centroids, ctx.temperature.get(), inp, W, G, kernel, stride, pad,
                                                   ctx.needs_input_grad[0])
        dbias = _b._bias_gradient(G) if ctx.has_bias and ctx.needs_input_grad[4] else None
        return dinp, dP, dt.reshape(temperature.shape), None, dbias, None, None, None, None, None


class SoftPQConv2d(torch.nn.Module):
    """A convolution replaced by table lookup, in training form.  W is the convolution's weight as the
    matrix [Cin*kh*kw, Cout] (rows ordered (ci, r, s)); sub-vector c covers columns [c*V, (c+1)*V)."""

    def __init__(self, centroids, W, kernel, stride=1, pad=0, bias=None, temperature=1.0,
                 table_dtype=_b.TABLE_I8):
        super().__init__()
        self.centroids = torch.nn.Parameter(centroids.clone())
        self.temperature = torch.nn.Parameter(torch.tensor(float(temperature), device=centroids.device))
        self.register_buffer("W", W.clone())
        self.bias = None if bias is None else torch.nn.Parameter(bias.clone())
        self.kernel, self.stride, self.pad = kernel, stride, pad
        self.table_dtype = table_dtype

    def forward(self, inp):
        return _SoftPQConv2dFn.apply(inp, self.centroids, self.temperature, self.W, self.bias,
                                     self.table_dtype, self.kernel, self.stride, self.pad,
                                     _host_temperature(inp, self.centroids, self.temperature, self.W, self.bias))
