"""PyTorch autograd over the C ABI (Section 1 states that the paper's library takes part in PyTorch's automatic
differentiation): thin ``torch.autograd.Function`` wrappers whose forward is ``sigkernel_fwd`` /
``sigkernel_gram`` and whose backward is ``sigkernel_bwd`` / ``sigkernel_gram`` with the upstream gradient
(Section 3.4: exact gradients of the discrete scheme).  Argument marshalling only; no arithmetic of the
method happens here.

    k = sig_kernel(x, y, lam1, lam2, flags)          # x[B,L1,d], y[B,L2,d] -> k[B]
    K = sig_kernel_gram(X, Y, lam1, lam2, flags)     # X[N,L1,d], Y[M,L2,d] -> K[N,M]
    K = sig_kernel_gram(X, None, lam1, lam2, flags)  # symmetric case K(X, X)
    loss = sig_mmd2(X, Y, lam1, lam2, flags)         # squared MMD between two sets of paths, one library call
    S = signature(x, N, flags)                       # x[B,L,d] -> truncated signatures [B, entries] (Section 2)

A time grid of the caller's own (Section 4 defines the time-augmented path as (x_{t_i}, t_i) and fixes no grid; the
library's flag takes t_i = i/(L-1)) is an ordinary channel: ``with_times(x, t)`` appends it, and the wrappers below take
``times=`` / ``times_x=, times_y=`` and do that for the caller.

The gradients are first-order only (the backward pass is not itself differentiable).

A forward call on inputs that require gradients keeps what it sweeps for its backward call where the launch mode has such a
form, and for few pairs also makes the adjoint sweep, beside its own.  It does so whether or not a backward call follows:
evaluate under ``torch.no_grad()``.  Under saved-tensor hooks (checkpoints, ``save_on_cpu``) it keeps nothing.

Each call goes to the same wrapper in native code first (csrc/sk_torch.cpp: the same library calls as nodes of PyTorch's
graph; the classes below cost a short training pass 20 to 90 us of host time).  It leaves to the classes what is not the
ordinary case: tracers and function transforms, forward gradients, kept workspaces above _KEEP_LIMIT, and everything that
is an error.
"""
import threading
import weakref

import torch

from . import binding as sk

sk.load()
from . import _native  # noqa: E402  (needs the library, and raises if it has not been built)


# Bytes of workspace a forward call may hold on to for its backward call, as long as its graph lives.  A sweep that takes
# more is kept while all such sweeps of the live graphs together take at most _KEEP_LARGE bytes on their device, and its
# workspace is given back by the first backward call.  Training steps without and with it: 32 pairs of 2048 points, order 2
# (1.6 GiB) 6.54 and 5.20 ms; lead-lag Grams of 128 x 128 paths of 101 points, d = 4 (1.5 GiB) 1.77 and 1.61 ms, K(X, X) of the
# same 0.99 and 0.92 ms.
# Smaller ones of the native calls come to at most _KEEP_ALL together, an eighth of a device's memory: a program that holds
# thousands of graphs before it calls backward would otherwise run out of memory for workspaces it can do without.
_KEEP_LIMIT = 1 << 30
_KEEP_LARGE = 1 << 32
_KEEP_ALL = 36 << 30

_large_lock = threading.RLock()   # (taken again if a tensor is collected while it is held)
_large_held = {}                  # device: bytes of the live workspaces above _KEEP_LIMIT


def _give_back(device, nbytes):
    with _large_lock:
        _large_held[device] -= nbytes


def _keep_workspace(nbytes, device):
    """A workspace of `nbytes` to keep for the backward call, or None: it exceeds what may be kept, or the device has no room
    for it (the calls go on without one)."""
    nbytes = max(int(nbytes), 256)
    if nbytes <= _KEEP_LIMIT:
        try:
            return torch.empty(nbytes, dtype=torch.uint8, device=device)
        except torch.OutOfMemoryError:
            return None
    key = str(device)
    with _large_lock:
        if _large_held.get(key, 0) + nbytes > _KEEP_LARGE:
            return None
        _large_held[key] = _large_held.get(key, 0) + nbytes
    try:
        ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    except torch.OutOfMemoryError:
        _give_back(key, nbytes)
        return None
    weakref.finalize(ws, _give_back, key, nbytes).atexit = False
    return ws


def _kept(ctx, x, y, lam1, lam2, flags, gram=False, symmetric=False):
    """A workspace of this call's own if it wants gradients, the launch mode hands what it sweeps to the backward call (the grid
    the paper's backward pass takes over from its forward pass, here as checkpoints), and that much may be kept; else None.
    ctx.kept: the flags of that form, forward and backward."""
    ctx.at = (x.data_ptr(), y.data_ptr())
    # (through saved-tensor hooks, checkpoints among them, the backward call may get other paths)
    if not any(ctx.needs_input_grad[:1 if symmetric else 2]) or _native.saving_through_hooks():
        return None
    N, L1, d = x.shape
    M, L2 = y.shape[:2]
    try:
        nbytes, *ctx.kept = _native.kept_form(gram, symmetric, N, M if gram else 0, L1, L2, d, lam1, lam2, flags, sk._dt(x))
    except TypeError:       # (orders or flags that are no integers: the call itself says so)
        return None
    return _keep_workspace(nbytes, x.device) if nbytes else None


def _take_workspace(ctx, x, y):
    """The workspace the forward call kept, or None.  A large one is taken out of the graph: a further backward call through
    it sweeps forward itself.  A call whose saved paths lie elsewhere than the forward call's (their data have been set) goes
    without: the library would take the sweeps for another call's."""
    ws = ctx.ws
    if ws is None:
        return None
    if ws.numel() > _KEEP_LIMIT:
        ctx.ws = None
    return ws if ctx.at == (x.data_ptr(), y.data_ptr()) else None


class _PairKernel(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, y, lam1, lam2, flags):
        x = x.contiguous()
        y = y.contiguous()
        ctx.save_for_backward(x, y)
        ctx.args = (lam1, lam2, flags)
        ctx.ws = _kept(ctx, x, y, lam1, lam2, flags)
        if ctx.ws is not None:
            return sk.sigkernel_fwd(x, y, lam1, lam2, flags | ctx.kept[0], ws=ctx.ws)
        return sk.sigkernel_fwd(x, y, lam1, lam2, flags)

    @staticmethod
    def backward(ctx, grad_k):
        x, y = ctx.saved_tensors
        lam1, lam2, flags = ctx.args
        want_x, want_y = ctx.needs_input_grad[0], ctx.needs_input_grad[1]
        if not (want_x or want_y):
            return None, None, None, None, None
        ws = _take_workspace(ctx, x, y)
        if ws is not None:
            _, gx, gy = sk.sigkernel_bwd(x, y, grad_k.contiguous(), lam1, lam2, flags | ctx.kept[1],
                                         want_x=want_x, want_y=want_y, ws=ws)
        else:
            _, gx, gy = sk.sigkernel_bwd(x, y, grad_k.contiguous(), lam1, lam2, flags, want_x=want_x, want_y=want_y)
        return gx, gy, None, None, None


class _GramKernel(torch.autograd.Function):
    @staticmethod
    def forward(ctx, X, Y, lam1, lam2, flags):
        X = X.contiguous()
        Y = Y.contiguous()
        ctx.save_for_backward(X, Y)
        ctx.args = (lam1, lam2, flags)
        ctx.ws = _kept(ctx, X, Y, lam1, lam2, flags, gram=True)
        if ctx.ws is not None:
            return sk.sigkernel_gram(X, Y, None, lam1, lam2, flags | ctx.kept[0], ws=ctx.ws)
        return sk.sigkernel_gram(X, Y, None, lam1, lam2, flags)

    @staticmethod
    def backward(ctx, grad_K):
        X, Y = ctx.saved_tensors
        lam1, lam2, flags = ctx.args
        ws = _take_workspace(ctx, X, Y)
        if ws is not None:
            _, gX, gY = sk.sigkernel_gram(X, Y, grad_K.contiguous(), lam1, lam2, flags | ctx.kept[1], ws=ws)
        else:
            _, gX, gY = sk.sigkernel_gram(X, Y, grad_K.contiguous(), lam1, lam2, flags)
        return (gX if ctx.needs_input_grad[0] else None), (gY if ctx.needs_input_grad[1] else None), None, None, None


class _GramKernelSym(torch.autograd.Function):
    @staticmethod
    def forward(ctx, X, lam1, lam2, flags):
        X = X.contiguous()
        ctx.save_for_backward(X)
        ctx.args = (lam1, lam2, flags)
        ctx.ws = _kept(ctx, X, X, lam1, lam2, flags, gram=True, symmetric=True)
        if ctx.ws is not None:
            return sk.sigkernel_gram(X, X, None, lam1, lam2, flags | ctx.kept[0], ws=ctx.ws)
        return sk.sigkernel_gram(X, X, None, lam1, lam2, flags)

    @staticmethod
    def backward(ctx, grad_K):
        (X,) = ctx.saved_tensors
        lam1, lam2, flags = ctx.args
        ws = _take_workspace(ctx, X, X)
        keep = ctx.kept[1] if ws is not None else 0
        _, gX, _ = sk.sigkernel_gram(X, X, grad_K.contiguous(), lam1, lam2, flags | keep, ws=ws)   # total derivative
        return gX, None, None, None


class _Mmd2(torch.autograd.Function):
    @staticmethod
    def forward(ctx, X, Y, lam1, lam2, flags):
        X = X.contiguous()
        Y = Y.contiguous()
        want_x, want_y = ctx.needs_input_grad[0], ctx.needs_input_grad[1]
        loss, gX, gY = sk.sigkernel_mmd2(X, Y, lam1, lam2, flags, want_x=want_x, want_y=want_y)
        ctx.save_for_backward(*[g for g in (gX, gY) if g is not None])
        ctx.have = (gX is not None, gY is not None)
        return loss[0]

    @staticmethod
    def backward(ctx, grad_loss):
        saved = list(ctx.saved_tensors)
        gX = saved.pop(0) if ctx.have[0] else None
        gY = saved.pop(0) if ctx.have[1] else None
        return (None if gX is None else gX * grad_loss), (None if gY is None else gY * grad_loss), None, None, None


class _Signature(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, N, flags):
        x = x.contiguous()
        out = sk.signature_fwd(x, N, flags)
        ctx.save_for_backward(x, out)
        ctx.args = (N, flags)
        return out

    @staticmethod
    def backward(ctx, grad_out):
        x, out = ctx.saved_tensors
        N, flags = ctx.args
        return sk.signature_bwd(x, grad_out.contiguous(), N, flags, sig=out), None, None


def signature(x, N, flags=0, times=None):
    """Truncated signatures of device paths x[B,L,d] up to level N, levels 0..N flattened (signature_fwd);
    differentiable in x (signature_bwd, handed the signatures of the forward call).  times: a time grid of the
    caller's own, appended as the last channel."""
    if times is not None:
        x = with_times(x, times)
    out = _native.signature(x, N, flags)
    return _Signature.apply(x, N, flags) if out is None else out


def with_times(x, t):
    """x[..., L, d] with the channel t appended: t[L] (one grid for every path) or t[..., L]."""
    t = torch.as_tensor(t, dtype=x.dtype, device=x.device)
    t = t.expand(x.shape[:-1]) if t.dim() == 1 else t
    return torch.cat([x, t.unsqueeze(-1)], dim=-1)


def sig_mmd2(X, Y, lam1=0, lam2=0, flags=0):
    """mean K(X,X) - 2 mean K(X,Y) + mean K(Y,Y) for device tensors X[N,L1,d], Y[M,L2,d] (sigkernel_mmd2: value and
    gradients in one call, the upstream weights never leave the GPU); differentiable in X and Y."""
    out = _native.mmd2(X, Y, lam1, lam2, flags)
    return _Mmd2.apply(X, Y, lam1, lam2, flags) if out is None else out


def sig_kernel(x, y, lam1=0, lam2=0, flags=0, times_x=None, times_y=None):
    """k[b] = k(x[b], y[b]) for device tensors x[B,L1,d], y[B,L2,d]; differentiable in x and y.  times_x, times_y: time
    grids of the caller's own (both or neither), appended as the last channel of each side."""
    if (times_x is None) != (times_y is None):
        raise ValueError("give time grids for both sides or for neither")
    if times_x is not None:
        x, y = with_times(x, times_x), with_times(y, times_y)
    out = _native.pair(x, y, lam1, lam2, flags, _KEEP_LIMIT, _KEEP_ALL)
    return _PairKernel.apply(x, y, lam1, lam2, flags) if out is None else out


def sig_kernel_gram(X, Y=None, lam1=0, lam2=0, flags=0, times_x=None, times_y=None):
    """K[n,m] = k(X[n], Y[m]); Y = None is the symmetric case K(X, X); differentiable in X and Y.  times_x (and times_y
    when Y is given): time grids of the caller's own, appended as the last channel."""
    if times_x is not None:
        X = with_times(X, times_x)
        if Y is not None:
            if times_y is None:
                raise ValueError("give time grids for both sides or for neither")
            Y = with_times(Y, times_y)
    elif times_y is not None:
        raise ValueError("give time grids for both sides or for neither")
    out = _native.gram(X, Y, lam1, lam2, flags, _KEEP_LIMIT, _KEEP_ALL)
    if out is not None:
        return out
    if Y is None:
        return _GramKernelSym.apply(X, lam1, lam2, flags)
    return _GramKernel.apply(X, Y, lam1, lam2, flags)
