"""Binding over the C ABI in include/cnn.h (same names, argument marshalling only).

PyTorch supplies device memory (tensors) and the stream handle; every step of
the computation runs inside the library's HIP kernels.  The built library must
be present (python -m paper_1912_05234_amd.build): there is no fallback path.
The calls that a program repeats go through the extension module built from
csrc/torch_calls.cpp (5 us a call instead of 10), the others through ctypes.
"""
import ctypes
import importlib.util
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libcnn_mi355x.so")
CALLS_PATH = os.path.join(_PKG, "_calls.so")

NPARAM = 3898
PARAM_SHAPES = (("k1", (6, 5, 5)), ("b1", (6,)), ("k2", (12, 6, 5, 5)), ("b2", (12,)),
                ("fc", (10, 12, 1, 4, 4)), ("b", (10,)))

_vp, _i, _f, _sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t

# name -> (restype, argtypes); one entry per declaration in include/cnn.h
SIGNATURES = {
    "cnn_strerror": (ctypes.c_char_p, [_i]),
    "cnn_workspace_bytes": (_sz, [_i]),
    "cnn_init": (_i, [ctypes.POINTER(_vp), _vp, _sz, _i, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "cnn_destroy": (None, [_vp]),
    "cnn_get_weights": (_i, [_vp] * 7),
    "cnn_set_weights": (_i, [_vp] * 7),
    "cnn_forward": (_i, [_vp, _vp, _i, _vp]),
    "cnn_forward_activations": (_i, [_vp, _vp, _i, _vp, _vp, _vp, _vp, _vp]),
    "cnn_gradient": (_i, [_vp, _vp, _vp, _i, _vp, _vp]),
    "cnn_train_batch": (_i, [_vp, _vp, _vp, _i, _f, _vp]),
    "cnn_train_epoch": (_i, [_vp, _vp, _vp, _i, _i, _f, _vp]),
    "cnn_epoch_mode": (_i, [_vp, _i, ctypes.c_double, _i]),
    "cnn_epoch_status": (_i, [_vp]),
    "cnn_evaluate": (_i, [_vp, _vp, _vp, _i, _vp, _vp]),
    "cnn_profile_begin": (_i, [_vp, _i]),
    "cnn_profile_read": (_i, [_vp, _vp, _i, ctypes.POINTER(_i)]),
    "cnn_conv_fwd": (_i, [_vp, _vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_conv_bwd_input": (_i, [_vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_conv_fwd_valu": (_i, [_vp, _vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_conv_bwd_input_valu": (_i, [_vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_conv_fwd_bf16": (_i, [_vp, _vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_conv_bwd_input_bf16": (_i, [_vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_conv_bwd_weight_workspace_bytes": (_sz, [_i] * 7),
    "cnn_conv_bwd_weight_bf16_workspace_bytes": (_sz, [_i] * 7),
    "cnn_conv_bwd_weight_bf16": (_i, [_vp, _vp, _vp, _vp] + [_i] * 7 + [_vp, _sz, _vp]),
    "cnn_conv_bwd_weight": (_i, [_vp, _vp, _vp, _vp] + [_i] * 7 + [_vp, _sz, _vp]),
    "cnn_conv_bwd_weight_static": (_i, [_vp, _vp, _vp, _vp] + [_i] * 7 + [_vp]),
    "cnn_avgpool_fwd": (_i, [_vp, _vp, _i, _i, _i, _i, _vp]),
    "cnn_avgpool_bwd": (_i, [_vp, _vp, _i, _i, _i, _i, _vp]),
    "cnn_fc_fwd": (_i, [_vp, _vp, _vp, _vp, _i, _i, _i, _vp]),
    "cnn_fc_bwd_input": (_i, [_vp, _vp, _vp, _i, _i, _i, _vp]),
    "cnn_fc_bwd_weight_workspace_bytes": (_sz, [_i] * 3),
    "cnn_fc_bwd_weight": (_i, [_vp, _vp, _vp, _vp, _i, _i, _i, _vp, _sz, _vp]),
    "cnn_logistic_fwd": (_i, [_vp, _vp, _sz, _vp]),
    "cnn_logistic_bwd": (_i, [_vp, _vp, _vp, _sz, _vp]),
}

_lib = None
_calls = None


class CnnError(RuntimeError):
    def __init__(self, code, where):
        self.code = code
        msg = lib().cnn_strerror(code).decode()
        super().__init__("%s failed: %s (code %d)" % (where, msg, code))


def lib():
    """The loaded shared library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError("%s is missing: build it with `python -m paper_1912_05234_amd.build`; "
                               "there is no fallback implementation" % LIB_PATH)
        handle = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(handle, name)
            fn.restype, fn.argtypes = res, args
        _lib = handle
    return _lib


def _native():
    """The extension module over the same library; raises if it has not been built."""
    global _calls
    if _calls is None:
        lib()
        if not os.path.exists(CALLS_PATH):
            raise RuntimeError("%s is missing: build it with `python -m paper_1912_05234_amd.build`" % CALLS_PATH)
        spec = importlib.util.spec_from_file_location("_calls", CALLS_PATH)
        module = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(module)
        module.raise_through(_check)
        _calls = module
    return _calls


def _check(code, where):
    if code != 0:
        raise CnnError(code, where)


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _dev(t, dtype=torch.float32):
    if t is None:
        return None
    if not t.is_cuda or t.dtype != dtype or not t.is_contiguous():
        raise ValueError("expected a contiguous %s tensor on the GPU" % dtype)
    return t


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


class CNN:
    """Owns a library context plus the device workspace it lives in."""

    def __init__(self, weights, max_batch, device="cuda:0"):
        self.device = torch.device(device)
        self._index = -1 if self.device.index is None else self.device.index  # -1: the current one
        self.max_batch = int(max_batch)
        L = lib()
        nbytes = L.cnn_workspace_bytes(self.max_batch)
        self.workspace = torch.empty(nbytes, dtype=torch.uint8, device=self.device)
        w = {k: _dev(torch.as_tensor(v, dtype=torch.float32).contiguous().to(self.device))
             for k, v in weights.items()}
        self._ctx = ctypes.c_void_p()
        with torch.cuda.device(self.device):
            self._stream_obj = torch.cuda.current_stream()
            _check(L.cnn_init(ctypes.byref(self._ctx), _ptr(self.workspace), nbytes, self.max_batch,
                              *[_ptr(w.get(n)) for n, _ in PARAM_SHAPES], _stream()), "cnn_init")
            torch.cuda.current_stream().synchronize()  # the staging copies of `w` may now be freed

    def close(self):
        if self._ctx:
            lib().cnn_destroy(self._ctx)
            self._ctx = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def get_weights(self):
        out = {n: torch.empty(s, dtype=torch.float32, device=self.device) for n, s in PARAM_SHAPES}
        _check(lib().cnn_get_weights(self._ctx, *[_ptr(out[n]) for n, _ in PARAM_SHAPES]), "cnn_get_weights")
        return out

    def get_weights_flat(self):
        w = self.get_weights()
        return torch.cat([w[n].reshape(-1) for n, _ in PARAM_SHAPES])

    def set_weights(self, weights):
        w = {k: _dev(torch.as_tensor(v, dtype=torch.float32).contiguous().to(self.device))
             for k, v in weights.items()}
        _check(lib().cnn_set_weights(self._ctx, *[_ptr(w.get(n)) for n, _ in PARAM_SHAPES]), "cnn_set_weights")
        self._stream_obj.synchronize()

    def forward(self, images, yhat=None):
        return (_calls or _native()).forward(self._ctx.value, images, yhat, self._index)

    def forward_activations(self, images):
        images = _dev(images)
        B = images.shape[0]
        mk = lambda *s: torch.empty((B,) + s, dtype=torch.float32, device=self.device)
        a = {"c1": mk(6, 24, 24), "s1": mk(6, 12, 12), "c2": mk(12, 8, 8), "s2": mk(12, 4, 4), "y": mk(10)}
        _check(lib().cnn_forward_activations(self._ctx, _ptr(images), B, _ptr(a["c1"]), _ptr(a["s1"]),
                                             _ptr(a["c2"]), _ptr(a["s2"]), _ptr(a["y"])),
               "cnn_forward_activations")
        return a

    def gradient(self, images, labels):
        return (_calls or _native()).gradient(self._ctx.value, images, labels, self._index)

    def train_batch(self, images, labels, lr, loss_sum=None):
        return (_calls or _native()).train_batch(self._ctx.value, images, labels, lr, loss_sum)

    def train_epoch(self, images, labels, batch, lr, loss_sums=None):
        """One pass over `images` in consecutive batches of `batch` (the last may be shorter)."""
        images, labels = _dev(images), _dev(labels, torch.int32)
        if loss_sums is not None and loss_sums.numel() < -(-images.shape[0] // int(batch)):
            raise ValueError("loss_sums needs one float per step")
        _check(lib().cnn_train_epoch(self._ctx, _ptr(images), _ptr(labels), images.shape[0], int(batch),
                                     float(lr), _ptr(_dev(loss_sums))), "cnn_train_epoch")
        return loss_sums

    def epoch_mode(self, device_loop, wait_seconds=1.0, never_arrives=False):
        _check(lib().cnn_epoch_mode(self._ctx, int(device_loop), float(wait_seconds), int(never_arrives)),
               "cnn_epoch_mode")

    def epoch_status(self):
        """Waits for the stream; 0, or the (negative) code of a device-side loop that gave up."""
        return lib().cnn_epoch_status(self._ctx)

    def evaluate(self, images, labels):
        return (_calls or _native()).evaluate(self._ctx.value, images, labels, self._index)

    def profile_begin(self, capacity):
        _check(lib().cnn_profile_begin(self._ctx, int(capacity)), "cnn_profile_begin")

    def profile_read(self, capacity):
        """Per-step milliseconds of the fused forward+backward kernel (host list)."""
        buf = (ctypes.c_float * max(1, capacity))()
        n = ctypes.c_int(0)
        _check(lib().cnn_profile_read(self._ctx, ctypes.cast(buf, _vp), int(capacity), ctypes.byref(n)),
               "cnn_profile_read")
        return [buf[i] for i in range(n.value)]


# ---- per-operation entry points -------------------------------------------------
def conv_fwd(inp, k, bias=None, bf16=False, valu=False):
    return (_calls or _native()).conv_fwd(inp, k, bias, 1 if bf16 else 2 if valu else 0)


def conv_bwd_input(d_out, k, H, W, bf16=False, valu=False):
    return (_calls or _native()).conv_bwd_input(d_out, k, H, W, 1 if bf16 else 2 if valu else 0)


def conv_bwd_weight(inp, d_out, want_bias=True, workspace=True, bf16=False):
    """workspace=False passes none, which selects the kernel that needs no partial sums."""
    return (_calls or _native()).conv_bwd_weight(inp, d_out, bool(want_bias), bool(workspace), bool(bf16))


def conv_bwd_weight_static(inp, d_out, d_k, d_b=None):
    """cnn_conv_bwd_weight_static into the caller's d_k / d_b (this wrapper allocates nothing either)."""
    inp, d_out, d_k, d_b = _dev(inp), _dev(d_out), _dev(d_k), _dev(d_b)
    B, Cin, H, W = inp.shape
    Cout, Ho, Wo = d_out.shape[1:]
    KH, KW = H - Ho + 1, W - Wo + 1
    _check(lib().cnn_conv_bwd_weight_static(_ptr(inp), _ptr(d_out), _ptr(d_k), _ptr(d_b), B, Cin, H, W, Cout,
                                            KH, KW, _stream()), "cnn_conv_bwd_weight_static")
    return d_k, d_b


def avgpool_fwd(inp):
    return (_calls or _native()).avgpool_fwd(inp)


def avgpool_bwd(d_out):
    return (_calls or _native()).avgpool_bwd(d_out)


def fc_fwd(inp, w, bias=None):
    return (_calls or _native()).fc_fwd(inp, w, bias)


def fc_bwd_input(d_out, w):
    return (_calls or _native()).fc_bwd_input(d_out, w)


def fc_bwd_weight(inp, d_out, want_bias=True, workspace=True):
    return (_calls or _native()).fc_bwd_weight(inp, d_out, bool(want_bias), bool(workspace))


def logistic_fwd(x):
    return (_calls or _native()).logistic_fwd(x)


def logistic_bwd(y, d_y):
    return (_calls or _native()).logistic_bwd(y, d_y)
