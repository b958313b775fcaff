"""The functions of the extension module `_wush_call` through ctypes: the same arguments, the same C calls, the same
status codes.  binding.py takes them where the module was not built for the running Python (it needs that Python's headers and
a host compiler); the marshalling of a call then costs some 4 us more."""
from __future__ import annotations

from . import binding as b


def _fmt(fmt, layout):
    return fmt or b.default_fmt(layout=layout)


def _k(K, codes):
    return 2 * codes.shape[-1] if K is None else K


def quantize_act(X, T_blocks, Xq, Xs, fmt, dbg_Yt, stream):
    M, K = X.shape
    return b.lib().wush_quantize_act(b._ptr(X), M, K, X.stride(0), b._ptr(T_blocks), _fmt(fmt, b.WUSH_LAYOUT_CANONICAL),
                                     b._ptr(Xq), b._ptr(Xs), b._ptr(dbg_Yt), b._stream(stream))


def linear(Xq, Xs, Wq, Ws, Y, fmt, stream, K):
    M, N = Y.shape
    return b.lib().wush_linear(b._ptr(Xq), b._ptr(Xs), b._ptr(Wq), b._ptr(Ws), M, N, _k(K, Xq),
                               _fmt(fmt, b.WUSH_LAYOUT_CANONICAL), b._ptr(Y), Y.stride(0), b._stream(stream))


def layer_decode(X, T_blocks, Wq, Ws, Y, workspace, fmt, stream):
    M, K = X.shape
    return b.lib().wush_layer_decode(b._ptr(X), M, K, X.stride(0), b._ptr(T_blocks), b._ptr(Wq), b._ptr(Ws), Y.shape[1],
                                     _fmt(fmt, b.WUSH_LAYOUT_TILED), b._ptr(Y), Y.stride(0), b._ptr(workspace),
                                     b._nbytes(workspace), b._stream(stream))


def layer_decode_static(X, T_blocks, Wq, Ws, Y, fmt, stream):
    M, K = X.shape
    return b.lib().wush_layer_decode_static(b._ptr(X), M, K, X.stride(0), b._ptr(T_blocks), b._ptr(Wq), b._ptr(Ws),
                                            Y.shape[1], _fmt(fmt, b.WUSH_LAYOUT_TILED), b._ptr(Y), Y.stride(0),
                                            b._stream(stream))


def quantize_act_nvfp4(X, T16, tensor_scale, Xq, Xs, layout, dbg_Yt, stream):
    M, K = X.shape
    return b.lib().wush_quantize_act_nvfp4(b._ptr(X), M, K, X.stride(0), b._ptr(T16), b._ptr(tensor_scale), layout,
                                           b._ptr(Xq), b._ptr(Xs), b._ptr(dbg_Yt), b._stream(stream))


def linear_nvfp4(Xq, Xs, tsx, Wq, Ws, tsw, Y, layout, out_dtype, stream, K):
    M, N = Y.shape
    return b.lib().wush_linear_nvfp4(b._ptr(Xq), b._ptr(Xs), b._ptr(tsx), b._ptr(Wq), b._ptr(Ws), b._ptr(tsw), M, N,
                                     _k(K, Xq), layout, out_dtype, b._ptr(Y), Y.stride(0), b._stream(stream))


def quantize_act_int4(X, T_blocks, Xq, Xs, layout, dbg_Yt, stream):
    M, K = X.shape
    return b.lib().wush_quantize_act_int4(b._ptr(X), M, K, X.stride(0), b._ptr(T_blocks), layout, b._ptr(Xq), b._ptr(Xs),
                                          b._ptr(dbg_Yt), b._stream(stream))


def linear_int4(Xq, Xs, Wq, Ws, Y, layout, out_dtype, stream, K):
    M, N = Y.shape
    return b.lib().wush_linear_int4(b._ptr(Xq), b._ptr(Xs), b._ptr(Wq), b._ptr(Ws), M, N, _k(K, Xq), layout, out_dtype,
                                    b._ptr(Y), Y.stride(0), b._stream(stream))
