"""Shared test plumbing: moving bf16 bit patterns between numpy and the GPU, and
the parity rule. No arithmetic of the method lives here."""
import ctypes

import numpy as np


def to_gpu(bits):
    """uint16 bf16 bit patterns -> torch.bfloat16 tensor on cuda:0 (same bits)."""
    import torch
    a = np.ascontiguousarray(bits, dtype=np.uint16)
    return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).to("cuda:0")


def to_bits(t):
    """torch.bfloat16 tensor -> uint16 bit patterns on the host."""
    import torch
    return t.detach().contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


# |gpu - ref| <= 1e-2 * |ref| + 1e-3 per element, ref the unrounded fp64 oracle
# value, gpu the bf16 output decoded exactly. bf16 rounding alone costs up to
# 2^-8 = 0.39 % relative; fp32 accumulation adds ~1e-6.
RTOL = 1e-2
ATOL = 1e-3


def assert_parity(gpu_f64, ref_f64, what):
    gpu_f64 = np.asarray(gpu_f64, dtype=np.float64)
    ref_f64 = np.asarray(ref_f64, dtype=np.float64)
    assert gpu_f64.shape == ref_f64.shape, (what, gpu_f64.shape, ref_f64.shape)
    both_nan = np.isnan(gpu_f64) & np.isnan(ref_f64)
    same_inf = np.isinf(ref_f64) & (gpu_f64 == ref_f64)
    with np.errstate(invalid="ignore"):
        err = np.abs(gpu_f64 - ref_f64)
        ok = (err <= RTOL * np.abs(ref_f64) + ATOL) | both_nan | same_inf
    if not ok.all():
        bad = np.argwhere(~ok)
        i = tuple(bad[0])
        raise AssertionError("%s: %d of %d elements out of tolerance; first at %s: gpu=%r ref=%r"
                             % (what, len(bad), ok.size, i, gpu_f64[i], ref_f64[i]))


class _KernelNode(ctypes.Structure):
    """hipKernelNodeParams"""
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def captured_grids(stream, call):
    """The workgroups of each kernel that call() launches (see captured_kernels)."""
    return [grid for _, grid in captured_kernels(stream, call)]


def captured_kernels(stream, call):
    """(function, workgroups) of each kernel that call() launches, found by capturing them (nothing runs). call()
    works on `stream` and on streams it forks from and joins into it, and allocates nothing."""
    import paper_2505_11329_amd as tw
    hip = tw.lib()      # a symbol of a library it was linked against is found through it
    handle, graph = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(handle, 1) == 0        # hipStreamCaptureModeThreadLocal
    try:
        call()
    finally:
        ended = hip.hipStreamEndCapture(handle, ctypes.byref(graph))
    assert ended == 0
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    kernels = []
    for node in nodes:
        kind, p = ctypes.c_int(-1), _KernelNode()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value == 0:     # hipGraphNodeTypeKernel
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            kernels.append((p.func, p.grid[0]))
    assert hip.hipGraphDestroy(graph) == 0
    return kernels
