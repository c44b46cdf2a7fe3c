"""Which kernel a call launches: the call is recorded into a HIP graph (nothing runs) and the graph's nodes are read."""
import ctypes

import torch

from paper_2605_26266_amd import binding as B

SIXTEEN_BIT, FP32 = 256, 512      # threads of a workgroup of the matrix-core kernels; the vector kernel has 64 or 128


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNode(ctypes.Structure):      # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3), ("params", ctypes.c_void_p),
                ("shared_bytes", ctypes.c_uint32)]


def attention_threads(cache, start, length, q, k, v, out, causal=False, correction=1, workspace=None):
    """Threads per workgroup of the first kernel of the call (its graph is never launched)."""
    hip, graph, stream = B.lib(), ctypes.c_void_p(), torch.cuda.Stream()
    handle = ctypes.c_void_p(int(stream.cuda_stream))
    heads, dim = cache.desc.num_heads, cache.desc.head_dim
    n_cur = 0 if k is None else k.shape[0]
    opts = B.kvq_attention_opts(q.shape[1] // heads, int(causal), q.stride(0), q.stride(1))
    st, sh = (k.stride(0), k.stride(1)) if n_cur else (heads * dim, dim)
    assert hip.hipStreamBeginCapture(handle, 1) == 0       # (of this thread)
    status = hip.kvq_chunk_attention_ws(
        cache.handle, start, length, q.data_ptr(), k.data_ptr() if n_cur else None, v.data_ptr() if n_cur else None, q.shape[0], n_cur,
        st, sh, 0.0, correction, ctypes.byref(opts), out.data_ptr(), None, None if workspace is None else workspace.data_ptr(),
        0 if workspace is None else workspace.numel(), handle)
    assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0 and status == B.KVQ_OK
    count = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0 and count.value >= 1
    nodes, node = (ctypes.c_void_p * count.value)(), _KernelNode()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(nodes[0]), ctypes.byref(node)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return node.block.x
