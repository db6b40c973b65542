"""Names of the GPU kernels that a call launches, for tests of which kernel a shape takes."""
import ctypes as C
import re

import torch


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNode(C.Structure):                            # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p), ("lds", C.c_uint32)]


def _runtime():
    """The HIP runtime of this process (not another copy of it)."""
    with open("/proc/self/maps") as f:
        hip = C.CDLL(next(line.split()[-1] for line in f if "libamdhip64.so" in line))
    hip.hipKernelNameRefByPtr.restype = C.c_char_p
    return hip


def kernels_of(call):
    """`call` runs once on the current stream, then its launches on a stream of their own are recorded into a graph, whose nodes
    name them; the graph is not run."""
    call()
    torch.cuda.synchronize()
    hip, stream, graph, n = _runtime(), torch.cuda.Stream(), C.c_void_p(), C.c_size_t()
    on = C.c_void_p(stream.cuda_stream)
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(on, 2) == 0       # relaxed: other threads may allocate meanwhile
        try:
            call()
        finally:
            assert hip.hipStreamEndCapture(on, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    names = []
    for node in nodes:
        kind, params = C.c_int(), _KernelNode()
        assert hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0
        if kind.value == 0:                                # a kernel
            assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(params)) == 0
            names.append(hip.hipKernelNameRefByPtr(C.c_void_p(params.func), on).decode())
    assert hip.hipGraphDestroy(graph) == 0
    return names


def layer_kernels(cas, cfg, weights, hidden, assignment, mask_kind=None, positions=None, fused_qkv=False):
    """Kernels of one layer on numpy inputs; fused_qkv as in layer_forward_numpy."""
    plan = cas.cascade_plan_create(cfg.batch, cfg.seq_len, cfg.n_shards, assignment, positions,
                                   cas.MASK_CAUSAL if mask_kind is None else mask_kind)
    desc = cas.make_layer_desc(cfg)
    t = {k: cas.to_device(v, cfg.dtype) for k, v in weights.items()}
    for names in (("wq", "wk", "wv"), ("bq", "bk", "bv")) if fused_qkv else ():
        if names[0] in t:
            parts = torch.cat([t[n] for n in names]).split([len(t[n]) for n in names])
            t.update(zip(names, parts))
    h = cas.to_device(hidden, cfg.dtype)
    out, w = torch.empty_like(h), cas.make_layer_weights(t)
    ws = cas.new_workspace(cas.cascade_layer_workspace_bytes(plan, desc))
    return kernels_of(lambda: cas.cascade_layer_forward(plan, desc, w, h, out, ws))


def gemm_tiles(names):
    """Rows and columns of the tiles of the MFMA GEMMs among `names`."""
    found = (re.search(r"gemm[23]_kernelILi(\d+)ELi(\d+)E", n) for n in names)
    return [(int(m[1]), int(m[2])) for m in found if m]


def split_tiles(names):
    """Tiles of the reductions in parts: of the GEMMs in front of the kernels that add the planes."""
    return [tile for i, n in enumerate(names) if "splitk_" in n for tile in gemm_tiles(names[i - 1:i])]
