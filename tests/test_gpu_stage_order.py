"""What waits for what in a stage's backward pass: its launches are captured into a graph, which is read and never run."""
import ctypes as C
import re

import numpy as np
import pytest
import torch

from paper_2502_19913_amd import binding as sp
from paper_2502_19913_amd import synth

pytestmark = pytest.mark.gpu


class Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class KernelParams(C.Structure):
    _fields_ = [("block", Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", Dim3), ("params", C.c_void_p), ("lds", C.c_uint32)]


def captured(stream, work):
    """Kernels of `work` in the order of their launches, and for each the set of those it has to wait for."""
    hip = C.CDLL([m.split()[-1] for m in open("/proc/self/maps") if "libamdhip64" in m][0])   # the runtime in use
    hip.hipKernelNameRefByPtr.restype = C.c_char_p

    def ok(rc):
        assert rc == 0, rc
    ptr = lambda v: C.c_void_p(v)
    graph = C.c_void_p()
    ok(hip.hipStreamBeginCapture(ptr(stream.cuda_stream), C.c_int(2)))
    try:
        work()
    finally:
        ok(hip.hipStreamEndCapture(ptr(stream.cuda_stream), C.byref(graph)))
    n = C.c_size_t()
    ok(hip.hipGraphGetNodes(graph, None, C.byref(n)))
    nodes = (C.c_void_p * n.value)()
    ok(hip.hipGraphGetNodes(graph, nodes, C.byref(n)))
    m = C.c_size_t()
    ok(hip.hipGraphGetEdges(graph, None, None, C.byref(m)))
    src, dst = (C.c_void_p * m.value)(), (C.c_void_p * m.value)()
    ok(hip.hipGraphGetEdges(graph, src, dst, C.byref(m)))
    names, at = [], {v: i for i, v in enumerate(nodes)}
    for v in nodes:
        p = KernelParams()
        ok(hip.hipGraphKernelNodeGetParams(ptr(v), C.byref(p)))   # every node is a kernel
        names.append(hip.hipKernelNameRefByPtr(ptr(p.func), ptr(stream.cuda_stream)).decode())
    direct = [set() for _ in nodes]
    for a, b in zip(src, dst):
        direct[at[b]].add(at[a])
    before = []
    for i in range(len(nodes)):   # a launch comes after what it waits for
        assert all(j < i for j in direct[i])
        before.append(direct[i].union(*(before[j] for j in direct[i])))
    ok(hip.hipGraphDestroy(graph))
    return names, before


# rows, width, hidden: products one by one and, of fewer operations, in one launch a layer; few operations but large outputs
@pytest.mark.parametrize("dtype,rows,d,hidden,launches", [("bf16", 1024, 1024, 2816, 4), ("f32", 1024, 512, 1408, 4), ("bf16", 64, 256, 512, 1),
                                                          ("f32", 128, 256, 512, 1), ("bf16", 16, 4096, 11008, 4)])
def test_the_gradient_chain_waits_for_no_weight_gradient_too_early(dtype, rows, d, hidden, launches):
    """Beside the chain, weight gradients may fall a layer behind: what ends a layer (its last norm, which writes the gradient
    of the layer below over what the layer above had for its own) waits for the layers two and more above and for the first
    launch of the layer above, and for none of its own layer."""
    layers = 6 if d < 4096 else 3
    cfg = dict(synth.CONFIGS["c1"], dim=d, n_heads=d // 64, n_kv_heads=d // 64, hidden=hidden, vocab=512, n_stages=2, layers_per_stage=layers,
               seq_len=rows, seqs_per_mb=1, n_mb=1, dtype=dtype, local_stage_begin=1, local_stage_count=1, has_embed=0, has_head=0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        dt = sp.torch_dtype(cfg)
        params = torch.zeros(sp.param_count(cfg), dtype=dt, device="cuda")
        grads = torch.zeros(params.numel(), device="cuda")
        act = torch.zeros(rows * d, dtype=dt, device="cuda")
        ctx = sp.Context(cfg, 1, 1, stream=stream)
        try:
            ctx.stage_fwd(1, params, act, [0])
            stream.synchronize()
            names, before = captured(stream, lambda: ctx.stage_bwd(1, params, act, [0], grads))
        finally:
            ctx.close()
    weight = [i for i, s in enumerate(names) if re.search(r"k_gemm_(f32_)?grads|k_gemm_(mfma|ring|f32|f32_few)(ILi2E|<2,)", s)]
    norms = [i for i, s in enumerate(names) if "k_rmsnorm_bwd" in s]
    assert len(weight) == launches * layers and len(norms) == 2 * layers, names
    for n in range(layers):
        waits = {weight.index(i) for i in before[norms[2 * n + 1]] if i in weight}
        assert waits == set(range(launches * (n - 1) + 1 if n else 0)), (n, waits)
    assert before[-1] == set(range(len(names) - 1))   # the last launch follows all others
