"""The weight gradients of a layer in one launch, against one launch each and against 64 bits."""
import ctypes as C
import re

import numpy as np
import pytest
import torch

from paper_2502_19913_amd import binding as sp
from paper_2502_19913_amd import synth
from tests.gpuharness import maxerr, relerr, round_bf16, run
from tests.test_gpu_stage_order import captured

pytestmark = pytest.mark.gpu


class Item(C.Structure):   # GradItem
    _fields_ = [("M", C.c_int64), ("N", C.c_int64), ("A", C.c_void_p), ("B", C.c_void_p), ("C", C.c_void_p)]


# width, hidden, width of q|k|v, rows; edges of the tiles that the launch takes.  float: widths with and without remainders (unaligned
# rows), a step and a part of one, whole and half runs of 64 k; 32-tiles at more than two and at most two a compute
# unit.  bf16: one run of the reduction a tile and several.
@pytest.mark.parametrize("dtype,d,h,nq,rows,tile", [
    ("f32", 32, 64, 80, 33, (16, 16)), ("f32", 64, 128, 160, 320, (16, 16)), ("f32", 31, 67, 81, 99, (16, 16)),
    ("f32", 228, 456, 456, 420, (32, 32)), ("f32", 227, 457, 455, 421, (32, 32)), ("f32", 136, 272, 392, 100, (32, 32)),
    ("f32", 137, 271, 393, 65, (32, 32)), ("f32", 200, 600, 584, 200, (64, 64)),
    ("f32", 201, 601, 583, 97, (64, 64)), ("f32", 264, 792, 776, 100, (128, 64)), ("f32", 263, 793, 775, 97, (128, 64)),
    ("f32", 544, 1088, 1616, 132, (128, 128)), ("f32", 543, 1087, 1615, 65, (128, 128)),
    ("bf16", 32, 64, 80, 33, (64,)), ("bf16", 64, 128, 160, 1000, (64,)), ("bf16", 392, 1176, 1160, 200, (128,)),
    ("bf16", 264, 792, 776, 2000, (128,)), ("bf16", 520, 1560, 1544, 100, (256,)), ("bf16", 520, 1560, 1544, 4100, (256,)),
])
def test_weight_gradients_in_one_launch(dtype, d, h, nq, rows, tile):
    code, dt = (sp.SP_F32, torch.float32) if dtype == "f32" else (sp.SP_BF16, torch.bfloat16)
    rnd = round_bf16 if dtype == "bf16" else (lambda x: x)
    shapes = [(d, h), (2 * h, d), (d, d), (nq, d)]
    a = [rnd(synth.normal(91, f"wa{i}{rows}", (rows, m))) for i, (m, _) in enumerate(shapes)]
    b = [rnd(synth.normal(92, f"wb{i}{rows}", (rows, n))) for i, (_, n) in enumerate(shapes)]
    guard = 64
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        on = lambda x: torch.from_numpy(x).cuda().to(dt)
        da, db = [on(x) for x in a], [on(x) for x in b]
        bufs = [torch.full((m * n + guard,), 0.5, device="cuda") for m, n in shapes]
        each = [torch.full((m, n), 0.5, device="cuda") for m, n in shapes]
        items = (Item * 4)(*[Item(m, n, x.data_ptr(), y.data_ptr(), c.data_ptr()) for (m, n), x, y, c in zip(shapes, da, db, bufs)])

        def together():
            rc = sp.lib()._ZN2sp10gemm_gradsEP12ihipStream_tilRA4_KNS_8GradItemE(C.c_void_p(stream.cuda_stream), C.c_int(code), C.c_int64(rows), items)
            assert rc == 0
        together()
        for x, y, c in zip(da, db, each):
            sp.gemm(2, x, y, c, stream=stream)
        stream.synchronize()
        got = [c.cpu().numpy() for c in bufs]
        single = [c.cpu().numpy() for c in each]
        names, _ = captured(stream, together)   # never run
    assert len(names) == 1 and re.search(r"k_gemm_(f32_)?grads", names[0]), names
    edges = tuple(int(x) for x in re.findall(r"\d+", names[0].split("grads")[1])[:len(tile)])
    assert edges == tile, names
    for i, (m, n) in enumerate(shapes):
        c = got[i][:m * n].reshape(m, n)
        assert np.all(got[i][m * n:] == 0.5), i
        if dtype == "f32":
            assert np.array_equal(c, single[i]), i
        # sums of K products of unit normals in float: about sqrt(K) 2^-24 of the largest, 4e-6 at 4100; products themselves are exact
        want = 0.5 + a[i].astype(np.float64).T @ b[i].astype(np.float64)
        assert relerr(c, want) < 2e-5 and maxerr(c, want) < 2e-5, (i, relerr(c, want), maxerr(c, want))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_small_stage_has_the_gradients_of_one_without_a_second_stream(dtype):
    """Five layers whose gradients are formed together, beside the chain and in it: the buffers of a layer are written again two
    layers on.  In float, matrices have the same bits; what is added in the order in which workgroups end (gains; in bf16 all) is
    a few sums of floats off."""
    cfg = dict(synth.CONFIGS["c1"], dim=128, n_heads=2, n_kv_heads=2, hidden=320, n_stages=2, layers_per_stage=5, seq_len=96, seqs_per_mb=2, n_mb=1,
               dtype=dtype, local_stage_begin=1, local_stage_count=1, has_embed=0, has_head=0)
    named = synth.make_params(cfg, 9, 0.1, 0.05)
    x = synth.make_activations(cfg, 9); dy = synth.make_upstream_grad(cfg, 9)
    paths, lens = np.array([[0, 1]], np.int32), np.array([2], np.int32)
    line, beside = (run(cfg, named, paths, lens, x_in=x, dy_in=dy, side_stream=side) for side in (0, 2))
    assert np.array_equal(line["y"], beside["y"]) and np.array_equal(line["dx"], beside["dx"])
    for k, g in line["grads"].items():
        if dtype == "f32" and g.ndim == 2:
            assert np.array_equal(g, beside["grads"][k]), k
        else:
            assert relerr(g, beside["grads"][k]) < 1e-5, k
