"""RMSNorm backward where its wavefronts are divided by the width of a row, and the one fold of a stage's gain gradients."""
import numpy as np
import pytest
import torch

from oracle import skippipe_oracle as orc
from paper_2502_19913_amd import binding as sp
from paper_2502_19913_amd import synth
from tests.gpuharness import cosine, maxerr, relerr, round_bf16, run

pytestmark = pytest.mark.gpu

# widths at the edges of one, two and four wavefronts per row; 185 rows leave a remainder in rounds of 16, 8 and 4 rows
# and are enough for partial sums; 5 layers are 10 norms, more than one fold takes; 3 rows add without partial sums
CASES = [("bf16", 504, 4, 1, 37), ("bf16", 512, 8, 2, 37), ("bf16", 520, 4, 1, 37), ("bf16", 1024, 16, 1, 37),
         ("bf16", 1032, 6, 1, 37), ("bf16", 288, 6, 5, 37), ("f32", 64, 4, 5, 37), ("bf16", 520, 4, 1, 3)]


@pytest.mark.parametrize("dtype,dim,heads,layers,seq", CASES)
def test_stage_gradients_over_row_widths(dtype, dim, heads, layers, seq):
    seqs = 5 if seq > 3 else 1
    cfg = dict(synth.CONFIGS["c1"], dim=dim, n_heads=heads, n_kv_heads=heads, hidden=96, n_stages=2, layers_per_stage=layers,
               seq_len=seq, seqs_per_mb=seqs, n_mb=1, dtype=dtype, local_stage_begin=1, local_stage_count=1, has_embed=0, has_head=0)
    named = synth.make_params(cfg, 5, gain_jitter=0.02, std=0.02)
    x = synth.normal(6, f"ns{dim}", (1, seq * seqs, dim))
    dy = synth.normal(7, f"nd{dim}", (1, seq * seqs, dim))
    if dtype == "bf16":
        named, x, dy = {k: round_bf16(v) for k, v in named.items()}, round_bf16(x), round_bf16(dy)
    paths, lens = np.array([[0, 1]], np.int32), np.array([2], np.int32)
    ref = orc.run_paths(cfg, named, paths, lens, x_in=x, dy_in=dy, dtype=np.float64)
    got = run(cfg, named, paths, lens, x_in=x, dy_in=dy)
    for name, g in ref["grads"].items():
        if dtype == "f32":   # float sums against 64-bit ones
            assert relerr(got["grads"][name], g) < 1e-4 and maxerr(got["grads"][name], g) < 1e-4, name
        else:                # a few roundings of 2^-9 per layer: the bounds of the other bfloat16 comparisons
            assert cosine(got["grads"][name], g) >= 0.999 and maxerr(got["grads"][name], g) < 5e-2, (name, maxerr(got["grads"][name], g))
    assert relerr(got["dx"], ref["dx"]) < (1e-4 if dtype == "f32" else 2e-2)

@pytest.mark.parametrize("dim,heads", [(64, 4), (520, 4)])
def test_gain_gradient_fold_is_timed_with_the_norms(dim, heads):
    # two norms a layer and one fold of the stage's partial sums, all of the RMSNorm-backward class
    cfg = dict(synth.CONFIGS["c1"], dim=dim, n_heads=heads, n_kv_heads=heads, hidden=96, n_stages=2, layers_per_stage=2,
               seq_len=37, seqs_per_mb=5, n_mb=1, dtype="bf16", local_stage_begin=1, local_stage_count=1, has_embed=0, has_head=0)
    params = sp.pack_params(cfg, synth.make_params(cfg, 5), "cuda")
    grads = torch.zeros(params.numel(), device="cuda")
    act = torch.zeros(185 * dim, device="cuda", dtype=torch.bfloat16); dact = act.clone()
    ctx = sp.Context(cfg, 1, 1)
    try:
        ctx.stage_fwd(1, params, act, [0])
        sp.prof_begin()
        ctx.stage_bwd(1, params, dact, [0], grads)
        cls = sp.prof_end()["rmsnorm_bwd"]
    finally:
        ctx.close()
    assert cls["launches"] == 5 and cls["flops"] == 4 * 4.0 * 185 * dim * 2
