"""The float mode's matrix-core kernels at the edges of their tiles, against the CPU checker's definitions."""
import numpy as np
import pytest
import torch

from oracle import skippipe_oracle as orc
from paper_2502_19913_amd import binding as sp
from paper_2502_19913_amd import synth
from tests.gpuharness import maxerr, relerr, round_bf16, run

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


# A float sum of K products of unit normals carries a relative rounding error of about sqrt(K) 2^-24 or less: 2e-6 at
# K = 1100.  The bounds allow ten times that over the tensor, and over the largest entry.
PRODUCTS = [  # M, N, K: 16-tiles and one entry; remainders in every dimension that are no multiple of 4 (unaligned
    # access); 64- and 128 x 64-tiles; a reduction of one step, of one group past a step, and of many
    (1, 1, 1), (33, 31, 17), (70, 50, 35), (130, 66, 300), (1100, 515, 33), (1030, 1100, 515), (2048, 2052, 36),
    (2049, 2047, 65), (516, 260, 1100), (36, 68, 4100),
]
# 128-tiles, with and without remainders that are no multiple of 4; 16-tiles of reductions that end around a step; 32-tiles of one step
# and a part, of a run and a part, and of many, at most two a compute unit and (the last two) more; aligned 64- and 128 x 64-tiles.  tests/test_host.py checks this against the dispatch.
PRODUCTS += [(2048, 2048, 36), (2183, 1351, 33), (2047, 2045, 67), (4096, 2048, 36), (4095, 2047, 33),
             (40, 36, 224), (40, 36, 256), (39, 35, 287), (40, 36, 292), (40, 36, 321),
             (516, 772, 36), (515, 771, 35), (600, 700, 100), (513, 770, 97), (512, 768, 292), (1100, 516, 36), (1600, 768, 132), (772, 772, 520), (775, 773, 519)]


@pytest.mark.parametrize("M,N,K", PRODUCTS)
def test_float_products(M, N, K):
    a = synth.normal(41, f"fa{M}{N}{K}", (M, K)); b = synth.normal(42, f"fb{M}{N}{K}", (N, K)); r = synth.normal(43, f"fr{M}{N}{K}", (M, N))
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    guard = 64
    buf = torch.full((M * N + guard,), 7.0, device="cuda")      # entries past the product must stay as they were
    c = buf[:M * N].view(M, N)
    for op, want in ((0, ref + r), (1, ref), (2, ref + 7.0)):
        buf.fill_(7.0)
        if op == 0:
            sp.gemm(0, dev(a), dev(b), c, dev(r))
        elif op == 1:
            sp.gemm(1, dev(a), dev(b.T), c)
        else:
            sp.gemm(2, dev(a.T), dev(b.T), c)
        got = c.cpu().numpy()
        assert relerr(got, want) < 2e-5 and maxerr(got, want) < 2e-5, (op, relerr(got, want), maxerr(got, want))
        assert torch.all(buf[M * N:] == 7.0), op


ATTENTION = [  # B, T, H, Hkv, hd: every compiled head dimension, at it and below it (zero columns, odd and unaligned
    # widths); sequences of one row, one tile of 32 short of, at and past a row, one block of 64 likewise, several
    (1, 1, 1, 1, 2), (2, 31, 2, 1, 32), (1, 33, 3, 3, 10), (2, 64, 2, 2, 48), (1, 65, 4, 2, 40), (1, 129, 2, 1, 64),
    (2, 63, 2, 2, 80), (1, 130, 6, 2, 96), (1, 97, 2, 1, 128), (1, 66, 2, 2, 113), (1, 100, 2, 1, 200), (1, 70, 2, 2, 256),
]


@pytest.mark.parametrize("B,T,H,Hkv,hd", ATTENTION)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_of_any_head_dimension(B, T, H, Hkv, hd, dtype):
    # Float: sums of up to hd or T products, exponentials of arguments below 30 in magnitude (relative error about
    # 30 * 2^-24): 2e-5 leaves a factor of ten.  bf16 storage: one rounding (2^-9) of o, and dO.o formed from that
    # rounded o; the head dimensions 64 and 128 also round probabilities.  Entries near zero carry their neighbours' errors.
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = (lambda a: a) if dtype == "f32" else round_bf16
    nq = (H + 2 * Hkv) * hd
    qkv = rnd(synth.normal(51, f"q{B}{T}{H}{hd}", (B * T, nq))); do = rnd(synth.normal(52, f"o{B}{T}{H}{hd}", (B * T, H * hd)))
    part = lambda lo, n: np.ascontiguousarray(qkv[:, lo * hd:(lo + n) * hd]).reshape(B * T, n, hd).astype(np.float64)
    q, k, v = part(0, H), part(H, Hkv), part(H + Hkv, Hkv)
    o_ref = orc.attention_fwd(q, k, v, B, T).reshape(B * T, -1)
    grads = orc.attention_bwd(do.reshape(B * T, H, hd).astype(np.float64), q, k, v, B, T)
    ref = np.concatenate([g.reshape(B * T, -1) for g in grads], axis=1)
    x = dev(qkv).to(dt)
    o = torch.empty((B * T, H * hd), dtype=dt, device="cuda"); lse = torch.empty((B, H, T), device="cuda")
    sp.attention_fwd(x, o, lse, B, T, H, Hkv, hd)
    dx = torch.empty_like(x); delta = torch.empty(B * H * T, device="cuda")
    sp.attention_bwd(x, o, lse, dev(do).to(dt), dx, delta, B, T, H, Hkv, hd)
    tol, worst = (2e-5, 5e-5) if dtype == "f32" else (2e-2, 4e-2)
    assert relerr(o.float().cpu().numpy(), o_ref) < tol and maxerr(o.float().cpu().numpy(), o_ref) < worst
    got = dx.float().cpu().numpy()
    assert relerr(got, ref) < tol and maxerr(got, ref) < worst, (relerr(got, ref), maxerr(got, ref))

# N, K: the 50M-shape products; widths and depths that are no multiple of 4 or 16; rows: some of them alone leave the chip
# idle in tiles of 64 (fewer than 128 of those), all of them take tiles of 64 or (last) of 128
@pytest.mark.parametrize("N,K,few,rows", [(288, 768, 1000, 2100), (768, 288, 65, 1100), (70, 35, 33, 6000), (288, 49, 17, 2100),
                                          (512, 65, 300, 16384)])
def test_float_rows_do_not_depend_on_their_number(N, K, few, rows):
    # forward and input-gradient products are row-wise: a microbatch alone and in a group has the same bits
    a = dev(synth.normal(44, f"ra{N}{K}", (rows, K))); b = dev(synth.normal(45, f"rb{N}{K}", (N, K))); r = dev(synth.normal(46, f"rr{N}{K}", (rows, N)))
    gu = dev(synth.normal(47, f"rg{N}{K}", (rows, 2 * N)))
    wgu = torch.cat([b, b.flip(0)])
    bt = b.t().contiguous()
    out = []
    for n in (rows, few):
        empty = lambda w: torch.empty((n, w), device="cuda")
        c0, c1, up, act, dgu = empty(N), empty(N), empty(2 * N), empty(N), empty(2 * N)
        sp.gemm(0, a[:n], b, c0, r[:n])
        sp.gemm(1, a[:n], bt, c1)
        sp.ffn_up_fwd(a[:n], wgu, up, act)
        sp.ffn_down_bwd(a[:n], bt, gu[:n], dgu, empty(N))
        out.append([x[:few].cpu().numpy() for x in (c0, c1, up, act, dgu)])
    for name, x, y in zip(("op 0", "op 1", "gate|up", "act", "d(gate)|d(up)"), *out):
        assert np.array_equal(x, y), (name, relerr(x, y))


def test_float_stage_does_not_depend_on_grouping():
    # 1024 rows alone leave the chip idle in tiles of 64, three microbatches together do not
    cfg = dict(synth.CONFIGS["c1"], dim=288, n_heads=6, n_kv_heads=6, hidden=768, n_stages=2, layers_per_stage=1, seq_len=256, seqs_per_mb=4,
               n_mb=3, local_stage_begin=1, local_stage_count=1, has_embed=0, has_head=0)
    named = synth.make_params(cfg, 8, 0.1, 0.05)
    x = synth.make_activations(cfg, 8); dy = synth.make_upstream_grad(cfg, 8)
    paths, lens = np.array([[0, 1]] * 3, np.int32), np.array([2] * 3, np.int32)
    a = run(cfg, named, paths, lens, x_in=x, dy_in=dy)
    b = run(cfg, named, paths, lens, x_in=x, dy_in=dy, regroup=lambda plan: [(pos, st, [mb]) for pos, st, mbs in plan for mb in mbs])
    assert np.array_equal(a["y"], b["y"]) and np.array_equal(a["dx"], b["dx"])
    for k in a["grads"]:
        assert relerr(a["grads"][k], b["grads"][k]) < 1e-5, k

def attention(qkv, do, dtype, B, T, H, Hkv, hd, o=None):
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    x = dev(qkv).to(dt)
    out = torch.empty((B * T, H * hd), dtype=dt, device="cuda"); lse = torch.empty((B, H, T), device="cuda")
    sp.attention_fwd(x, out, lse, B, T, H, Hkv, hd)
    dx = torch.empty_like(x); delta = torch.empty(B * H * T, device="cuda")
    sp.attention_bwd(x, out, lse, dev(do).to(dt), dx, delta, B, T, H, Hkv, hd)
    return out.float().cpu().numpy(), dx.float().cpu().numpy().reshape(B * T, H + 2 * Hkv, hd)


# two sets of wavefronts (hd <= 48) and one; a hidden dimension below its compiled size; a group of query heads
@pytest.mark.parametrize("T,H,Hkv,hd", [(130, 2, 2, 48), (77, 2, 1, 10), (130, 2, 1, 96), (70, 2, 2, 200)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_attention_is_causal_for_non_finite_values(T, H, Hkv, hd, dtype, bad):
    # a key or value that is not finite reaches the queries that see it and no earlier one; a query or upstream gradient
    # that is not finite reaches the keys it sees and no later one
    rnd = (lambda a: a) if dtype == "f32" else round_bf16
    qkv = rnd(synth.normal(61, f"nq{T}{hd}", (T, (H + 2 * Hkv) * hd))); do = rnd(synth.normal(62, f"no{T}{hd}", (T, H * hd)))
    o0, d0 = attention(qkv, do, dtype, 1, T, H, Hkv, hd)
    # sums over the same values in another order where they are formed anew: the bounds of the test above
    same = lambda got, want: np.isfinite(got).all() and relerr(got, want) < (2e-5 if dtype == "f32" else 2e-2)
    at, col = 37, 3
    other = np.arange(hd) != col
    p = qkv.copy(); p[at, (H + Hkv) * hd + col] = bad            # v: one column of the outputs, from its position on
    o, d = attention(p, do, dtype, 1, T, H, Hkv, hd)
    assert same(o[:at], o0[:at]) and not np.isfinite(o[at:, col]).any() and same(o[at:, :hd][:, other], o0[at:, :hd][:, other])
    assert same(d[:at, :H], d0[:at, :H])                         # dq
    p = qkv.copy(); p[at, H * hd + col] = bad                    # k
    o, d = attention(p, do, dtype, 1, T, H, Hkv, hd)
    assert same(o[:at], o0[:at]) and same(d[:at, :H], d0[:at, :H])
    p = qkv.copy(); p[at, col] = bad                             # q of head 0
    o, d = attention(p, do, dtype, 1, T, H, Hkv, hd)
    assert same(np.delete(o, at, 0), np.delete(o0, at, 0)) and not np.isfinite(o[at, :hd]).any()
    assert same(np.delete(d, at, 0)[:, :H], np.delete(d0, at, 0)[:, :H]) and same(d[at + 1:, H:], d0[at + 1:, H:])
    p = do.copy(); p[at, col] = bad                              # upstream gradient of head 0
    o, d = attention(qkv, p, dtype, 1, T, H, Hkv, hd)
    assert same(d[at + 1:, H:], d0[at + 1:, H:]) and not np.isfinite(d[:at + 1, H + Hkv, col]).any()
    assert same(d[:at + 1, H + Hkv][:, other], d0[:at + 1, H + Hkv][:, other])   # dv's other columns

# whole tiles of 32 keys that no query attends to: the first of a wavefront's walk (one set of wavefronts: keys 0 .. 31;
# two sets: also keys 32 .. 63) and a later one
@pytest.mark.parametrize("hd", [40, 96])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lo", [0, 32, 64])
def test_attention_over_keys_of_weight_zero(hd, dtype, lo):
    T, H = 160, 2
    rnd = (lambda a: a) if dtype == "f32" else round_bf16
    qkv = rnd(synth.normal(63, f"iq{hd}", (T, 3, H, hd)).reshape(T, -1)).reshape(T, 3, H, hd)
    qkv[:, 0, :, 0] = 1.0
    qkv[lo:lo + 32, 1, :, 0] = -np.inf                            # their scores are -inf: weight 0
    o, _ = attention(qkv.reshape(T, -1), np.zeros((T, H * hd), np.float32), dtype, 1, T, H, H, hd)
    q, k, v = (qkv[:, i].astype(np.float64) for i in range(3))
    s = np.stack([q[:, h] @ np.where(np.isinf(k[:, h]), 0, k[:, h]).T for h in range(H)]) / np.sqrt(hd)
    s[:, :, lo:lo + 32] = -np.inf
    s = np.where(np.tril(np.ones((T, T), bool)), s, -np.inf)
    rows = np.arange(32 if lo == 0 else 0, T)                     # a row that sees no other key has no result
    p = np.exp(s[:, rows] - s[:, rows].max(-1, keepdims=True)); p /= p.sum(-1, keepdims=True)
    ref = np.stack([p[h] @ v[:, h] for h in range(H)], 1).reshape(len(rows), -1)
    assert relerr(o[rows], ref) < (2e-5 if dtype == "f32" else 1e-2), relerr(o[rows], ref)

# few tiles and a long reduction: tiles of 64 and of 32, and ones that leave remainders
@pytest.mark.parametrize("M,N,K", [(864, 288, 4096), (288, 288, 1000), (1024, 1024, 3072), (70, 66, 2049)])
def test_float_weight_gradients_are_repeatable(M, N, K):
    # in float every entry is summed in one order and added once: the same bits on every run
    a = dev(synth.normal(48, f"pa{M}{K}", (K, M))); b = dev(synth.normal(49, f"pb{N}{K}", (K, N))); c0 = dev(synth.normal(50, f"pc{M}{N}", (M, N)))
    got = []
    for _ in range(6):
        c = c0.clone()
        sp.gemm(2, a, b, c)
        got.append(c.cpu().numpy())
    assert all(np.array_equal(g, got[0]) for g in got[1:])
    want = a.cpu().numpy().astype(np.float64).T @ b.cpu().numpy().astype(np.float64) + c0.cpu().numpy()
    assert relerr(got[0], want) < 2e-5 and maxerr(got[0], want) < 2e-5


@pytest.mark.parametrize("op,M,N,K", [(0, 128, 288, 768), (1, 1000, 288, 1536), (0, 2048, 288, 768), (0, 2048, 2048, 2048), (2, 864, 288, 4096),
                                      (2, 1024, 1024, 3072), (2, 4096, 2048, 1024)])
def test_float_products_lose_little_over_long_reductions(op, M, N, K):
    # runs of 64 k (16 instructions), then K / 64 runs: about 3.6e-8 (16 + K / 64)^0.5 at most, 3.2e-7 at K = 4096; one
    # chain over the whole reduction would be 5e-7 at K = 768 and 1.1e-6 at 4096
    a = synth.normal(64, f"la{M}{K}", (M, K)); b = synth.normal(65, f"lb{N}{K}", (N, K))
    c = torch.zeros((M, N), device="cuda")
    sp.gemm(op, dev(a.T if op == 2 else a), dev(b if op == 0 else b.T), c)
    err = relerr(c.cpu().numpy(), a.astype(np.float64) @ b.astype(np.float64).T)
    assert err < 3.6e-8 * np.sqrt(16 + K / 64), err


# 64-tiles alone on their CUs and 128 x 64-tiles, one step and a run and a half; with and without remainders; the smallest
@pytest.mark.parametrize("M,N,K", [(1024, 1024, 96), (1023, 1021, 97), (2048, 1024, 32), (2048, 1024, 96), (2047, 1023, 95), (5, 3, 2), (36, 32, 33), (1600, 768, 132)])
def test_float_products_of_values_at_the_ends_of_the_range(M, N, K):
    # operands are split into bfloat16 parts: values that have none, that round past the largest one, and that are so
    # small that products vanish give what float products of them give, and reach no other row or column
    a = synth.normal(66, f"ea{M}{N}{K}", (M, K)); b = synth.normal(67, f"eb{M}{N}{K}", (N, K))
    b[N // 2] *= 1e-30
    # a value that rounds past the largest bfloat16; no partial sum may pass the largest float (its order would decide)
    a[M // 3, K // 2] = 3.4028e38; b[:, K // 2] = 0; b[N // 2, K // 2] = 1e-3
    a[M // 2, 0] = np.inf; a[M - 1, K - 1] = np.nan; b[0, K - 1] = -np.inf
    a[0] *= 1e-25
    with np.errstate(over="ignore", invalid="ignore"):
        ref = a.astype(np.float64) @ b.astype(np.float64).T
        ref32 = ref.astype(np.float32)
    for op in (0, 1, 2):
        c = torch.zeros((M, N), device="cuda")
        sp.gemm(op, dev(a.T if op == 2 else a), dev(b if op == 0 else b.T), c)
        got = c.cpu().numpy()
        fin = np.isfinite(ref32)
        assert np.array_equal(np.isfinite(got), fin) and np.array_equal(np.isnan(got), np.isnan(ref32)), op
        assert np.array_equal(got[~fin & ~np.isnan(ref32)], ref32[~fin & ~np.isnan(ref32)]), op
        # rows have scales of their own: against the largest product of an entry, ten times sqrt(K) 2^-24
        with np.errstate(over="ignore", invalid="ignore"):
            size = np.sqrt((a.astype(np.float64) ** 2) @ (b.astype(np.float64) ** 2).T)
        assert np.all(np.abs(got[fin] - ref[fin]) <= 6e-7 * np.sqrt(K) * size[fin] + 1e-37), op


# rows: few take tiles of 16, whose wavefronts form the runs of 64 k in turn (one run less than eight, eight, one more, several
# rounds, a run of one step), the others tiles of 32, 64, 128 x 64 and 128
@pytest.mark.parametrize("N,K,few,rows", [(288, 448, 33, 700), (288, 512, 64, 5000), (288, 576, 16, 700), (70, 1569, 50, 20000), (288, 1536, 64, 1024), (512, 65, 1, 9000)])
def test_float_rows_have_the_bits_of_larger_tiles_in_tiles_of_16(N, K, few, rows):
    a = dev(synth.normal(68, f"qa{N}{K}", (rows, K))); b = dev(synth.normal(69, f"qb{N}{K}", (N, K))); r = dev(synth.normal(70, f"qr{N}{K}", (rows, N)))
    gu = dev(synth.normal(71, f"qg{N}{K}", (rows, 2 * N))); wgu = torch.cat([b, b.flip(0)]); bt = b.t().contiguous()
    assert sp.gemm_shape(sp.SP_F32, 0, few, N, K)[0] == 16 and sp.gemm_shape(sp.SP_F32, 0, rows, N, K)[0] > 16
    out = []
    for n in (rows, few):
        empty = lambda w: torch.empty((n, w), device="cuda")
        c0, c1, up, act, dgu = empty(N), empty(N), empty(2 * N), empty(N), empty(2 * N)
        sp.gemm(0, a[:n], b, c0, r[:n])
        sp.gemm(1, a[:n], bt, c1)
        sp.ffn_up_fwd(a[:n], wgu, up, act)
        sp.ffn_down_bwd(a[:n], bt, gu[:n], dgu, empty(N))
        out.append([x[:few].cpu().numpy() for x in (c0, c1, up, act, dgu)])
    for name, x, y in zip(("op 0", "op 1", "gate|up", "act", "d(gate)|d(up)"), *out):
        assert np.array_equal(x, y), (name, relerr(x, y))
    want = a[:few].double() @ b.double().T
    assert relerr(out[1][1], want.cpu().numpy()) < 2e-5


# a last step that is not full (16-byte access, and not), in tiles of 16, 32, 64, 128 x 64 and 128
@pytest.mark.parametrize("M,N,K", [(33, 40, 36), (512, 768, 292), (1100, 516, 36), (1100, 515, 35), (2048, 1024, 100), (2183, 1352, 36), (2183, 1352, 260)])
def test_float_rows_keep_their_bits_beside_rows_that_are_not_finite(M, N, K):
    # a row runs on into the next one past the end of k: nothing of that may reach it, not even the order of its sums
    a = dev(synth.normal(72, f"ka{M}{K}", (M, K))); b = dev(synth.normal(73, f"kb{N}{K}", (N, K)))
    gu = dev(synth.normal(74, f"kg{M}{N}", (M, 2 * N))); bt = b.t().contiguous(); wgu = torch.cat([b, b.flip(0)])
    bad = torch.arange(M, device="cuda") % 3 == 1
    out = []
    for poison in (False, True):
        if poison:
            a[bad] = float("nan")
        empty = lambda w: torch.empty((M, w), device="cuda")
        c0, c1, up, act, dgu = empty(N), empty(N), empty(2 * N), empty(N), empty(2 * N)
        sp.gemm(0, a, b, c0)
        sp.gemm(1, a, bt, c1)
        sp.ffn_up_fwd(a, wgu, up, act)
        sp.ffn_down_bwd(a, bt, gu, dgu, empty(N))
        out.append([x[~bad] for x in (c0, c1, up, act, dgu)])
    for name, x, y in zip(("op 0", "op 1", "gate|up", "act", "d(gate)|d(up)"), *out):
        assert torch.equal(x, y), name


@pytest.mark.parametrize("M,N,K", [(33, 40, 4096), (1030, 1100, 3072), (2048, 2048, 2051)])
def test_float_products_formed_anew_lose_no_more_than_others(M, N, K):
    # a factor that rounds past the largest bfloat16 has no finite parts, and all its row's entries are formed again from the
    # floats: in runs of 64 k too (bound: test_float_products_lose_little_over_long_reductions)
    a = synth.normal(75, f"ma{M}{K}", (M, K)); b = synth.normal(76, f"mb{N}{K}", (N, K))
    a[M // 2:, K // 3] = 3.4e38; b[:, K // 3] *= np.float32(1e-38)
    want = a.astype(np.float64) @ b.astype(np.float64).T
    for op in (0, 1, 2):
        c = torch.zeros((M, N), device="cuda")
        sp.gemm(op, dev(a.T if op == 2 else a), dev(b if op == 0 else b.T), c)
        err = relerr(c[M // 2:].cpu().numpy(), want[M // 2:])
        assert err < 3.6e-8 * np.sqrt(16 + K / 64), (op, err)


def least_ms(*works):
    """The least of six timings of each."""
    best = []
    for work in works:
        took = []
        for _ in range(6):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            t[0].record()
            work()
            t[1].record()
            torch.cuda.synchronize()
            took.append(t[0].elapsed_time(t[1]))
        best.append(min(took))
    return best


@pytest.mark.parametrize("op", [0, 1, 2])
def test_float_products_of_nan_take_little_longer_than_others(op):
    # a pass that has diverged is NaN throughout: such entries are settled by the first run of k, at a few per cent of a product
    # (1.1 to 1.3 times the time of a finite one; 12 to 18 times when every entry took the whole reduction); four leaves room
    M, N, K = 4096, 1024, 2816
    a = dev(synth.normal(77, "na", (M, K) if op < 2 else (K, M))); b = dev(synth.normal(78, "nb", (N, K) if op == 0 else (K, N)))
    c = torch.zeros((M, N), device="cuda"); nan = torch.full_like(a, float("nan"))
    best = least_ms(lambda: sp.gemm(op, a, b, c), lambda: sp.gemm(op, nan, b, c))
    assert torch.isnan(c).all() and best[1] < 4 * best[0], best


# strided widths of one to five columns (a load of four reaches past the row), reductions that end with, before and after a step,
# in tiles of 16 and larger; pointers off by 4, 8 and 12 bytes; rows so long that a tile of theirs passes 31 bits
@pytest.mark.parametrize("M,N,K,off", [(20000, 1, 64, 0), (20000, 2, 65, 1), (3, 9000, 96, 2), (5000, 5, 33, 3), (1, 2, 99, 1), (1030, 513, 64, 1),
                                       (2048, 1026, 160, 2), (2049, 2050, 97, 3), (9, 130, 224, 1), (2, 3, (1 << 22) + 5, 0)])
def test_float_products_at_any_alignment(M, N, K, off):
    a = synth.normal(79, f"ga{M}{N}", (M, K)); b = synth.normal(80, f"gb{M}{N}", (N, K)); r = synth.normal(81, f"gr{M}{N}", (M, N))
    guard = 64

    def put(x):   # `off` floats into its buffer, with NaN on both sides
        buf = torch.full((x.size + off + guard,), float("nan"), device="cuda")
        buf[off:off + x.size] = dev(x).view(-1)
        return buf[off:off + x.size].view(*x.shape)
    want = a.astype(np.float64) @ b.astype(np.float64).T
    for op, ref in ((0, want + r), (1, want), (2, want + r)):
        if op == 2 and K > 1 << 22:
            continue
        c = put(r)
        if op == 0:
            sp.gemm(0, put(a), put(b), c, put(r))
        else:
            sp.gemm(op, put(a if op == 1 else np.ascontiguousarray(a.T)), put(np.ascontiguousarray(b.T)), c)
        got = c.cpu().numpy()
        assert relerr(got, ref) < 2e-5 and maxerr(got, ref) < 2e-5, (op, relerr(got, ref), maxerr(got, ref))


def test_float_products_of_far_operands():
    # k-strided widths past 2^24: no buffer load reaches the tile's last rows
    torch.manual_seed(82)
    W = (1 << 24) + 3
    a = torch.randn(W, 33, device="cuda"); b = torch.randn(2, 33, device="cuda")
    want = a @ b.t()
    at = a.t().contiguous()
    c = torch.zeros((W, 2), device="cuda")
    sp.gemm(2, at, b.t().contiguous(), c)
    assert float((c - want).norm() / want.norm()) < 1e-5
    c = torch.zeros((2, W), device="cuda")
    sp.gemm(1, b, at, c)
    assert float((c.t() - want).norm() / want.norm()) < 1e-5
    h, d, R = 2, (1 << 22) + 8, 3       # a SwiGLU tile
    hn = torch.randn(R, d, device="cuda"); w = torch.randn(2 * h, d, device="cuda") / d ** 0.5
    gu, act = torch.empty(R, 2 * h, device="cuda"), torch.empty(R, h, device="cuda")
    sp.ffn_up_fwd(hn, w, gu, act)
    ref = (hn.double() @ w.double().t())
    lim = 3.6e-8 * (16 + d / 64) ** 0.5   # as in test_float_products_lose_little_over_long_reductions: 9.2e-6
    assert float((gu - ref).norm() / ref.norm()) < lim
    # two factors, and silu at most doubles the relative error of values of order one
    assert float((act - torch.nn.functional.silu(ref[:, :h]) * ref[:, h:]).norm() / act.norm()) < 4 * lim


def test_float_weight_gradients_of_odd_widths_take_no_longer_than_of_even_ones():
    # 999 columns leave rows unaligned: 5.4 times the time of 1024 when they were loaded one by one, 1.0 times now
    K, N = 5632, 1024
    works = []
    for M in (1024, 999):
        a, b, c = torch.randn(K, M, device="cuda"), torch.randn(K, N, device="cuda"), torch.zeros(M, N, device="cuda")
        works.append(lambda a=a, b=b, c=c: sp.gemm(2, a, b, c))
    even, odd = least_ms(*works)
    assert odd < 2 * even, (odd, even)


@pytest.mark.parametrize("late", [True, False])
@pytest.mark.parametrize("dtype,hd", [("f32", 16), ("f32", 48), ("f32", 80), ("f32", 128), ("bf16", 16), ("bf16", 48), ("bf16", 80)])
def test_attention_weights_below_the_smallest_normal_float(dtype, hd, late):
    """Weights of e^-90 that meet values of 1e30.  late: the largest score (key 70) is met after sums have been formed, which are
    scaled down by as much.  Scores carry 90 * 2^-24 times a few, a float weight at most 2^-150 of 2^-130: 1e-4 leaves a factor of
    three.  In bf16 a weight is multiplied to 2^-134 (1/16 of this one), and results round to 2^-9."""
    T, top = 100, 70 if late else 0
    rnd = round_bf16 if dtype == "bf16" else (lambda a: a.astype(np.float32))
    q, k, v, do = (np.zeros((T, hd)) for _ in range(4))
    q[:, 0] = 20
    k[:, 0] = -4.5 * np.sqrt(hd); k[top] = 0
    v[1, 2] = 1e30                                  # forward: a row that sees key `top` has e^-90 of this
    qkv = rnd(np.concatenate([q, k, v], 1))
    tol = 1e-4 if dtype == "f32" else 1 / 16 + 2.0 ** -8
    close = lambda x, want: np.all(np.abs(x - want) <= tol * np.abs(want))
    parts = lambda: [np.ascontiguousarray(qkv[:, i * hd:(i + 1) * hd]).reshape(T, 1, hd).astype(np.float64) for i in range(3)]
    want = orc.attention_fwd(*parts(), 1, T).reshape(T, hd)
    assert 0 < want[80, 2] < 1e-8
    got, _ = attention(qkv, np.zeros((T, hd)), dtype, 1, T, 1, 1, hd)
    assert close(got, want), (got[[1, 69, 70, 99], 2], want[[1, 69, 70, 99], 2])
    v[:] = 0; v[:, 3] = 1; v[top] = 0
    qkv = rnd(np.concatenate([q, k, v], 1))
    do[80, 3] = 1e30
    do = rnd(do)
    grads = orc.attention_bwd(do.reshape(T, 1, hd).astype(np.float64), *parts(), 1, T)
    want = np.concatenate([g.reshape(T, hd) for g in grads], 1)
    assert 0 < abs(want[5, 2 * hd + 3]) < 1e-8 and 0 < abs(want[5, hd]) < 1e-8 and 0 < abs(want[80, 0]) < 1e-5
    got = attention(qkv, do, dtype, 1, T, 1, 1, hd)[1].reshape(T, -1)
    assert close(got, want), [(got[at], want[at]) for at in ((5, 2 * hd + 3), (5, hd), (80, 0))]
