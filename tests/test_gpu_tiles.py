"""Launch shapes the size rules choose between: the Patch, aligner and fold products on 256- and
128-wide tiles and on the deep copy ring, and the Reuse decode's channel chunks, at sizes on each side
of every rule, against the fp64 oracle (bf16 bar)."""
import pytest
import torch

import paper_2606_07684_amd as scd
from synth import workloads as W
from tests import parity_util as U
from tests import test_gpu_fit as F

pytestmark = pytest.mark.gpu
BF16_TOL = U.TOL["bf16"]


def _patch(name, heads, head_dim, d_model, tokens, layers, **kw):
    return W.Workload(name, layers, d_model, heads, head_dim, tokens, (32,) * layers,
                      tuple(range(layers)), 5e5, "bf16", with_bias=True, **kw)


# (KV heads, head_dim, d_model, request lengths, Patch layers): contractions of 1 to 9 steps of 64
# around both rings' depths; 128-wide tiles up to one per CU (deep ring), up to two per CU, and
# 256-wide tiles; full and ragged last tiles.
PATCH = [
    (8, 128, 64, (1, 127), 1),        # deep ring, one step, one full token tile
    (2, 64, 320, (129,), 2),          # deep ring, 5 steps, one token in the second tile
    (8, 64, 576, (300, 33), 2),       # deep ring, 9 steps, d_h = 64
    (8, 128, 256, (333, 267), 4),     # two per CU (5 token tiles x 64), 4 steps
    (16, 64, 192, (600,), 4),         # two per CU, d_h = 64, 3 steps
    (8, 128, 128, (700, 380), 4),     # 256-wide (5 token tiles x 32), d_h = 128
    (16, 64, 448, (1025,), 4),        # 256-wide, one token in the last tile, d_h = 64
]


@pytest.mark.parametrize("heads,head_dim,d_model,tokens,layers", PATCH)
def test_patch_tiles(heads, head_dim, d_model, tokens, layers):
    wl = _patch(f"tiles_{heads}_{head_dim}_{d_model}", heads, head_dim, d_model, tokens, layers)
    dev = torch.device("cuda")
    inp = W.Inputs(wl, dev, encode=False, decode=False)
    rope = scd.scd_rope_table(U.model_of(wl), wl.max_position)
    out = U.run_gpu(wl, inp, rope, which=("patch",), fill=float("nan"))
    U.assert_within(U.compare_all(wl, inp, out), BF16_TOL, wl.name)


# Folds: hidden widths that end inside a tile and inside a 16-byte chunk group, d_model of one and
# many steps, and a d_model that is not whole steps (the vector-unit product).
@pytest.mark.parametrize("heads,head_dim,d_model,hidden,layers", [
    (2, 64, 64, 16, 1), (2, 128, 320, 144, 2), (8, 128, 192, 1040, 4), (8, 128, 128, 4112, 4),
    (2, 64, 96, 80, 1)])
def test_fold_tiles(heads, head_dim, d_model, hidden, layers):
    wl = _patch(f"fold_{d_model}_{hidden}", heads, head_dim, d_model, (70,), layers,
                aligner_hidden=hidden)
    pc = U.PatchFromCodes(wl)
    U.assert_within({**pc.fold_errors(), **pc.cache_errors(list(range(wl.n_tokens)))}, BF16_TOL,
                    wl.name)


# Reuse decode at 8 KV heads of 128 (w = 1024): chunks of 128, 256 and 512 channels for ranks up to 128
# (512 at rank 32 with two workgroups per CU and with one), of 128 and 256 for rank 256;
# test_launch_rules.test_decode_chunks names the chunk of each.
@pytest.mark.parametrize("rank,tokens,layers", [
    (128, 40, 2), (128, 1999, 7), (128, 8192, 4), (256, 333, 2), (256, 5000, 2), (64, 500, 3),
    (64, 31000, 2), (64, 40000, 2), (32, 9000, 4), (32, 31000, 2), (32, 40000, 2)])
def test_decode_chunks(rank, tokens, layers):
    wl = W.Workload(f"chunks_{rank}_{tokens}", layers, 256, 8, 128, (tokens - 7, 7),
                    (rank,) * layers, (), 5e5, "bf16")
    dev = torch.device("cuda")
    inp = W.Inputs(wl, dev, encode=False, patch=False)
    rope = scd.scd_rope_table(U.model_of(wl), wl.max_position)
    out = U.run_gpu(wl, inp, rope, which=("decode",), fill=float("nan"))
    errs = U.compare_all(wl, inp, out, U.sample_tokens(wl))
    assert all(bool(torch.isfinite(t).all()) for l in inp.R for t in (out["k_cache"][l], out["v_cache"][l]))
    U.assert_within(errs, BF16_TOL, wl.name)


# The generic kernel's workgroup shapes (fp32, and bf16 with heads of 32): enough rows for four 32 x 64
# waves per workgroup, fewer (contraction split by 4) and few (split by 8), each with deRoPE, offsets,
# biases and rotated output; contractions that end inside a step (ranks 16 and 48).
@pytest.mark.parametrize("dtype,heads,head_dim", [("f32", 8, 64), ("f32", 4, 128), ("bf16", 16, 32)])
@pytest.mark.parametrize("tokens", [(4000, 101), (970, 30), (33,)])
def test_generic_shapes(dtype, heads, head_dim, tokens):
    wl = W.Workload(f"generic_{dtype}_{head_dim}", 5, 160, heads, head_dim, tokens,
                    (48, 16, 64, 64, 48), (0,), 1e4, dtype, with_bias=True,
                    pos0=tuple(11 * i + 3 for i in range(len(tokens))), ranks_v=(16, 48, 64, 80, 16))
    dev = torch.device("cuda")
    inp = W.Inputs(wl, dev)
    rope = scd.scd_rope_table(U.model_of(wl), wl.max_position)
    out = U.run_gpu(wl, inp, rope, fill=float("nan"))
    U.assert_within(U.compare_all(wl, inp, out), U.TOL[dtype], wl.name)


# The staged tiles of the bf16 decode and Patch off the specialised kernels' shapes: rows that end inside a
# tile (192 and 160 columns), heads of 32, 64 and 128, more than 256 requests (some empty) with start
# positions, ranks that end inside a contraction step, with and without offsets and biases.
@pytest.mark.parametrize("heads,head_dim,d_model,tokens,layers,ranks,mu", [
    (3, 64, 96, (1500, 559), 6, (16, 48, 96, 128, 176, 192), True),
    (5, 32, 160, (1999,), 6, (32, 80, 160, 16, 128, 64), False),
    (8, 128, 64, tuple(i % 13 for i in range(300)), 3, (112, 256, 64), True)])
def test_staged_tiles(heads, head_dim, d_model, tokens, layers, ranks, mu):
    wl = W.Workload(f"staged_{heads}_{head_dim}", layers, d_model, heads, head_dim, tokens, ranks, (0,) if d_model > 64
                    else (), 1e4, "bf16", with_bias=mu, with_mu=mu, pos0=tuple(5 * i for i in range(len(tokens))))
    dev = torch.device("cuda")
    inp = W.Inputs(wl, dev, encode=False)
    rope = scd.scd_rope_table(U.model_of(wl), wl.max_position)
    out = U.run_gpu(wl, inp, rope, which=("decode", "patch"), fill=float("nan"))
    U.assert_within(U.compare_all(wl, inp, out), BF16_TOL, wl.name)


# Ranks that are odd multiples of 16 on the bf16 decode (instances of their own): chunks of 256 channels,
# and of 512 at w = 1024.
@pytest.mark.parametrize("heads,head_dim,tokens,ranks,ranks_v", [
    (4, 64, (300, 77), (16, 48, 80), (112, 16, 48)), (4, 64, (300, 77), (144, 176, 208), (240, 16, 144)),
    (8, 128, (65000, 700), (16, 48, 112), (48, 112, 16))])
def test_decode_odd_ranks(heads, head_dim, tokens, ranks, ranks_v):
    wl = W.Workload(f"odd_{ranks[0]}", 3, 256, heads, head_dim, tokens, ranks, (), 5e5, "bf16",
                    ranks_v=ranks_v)
    dev = torch.device("cuda")
    inp = W.Inputs(wl, dev, encode=False, patch=False)
    rope = scd.scd_rope_table(U.model_of(wl), wl.max_position)
    out = U.run_gpu(wl, inp, rope, which=("decode",), fill=float("nan"))
    assert all(bool(torch.isfinite(t).all()) for l in inp.R for t in (out["k_cache"][l], out["v_cache"][l]))
    U.assert_within(U.compare_all(wl, inp, out, U.sample_tokens(wl)), BF16_TOL, wl.name)


# bf16 encode: the resident kernel with whole-layer shares (one and several code blocks), its balanced
# list crossing layers (several chunks, and one), 1 to 4 code blocks of 32, with and without offsets;
# the streamed kernel with 127-row tiles; Patch codes on either side of the split contraction
# (test_launch_rules.test_encode_resident names the kernel of each).
@pytest.mark.parametrize("heads,head_dim,shared,tokens,layers,ranks,mu", [
    (8, 128, False, (300, 3), 3, (128, 256, 96), True),
    (8, 128, False, (5000,), 3, (128, 192, 128), True),
    (2, 128, False, (9000, 100), 9, (64,) * 9, True),
    (4, 64, False, (9001,), 9, (96,) * 9, False),
    (4, 128, False, (700,), 4, (128, 32, 96, 48), True),
    (8, 128, True, (2999,), 4, (128, 128, 32, 32), True),
    (2, 64, False, (1,), 2, (16, 112), False),
    (4, 128, False, (20000, 20000), 3, (128,) * 3, True),
    (4, 128, False, (30100,), 4, (96,) * 4, True),
    (4, 64, False, (33000,), 5, (96,) * 5, False),
    (8, 128, True, (16385,), 5, (32,) * 5, True),
    (8, 128, True, (16000, 385), 5, (64,) * 5, False)])
def test_encode_shapes(heads, head_dim, shared, tokens, layers, ranks, mu):
    wl = W.Workload(f"encode_{heads}_{tokens[0]}", layers, 384, heads, head_dim, tokens, ranks, (0,),
                    5e5, "bf16", basis_width=head_dim if shared else None, with_mu=mu,
                    pos0=tuple(9 * i for i in range(len(tokens))))
    dev = torch.device("cuda")
    inp = W.Inputs(wl, dev, decode=False, patch=False)
    rope = scd.scd_rope_table(U.model_of(wl), wl.max_position)
    out = U.run_gpu(wl, inp, rope, which=("encode",))
    rows = U.sample_tokens(wl) if wl.n_tokens > 10000 else None
    U.assert_within(U.compare_all(wl, inp, out, rows), BF16_TOL, wl.name)


# An infinite offset entry reaches every code as minus infinity times its encoder weight's sign, and
# nothing becomes NaN: on the streamed kernel (w = 1024, rank 256), the resident one (w = 256) and the
# generic one (heads of 32; fp32), keys and values.
@pytest.mark.parametrize("dtype,heads,head_dim,rank,tokens", [
    ("bf16", 8, 128, 256, 17000), ("bf16", 2, 128, 64, 300), ("bf16", 4, 32, 32, 300), ("f32", 4, 64, 32, 300)])
def test_encode_infinite_offset(dtype, heads, head_dim, rank, tokens):
    wl = W.Workload(f"inf_{dtype}_{rank}", 1, 256, heads, head_dim, (tokens,), (rank,), (), 5e5, dtype,
                    with_mu=True)
    inp = W.Inputs(wl, torch.device("cuda"), decode=False, patch=False)
    col = head_dim // 2 + 5
    for mu in (inp.mu_k[0], inp.mu_v[0]):
        mu[col] = float("inf")
    out = U.run_gpu(wl, inp, scd.scd_rope_table(U.model_of(wl), wl.max_position), which=("encode",))
    for z, w in ((out["z_k"][0], inp.w_enc_k[0]), (out["z_v"][0], inp.w_enc_v[0])):
        assert bool((w[:, col] != 0).all())
        assert torch.equal(z.float(), (-torch.inf * w[:, col].float().sign()).expand(z.shape))


# The fit's tridiagonal steps: row registers of 8, 16, 24 and 32 per lane (trailing blocks of up to 512,
# 1024, 1536 and 2047 rows, each entered and left inside one fit), 4 rows per workgroup and, above 3072
# rows over the layers, 8; widths whose last workgroup and last lane registers are partly filled.
@pytest.mark.parametrize("heads,head_dim,tokens,layers", [
    (3, 64, (400, 61), 1), (9, 64, (1201,), 1), (13, 64, (1701,), 2), (9, 64, (1201,), 3)])
def test_fit_tridiagonal_shapes(heads, head_dim, tokens, layers):
    wl = W.Workload(f"fit_{heads}_{layers}", layers, 256, heads, head_dim, tokens, (32,) * layers, (),
                    5e5, "bf16", ranks_v=(32,) * layers)
    dev = torch.device("cuda")
    R, a_in, b_in, rope = F._setup(wl, "v", dev)
    lam = F._lam(wl)
    w_enc, w_dec, mu_enc, mu_dec, _, _ = scd.fit_reuse(U.model_of(wl), U.batch_of(wl, dev), rope,
                                                       scd.FIT_VALUES, a_in, b_in, lam, center=True)
    errs = {}
    for l in R:
        want = F._oracle_fit(wl, "v", a_in, b_in, l, lam)
        for name, got, ref in zip(("w_enc", "w_dec", "mu_enc", "mu_dec"),
                                  (w_enc[l], w_dec[l], mu_enc[l], mu_dec[l]), want):
            errs[(name, l)] = U.max_abs_rel(U.f64(got), ref)
    U.assert_within(errs, BF16_TOL, wl.name)
