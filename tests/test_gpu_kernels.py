"""Kernels and dispatch branches at the sizes where they can go wrong (tile edges, remainders, the
two sides of a dispatch line), as whole passes against the float64 oracle.  Tolerances: the
harness's, per tensor and request."""
import numpy as np
import pytest
import torch

import gen
import oracle
from paper_2603_02565_amd import flasheval as fe
from tests import bf16_error_model
from tests.gpu_harness import make_evaluator, min_argmax, normwise, rtol_for, run_pass
from tests.test_gpu_linear import _amplify

pytestmark = pytest.mark.gpu


def check_pass(c, W=None, I=None, requests=None):
    W, I = W or gen.make_weights(c), I or gen.make_inputs(c)
    out = run_pass(c, W, I)
    tol = rtol_for(c)
    for b, ref in oracle.evaluate_cached(c, W, I, requests=requests, stages=True).items():
        for l in range(c.n_layers):
            if c.attention == "linear":
                st = oracle.linear_kv_state(ref["kv"][l][0], ref["kv"][l][1], c.n_heads)
                assert normwise(out["kv"][l, b], st) <= tol, ("linear state", b, l)
            else:
                for j in range(2):
                    assert normwise(out["kv"][l, j, b], ref["kv"][l][j]) <= tol, ("kv", b, l, j)
        U = len(ref["uniq"])
        assert out["n_uniq"][b] == U and np.array_equal(out["uniq"][b, :U], ref["uniq"])
        assert np.array_equal(out["slot"][b], ref["slot"])
        assert normwise(out["H"][b, :U], ref["H"]) <= tol, ("H", b)
        assert not out["H"][b, U:].any()
        assert normwise(out["seq"][b], ref["seq"]) <= tol, ("seq", b)
        assert normwise(out["Cp"][b], ref["Cp"]) <= tol, ("Cp", b)
        # few lists: a score's own size says nothing about its error (its d terms may cancel), so it
        # is bounded by the propagated C' error plus the fp32 dot product's rounding
        w, Cg = np.abs(W["head.w"].astype(np.float64)), out["Cp"][b].astype(np.float64)
        bound = np.abs(Cg - ref["Cp"]) @ w + (c.d + 2) * 2.0 ** -24 * (np.abs(Cg) @ w + abs(float(W["head.b"][0])))
        assert np.all(np.abs(out["scores"][b] - ref["scores"]) <= bound), ("scores", b)
        assert out["best"][b] == min_argmax(out["scores"][b])
    return out


@pytest.mark.parametrize("B,T,K,L,ffn", [
    (1, 1, 2, 3, 2048),      # one context row: a single row of a 32-row block
    (1, 33, 5, 7, 384),      # FFN width that does not divide over four waves: tiles for few rows
    (2, 130, 9, 7, 1024),    # rows between the two forms, padded item rows
    (1, 257, 4, 3, 128),     # two stages of the tile loop (the shortest), 64-row remainder of one
    (1, 700, 33, 9, 640),    # above the line at N = 1536, below it at N = 512
])
def test_wide_products(B, T, K, L, ffn):
    check_pass(gen.config(4, B=B, T=T, K=K, L=L, ffn=ffn, n_layers=1, vocab=600, M=600))


def test_wide_request_independent_of_batch():
    """Wide models: few rows take one product kernel, many the other (one request's 144 item and 16 list
    rows against those of 24 requests), and head width 64 one or two query tiles per wave.  A request's
    results have the same bits whoever shares the batch."""
    c = gen.config(4, B=24, T=300, K=16, L=9, n_layers=1, vocab=600, M=600)
    W, I = gen.make_weights(c), gen.make_inputs(c)
    whole = run_pass(c, W, I)
    for b in (0, 23):
        one = run_pass(c, W, {k: None if v is None else v[b:b + 1] for k, v in I.items()})
        assert np.array_equal(one["kv"][:, :, 0], whole["kv"][:, :, b]), ("kv", b)
        for k in ("H", "seq", "Cp", "scores"):
            assert np.array_equal(one[k][0], whole[k][b]), (k, b)


def context_kv(c, W, x):
    """kv of fe_encode_context for context rows x [B][T][d] (bf16, on the GPU), as its own bits."""
    ev = make_evaluator(c, W)
    bufs = ev.allocate(x.shape[0], c.T, c.M, c.K, c.L)
    fe.fe_encode_context(ev.handle, x.shape[0], c.T, x, None, bufs["kv"], bufs["ws"])
    kv = bufs["kv"].view(c.n_layers, 2, x.shape[0], c.T, c.d).clone()
    torch.cuda.synchronize()
    ev.close()
    return kv


def test_context_independent_of_batch():
    """Head width 64: one query tile per wave for one request (8 workgroups of two), two for 64 of
    them (512).  A request's context cache has the same bits either way."""
    c = gen.config(1, B=64, T=400, d=128, n_heads=2, ffn=512, n_layers=1)
    W = gen.make_weights(c)
    x = torch.from_numpy(gen.make_inputs(c)["x"]).cuda().bfloat16()
    kv = context_kv(c, W, x)
    for b in (0, 37, 63):
        assert torch.equal(context_kv(c, W, x[b:b + 1].contiguous())[:, :, 0], kv[:, :, b]), b


def tiles_per_wave(d, H, B, T):
    """Query tiles per wave of the chunked attention over B contexts of T rows (the launcher's rule)."""
    groups = lambda qt: -(-T // (64 * qt)) * H * B
    return 8 if d // H == 32 and groups(8) >= 512 else 2 if groups(2) >= 512 else 1


@pytest.mark.parametrize("d,H,B,T,tiles", [
    (128, 4, 1, 257, 1),     # a last chunk of one key
    (128, 2, 1, 300, 1),     # head width 64
    (128, 2, 64, 400, 2),    # head width 64, a last chunk of 16 keys
    (256, 8, 16, 513, 2),    # head width 32
    (128, 4, 64, 520, 8),    # the last tiles without queries
])
def test_attention_reference_moves(d, H, B, T, tiles):
    """Peaked scores (queries and keys 16 times the usual size: a row's weights differ by up to 2^60), so
    the softmax reference of the chunked attention moves in later chunks.  Against the float64 network
    with the values rounded that the GPU path stores in bf16 (a rounding of a query changes such scores,
    so the exact network's probabilities are others: its cache is off by up to 3e-2).  What is left are
    probabilities rounded relative to another reference and single roundings the other way, 2^-9 each in
    front of a residual stream of the same size (leaving either out of the network moves its cache by 1e-3
    to 2.6e-3), and the cache's own rounding (2^-8 of a value at most); the bound is their sum.  A sum or
    an output that is not rescaled when the reference moves is off by 0.4 and more.  Encoded with its
    rows in the opposite order, where the reference moves elsewhere, the context is held to the same bound."""
    assert tiles_per_wave(d, H, B, T) == tiles
    c = gen.config(1, B=B, T=T, d=d, n_heads=H, ffn=4 * d, n_layers=1)
    W = dict(gen.make_weights(c))
    w = W["ctx.0.wqkv"].copy()
    w[:, : 2 * d] *= 16      # powers of two: the values stay bf16 numbers
    w[:, 2 * d:] *= 4
    W["ctx.0.wqkv"] = w
    W["ctx.0.wo"] = W["ctx.0.wo"] * 4
    I = gen.make_inputs(c)
    x = torch.from_numpy(I["x"]).cuda().bfloat16()
    there, back = context_kv(c, W, x).float(), context_kv(c, W, x.flip(1).contiguous()).float().flip(3)
    m = bf16_error_model.Model(c, W, bf16_error_model.POINTS)
    for b in (0, B - 1):
        Q = m.ln(m.stack(np.asarray(I["x"][b], np.float64), "ctx", True), "ctx.lnf")
        for j, s in enumerate("kv"):
            ref = Q @ m.w("ctx.kv.0.w" + s) + m.w("ctx.kv.0.b" + s)
            for got in (there, back):
                assert normwise(got[0, j, b].cpu().numpy(), ref) <= 1e-2, (b, s)


@pytest.mark.parametrize("d,H,B,T,M,K,L,ffn", [
    (32, 1, 1, 1, 5, 1, 1, 32),       # one row; a step of 32 k values
    (64, 1, 1, 65, 63, 9, 6, 160),    # one row above a tile; k = 160: a short second step
    (128, 4, 2, 64, 40, 33, 3, 128),  # exact tiles and steps, padded item rows
    (256, 4, 1, 63, 20, 7, 4, 288),   # LayerNorm rows of two steps
    (512, 8, 1, 20, 70, 5, 13, 64),   # LayerNorm rows of four steps
])
def test_fp32_products(d, H, B, T, M, K, L, ffn):
    check_pass(gen.config(1, B=B, T=T, M=M, K=K, L=L, d=d, n_heads=H, ffn=ffn, n_layers=2, dtype="f32"))


@pytest.mark.parametrize("d,H,B,T,M,K,L,dtype", [
    (128, 4, 1, 1, 5, 1, 2, "bf16"),        # one row of a 32-row block
    (128, 2, 2, 33, 40, 31, 3, "bf16"),     # head width 64; one row above a block, one below
    (256, 8, 32, 601, 90, 33, 5, "bf16"),   # a last block of 25 rows
    (64, 1, 2, 65, 64, 32, 4, "f32"),       # fp32 rows of 64, padded item rows, an exact block
    (32, 1, 3, 31, 20, 7, 3, "f32"),
])
def test_linear_attention_blocks(d, H, B, T, M, K, L, dtype):
    check_pass(gen.config(1, B=B, T=T, M=M, K=K, L=L, d=d, n_heads=H, ffn=4 * d, n_layers=1, dtype=dtype, attention="linear"))


@pytest.mark.parametrize("d,H,B,dtype", [(128, 4, 64, "bf16"), (128, 2, 128, "bf16"), (64, 2, 128, "f32"), (64, 1, 256, "f32")])
def test_linear_attention_walk(d, H, B, dtype):
    """Waves that walk two blocks of 32 rows: 1030 element rows are 33 blocks, so the last wave has one,
    of six rows.  Every element is listed, and attention dominates its block, so each row of H shows its
    own block's work; the context's 1030 rows take the same walk."""
    U = 1030
    assert 2 * 4096 <= -(-U // 32) * B * H < 3 * 4096     # blocks per wave: two
    c = gen.config(1, B=B, T=U, M=U, K=103, L=10, d=d, n_heads=H, ffn=2 * d, n_layers=1, dtype=dtype, attention="linear")
    W, I = _amplify(gen.make_weights(c), 1), dict(gen.make_inputs(c))
    r = np.random.default_rng(2)
    I["lists"] = np.stack([r.permutation(U).reshape(103, 10) for _ in range(B)]).astype(np.int32)
    check_pass(c, W, I, requests=[0, B // 2, B - 1])
