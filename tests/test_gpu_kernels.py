"""Kernels and dispatch branches at the sizes where they can go wrong (tile edges, remainders, the
two sides of a dispatch line), as whole passes against the float64 oracle.  Tolerances: the
harness's, per tensor and request."""
import numpy as np
import pytest
import torch

import gen
import oracle
from paper_2603_02565_amd import flasheval as fe
from tests.gpu_harness import make_evaluator, min_argmax, normwise, rtol_for, run_pass

pytestmark = pytest.mark.gpu


def check_pass(c):
    W, I = gen.make_weights(c), gen.make_inputs(c)
    out = run_pass(c, W, I)
    tol = rtol_for(c)
    for b, ref in oracle.evaluate_cached(c, W, I, stages=True).items():
        if c.attention == "softmax":
            for l in range(c.n_layers):
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


@pytest.mark.parametrize("d,H,B,T", [
    (128, 4, 1, 257),     # one query tile per wave; a last chunk of one key
    (128, 2, 1, 300),     # head width 64
    (128, 2, 64, 383),    # head width 64, two tiles per wave
    (256, 8, 16, 513),    # two tiles per wave
    (128, 4, 64, 520),    # eight tiles per wave, the last ones without queries
])
def test_attention_reference_moves(d, H, B, T):
    """Peaked scores (queries and keys 25 times the usual size: a row's scores differ by up to 2^100
    in weight), so the softmax reference of the chunked attention moves in later chunks.  The
    context is encoded twice, its rows in the opposite order the second time: each row meets the
    keys in the other order, so its reference moves elsewhere, and its result is the same but for
    the bf16 rounding of probabilities and output (2^-9 each and side, in front of a residual
    stream of the same size; the harness's 2e-2 is four times that)."""
    c = gen.config(1, B=B, T=T, d=d, n_heads=H, ffn=4 * d, n_layers=1)
    W = dict(gen.make_weights(c))
    w = W["ctx.0.wqkv"].copy()
    w[:, : 2 * d] *= 25
    w[:, 2 * d:] *= 4
    W["ctx.0.wqkv"] = w
    W["ctx.0.wo"] = W["ctx.0.wo"] * 4
    ev = make_evaluator(c, W)
    x = torch.from_numpy(gen.make_inputs(c)["x"]).cuda().bfloat16()
    kv = []
    for rows in (x, x.flip(1).contiguous()):
        bufs = ev.allocate(c.B, c.T, c.M, c.K, c.L)
        fe.fe_encode_context(ev.handle, c.B, c.T, rows, None, bufs["kv"], bufs["ws"])
        kv.append(bufs["kv"].float().view(2, B, T, d))
    a, b = kv[0], kv[1].flip(2)
    assert torch.isfinite(a).all()
    assert (a - b).abs().max() <= rtol_for(c) * a.abs().max()


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
    (256, 8, 32, 601, 90, 33, 5, "bf16"),   # several blocks per wave, the last one of 25 rows
    (64, 1, 2, 65, 64, 32, 4, "f32"),       # fp32 rows of 64, padded item rows, an exact block
    (32, 1, 3, 31, 20, 7, 3, "f32"),
])
def test_linear_attention_blocks(d, H, B, T, M, K, L, dtype):
    check_pass(gen.config(1, B=B, T=T, M=M, K=K, L=L, d=d, n_heads=H, ffn=4 * d, n_layers=1, dtype=dtype, attention="linear"))
