"""Kernels and dispatch branches at the sizes where they can go wrong (tile edges, remainders, the
two sides of a dispatch line), as whole passes against the float64 oracle.  Tolerances: the
harness's, per tensor and request."""
import numpy as np
import pytest

import gen
import oracle
from tests.gpu_harness import min_argmax, normwise, rtol_for, run_pass

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
