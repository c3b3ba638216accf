"""GPU: spans of steep spectrum, short and long: singular values falling by 4 decades with bfloat16
storage (whose rounding hides what is below), by 2.5 and by 10 and 12 with float32 (components below
1e-5 of the largest are not kept).

The rows of Vt that a span keeps are orthonormal to their storage rounding, however small their
singular value: with unit roundoff u = 2^-8 (bfloat16) or 2^-24 (float32) a stored row is off by
at most u of its length (entrywise rounding), so two rows' product by at most 2 u + u^2; 1e-8 is left
for the factorisation itself.

Reconstruction as in every other build test: 1.25 x the optimal error (2 x without an iteration)
plus 2^-7 or 1e-5 of the span's norm.  With float32 storage the sums of P = Y^T X, in float32 of
terms up to s_1^2, show too: an error of about 2^-22 s_1^2 in P is one of 2^-22 s_1^2 / s_i^2 in row i of
Vt, so of 2^-22 s_1^2 / s_i in the product, for each of k components."""

import math

import numpy as np
import pytest

import oracle
from synth import make_prefill
from tests.gpu_common import banner
from tests.test_gpu_build import S, _build  # noqa: F401

pytestmark = pytest.mark.gpu
LENGTHS = [31, 200, 1500]


@pytest.mark.parametrize("dtype,d,rank,sketch,power,heads,decades", [
    ("bf16", 128, 32, 40, 1, 100, 4), ("bf16", 128, 24, 40, 0, 100, 4), ("bf16", 64, 32, 40, 1, 100, 4),
    ("bf16", 128, 32, 40, 1, 2, 4), ("f32", 128, 32, 40, 1, 100, 2.5), ("f32", 64, 16, 24, 2, 2, 2.5),
    ("f32", 128, 32, 40, 1, 100, 12), ("f32", 64, 32, 40, 1, 2, 10)])
def test_steep_spectrum(S, dtype, d, rank, sketch, power, heads, decades):  # noqa: F811
    banner(f"steep spectrum {dtype} d{d} r{rank} l{sketch} p{power} heads {heads} decades {decades}")
    n = sum(LENGTHS) + len(LENGTHS)
    p = make_prefill(1, heads, d, [n], dtype=dtype, true_rank=4, sketch=sketch, seed=84)
    p.surprisal[:] = 1.0
    end = np.cumsum([L + 1 for L in LENGTHS]) - 1
    p.surprisal[0, end] = 9.0
    rng = np.random.default_rng(5)
    some = sorted({0, 1, heads - 1})
    for g in some:
        for i, L in enumerate(LENGTHS):
            for rows in (p.keys, p.values):
                k = min(L, d)
                q = [np.linalg.qr(rng.standard_normal((m, k)))[0] for m in (L, d)]
                X = (q[0] * 10.0 ** -np.linspace(0, decades, k)) @ q[1].T * math.sqrt(L)
                rows[0, g, end[i] - L:end[i]] = oracle.narrow(X, dtype)
    got, _, lay = _build(S, p, dict(rank=rank, sketch=sketch, min_span=2, window=0, power=power, Hkv=heads, d=d))
    spans = [s for s in oracle.segment(p.surprisal[0], n, 1.0, 2, 0)[1]]
    assert [L for _, L in spans] == LENGTHS
    u, rec = (2.0 ** -8, 2.0 ** -7) if dtype == "bf16" else (2.0 ** -24, 1e-5)
    worst, least = 0.0, 1.0
    for g in some:
        for i, (s0, L) in enumerate(spans):
            w = int(lay["block_rank"][0, g, i])
            blk = oracle.read_span_block(got["factors"], int(lay["block_off"][0, g, i]), L, w & 0xFFFF, d, dtype, w >> 16)
            for side, rows in (("K", p.keys), ("V", p.values)):
                X = oracle.widen(rows[0, g, s0:s0 + L], dtype)
                sg, Vt = blk["s" + side], blk["Vt" + side]
                Vt = Vt[sg > 0]
                e = np.abs(Vt @ Vt.T - np.eye(len(Vt))).max()
                worst, least = max(worst, e), min(least, sg[sg > 0].min() / sg.max())
                assert e <= 2 * u + u * u + 1e-8, (g, L, side, e)
                opt = math.sqrt(np.sum(np.linalg.svd(X, compute_uv=False)[min(L, d, rank):] ** 2))
                err = np.linalg.norm(X - oracle.reconstruct(blk["U" + side], sg, blk["Vt" + side]))
                sums = 0.0 if dtype == "bf16" else 2.0 ** -22 * math.sqrt(len(Vt)) * sg.max() ** 2 / sg[sg > 0].min()
                assert err <= (1.25 if power else 2.0) * opt + rec * np.linalg.norm(X) + sums, (g, L, side, err, opt)
    banner(f"worst product of two rows {worst:.2e}, smallest kept singular value {least:.1e} of the largest")
