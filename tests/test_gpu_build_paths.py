"""GPU: the builder's factorisation at the edges of its tiles (16 tokens, 16 sketch columns)
and on both sides of the rule that gives a span side one wave or four, against the optimal
truncated SVD; the segmentation past one 65536-token tile at an unaligned length.

Bound: 1.25 x the optimal error (2 x without a subspace iteration) plus the storage rounding of
the three factors, 2^-7 (bfloat16) or 1e-5 (float32) of the span's norm, as for every other
build test here."""

import math

import numpy as np
import pytest

import oracle
from synth import make_prefill
from tests.gpu_common import banner
from tests.test_gpu_build import S, _bdims, _build, _check_segments, _segment  # noqa: F401

pytestmark = pytest.mark.gpu
LENGTHS = [15, 16, 17, 3, 31, 32, 33, 64, 65, 130, 2, 257]

# dtype, d, rank, sketch, power, heads: 2 x heads x 12 span sides (more than 512: one wave each)
CASES = [("bf16", 128, 32, 40, 1, 2), ("bf16", 128, 24, 32, 1, 24), ("f32", 64, 8, 16, 2, 24),
         ("f32", 128, 32, 40, 1, 1), ("bf16", 64, 40, 40, 2, 24), ("f32", 128, 12, 18, 1, 22),
         ("bf16", 64, 16, 34, 1, 2), ("f32", 64, 24, 32, 0, 1)]


@pytest.mark.parametrize("dtype,d,rank,sketch,power,heads", CASES)
def test_factor_tiles(S, dtype, d, rank, sketch, power, heads):  # noqa: F811
    banner(f"factors {dtype} d{d} r{rank} l{sketch} heads {heads}")
    n = sum(LENGTHS) + len(LENGTHS)
    p = make_prefill(1, heads, d, [n], dtype=dtype, true_rank=min(rank, 20), noise=0.05, sketch=sketch, seed=81)
    p.surprisal[:] = 1.0
    at = np.cumsum([L + 1 for L in LENGTHS]) - 1
    p.surprisal[0, at] = 9.0
    c = dict(rank=rank, sketch=sketch, min_span=2, window=0, power=power, Hkv=heads, d=d)
    zero = {int(at[i - 1]) + 1: L for i, L in enumerate(LENGTHS) if L in (3, 130)}   # keys of zeros: a
    for s0, L in zero.items():                              # span inside the sketch and one past it
        assert p.keys[0, :, s0:s0 + L].any()
        p.keys[0, :, s0:s0 + L] = 0
    p.values[0, :, at[7] + 1:at[8] + 1] = p.values[0, :, at[7] + 1:at[7] + 2]   # and one of equal rows
    got, seg, lay = _build(S, p, c)
    _check_segments(seg, p, 1.0, 2, 0, "lengths")
    _, spans = oracle.segment(p.surprisal[0], n, 1.0, 2, 0)
    assert len(spans) >= len(LENGTHS) - 1
    assert zero.items() <= dict(spans).items()
    rec = 2.0 ** -7 if dtype == "bf16" else 1e-5
    for g in sorted({0, heads // 2, heads - 1}):
        for i, (s0, L) in enumerate(spans):
            w = int(lay["block_rank"][0, g, i])
            blk = oracle.read_span_block(got["factors"], int(lay["block_off"][0, g, i]), L, w & 0xFFFF, d, dtype, w >> 16)
            if s0 in zero:
                assert all(np.all(blk[name + "K"] == 0) for name in ("U", "s", "Vt")), (i, L)
            for side, src in (("K", p.keys), ("V", p.values)):
                X = oracle.widen(src[0, g, s0:s0 + L], dtype)
                opt = math.sqrt(np.sum(np.linalg.svd(X, compute_uv=False)[min(L, d, rank):] ** 2))
                err = np.linalg.norm(X - oracle.reconstruct(blk["U" + side], blk["s" + side], blk["Vt" + side]))
                assert err <= (1.25 if power else 2.0) * opt + rec * np.linalg.norm(X) + 1e-30, (i, L, side, err, opt)


@pytest.mark.parametrize("n", [65535, 65537, 70001])
def test_segment_past_one_tile(S, n):  # noqa: F811
    banner(f"segment {n}")
    p = make_prefill(2, 1, 64, [n, n - 3], dtype="bf16", spike_every=170, true_rank=2, seed=82)
    _check_segments(_segment(S, _bdims(S, p, 1, 64, min_span=3, window=77), p), p, 1.0, 3, 77, n)


@pytest.mark.parametrize("n,spikes,min_span", [(20000, [], 20001), (20000, [64, 97, 130, 9000, 9001, 9067], 20000),
                                               (3000, [31, 64, 98, 1500], 33), (70001, [65535, 65536], 65535)])
def test_segment_long_runs_of_anchors(S, n, spikes, min_span):  # noqa: F811
    """Runs shorter than min_span up to a whole sequence: one lane writes a run of up to 32 tokens, its
    wave a longer one."""
    banner(f"anchor runs {n} min_span {min_span}")
    p = make_prefill(2, 1, 64, [n, max(1, n // 3)], dtype="bf16", true_rank=2, seed=85)
    p.surprisal[:] = 1.0
    for b in range(2):
        p.surprisal[b, [t for t in spikes if t < int(p.n_tokens[b])]] = 50.0
    _check_segments(_segment(S, _bdims(S, p, 1, 64, min_span=min_span, window=2), p), p, 1.0, min_span, 2, n)
